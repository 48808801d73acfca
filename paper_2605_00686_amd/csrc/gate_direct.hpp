// Gate of bf16 problems of few tokens: exact fp64 logits of all experts, a task per CU (paper section 2.1 step 1).
//
// With few tokens what a gate task costs is not its arithmetic but its chain of steps, and the screen (gate.hpp) has a long one:
// approximate logits, bounds, threshold, candidates, exact logits, selection.  Here a task has 1 to kDirectTokens tokens, so that there
// is at most one task per CU, and goes over the gate weights once, as they lie in memory: a thread takes 8 experts (16
// bytes of a row) and every RL-th group of four rows, the next 8 rows' loads in flight while it multiplies these on the vector
// ALU (bf16 products are exact in fp64; its fp64 rate is the matrix cores').  The threads' partial sums meet in LDS.  In the
// megakernel the experts are cut into parts where that keeps more CUs busy; the part that finishes last selects.
// Bound: three instructions per weight (shift or mask, conversion to fp64, which runs at full rate, and the product; one more per
// further token), of 5.5 cycles each with one wavefront per SIMD, and the chain of steps around them.
#pragma once
#include "common.hpp"
#include "gate.hpp"

namespace moe {

constexpr int kGateDirect = 7;  // this gate's number among the gate variants (see gate_variant)
constexpr int kDirectTokens = 4;
constexpr int kDirectSplitTokens = 128;           // more tokens are one task per CU, or nearly, as they are
constexpr int kDirectMaxParts = 8;
// Partial sums of a logit from which on the standalone gate adds them up in two steps (inside the layer, where few-token tasks have
// as many, it made no difference).  moe_route of 1024 tokens x 16 experts of d 512 7.8 -> 7.0 us, 300 x 8 of 512 8.9 -> 6.2.
constexpr int kDirectRuns = 64;
// Threads of a task of the standalone gate: two wavefronts per SIMD where there are enough weights for them, 256 / 512 threads, us: 128 tokens x 128
// experts of d 7168 44.0 / 38.8, 256 x 256 of 4096 49.4 / 43.5, 1024 x 128 of 2048 28.0 / 27.0, 128 x 32 of 7168 15.7 / 14.3; the other way 1024 x 24 of
// 4096 17.1 / 18.2, 1024 x 16 of 512 7.8 / 9.3.  (No warming of the L2 in either: it is a trip to memory before the first load, and the
// tasks' own loads find each other's lines; 8 tokens x 128 of 2048 19.7 -> 16.9, 8 x 256 of 4096 54.7 -> 42.3.)
__host__ __device__ inline int direct_threads_alone(int E, int d) { return (long long)E * d > 1 << 17 ? 512 : 256; }
constexpr size_t kDirectLds = 96 * 1024;  // of a task's tokens as fp32
__host__ __device__ inline int direct_tokens(int T) { return T <= 256 ? 1 : T <= 512 ? 2 : kDirectTokens; }
// Whether a gate takes this form (x and Wg may start anywhere: the loads accept any address).  Gate end inside the layer, the screen's / this one's,
// us: E 128, d 2048 8 tokens 29 / 17, 128 30 / 22, 512 31 / 29, 513 31 / 40; E 32, d 7168 128 tokens 41 / 21, 512 47 / 27; E 48, d 1024 1024 tokens
// 26 / 19; E 64, d 2048 256 24 / 18, 513 28 / 31; E 128, d 7168 512 71 / 61; E 256, d 4096 256 60 / 56, 512 62 / 67; E 256, d 2048 512 42 / 41; E 128,
// d 512 1024 27 / 23.  Alone (the screen goes over the weights twice there): E 128, d 2048 8 tokens 37 / 17, 1024 38 / 27; E 256, d 2048 1024
// tokens 54 / 43; E 256, d 4096 1024 85 / 83.
__host__ __device__ inline bool gate_is_direct(int T, int E, int d, bool alone) {
    const long long work = (long long)E * d, most = T <= 256 || (T <= 512 && E <= 128) ? 1 << 20 : T <= 512 || alone ? 1 << 19 : 1 << 16;
    return E % 8 == 0 && T <= 256 * kDirectTokens && (size_t)direct_tokens(T) * d * 4 <= kDirectLds && work <= most;
}
// Parts of a task in the megakernel: as many as there are CUs for, of at least 16 experts, where that is worth handing the logits
// over (3 us): 8 tokens of E 128, d 2048 21.7 us in one part, 17.0 in 8; E 64, d 2048 14.7 and, in 4, 16.2
__host__ __device__ inline int direct_parts(int T, int E, int d) {
    if (T > kDirectSplitTokens || (long long)E * d < 1 << 18) return 1;
    int S = 256 / T;
    if (S > E / 16) S = E / 16;
    if (S > kDirectMaxParts) S = kDirectMaxParts;
    return S > 1 ? S : 1;
}
// Threads that share a piece's column: as many as the largest part has room for, in every part, so that every expert's sum has
// the same order.  Experts with the same weights have the same logit then, and the lower id comes first.
__host__ __device__ inline int direct_threads(int E, int parts, int threads) { return threads / ((E / 8 + parts - 1) / parts); }
__host__ __device__ inline size_t direct_lds_bytes(int E, int d, int threads) {
    const size_t rows = (size_t)kDirectTokens * d * 4 < kDirectLds ? (size_t)kDirectTokens * d * 4 : kDirectLds;
    const size_t part = (size_t)kDirectTokens * threads * 64;
    return kMaxExperts * 4 + (rows > part ? rows : part) + (size_t)kDirectTokens * E * 8 + kDirectTokens * 32 * 4;
}

// Token t's results from its choices, position j in lane j of a wavefront: expert e (-1: none) with logit v
__device__ __forceinline__ void finish_token(const KArgs &a, int t, int e, double v, int *cnt, bool do_hist) {
    const int lane = threadIdx.x & 63, k = a.k;
    const double m = __shfl(v, 0, 64), ex = lane < k ? exp(v - m) : 0.0;
    double sum = ex;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (t < a.T && lane < k) {
        store_through(&a.idx[(size_t)t * k + lane], e);
        store_through(&a.w[(size_t)t * k + lane], (float)(ex / sum));
        if (do_hist) count_choice(a, cnt, t, e);
    }
}

// Top-k of one token's exact logits lg[E] (LDS) by one wavefront, softmax over them; e_at, v_at: 32 entries each in LDS.  Position j is the
// lowest expert that exactly j logits beat (larger, or equal and lower id), or -1 where there is none (logits that are no
// numbers beat none and are beaten by none).
__device__ __forceinline__ void select_wave(const KArgs &a, int t, const double *lg, int *e_at, double *v_at, int *cnt, bool do_hist) {
    const int lane = threadIdx.x & 63, E = a.E, k = a.k;
    double v[4];
    u64 key[4];  // order-preserving; 0 past the last expert
    bool odd = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = lane + 64 * q;
        v[q] = e < E ? lg[e] : 0.0;
        odd = odd || v[q] != v[q];
        const u64 u = (u64)__double_as_longlong(v[q] + 0.0);  // (-0 is 0)
        key[q] = e < E ? ((long long)u < 0 ? ~u : u | 0x8000000000000000ull) : 0ull;
    }
    if (lane < k) e_at[lane] = -1, v_at[lane] = -__builtin_huge_val();
    wave_lds_order();
    if (__any(odd)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = lane + 64 * q;
            int rank = e < E ? 0 : (1 << 20);
            for (int c = 0; c < E; ++c) rank += (lg[c] > v[q] || (lg[c] == v[q] && c < e)) ? 1 : 0;
            for (int j = 0; j < k; ++j) {
                const u64 m = __ballot(rank == j);
                if (lane == 0 && m != 0ull && e_at[j] < 0) {
                    e_at[j] = 64 * q + __ffsll((long long)m) - 1;
                    v_at[j] = lg[e_at[j]];
                }
            }
        }
        wave_lds_order();
    } else {
        // K: the k-th largest key, or a smaller number that still parts the keys at k: bisection, over as soon as exactly k keys reach K
        u64 K = 1ull, hi = ~0ull;  // count(>= K) >= k > count(>= hi)
        int n = E;
        while (n != k && hi - K > 1ull) {
            const u64 mid = K + ((hi - K) >> 1);
            int m = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) m += __popcll(__ballot(key[q] >= mid));
            if (m >= k)
                K = mid, n = m;
            else
                hi = mid;
        }
        // those above K, then ties at K in expert order, into the list
        int above = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) above += __popcll(__ballot(key[q] > K));
        int pos = 0, ties = n == k ? k : k - above;  // (exactly k keys: all of them go in)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool tie = n != k && key[q] == K, in0 = n == k ? key[q] >= K : key[q] > K;
            const u64 mt = __ballot(tie);
            const bool in = in0 || (tie && (int)__popcll(mt & ((1ull << lane) - 1ull)) < ties);
            ties -= (int)__popcll(mt);
            const u64 m = __ballot(in);
            if (in) {
                const int at = pos + (int)__popcll(m & ((1ull << lane) - 1ull));
                e_at[at] = lane + 64 * q;
                v_at[at] = v[q];
            }
            pos += (int)__popcll(m);
        }
        wave_lds_order();
        // their order
        const double mine = lane < k ? v_at[lane] : 0.0;
        const int my_e = lane < k ? e_at[lane] : 0;
        int rank = 0;
        for (int c = 0; c < k; ++c) {
            const double ov = v_at[c];
            rank += (ov > mine || (ov == mine && e_at[c] < my_e)) ? 1 : 0;
        }
        wave_lds_order();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane < k) e_at[rank] = my_e, v_at[rank] = mine;
        wave_lds_order();
    }
    finish_token(a, t, lane < k ? e_at[lane] : -1, lane < k ? v_at[lane] : -__builtin_huge_val(), cnt, do_hist);
}

// Part `slice` of S of a task (the experts are cut by pieces of 8 into S parts): tokens [t0, t0 + TOK): idx and w written, choices counted in cnt (LDS, zeroed) if do_hist.  lds: behind cnt, 16-byte aligned.
// NT: threads of the workgroup.  ALONE: the standalone gate's.
template <int TOK, int NT, bool ALONE>
__device__ __forceinline__ void route_direct(const KArgs &a, int t0, int slice, int S, char *lds, int *cnt, bool do_hist) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.d;
    const int p0 = a.E / 8 * slice / S, ppr = a.E / 8 * (slice + 1) / S - p0;  // the part's pieces of a row
    const int E = 8 * ppr, RL = a.gate_direct;        // its experts; threads that share a piece's column (direct_threads)
    const int rl = tid / ppr, p = tid - rl * ppr;
    float *xs = (float *)lds;                         // [TOK][d]
    double *part = (double *)lds;                     // [RL][TOK][E], in their place
    const size_t rows = (size_t)TOK * d * 4, parts = (size_t)RL * TOK * E * 8;
    double *lg = (double *)(lds + (rows > parts ? rows : parts));  // [TOK][E], in the end of all experts
    int *at = (int *)(lg + TOK * a.E);                // [TOK][32] (see select_wave)
    const char *Wg = (const char *)a.Wg;
    MOE_TT_BEGIN();
    constexpr int G = 2;                              // groups of four rows per batch
    const int n_groups = d / 4, nb = (n_groups + RL * G - 1) / (RL * G);
    const bool active = rl < RL;
    u32x4_t wa[4 * G], wb[4 * G];
    auto load = [&](u32x4_t(&w)[4 * G], int b) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int row = 4 * min(min(rl, RL - 1) + RL * (b * G + g), n_groups - 1);
#pragma unroll
            for (int u = 0; u < 4; ++u) w[4 * g + u] = load16_unaligned(Wg, ((u32)(row + u) * (u32)a.E + 8u * (u32)(p0 + p)) * 2u);
        }
    };
    load(wa, 0);
    // the tokens' rows, as fp32
    for (int q = tid; q < TOK * d / 8; q += NT) {
        const int t = q / (d / 8), c = q - t * (d / 8);
        const u32x4_t v = load16_unaligned((const char *)a.x + (size_t)min(t0 + t, a.T - 1) * d * 2, 16u * (u32)c);
        f32x4_t lo, hi;
        lo[0] = __uint_as_float(v[0] << 16), lo[1] = __uint_as_float(v[0] & 0xffff0000u);
        lo[2] = __uint_as_float(v[1] << 16), lo[3] = __uint_as_float(v[1] & 0xffff0000u);
        hi[0] = __uint_as_float(v[2] << 16), hi[1] = __uint_as_float(v[2] & 0xffff0000u);
        hi[2] = __uint_as_float(v[3] << 16), hi[3] = __uint_as_float(v[3] & 0xffff0000u);
        *(f32x4_t *)(xs + t * d + 8 * c) = lo;
        *(f32x4_t *)(xs + t * d + 8 * c + 4) = hi;
    }
    __syncthreads();
    MOE_TT(a.ctrl, 44);
    double acc[TOK][8];
#pragma unroll
    for (int t = 0; t < TOK; ++t)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[t][c] = 0.0;
    // (a group past the end, in the last batch, is the last one again with zeros in the place of both operands)
    auto multiply = [&](const u32x4_t(&w)[4 * G], int b, bool last) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int group = min(rl, RL - 1) + RL * (b * G + g);
            const u32 keep = !last || group < n_groups ? ~0u : 0u;
            f32x4_t xv[TOK];
#pragma unroll
            for (int t = 0; t < TOK; ++t) xv[t] = *(const f32x4_t *)(xs + t * d + 4 * min(group, n_groups - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                double xd[TOK];
#pragma unroll
                for (int t = 0; t < TOK; ++t) xd[t] = (double)__uint_as_float(__float_as_uint(xv[t][u]) & keep);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const u32 ww = w[4 * g + u][c] & keep;
                    const double lo = (double)__uint_as_float(ww << 16), hi = (double)__uint_as_float(ww & 0xffff0000u);
#pragma unroll
                    for (int t = 0; t < TOK; ++t) {
                        acc[t][2 * c] = fma(lo, xd[t], acc[t][2 * c]);
                        acc[t][2 * c + 1] = fma(hi, xd[t], acc[t][2 * c + 1]);
                    }
                }
            }
        }
    };
    for (int b = 0; b < nb; b += 2) {
        if (b + 1 < nb) load(wb, b + 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(wa, b, b + 1 == nb);
        if (b + 2 < nb) load(wa, b + 2);
        __builtin_amdgcn_sched_barrier(0);
        if (b + 1 < nb) multiply(wb, b + 1, b + 2 == nb);
    }
    __syncthreads();
    if (active) {
#pragma unroll
        for (int t = 0; t < TOK; ++t)
#pragma unroll
            for (int c = 0; c < 8; ++c) part[(rl * TOK + t) * E + 8 * p + c] = acc[t][c];
    }
    __syncthreads();
    // The RL partial sums of a logit: many of them in 2, 4, 8 or 16 runs first, a thread each, whose sums take the place of a run's first
    const int n_out = TOK * E;
    const int lr = !ALONE || RL < kDirectRuns || 2 * n_out > NT ? 0 : min(4, 31 - __clz(NT / n_out)), runs = 1 << lr;  // (RL >= 64 > runs)
    if (lr > 0) {
        const int g = tid / n_out, i = tid - g * n_out;
        if (g < runs) {
            const int r0 = RL * g >> lr, r1 = RL * (g + 1) >> lr;
            double v = 0.0;
#pragma unroll 8
            for (int r = r0; r < r1; ++r) v += part[r * n_out + i];
            part[r0 * n_out + i] = v;
        }
        __syncthreads();
    }
    for (int i = tid; i < n_out; i += NT) {
        const double s = a.bias ? (double)a.bias[8 * p0 + i % E] : 0.0;
        double v = 0.0;
        const int n = lr > 0 ? runs : RL, step = lr > 0 ? RL : 1;
#pragma unroll 8
        for (int r = 0; r < n; ++r) v += part[(step * r >> lr) * n_out + i];
        lg[i] = s + v;
    }
    __syncthreads();
    MOE_TT(a.ctrl, 45);
    if (S > 1) {  // the other parts' logits: whichever part of the block finishes last goes on
        double *all = a.gate_partial + (size_t)t0 * a.E;  // [tokens][E]
        for (int i = tid; i < TOK * E; i += NT) {
            const int t = i / E;
            if (t0 + t < a.T) store_through(&all[(size_t)t * a.E + 8 * p0 + i - t * E], lg[i]);
        }
        sync_stores();
        if (tid == 0) {
            at[0] = atomicAdd(&a.gate_parts[t0 / TOK], 1u) == (u32)(S - 1) ? 1 : 0;
            if (at[0]) fence_acquire(0);
        }
        __syncthreads();
        const bool last = uniform(at[0]) != 0;
        __syncthreads();
        if (!last) return;
        for (int i = tid; i < TOK * a.E; i += NT) lg[i] = all[min(i, (a.T - t0) * a.E - 1)];
        __syncthreads();
    }
    if (a.E <= 64) {  // the rank of every logit, a thread each (E steps of LDS reads; the bisection takes about 2 us more)
        if (tid < TOK * 32) at[tid] = 0x7fffffff;
        __syncthreads();
        for (int i = tid; i < TOK * a.E; i += NT) {
            const int t = i / a.E, e = i - t * a.E;
            const double v = lg[i];
            int rank = 0;
#pragma unroll 8
            for (int c = 0; c < a.E; ++c) {
                const double ov = lg[t * a.E + c];
                rank += (ov > v || (ov == v && c < e)) ? 1 : 0;
            }
            if (rank < a.k) atomicMin(&at[t * 32 + rank], e);
        }
        __syncthreads();
        for (int t = wave; t < TOK; t += NT / 64) {
            const int found = lane < a.k ? at[t * 32 + lane] : 0x7fffffff, e = found < a.E ? found : -1;
            finish_token(a, t0 + t, e, e >= 0 ? lg[t * a.E + e] : -__builtin_huge_val(), cnt, do_hist);
        }
        return;
    }
    // a wavefront per token
    for (int t = wave; t < TOK; t += NT / 64) select_wave(a, t0 + t, lg + t * a.E, at + t * 32, (double *)lds + t * 32, cnt, do_hist);
}

}  // namespace moe
