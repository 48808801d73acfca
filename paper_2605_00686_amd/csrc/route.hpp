// Gate: fp64-accumulated logits, wavefront top-k, softmax over the chosen k
// (paper section 2.1 step 1), plus the per-block / per-destination histograms
// that feed the dispatch plan.
#pragma once
#include "common.hpp"
#include "gate.hpp"
#include "gate_direct.hpp"

namespace moe {

typedef __attribute__((ext_vector_type(4))) double f64x4_t;

// How a gate task lays out its work.  The gate weights and the task's 16 rows
// of x pass through LDS in chunks of KC reduction indices (weights: row stride
// RS bytes, x: row stride XRS bytes), two buffers, the next chunk in flight
// while this one multiplies.  A chunk is made as large as LDS allows (72 KB in
// all, so that two workgroups still share a CU): its multiplications then
// outlast the trip to memory of the next one.  The E/16 expert blocks are dealt
// to `groups` groups of wavefronts, and the `parts` wavefronts of a group take
// alternate 16-index pieces of every chunk.
constexpr int kRouteLds = 72 * 1024;
constexpr int kRouteMaxKC = 512;
struct RouteShape {
    int RS, XRS, KC, nb, groups, parts, nbw;
};
__host__ __device__ inline RouteShape route_shape(int E, int elem_size) {
    RouteShape r;
    r.RS = (E * elem_size + 15) / 16 * 16;
    const int budget = (kRouteLds - kRouteTokens * E * 8) / 2;  // bytes per buffer
    r.KC = budget / (r.RS + kRouteTokens * elem_size) / 16 * 16;
    if (r.KC > kRouteMaxKC) r.KC = kRouteMaxKC;
    if (r.KC < 16) r.KC = 16;
    r.XRS = r.KC * elem_size;
    r.nb = (E + 15) / 16;
    r.groups = r.nb >= 4 ? 4 : r.nb >= 2 ? 2 : 1;
    r.parts = 4 / r.groups;
    r.nbw = (r.nb + r.groups - 1) / r.groups;
    return r;
}
__host__ __device__ inline size_t route_stage_bytes(const RouteShape &r) {
    return (size_t)r.KC * r.RS + (size_t)kRouteTokens * r.XRS;
}
__host__ __device__ inline size_t route_smem_bytes(int E, int elem_size) {
    const RouteShape r = route_shape(E, elem_size);
    return (size_t)kRouteTokens * E * 8 + 2 * route_stage_bytes(r);  // logits [16][E] f64 + two chunks
}

// (value, index) argmax step: larger value wins, equal values -> lower index
__device__ __forceinline__ void argmax_merge(double &v, int &i, double ov, int oi) {
    if (ov > v || (ov == v && oi < i)) {
        v = ov;
        i = oi;
    }
}

template <typename ET>
struct RouteLoad;
template <>
struct RouteLoad<bf16_t> {
    typedef uint2 x4_t;  // four consecutive bf16
    static __device__ __forceinline__ double get(const x4_t &v, int s) {
        const u32 w = (s < 2) ? v.x : v.y;
        return (double)__uint_as_float((s & 1) ? (w & 0xffff0000u) : (w << 16));
    }
    // value of the raw element, or 0.0 when keep == 0 (keep is 0 or ~0: no branch around the load)
    static __device__ __forceinline__ double to_double(bf16_t r, u32 keep) {
        return (double)__uint_as_float(((u32)r << 16) & keep);
    }
};
template <>
struct RouteLoad<float> {
    typedef float4 x4_t;
    static __device__ __forceinline__ double get(const x4_t &v, int s) {
        return (double)(s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w);
    }
    static __device__ __forceinline__ double to_double(float r, u32 keep) {
        return (double)__uint_as_float(__float_as_uint(r) & keep);
    }
};

// Logits of tokens [t0, t0+16) into lg[16][E] (LDS, fp64) with the fp64 matrix
// cores: D[token][expert] += x[token][k] * Wg[k][expert], 16 x 16 x 4 per
// instruction.  bf16/fp32 inputs convert exactly and their products are exact
// in fp64, so the only rounding is the fp64 accumulation.  Lane l feeds token
// (or expert) l % 16 and reduction index 4*(l / 16) + s within a piece of 16.
// Both operands come through LDS: wide coalesced loads one chunk ahead, double
// buffered, one barrier per chunk.  Wavefronts of different groups own
// different experts; the PARTS wavefronts of a group add their partial sums
// into LDS one after the other (fixed order: deterministic).
// Only the reduction indices [k_begin, k_end) are summed (both multiples of 16), in chunks of up to
// RouteShape::KC; the bias is added if add_bias.
template <typename ET, int NBW, int PARTS>
__device__ __forceinline__ void route_logits(const KArgs &a, int t0, char *smem, int k_begin, int k_end, bool add_bias) {
    typedef RouteLoad<ET> L;
    typedef typename L::x4_t x4_t;
    constexpr int ES = (int)sizeof(ET);
    constexpr int GROUPS = 4 / PARTS;
    constexpr int MAXPW = 7, MAXPX = 8;  // 16-byte pieces of a chunk per thread (the most route_shape() can ask for)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int E = a.E, d = a.d;
    const RouteShape rs = route_shape(E, ES);
    const int li = lane & 15, kq = lane >> 4;
    const int g = wave % GROUPS, part = wave / GROUPS;
    double *lg = (double *)smem;  // [16][E]
    char *stage = smem + (size_t)kRouteTokens * E * 8;
    const int stage_bytes = (int)route_stage_bytes(rs);
    const int x_off = rs.KC * rs.RS;  // x rows follow the weight rows of a buffer
    const char *x = (const char *)a.x;
    const char *Wg = (const char *)a.Wg;
    const int row_bytes = E * ES;
    const bool wide = (row_bytes % 16) == 0;
    const int ppr = row_bytes / 16;

    // this wavefront's expert columns; lanes past E read a valid column and are masked
    u32 keep[NBW];
    int col_off[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
        const int e = (g + b * GROUPS) * 16 + li;
        keep[b] = e < E ? ~0u : 0u;
        col_off[b] = (e < E ? e : 0) * ES;
    }
    f64x4_t acc[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b) acc[b] = f64x4_t{0.0, 0.0, 0.0, 0.0};

    u32x4_t prew[MAXPW], prex[MAXPX];
    auto fetch = [&](int c) __attribute__((always_inline)) {  // chunk c -> registers
        const int k0 = k_begin + c * rs.KC, rows = min(rs.KC, k_end - k0);
        if (wide) {
#pragma unroll
            for (int i = 0; i < MAXPW; ++i) {
                const int q = tid + i * kThreads;
                if (q < rows * ppr) prew[i] = *(const u32x4_t *)(Wg + (size_t)(k0 + q / ppr) * row_bytes + (q % ppr) * 16);
            }
        }
        const int ppx = rows * ES / 16;
#pragma unroll
        for (int i = 0; i < MAXPX; ++i) {
            const int q = tid + i * kThreads;
            if (q < kRouteTokens * ppx) {
                const int tok = min(t0 + q / ppx, a.T - 1);
                prex[i] = *(const u32x4_t *)(x + ((size_t)tok * d + k0) * ES + (q % ppx) * 16);
            }
        }
    };
    auto store = [&](int c, int buf) __attribute__((always_inline)) {  // registers -> LDS buffer
        const int k0 = k_begin + c * rs.KC, rows = min(rs.KC, k_end - k0);
        char *dst = stage + buf * stage_bytes;
        if (wide) {
#pragma unroll
            for (int i = 0; i < MAXPW; ++i) {
                const int q = tid + i * kThreads;
                if (q < rows * ppr) *(u32x4_t *)(dst + (q / ppr) * rs.RS + (q % ppr) * 16) = prew[i];
            }
        } else {  // odd row sizes (tiny expert counts): element by element, straight from global memory
            for (int q = tid; q < rows * E; q += kThreads)
                *(ET *)(dst + (q / E) * rs.RS + (q % E) * ES) = *(const ET *)(Wg + ((size_t)(k0 + q / E) * E + q % E) * ES);
        }
        const int ppx = rows * ES / 16;
#pragma unroll
        for (int i = 0; i < MAXPX; ++i) {
            const int q = tid + i * kThreads;
            if (q < kRouteTokens * ppx) *(u32x4_t *)(dst + x_off + (q / ppx) * rs.XRS + (q % ppx) * 16) = prex[i];
        }
    };
    auto mul = [&](int c, int buf) __attribute__((always_inline)) {
        const int pieces = min(rs.KC, k_end - k_begin - c * rs.KC) / 16;
        const char *src = stage + buf * stage_bytes;
        const char *xs = src + x_off + li * rs.XRS + 4 * kq * ES;
        for (int u = part; u < pieces; u += PARTS) {
            const x4_t xv = *(const x4_t *)(xs + 16 * u * ES);
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
                const double av = L::get(xv, s2);
                const char *wrow = src + (16 * u + 4 * kq + s2) * rs.RS;
#pragma unroll
                for (int b = 0; b < NBW; ++b) {
                    const double bv = L::to_double(*(const ET *)(wrow + col_off[b]), keep[b]);
                    acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[b], 0, 0, 0);
                }
            }
        }
    };

    const int c_end = (k_end - k_begin + rs.KC - 1) / rs.KC;
    fetch(0);
    store(0, 0);
    __syncthreads();
    for (int c = 0; c < c_end; ++c) {
        const int buf = c & 1;
        if (c + 1 < c_end) fetch(c + 1);
        mul(c, buf);
        if (c + 1 < c_end) store(c + 1, buf ^ 1);
        __syncthreads();
    }
    // D layout: lane l, register v -> token 4*v + l/16, expert (block) l % 16
    for (int p2 = 0; p2 < PARTS; ++p2) {
        if (part == p2) {
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                const int e = (g + b * GROUPS) * 16 + li;
                if (e < E) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int t = 4 * v + kq;
                        const double prev = (p2 == 0) ? (add_bias && a.bias ? (double)a.bias[e] : 0.0) : lg[t * E + e];
                        lg[t * E + e] = prev + acc[b][v];
                    }
                }
            }
        }
        __syncthreads();
    }
}

// A gate split over its reduction gives every task a slice of whole 16-index pieces, at least
// kRouteMinSlice indices long: the most slices a reduction of length d can have.
constexpr int kRouteMinSlice = 128;
__host__ __device__ inline int route_max_slices(int d) { return d / kRouteMinSlice > 1 ? d / kRouteMinSlice : 1; }

template <typename ET>
__device__ __forceinline__ void route_logits_dispatch(const KArgs &a, int t0, char *smem, int k0, int k1, bool bias) {
    const RouteShape rs = route_shape(a.E, (int)sizeof(ET));
    if (rs.parts == 4)
        route_logits<ET, 1, 4>(a, t0, smem, k0, k1, bias);
    else if (rs.parts == 2) {
        if (rs.nbw == 1)
            route_logits<ET, 1, 2>(a, t0, smem, k0, k1, bias);
        else
            route_logits<ET, 2, 2>(a, t0, smem, k0, k1, bias);
    } else if (rs.nbw == 1)
        route_logits<ET, 1, 1>(a, t0, smem, k0, k1, bias);
    else if (rs.nbw == 2)
        route_logits<ET, 2, 1>(a, t0, smem, k0, k1, bias);
    else if (rs.nbw == 3)
        route_logits<ET, 3, 1>(a, t0, smem, k0, k1, bias);
    else
        route_logits<ET, 4, 1>(a, t0, smem, k0, k1, bias);
}

// Exact logits of all experts in lg[16][E] (LDS) -> top-k by k rounds of a 64-lane butterfly
// argmax on (value, index), softmax over the chosen k; each wavefront selects for its four
// tokens (wave, wave + 4, ...) at once, so that the four shuffle chains overlap.  Choices counted in cnt if do_hist.
// Logits that are no numbers: a position no expert can be given is -1, which count_choice and the dispatch report.
__device__ __forceinline__ void select_full(const KArgs &a, int t0, int TOK, const double *lg, int *cnt, bool do_hist) {
    constexpr int TPW = kRouteTokens / 4;
    const int E = a.E, k = a.k;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double NEG = -__builtin_huge_val();
    double v[TPW][4], my_v[TPW];
    int my_e[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int tl = wave + 4 * i;
        my_v[i] = 0.0;
        my_e[i] = -1;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[i][q] = (lane + 64 * q < E) ? lg[tl * E + lane + 64 * q] : NEG;
    }
    // The argmax rounds below need k logits that are numbers above -inf, which is also what marks the experts already
    // taken; a gate bias of -inf and logits that are no numbers can leave fewer.
    bool scarce = false;
    if (E > 64) {
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            int n = 0;
            u64 nan = 0ull;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                n += __popcll(__ballot(v[i][q] > NEG));
                nan |= __ballot(v[i][q] != v[i][q]);
            }
            scarce = scarce || n < k || nan != 0ull;
        }
    }
    if (E <= 64) {
        // one logit per lane: its output position is the number of logits that beat it (larger value, or
        // equal value and lower expert id: the order of the argmax rounds below), counted against
        // broadcast reads of the row; position j then goes to lane j.  E steps instead of k shuffle trees.
        int rank[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) rank[i] = lane < E ? 0 : (1 << 20);
        for (int c = 0; c < E; ++c) {
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const double ov = lg[(wave + 4 * i) * E + c];
                rank[i] += (ov > v[i][0] || (ov == v[i][0] && c < lane)) ? 1 : 0;
            }
        }
        for (int j = 0; j < k; ++j) {
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int src = __ffsll((long long)__ballot(rank[i] == j)) - 1;
                const double bv = __shfl(v[i][0], src, 64);
                if (lane == j) {
                    my_v[i] = bv;
                    my_e[i] = src;
                }
            }
        }
    } else if (scarce) {  // by rank, as for up to 64 experts: position j is the lowest expert that exactly j logits beat, or -1
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            int rank[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) rank[q] = lane + 64 * q < E ? 0 : (1 << 20);
            for (int c = 0; c < E; ++c) {
                const double ov = lg[(wave + 4 * i) * E + c];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    rank[q] += (ov > v[i][q] || (ov == v[i][q] && c < lane + 64 * q)) ? 1 : 0;
            }
            for (int j = 0; j < k; ++j) {
                int be = -1;
                double bv = NEG;
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    const u64 m = __ballot(rank[q] == j);
                    if (m != 0ull) {
                        const int src = __ffsll((long long)m) - 1;
                        bv = __shfl(v[i][q], src, 64);
                        be = src + 64 * q;
                    }
                }
                if (lane == j) {
                    my_v[i] = bv;
                    my_e[i] = be;
                }
            }
        }
    } else {
        for (int j = 0; j < k; ++j) {
            double bv[TPW];
            int bi[TPW];
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                bv[i] = v[i][0];
                bi[i] = lane;
#pragma unroll
                for (int q = 1; q < 4; ++q) argmax_merge(bv[i], bi[i], v[i][q], lane + 64 * q);
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
                for (int i = 0; i < TPW; ++i) {
                    const double ov = __shfl_xor(bv[i], off, 64);
                    const int oi = __shfl_xor(bi[i], off, 64);
                    argmax_merge(bv[i], bi[i], ov, oi);
                }
            }
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (bi[i] == lane + 64 * q) v[i][q] = NEG;
                if (lane == j) {
                    my_v[i] = bv[i];
                    my_e[i] = bi[i];
                }
            }
        }
    }
    // softmax over the k chosen logits
    double ex[TPW], sum[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const double m = __shfl(my_v[i], 0, 64);
        ex[i] = (lane < k) ? exp(my_v[i] - m) : 0.0;
        sum[i] = ex[i];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int i = 0; i < TPW; ++i) sum[i] += __shfl_xor(sum[i], off, 64);
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int tl = wave + 4 * i, t = t0 + tl;
        if (tl < TOK && t < a.T && lane < k) {
            store_through(&a.idx[(size_t)t * k + lane], my_e[i]);
            store_through(&a.w[(size_t)t * k + lane], (float)(ex[i] / sum[i]));
            if (do_hist) count_choice(a, cnt, t, my_e[i]);
        }
    }
}

// The fallback of a screened task, a real call because it hardly ever runs: exact logits of all experts, selection, counts.
static __device__ __attribute__((noinline)) void route_fallback(KArgsAddr args, u32 smem_off, int t0, int TOK, int do_hist) {
    KArgs a = load_kernel_args(args);
    a.x = as_global((const char *)a.x);
    a.Wg = as_global((const char *)a.Wg);
    a.bias = as_global(a.bias);
    a.idx = as_global(a.idx);
    a.w = as_global(a.w);
    a.seg_cnt = as_global(a.seg_cnt);
    a.ctrl = as_global(a.ctrl);
    t0 = uniform(t0), TOK = uniform(TOK), do_hist = uniform(do_hist);
    char *smem = lds_at((u32)uniform((int)smem_off));
    route_logits_dispatch<bf16_t>(a, t0, smem + kMaxExperts * 4, 0, a.d, true);
    select_full(a, t0, TOK, (const double *)(smem + kMaxExperts * 4), (int *)smem, do_hist != 0);
}
// LDS of a gate task: the counts, then what its path needs
__host__ __device__ inline size_t gate_task_smem_bytes(int E, int d, int elem_size) {
    const size_t full = (size_t)kMaxExperts * 4 + route_smem_bytes(E, elem_size);
    const size_t screened = elem_size == 2 ? (size_t)gate_screened_lds(gate_variant(E, d)) : 0;
    const size_t direct = elem_size == 2 ? direct_lds_bytes(E, d, kThreads) : 0;
    const size_t most = full > screened ? full : screened;
    return most > direct ? most : direct;
}

// One gate task: the a.gate_tok tokens from t0 = task * a.gate_tok.  With a.Wg == NULL the routing is an input and only
// the histograms are produced (a task is then a whole permutation block).
// fp32 problems with few tokens (a decode-sized batch): few blocks of 16 and an idle GPU while they run, so the
// megakernel may split the gate: a.gate_split = S > 1 tasks per block, task = b*S + s sums slice s
// of the reduction and leaves its partial logits in the workspace; whichever task of a block
// finishes last adds the S partial sums in slice order (so the result does not depend on who that
// is) and goes on to the selection; the others are done.  s_slot: an int in LDS outside `smem`.
// WGT, wgt_ready: see route_screened.  NT: threads of the workgroup.
template <typename ET, int V, bool WGT, int NT, class WgtReady>
__device__ __forceinline__ void route_task(const KArgs &a, KArgsAddr args, int task, char *smem, bool do_hist, int *s_slot,
                                           WgtReady wgt_ready) {
    static_assert(NT == kThreads || V == kGateDirect, "the other gates' tasks are written for kThreads threads");
    const int E = a.E, k = a.k;
    // (the megakernel's bf16 problems with a gate have V > 0)
    const bool compute = (V > 0 || !WGT || sizeof(ET) == 4) && a.Wg != nullptr;
    const int S = (compute && a.gate_split > 1) ? a.gate_split : 1;
    const int block = task / S, slice = task % S;
    const int TOK = compute ? a.gate_tok : kPermBlock;
    const int t0 = block * TOK;
    int *cnt = (int *)smem;  // [E] choices of the task's tokens per expert
    char *lds = smem + kMaxExperts * 4;
    for (int e = threadIdx.x; e < E; e += NT) cnt[e] = 0;
    __syncthreads();
    MOE_TT_BEGIN();
    if (compute) {
        if constexpr (V == kGateDirect) {
            if (TOK == 1)
                route_direct<1, NT, !WGT>(a, t0, slice, S, lds, cnt, do_hist);
            else if (TOK == 2)
                route_direct<2, NT, !WGT>(a, t0, slice, S, lds, cnt, do_hist);
            else
                route_direct<kDirectTokens, NT, !WGT>(a, t0, slice, S, lds, cnt, do_hist);
        } else if constexpr (V > 0) {
            if (!a.gate_screens || !route_screened<V, WGT>(a, t0, TOK, smem, do_hist, wgt_ready)) {
                route_fallback(args, lds_offset(smem), t0, TOK, do_hist ? 1 : 0);
                __syncthreads();
            }
        } else {
            const int pieces = a.d / 16;  // slice s of S: pieces [pieces * s / S, pieces * (s + 1) / S)
            route_logits_dispatch<ET>(a, t0, lds, 16 * (int)((long long)pieces * slice / S),
                                      16 * (int)((long long)pieces * (slice + 1) / S), S == 1);
            if (S > 1) {
                double *lg = (double *)lds;
                const size_t per = (size_t)kRouteTokens * E;
                double *mine = a.gate_partial + ((size_t)block * S + slice) * per;
                for (int i = threadIdx.x; i < (int)per; i += kThreads) store_through(&mine[i], lg[i]);
                sync_stores();
                if (threadIdx.x == 0) {
                    const u32 before = atomicAdd(&a.gate_parts[block], 1u);
                    *s_slot = (before == (u32)(S - 1)) ? 1 : 0;
                    if (*s_slot) fence_acquire(0);
                }
                __syncthreads();
                if (!*s_slot) return;
                // (the partial sums come from memory: all S loads of two logits are issued before the first
                // addition; one load at a time, the S round trips of a logit would come one after the other)
                const double *all = a.gate_partial + (size_t)block * S * per;
                constexpr int MAXS = 16, EU = 2;  // S <= MAXS (the host's limit)
                for (int i0 = threadIdx.x; i0 < (int)per; i0 += kThreads * EU) {
                    double part[EU][MAXS];
#pragma unroll
                    for (int u = 0; u < EU; ++u) {
                        const int i = min(i0 + u * kThreads, (int)per - 1);
#pragma unroll
                        for (int s2 = 0; s2 < MAXS; ++s2)
                            if (s2 < S) part[u][s2] = all[(size_t)s2 * per + i];
                    }
#pragma unroll
                    for (int u = 0; u < EU; ++u) {
                        const int i = i0 + u * kThreads;
                        if (i < (int)per) {
                            double v = a.bias ? (double)a.bias[i % E] : 0.0;
#pragma unroll
                            for (int s2 = 0; s2 < MAXS; ++s2)
                                if (s2 < S) v += part[u][s2];
                            lg[i] = v;
                        }
                    }
                }
                __syncthreads();
            }
            select_full(a, t0, TOK, (const double *)lds, cnt, do_hist);
        }
    } else {
        for (int q = threadIdx.x; q < TOK * k; q += NT) {
            const int t = t0 + q / k;
            if (t < a.T) count_choice(a, cnt, t, a.idx[(size_t)t0 * k + q]);
        }
    }
    if (do_hist) {
        // The task's tokens lie in one permutation block: the non-zero counts are added to the block's histogram with
        // few, uncontended global atomics.  The per-destination counts come from the block histograms in the plan
        // whenever destinations are whole blocks; else they were counted slot by slot.
        __syncthreads();
        int32_t *bh = a.blk_hist + (size_t)(t0 / kPermBlock) * E;
        for (int e = threadIdx.x; e < E; e += NT)
            if (cnt[e] != 0) atomicAdd(&bh[e], cnt[e]);
    }
    MOE_TT(a.ctrl, 33);
}

}  // namespace moe
