// Gate of bf16 problems: screen in bf16, decide in fp64 (paper section 2.1 step 1).
//
// The fp64 units retire a few per cent of what the bf16 matrix cores do, and exact
// logits of all E experts would be nearly all of a gate task.  Only the k largest
// matter, so a task first computes every logit approximately on the bf16 matrix cores
// together with a rigorous bound on its error, keeps the experts that could be among
// the k largest, and computes exact fp64 logits for those few only.  The result is
// identical to selecting on exact logits of all experts:
//   approximate  L~[t,e] = sum_i x*w (fp32 accumulation of exact products) + bias
//   bound        eps[t,e] >= |L~ - L|, from A[t,e] = sum_i |x|*|w| (second MFMA on the
//                magnitudes): every one of the d additions rounds (or truncates) by at
//                most 2^-23 of a partial sum that is at most A, so |L~ - L| <= d * 2^-23 * A
//                and twice that is taken, plus the rounding of the bias addition
//   threshold    tau[t] = the k-th largest of (L~ - eps): at least k experts have an exact
//                logit >= tau
//   candidates   {e : L~ + eps >= tau}: every expert whose exact logit reaches the k-th
//                largest exact logit is among them, ties included
// A row of zeros (a padded slot of a decode step) has the biases as its logits, exactly: no
// error bound, and of the experts that tie for the last places only the first are candidates.
// Other logits closer together than their error bounds make many candidates.  A task of 4 tokens
// has room for all E of each; if a token of a larger task has more than there is room for
// (kCandidates), or a logit or its bound is not finite (a NaN or an infinity in x or Wg: such
// bounds order nothing), the task falls back to exact logits for all experts.  An expert masked
// by a bias of -inf is no such case: its logit is -inf, exactly.
//
// First pass.  The reduction is split over the four wavefronts, which then work without
// barriers: each streams its slice of the gate weights, as they lie in memory ([d][E]),
// in chunks of KC reduction indices into LDS slots of its own, by direct global->LDS loads
// two or three chunks ahead (through registers, one chunk ahead, where the rows of Wg are
// unaligned: E is no multiple of 8, or Wg is a view that starts between 16-byte boundaries), and
// takes its MFMA operands from there with the transposing LDS read, those of the next chunk while
// this one multiplies.  The wavefronts' partial sums meet in LDS.
// Second pass, in the megakernel: rows of the transposed gate weights WgT[E][d], which the
// first front tasks of the kernel wrote to the workspace while the first passes ran, times
// the tokens' rows, straight from L2.  Standalone (no workspace): the weights are streamed
// again as in the first pass, the transposed pieces written back in their chunk's place as
// T[expert][index], and rows of T multiplied, four lanes per (token, candidate).
//
// Bound: with one wavefront per SIMD, the latency of a chunk where a task has few tokens, and
// the fp64 arithmetic of the second pass where it has 16; much of the rest is code that runs
// once per task and waits for its instructions, so it is kept short.
#pragma once
#include "common.hpp"

namespace moe {

constexpr int kCandidates = 1024;  // of a task: 64 per token of 16, 128 of 8, 256 of 4
constexpr int kGateSlots = 16;  // standalone second pass: candidates per group of lanes and sweep over the reduction

// The gate's code for a problem: 1 .. 6 = route_screened for bf16, by E and d; 0 = exact logits of all experts (fp32; also
// the code of tasks whose routing is an input)
__host__ __device__ inline int gate_variant(int E, int d) {
    return E <= 32 ? (d % 128 == 0 ? 1 : 6) : E <= 64 ? 2 : E <= 128 ? 3 : E <= 192 ? 4 : 5;
}
// Standalone gate: exact logits of all experts at once where the experts are few and the reduction short.  The screen pays a
// fixed 10 us for its two sweeps, threshold and selection, the more the more tokens a task has (see gate_tokens); the exact
// logits' cost grows with d and with the blocks of 16 experts, and is higher for rows of Wg that are no multiple of 16 bytes.
// moe_route, exact / screened, us:
//   E = 8    4096 tokens of d 2048 21.8 / 22.6, of d 4096 36.2 / 35.8; 1024 of d 1024 14.4 / 15.5, of d 2048 21.4 / 19.3
//   E = 12   4096 of d 1024 18.1 / 18.7, of d 2048 31.2 / 25.8
//   E = 24   4096 of d 640 16.3 / 17.0, of d 768 17.6 / 17.4; 2048 of d 384 12.3 / 13.6, of d 512 14.9 / 14.3; 128 of d 256 11.4 / 13.5
//   E = 48   4096 of d 256 15.2 / 15.5, of d 512 19.6 / 17.5; 2048 of d 256 14.9 / 15.0; 128 of d 256 14.9 / 13.3
//   E = 64   4096 of d 192 15.4 / 15.5, of d 256 17.4 / 16.0; 2048 of d 128 13.7 / 15.2; 128 of d 64 12.2 / 13.3, of d 128 13.7 / 13.6
//   E = 128  4096 of d 128 16.7 / 16.5, of d 192 18.6 / 17.7; 2048 of d 64 13.8 / 15.2; 128 of d 64 13.8 / 14.1, of d 128 16.6 / 14.5
__host__ __device__ inline bool route_exact(int T, int E, int d) {
    if (E <= 16) return d <= (T > 2048 && E % 8 == 0 ? 2048 : 1024);
    const int most = E <= 32 ? 640 : E <= 48 ? 384 : E <= 64 ? 192 : 128;
    return d <= (T > 2048 ? most : T > 1024 ? most * 3 / 4 : most / 2);
}
// Blocks of 16 experts (at most), reduction indices per chunk (divides d; about 8 KB of weights, so that the chunk's
// latency is spread over enough work), chunk slots per wavefront
template <int V>
struct GateCfg {
    static constexpr int NB = V == 1 || V == 6 ? 2 : V == 2 ? 4 : V == 3 ? 8 : V == 4 ? 12 : 16;
    static constexpr int KC = V == 1 ? 128 : V == 2 || V == 6 ? 64 : 32;
    static constexpr int NS = V == 2 || V == 3 || V == 6 ? 3 : 2;
    static constexpr int WBYTES = KC * NB * 32;                     // weights of a chunk, or T[16 * NB][KC]
    static constexpr int SLOT = WBYTES + kRouteTokens * KC * 2;     // ... and the tokens' x
    static constexpr int WAVE = NS * SLOT;
    // LDS: the task's expert counts, the bias, candidates, their exact logits, numbers of candidates, the wavefronts' slots
    static constexpr int O_BIAS = kMaxExperts * 4;
    static constexpr int O_CAND = O_BIAS + kMaxExperts * 4;
    static constexpr int O_EXACT = O_CAND + kCandidates * 4;
    static constexpr int O_NCAND = O_EXACT + kCandidates * 8;
    static constexpr int O_SLOTS = O_NCAND + 128;
    static constexpr int TOTAL = O_SLOTS + 4 * WAVE;
    static_assert(WAVE >= kRouteTokens * 16 * NB * 8, "a wavefront's approximate logits and magnitudes take its slots' place");
    static_assert(WAVE >= kGateSlots * 64 * 8, "so do its partial exact logits ...");
    static_assert(4 * WAVE >= kCandidates * 4 * 8, "... in either form of the second pass");
};
__host__ __device__ inline int gate_screened_lds(int variant) {
    switch (variant) {
        case 1: return GateCfg<1>::TOTAL;
        case 2: return GateCfg<2>::TOTAL;
        case 3: return GateCfg<3>::TOTAL;
        case 4: return GateCfg<4>::TOTAL;
        case 5: return GateCfg<5>::TOTAL;
        case 6: return GateCfg<6>::TOTAL;
        default: return 0;
    }
}
// Tokens per gate task: the fewest that make at most 256 tasks, one per CU, up to 16 (one MFMA row block): what a task reads
// of the weights does not shrink with its tokens, but its fp64 work does; a second task on some CUs costs more than that.
// Gate phase of the layer, 128 experts of d 2048, 4 / 8 / 16 tokens per task, us: 1024 tokens 39 / 44 / -, 1025 63 / 48 / 55, 2000
// 73 / 56 / 63, 2049 - / 71 / 66, 4096 - / 86 / 60.
__host__ __device__ inline int gate_tokens(int T) { return T > 2048 ? 16 : T > 1024 ? 8 : 4; }

constexpr int kWgtTile = 64;  // transposition tile: 64 reduction indices x 64 experts
__host__ __device__ inline int wgt_tasks(int d, int E) { return (d / kWgtTile) * ((E + kWgtTile - 1) / kWgtTile); }

// WgT[e][k0 .. k0+64) = Wg[k0 .. k0+64)[e] for 64 experts, through LDS.
__device__ __forceinline__ void wgt_task(const KArgs &a, int task, char *smem) {
    const int tid = threadIdx.x;
    const int E = a.E, d = a.d;
    const int ebn = (E + kWgtTile - 1) / kWgtTile;
    const int k0 = (task / ebn) * kWgtTile, e0 = (task % ebn) * kWgtTile;
    constexpr int LD = kWgtTile + 2;  // LDS row length in elements (odd number of dwords: column reads spread over banks)
    bf16_t *tile = (bf16_t *)smem;    // [64 k][LD]
    const bf16_t *Wg = (const bf16_t *)a.Wg;
    bf16_t *WgT = (bf16_t *)a.WgT;
    if ((E & 7) == 0) {
        // 16-byte pieces, all loads of a thread in flight together
        constexpr int PPT = kWgtTile * kWgtTile / 8 / kThreads;  // pieces per thread
        u32x4_t v[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int q = tid + kThreads * u, kk = q >> 3, e = e0 + (q & 7) * 8;
            v[u] = u32x4_t{0u, 0u, 0u, 0u};
            if (e < E) v[u] = *(const u32x4_t *)(Wg + (size_t)(k0 + kk) * E + e);
        }
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const int q = tid + kThreads * u, kk = q >> 3, pc = q & 7;
            u32 *dst = (u32 *)(tile + kk * LD + pc * 8);
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i] = v[u][i];
        }
    } else {
#pragma unroll 4
        for (int q = tid; q < kWgtTile * kWgtTile; q += kThreads) {
            const int kk = q / kWgtTile, ee = q % kWgtTile;
            tile[kk * LD + ee] = (e0 + ee < E) ? Wg[(size_t)(k0 + kk) * E + e0 + ee] : (bf16_t)0;
        }
    }
    __syncthreads();
    for (int q = tid; q < kWgtTile * kWgtTile / 8; q += kThreads) {
        const int ee = q >> 3, kp = (q & 7) * 8;
        u32x4_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = (u32)tile[(kp + 2 * i) * LD + ee] | ((u32)tile[(kp + 2 * i + 1) * LD + ee] << 16);
        if (e0 + ee < E) store_tile16((char *)(WgT + (size_t)(e0 + ee) * d + k0 + kp), make_uint4(o[0], o[1], o[2], o[3]));
    }
    __syncthreads();
}

__device__ __forceinline__ u32 float_key(float f) {  // order-preserving map of floats to unsigned integers
    const u32 u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// sum / maximum over the 16 lanes of a DPP row, in every lane of the row (row_ror by 8, 4, 2, 1)
template <int CTRL>
__device__ __forceinline__ int dpp16(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ int row_sum16(int v) {
    v += dpp16<0x128>(v);
    v += dpp16<0x124>(v);
    v += dpp16<0x122>(v);
    v += dpp16<0x121>(v);
    return v;
}
__device__ __forceinline__ u32 row_max16(u32 v) {
    v = max(v, (u32)dpp16<0x128>((int)v));
    v = max(v, (u32)dpp16<0x124>((int)v));
    v = max(v, (u32)dpp16<0x122>((int)v));
    v = max(v, (u32)dpp16<0x121>((int)v));
    return v;
}
template <int CTRL>
__device__ __forceinline__ double row_add_step(double v) {
    const int lo = dpp16<CTRL>(__double2loint(v)), hi = dpp16<CTRL>(__double2hiint(v));
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum16(double v) {
    v = row_add_step<0x128>(v);
    v = row_add_step<0x124>(v);
    v = row_add_step<0x122>(v);
    return row_add_step<0x121>(v);
}

// 16 bytes at a 2-byte aligned byte offset (a scalar base and a 32-bit offset: one address register)
__device__ __forceinline__ u32x4_t load16_unaligned(const char *base, u32 byte_offset) {
    u32x4_t v;
    __builtin_memcpy(&v, base + byte_offset, 16);
    return v;
}

// one more slot of token t for expert e: the task's count in LDS, and the destination's when the plan cannot derive it
__device__ __forceinline__ void count_choice(const KArgs &a, int *cnt, int t, int e) {
    if (e < 0 || e >= a.E) {
        set_error(a.ctrl, MOE_ERR_BAD_ROUTING);
    } else {
        atomicAdd(&cnt[e], 1);
        if (!a.seg_from_blocks) atomicAdd(&a.seg_cnt[(size_t)e * a.R + t / a.per_dest], 1);
    }
}

// LDS accesses of one wavefront are executed in program order; this keeps the compiler to it
__device__ __forceinline__ void wave_lds_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}
// 64 lanes x 16 bytes from base + voff to 1 KB of consecutive LDS at lds_addr (lane l: byte 16 * l); counted in vmcnt by
// hand, as in the GEMM main loop
__device__ __forceinline__ void load_lds16(const void *base, u32 voff, u32 lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(base)
                 : "m0", "memory");
}

// The gate weights into this XCD's L2, by all workgroups of the XCD together, each its share of the cache lines (16 bytes
// of each land in a KB of LDS nobody reads): every workgroup streams all of them, in step with the others, and would
// otherwise meet memory's latency at every chunk instead of once.  (Where workgroups run is only assumed: round-robin over
// the XCDs.)  The caller waits for the loads before it uses that KB.
__device__ __forceinline__ void gate_warm_l2(const KArgs &a, u32 lds_scratch, int wg, int n_wg) {
    if (!a.gate_screens) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u32 skip = (0u - (u32)(uintptr_t)a.Wg) & 15u;  // to the first aligned address
    const char *Wg = (const char *)a.Wg + skip;
    const long long lines = ((long long)a.d * a.E * 2 - skip) / 128;
    const int part = wg / kTileQueues, parts = (n_wg + kTileQueues - 1) / kTileQueues;
    const int l0 = (int)(lines * part / parts), l1 = (int)(lines * (part + 1) / parts);
    for (int l = l0 + wave * 64; l < l1; l += kThreads) load_lds16(Wg, (u32)min(l + lane, l1 - 1) * 128u, lds_scratch);
}

// Tokens [t0, t0 + TOK): idx and w written, choices counted in cnt if do_hist (LDS, zeroed).  Returns false, with nothing
// written, if the task must fall back to exact logits of all experts.  Uniform over the workgroup.
// WGT: the transposed gate weights are there once wgt_ready() returns true (called by all threads; false: the caller's
// problem is void).
template <int V, bool WGT, class WgtReady>
__device__ __forceinline__ bool route_screened(const KArgs &a, int t0, int TOK, char *smem, bool do_hist, WgtReady wgt_ready) {
    using G = GateCfg<V>;
    constexpr int NB = G::NB, KC = G::KC, NS = G::NS;
    constexpr int KK = KC / 32, CPR = KC / 8;  // MFMA steps and 16-byte pieces per x row of a chunk
    constexpr int NWP = KC * NB / 32;          // weight pieces per lane and chunk, at most
    constexpr int NXP = KC / 32;               // x pieces per lane and chunk; standalone second pass: pieces per lane
    // (opaque copies: what follows depends on nothing else, and the compiler would move all of it in front of the loop
    // over tasks, out to scratch memory)
    int tid = threadIdx.x, E = a.E;
    asm volatile("" : "+v"(tid), "+s"(E));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = a.d, k = a.k;
    const int li = lane & 15, kq = lane >> 4;
    const int ppr = (E + 7) / 8;                     // pieces per (padded) weight row
    int *cnt = (int *)smem;
    float *s_bias = (float *)(smem + G::O_BIAS);
    const int llpt = 8 - (31 - __clz(TOK)), lmc = llpt + 2;  // log2 of: threads, and candidates at most, per token
    int *cand = (int *)(smem + G::O_CAND);           // [TOK][1 << lmc] candidate experts
    double *exact = (double *)(smem + G::O_EXACT);   // [TOK][1 << lmc] their exact logits
    int *s_ncand = (int *)(smem + G::O_NCAND);       // [TOK]
    // the wavefront's chunk slots; after the first pass its partial logits [16][16 * NB] and sums of magnitudes
    char *wslots = smem + G::O_SLOTS + wave * G::WAVE;
    const u32 wslots_lds = lds_offset(wslots);
    const char *Wg = (const char *)a.Wg;
    const char *x = (const char *)a.x + (size_t)t0 * d * 2;
    const int nC = d / KC;
    const int c_begin = nC * wave / 4, c_end = nC * (wave + 1) / 4;
    const bool aligned = a.gate_rows_aligned != 0;
    MOE_TT_BEGIN();
    // piece p of row r of x (and of T) sits at p ^ swz(r); piece p of weight row r at (p + rot(r)) mod ppr: the 16
    // rows of an MFMA operand, and the 4 rows of a transposing read, then come from different banks (narrow rows: as is)
    auto swz = [](int r) { return KC == 32 ? (r >> 2) & 3 : KC == 64 ? (r >> 1) & 7 : r & 15; };
    auto rot = [&](int r) { return ppr >= 16 ? 2 * (r & 3) + (r & 8) : ppr >= 8 ? 2 * (r & 3) : 0; };

    // ---- what this lane loads of a chunk: the piece that belongs at its place of the slot (a place past the chunk's end
    // gets any piece: every chunk takes the same number of loads).  Unaligned: piece `lane + 64 * i` of the chunk in memory
    // order, put to its place by put_regs.
    u32 w_src[NWP], x_src[NXP];
    {
        const int drow = 64 / ppr, dpp = 64 - drow * ppr;  // from one of the lane's pieces to the next
        int row = lane / ppr, pp = lane - row * ppr;
#pragma unroll
        for (int i = 0; i < NWP; ++i) {
            int p = pp - (aligned ? rot(row) : 0);
            p += p < 0 ? ppr : 0;
            w_src[i] = (u32)(min(row, KC - 1) * E + 8 * p) * 2u;
            row += drow;
            pp += dpp;
            if (pp >= ppr) pp -= ppr, ++row;
        }
    }
#pragma unroll
    for (int i = 0; i < NXP; ++i) {
        const int q = lane + 64 * i, row = q / CPR, pp = q % CPR;
        x_src[i] = (u32)((min(t0 + (row & (TOK - 1)), a.T - 1) - t0) * d + 8 * (pp ^ swz(row))) * 2u;
    }
    u32x4_t R[NWP];  // unaligned: the next chunk's weights
    const u32 total = (u32)d * (u32)E * 2u;  // bytes of the gate weights
    auto load = [&](int c, int slot) __attribute__((always_inline)) {
        const char *wb = Wg + (size_t)c * KC * E * 2, *xb = x + (size_t)c * KC * 2;
        const u32 dst = wslots_lds + slot * G::SLOT;
        if (aligned) {
#pragma unroll
            for (int i = 0; i < NWP; ++i) load_lds16(wb, w_src[i], dst + 1024 * i);
        }
#pragma unroll
        for (int i = 0; i < NXP; ++i) load_lds16(xb, x_src[i], dst + G::WBYTES + 1024 * i);
    };
    auto fetch_regs = [&](int c) __attribute__((always_inline)) {
        const u32 o = (u32)c * (u32)(KC * E * 2);
#pragma unroll
        for (int i = 0; i < NWP; ++i) R[i] = load16_unaligned(Wg, min(o + w_src[i], total - 16u));
    };
    auto put_regs = [&](int c, char *st) __attribute__((always_inline)) {
        const u32 o = (u32)c * (u32)(KC * E * 2);
        const int drow = 64 / ppr, dpp = 64 - drow * ppr;
        int row = lane / ppr, pp = lane - row * ppr;
#pragma unroll
        for (int i = 0; i < NWP; ++i) {
            if (row < KC) {
                u32x4_t v = R[i];
                if (o + w_src[i] > total - 16u) {  // the weights' very last piece sticks out: it was loaded from further in front
                    const int sh = 8 * (int)(o + w_src[i] - (total - 16u));  // 16 .. 112 bits
                    const u64 lo = (u64)v[0] | ((u64)v[1] << 32), hi = (u64)v[2] | ((u64)v[3] << 32);
                    const u64 lo2 = sh < 64 ? (lo >> sh) | (hi << (64 - sh)) : hi >> (sh - 64);
                    const u64 hi2 = sh < 64 ? hi >> sh : 0ull;
                    v = u32x4_t{(u32)lo2, (u32)(lo2 >> 32), (u32)hi2, (u32)(hi2 >> 32)};
                }
                int p = pp + rot(row);
                p -= p >= ppr ? ppr : 0;
                *(u32x4_t *)(st + (row * ppr + p) * 16) = v;
            }
            row += drow;
            pp += dpp;
            if (pp >= ppr) pp -= ppr, ++row;
        }
    };
    {  // the wavefront's slice of the tokens' rows into the L2 (see gate_warm_l2): rows of at least 128 bytes
        const int lpr = ((c_end - c_begin) * KC * 2 + 127) / 128;  // cache lines per row
        for (int row = 0; row < TOK; ++row)
            for (int l = lane; l - lane < lpr; l += 64)
                load_lds16(x + (size_t)c_begin * KC * 2, (u32)((min(t0 + row, a.T - 1) - t0) * d * 2 + min(l, lpr - 1) * 128),
                           lds_offset(smem + G::O_EXACT));
    }
    static_assert(kThreads == kMaxExperts, "one bias per thread");
    s_bias[tid] = a.bias && tid < E ? a.bias[tid] : 0.f;
    // MFMA operands of a chunk: lane l feeds token (or expert) l % 16 and reduction indices 8 * (l / 16) .. + 7 of a step of
    // 32 (expert columns past the padded row read a valid piece and are masked in the end)
    int b_off[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int r4 = (lane & 15) >> 2;
        int p = min(2 * b + ((lane & 3) >> 1), ppr - 1) + rot(8 * kq + r4);
        p -= p >= ppr ? ppr : 0;
        b_off[b] = ((8 * kq + r4) * ppr + p) * 16 + (lane & 1) * 8;
    }
    struct Frag {
        u32x4_t x[KK], w[KK][NB];
    };
    auto read = [&](const char *st, Frag &f) __attribute__((always_inline)) {
        const char *xs = st + G::WBYTES + li * (KC * 2);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            f.x[kk] = *(const u32x4_t *)(xs + (((kk * 4 + kq) ^ swz(li)) * 16));
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const char *p = st + kk * 32 * ppr * 16 + b_off[b];
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3))) *)p);
                const s16x4_t hi =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3))) *)(p + 4 * ppr * 16));
                f.w[kk][b] = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        }
    };
    // use(operands, slot) on every chunk c of the wavefront's slice, with the operands of c + 1 on their way from LDS and
    // chunks up to c + NS - 1 on theirs from memory (past the end the last one again, so that the count of loads in
    // flight is always the same).  use() calls its last argument once it has no more need of the slot itself.
    auto sweep = [&](auto use) __attribute__((always_inline)) {
        Frag f0, f1;
#pragma unroll
        for (int u = 0; u < NS; ++u) load(min(c_begin + u, nC - 1), u);
        auto landed = [&](int c, char *st) __attribute__((always_inline)) {  // chunk c is in its slot
            if (aligned) {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * (NWP + NXP)) : "memory");
            } else {
                put_regs(c, st);
                fetch_regs(min(c + 1, nC - 1));
                // (the register loads just issued are younger than the chunk's x)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NWP) : "memory");
            }
            wave_lds_order();
        };
        if (!aligned) fetch_regs(min(c_begin, nC - 1));
        int slot = 0;
        if constexpr (NB > 8) {  // (two chunks' operands would not fit the registers: one after the other)
            for (int c = c_begin; c < c_end; ++c) {
                char *st = wslots + slot * G::SLOT;
                landed(c, st);
                read(st, f0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                use(f0, st, [&]() __attribute__((always_inline)) { load(min(c + NS, nC - 1), slot); });
                slot = slot + 1 == NS ? 0 : slot + 1;
            }
        } else {
            landed(min(c_begin, nC - 1), wslots);
            read(wslots, f0);
            for (int c = c_begin; c < c_end; c += 2) {
                auto body = [&](int cc, Frag &cur, Frag &nxt) __attribute__((always_inline)) {
                    char *st = wslots + slot * G::SLOT;
                    const int next = slot + 1 == NS ? 0 : slot + 1;
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the operands of cc have left its slot
                    use(cur, st, [&]() __attribute__((always_inline)) {
                        load(min(cc + NS, nC - 1), slot);
                        landed(min(cc + 1, nC - 1), wslots + next * G::SLOT);
                        read(wslots + next * G::SLOT, nxt);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    slot = next;
                };
                body(c, f0, f1);
                if (c + 1 < c_end) body(c + 1, f1, f0);
            }
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();  // (all slots are free: other things take their place)
    };

    // ---- first pass: D[token][expert] on the bf16 matrix cores (16 x 16 x 32), values and magnitudes
    {
        f32x4_t acc[NB], mag[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            mag[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
        const u32x4_t absmask = u32x4_t{0x7fff7fffu, 0x7fff7fffu, 0x7fff7fffu, 0x7fff7fffu};
        sweep([&](Frag &f, char *, auto go_on) __attribute__((always_inline)) {
            go_on();
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const u32x4_t xl = f.x[kk], xa = xl & absmask;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const u32x4_t wv = f.w[kk][b], wa = wv & absmask;
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, xl),
                                                                     __builtin_bit_cast(bf16x8_t, wv), acc[b], 0, 0, 0);
                    mag[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, xa),
                                                                     __builtin_bit_cast(bf16x8_t, wa), mag[b], 0, 0, 0);
                }
            }
        });
        // D layout: lane l, register v -> token 4 * (l / 16) + v, expert (block) l % 16
        float *Ls = (float *)wslots;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Ls[(4 * kq + v) * (16 * NB) + 16 * b + li] = acc[b][v];
                Ls[(kRouteTokens + 4 * kq + v) * (16 * NB) + 16 * b + li] = mag[b][v];
            }
    }
    __syncthreads();
    MOE_TT(a.ctrl, 40);

    // ---- threshold and candidates: 16 lanes per token, lane j holds experts j, j + 16, ...
    {
        const int tl = (tid >> 4) & (TOK - 1);  // (with fewer tokens than 16 the other lane rows repeat them)
        const float scale = (float)(d + 64) * (1.0f / 4194304.0f);  // (d + 64) * 2^-22
        const float *L0 = (const float *)(smem + G::O_SLOTS) + tl * (16 * NB) + li;
        // (the bias addition: |logit| is at most the sum of magnitudes plus |bias|, hence twice the latter)
        const float s_mag = 1.01f * (scale + 1.0f / 4194304.0f), s_add = 1.01f * 2.0f / 4194304.0f;
        u32 klo[NB], khi[NB], kmax = 0u;
        u32 mmax = 0u, lmax = 0u;  // largest bit pattern of a magnitude and of a logit: from 0x7f800000 on no finite number
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            float l = 0.f, mag = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                l += L0[w * (G::WAVE / 4) + 16 * q];
                mag += L0[w * (G::WAVE / 4) + kRouteTokens * 16 * NB + 16 * q];
            }
            const float bias = s_bias[(li + 16 * q) & (kMaxExperts - 1)];
            l += bias;
            mmax = max(mmax, __float_as_uint(mag));
            lmax = max(lmax, bias == -__builtin_huge_valf() ? 0u : __float_as_uint(l) & 0x7fffffffu);
            const float eps = fmaf(mag, s_mag, fmaf(fminf(fabsf(bias), 3.4e38f), s_add, 1e-30f));
            klo[q] = li + 16 * q < E ? float_key(l - eps) : 0u;
            khi[q] = li + 16 * q < E ? float_key(l + eps) : 0u;
            kmax = max(kmax, klo[q]);
        }
        bool zero = false;  // a row of zeros
        if (__builtin_expect(__any(mmax == 0u) != 0, 0)) {
            zero = row_max16(mmax) == 0u;  // (so far: no product large enough for fp32)
            const char *xr = x + (size_t)(min(t0 + tl, a.T - 1) - t0) * d * 2;
            u32 bits = 0u;
            for (int o = li * 16; o < 2 * d; o += 8 * 256) {
                u32x4_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *(const u32x4_t *)(xr + min(o + 256 * u, 2 * d - 16));
#pragma unroll
                for (int u = 0; u < 8; ++u) bits |= v[u][0] | v[u][1] | v[u][2] | v[u][3];
            }
            const u32 row_bits = row_max16(bits & 0x7fff7fffu);
            zero = zero && row_bits == 0u;
#pragma unroll
            for (int q = 0; q < NB; ++q)
                if (zero && li + 16 * q < E) {
                    klo[q] = khi[q] = float_key(0.f + s_bias[(li + 16 * q) & (kMaxExperts - 1)]);
                    kmax = max(kmax, klo[q]);
                }
        }
        // K: the k-th largest lower bound, or a smaller one that still parts the keys at k (what is needed is that at least
        // k lower bounds reach K): bisection between the largest key and none, over as soon as exactly k keys reach K
        u32 K = 0u, hi = row_max16(kmax) + 1u;  // count(>= K) >= k > count(>= hi)
        bool found = false;
        while (true) {
            const u32 mid = K + ((hi - K) >> 1);
            int n = 0;
#pragma unroll
            for (int q = 0; q < NB; ++q) n += klo[q] >= mid ? 1 : 0;
            n = row_sum16(n);
            if (!found) {
                if (n >= k)
                    K = mid;
                else
                    hi = mid;
                found = n == k || hi - K <= 1u;
            }
            if (__all(found)) break;
        }
        int before = 0;
        auto collect = [&](auto in) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const bool mine = in(q);
                const u32 m = (u32)(__ballot(mine) >> (lane & 48)) & 0xffffu;  // this token's 16 lanes
                const int pos = before + (int)__popc(m & ((1u << li) - 1u));
                if (mine && pos < (1 << lmc) && (tid >> 4) < TOK) cand[(tl << lmc) + pos] = li + 16 * q;
                before += (int)__popc(m);
            }
        };
        if (__builtin_expect(__any(zero) != 0, 0)) {
            int left = 0;  // places of a row of zeros left for the experts at K, in their order
#pragma unroll
            for (int q = 0; q < NB; ++q) left += klo[q] > K ? 1 : 0;
            left = k - row_sum16(left);
            collect([&](int q) __attribute__((always_inline)) {
                const bool in = khi[q] >= K && khi[q] != 0u, tie = zero && in && khi[q] == K;
                const u32 m = (u32)(__ballot(tie) >> (lane & 48)) & 0xffffu;
                const bool late = tie && (int)__popc(m & ((1u << li) - 1u)) >= left;
                left -= (int)__popc(m);
                return in && !late;
            });
        } else {
            collect([&](int q) __attribute__((always_inline)) { return khi[q] >= K && khi[q] != 0u; });
        }
        const bool odd = row_max16(max(mmax, lmax)) >= 0x7f800000u;
        if (li == 0 && (tid >> 4) < TOK) s_ncand[tl] = odd ? kCandidates + 1 : before;
    }
    __syncthreads();
    const int n_max = uniform((int)row_max16(li < TOK ? (u32)s_ncand[li] : 0u));
    MOE_TT(a.ctrl, 41);
    if (n_max > (1 << lmc)) {
        __syncthreads();
        return false;
    }

    if constexpr (WGT) {
        // ---- second pass, exact fp64 logits of the candidates: a wavefront takes every fourth group of four candidates of a
        // token (groups counted over all tokens, so that a token of many keeps all wavefronts busy), 512 reduction indices
        // per step (16 bytes per lane and row), UM steps' loads in flight
        if (!wgt_ready()) return true;
        constexpr int CG = 4, UM = 4;
        double *part = (double *)(smem + G::O_SLOTS);  // [TOK][1 << lmc][4]: sums over the 16 lanes of each DPP row
        const char *WgT = (const char *)a.WgT;
        const int nm = (d + 511) / 512;
        const int my_n = s_ncand[li & (TOK - 1)];
        int groups = 0;
        for (int tl = 0; tl < TOK; ++tl) {
            const int n = __builtin_amdgcn_readlane(my_n, tl);
            const char *xr = x + (size_t)(min(t0 + tl, a.T - 1) - t0) * d * 2;
            const int first = CG * ((wave - groups) & 3);
            groups += (n + CG - 1) / CG;
            for (int c0 = first; c0 < n; c0 += 4 * CG) {
                const char *wr[CG];
                double acc[CG];
#pragma unroll
                for (int i = 0; i < CG; ++i) {
                    wr[i] = WgT + (size_t)uniform(cand[(tl << lmc) + min(c0 + i, n - 1)]) * d * 2;
                    acc[i] = 0.0;
                }
                for (int m0 = 0; m0 < nm; m0 += UM) {
                    u32x4_t xv[UM], wv[UM][CG];
#pragma unroll
                    for (int u = 0; u < UM; ++u) {
                        const u32 off = 2u * (u32)min((m0 + u) * 512 + lane * 8, d - 8);
                        xv[u] = *(const u32x4_t *)(xr + off);
#pragma unroll
                        for (int i = 0; i < CG; ++i) wv[u][i] = *(const u32x4_t *)(wr[i] + off);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < UM; ++u) {
                        if ((m0 + u) * 512 < d) {
                            const u32 live = (m0 + u) * 512 + lane * 8 < d ? ~0u : 0u;
#pragma unroll
                            for (int p = 0; p < 4; ++p) {  // (products of bf16 numbers are exact in fp64)
                                const double xl = (double)__uint_as_float((xv[u][p] & live) << 16);
                                const double xh = (double)__uint_as_float(xv[u][p] & live & 0xffff0000u);
#pragma unroll
                                for (int i = 0; i < CG; ++i) {
                                    acc[i] = fma((double)__uint_as_float(wv[u][i][p] << 16), xl, acc[i]);
                                    acc[i] = fma((double)__uint_as_float(wv[u][i][p] & 0xffff0000u), xh, acc[i]);
                                }
                            }
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < CG; ++i) {
                    const double s = row_sum16(acc[i]);
                    if (li == 0 && c0 + i < n) part[((tl << lmc) + c0 + i) * 4 + kq] = s;
                }
            }
        }
        __syncthreads();
        {
            const int t = tid >> llpt, n = s_ncand[t];
            for (int c = tid & ((1 << llpt) - 1); c < n; c += 1 << llpt) {
                const int i = (t << lmc) + c;
                exact[i] = (double)s_bias[cand[i]] + ((part[4 * i] + part[4 * i + 1]) + (part[4 * i + 2] + part[4 * i + 3]));
            }
        }
        __syncthreads();
    } else {
        // ---- second pass, standalone: four lanes per (token, candidate); a group of lanes belongs to one token and takes
        // every (16 / TOK)-th of its candidates, up to kGateSlots of them per sweep over the reduction
        const int gi = lane >> 2, j = lane & 3;
        const int tl = gi & (TOK - 1), sub = gi / TOK, gpt = 16 / TOK;
        const int n = s_ncand[tl];
        double acc[kGateSlots];
        for (int base = 0; base < n_max; base += kGateSlots * gpt) {
            int eoff[kGateSlots];  // the candidate's row of T, with the swizzle in the lowest bits
#pragma unroll
            for (int s = 0; s < kGateSlots; ++s) {
                const int e = cand[(tl << lmc) + min(base + sub + s * gpt, n - 1)];
                eoff[s] = e * (KC * 2) + ((j ^ swz(e)) * 16);
                acc[s] = 0.0;
            }
            const int ns = min((n_max - base + gpt - 1) / gpt, kGateSlots);  // slots any group needs
            sweep([&](Frag &f, char *st, auto go_on) __attribute__((always_inline)) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk)
                        *(u32x4_t *)(st + (16 * b + li) * (KC * 2) + (((kk * 4 + kq) ^ swz(li)) * 16)) = f.w[kk][b];
                wave_lds_order();
                const char *xs = st + G::WBYTES + tl * (KC * 2);
#pragma unroll
                for (int pp = 0; pp < NXP; ++pp) {
                    const u32x4_t xv = *(const u32x4_t *)(xs + (((j + 4 * pp) ^ swz(tl)) * 16));
                    double xd[8];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        xd[2 * i] = (double)__uint_as_float(xv[i] << 16);
                        xd[2 * i + 1] = (double)__uint_as_float(xv[i] & 0xffff0000u);
                    }
#pragma unroll
                    for (int s = 0; s < kGateSlots; s += 2) {
                        if (s < ns) {  // two at a time: two independent chains for the fp64 unit
                            const u32x4_t w0 = *(const u32x4_t *)(st + (eoff[s] ^ (64 * pp)));
                            const u32x4_t w1 = *(const u32x4_t *)(st + (eoff[s + 1] ^ (64 * pp)));
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                acc[s] = fma((double)__uint_as_float(w0[i] << 16), xd[2 * i], acc[s]);
                                acc[s + 1] = fma((double)__uint_as_float(w1[i] << 16), xd[2 * i], acc[s + 1]);
                                acc[s] = fma((double)__uint_as_float(w0[i] & 0xffff0000u), xd[2 * i + 1], acc[s]);
                                acc[s + 1] = fma((double)__uint_as_float(w1[i] & 0xffff0000u), xd[2 * i + 1], acc[s + 1]);
                            }
                        }
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // T has been read
                go_on();
            });
            // the lanes' and the wavefronts' parts, in their order
            double *part = (double *)wslots;  // [slot][lane]
#pragma unroll
            for (int s = 0; s < kGateSlots; ++s) part[s * 64 + lane] = acc[s];
            __syncthreads();
            const int t = tid >> llpt, c_end = min(s_ncand[t], base + kGateSlots * gpt);
            for (int c = base + (tid & ((1 << llpt) - 1)); c < c_end; c += 1 << llpt) {
                const int i = (t << lmc) + c, cs = c - base;
                const int at = (cs / gpt) * 64 + (t + TOK * (cs % gpt)) * 4;
                double v = (double)s_bias[cand[i]];
                for (int w = 0; w < 4; ++w) {
                    const double *pw = (const double *)(smem + G::O_SLOTS + w * G::WAVE) + at;
                    v += (pw[0] + pw[1]) + (pw[2] + pw[3]);
                }
                exact[i] = v;
            }
            __syncthreads();
        }
    }
    MOE_TT(a.ctrl, 42);

    // ---- select: the output position of a candidate is the number of candidates that beat it (larger logit, or equal
    // and lower expert id); softmax over the k selected.  16 lanes per token (more where the candidates ask for it), lane j
    // holds candidates j, j + lanes, ...
    {
        constexpr int CPL = kCandidates / kThreads;  // candidates per lane, at most
        const int ll = n_max <= 16 * CPL ? 4 : llpt, lpt = 1 << ll;
        const int tl = tid >> ll, lj = tid & (lpt - 1);
        const bool live = tl < TOK && t0 + tl < a.T;
        const int n = live ? s_ncand[tl] : 0;
        const double *ev = exact + ((live ? tl : 0) << lmc);
        const int *ce = cand + ((live ? tl : 0) << lmc);
        double top = -__builtin_huge_val(), sum = 0.0;
        // (four at a time: their reads of LDS are then in flight together)
        for (int c = 0; c < n_max; c += 4)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (c + u < n) top = fmax(top, ev[c + u]);
        // two rounds over the lane's candidates: ranks (kept in cand's upper bits) and the softmax's sum, then the results
        int rk[CPL];
        double ex[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            rk[q] = 1 << 20;
            ex[q] = 0.0;
            if (lpt * q < n_max) {
                const int ci = min(lj + lpt * q, max(n - 1, 0));
                const double v = ev[ci];
                const int e = ce[ci];
                int rank = 0;
                for (int c = 0; c < n_max; c += 4) {
                    double ov[4];
                    int oe[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) ov[u] = ev[c + u], oe[u] = ce[c + u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) rank += (c + u < n && (ov[u] > v || (ov[u] == v && oe[u] < e))) ? 1 : 0;
                }
                if (lj + lpt * q < n && rank < k) {
                    rk[q] = rank;
                    ex[q] = exp(v - top);
                }
                sum += ex[q];
            }
        }
        sum = row_sum16(sum);
        for (int off = 16; off < lpt; off <<= 1) sum += __shfl_xor(sum, off, 64);
#pragma unroll
        for (int q = 0; q < CPL; ++q)
            if (lpt * q < n_max && rk[q] < k) {
                const int e = ce[lj + lpt * q];
                store_through(&a.idx[(size_t)(t0 + tl) * k + rk[q]], e);
                store_through(&a.w[(size_t)(t0 + tl) * k + rk[q]], (float)(ex[q] / sum));
                if (do_hist) count_choice(a, cnt, t0 + tl, e);
            }
    }
    MOE_TT(a.ctrl, 43);
    return true;
}

}  // namespace moe
