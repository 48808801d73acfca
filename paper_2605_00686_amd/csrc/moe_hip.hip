// C ABI of the MoE hot path for MI355X (gfx950): argument validation, workspace
// layout, kernel selection and launches.  Declarations and contracts live in
// include/moe.h.
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "dispatch.hpp"
#include "expert.hpp"
#include "route.hpp"

namespace moe {

// ------------------------------------------------------------------ kernels
__global__ __launch_bounds__(kThreads) void k_zero(u32 *p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

template <typename ET, int V, int NT>
__global__ __launch_bounds__(NT, 1) void k_route(KArgs a, int do_hist) {
    extern __shared__ __align__(16) char smem[];
    __shared__ int s_slot;
    if constexpr (V > 0 && V != kGateDirect) gate_warm_l2(a, lds_offset(smem + GateCfg<V>::O_EXACT), blockIdx.x, gridDim.x);
    route_task<ET, V, false, NT>(a, kernel_args_address(), blockIdx.x, smem, do_hist != 0, &s_slot, [] { return false; });
}

__global__ __launch_bounds__(kThreads) void k_plan(KArgs a) {
    extern __shared__ __align__(16) char smem[];
    plan_task(a, smem);
}

template <typename ET>
__global__ __launch_bounds__(kThreads) void k_perm(KArgs a) {
    extern __shared__ __align__(16) char smem[];
    if (a.ctrl->error.v == 0) perm_task<ET>(a, blockIdx.x, smem, a.blk_base + (size_t)blockIdx.x * a.E, a.counts);
}

// standalone dispatch, short form (see block_hist_task): histograms go to blk_base, which nothing
// else reads in this form, and nothing that must be zero between calls is touched
__global__ __launch_bounds__(kThreads) void k_block_hist(KArgs a) {
    extern __shared__ __align__(16) char smem[];
    block_hist_task(a, blockIdx.x, a.blk_base, smem);
}
template <typename ET>
__global__ __launch_bounds__(kThreads) void k_block_perm(KArgs a) {
    extern __shared__ __align__(16) char smem[];
    block_perm_task<ET>(a, blockIdx.x, a.blk_base, smem);
}

__global__ __launch_bounds__(kThreads) void k_gather(KArgs a, size_t row_bytes) {
    if (a.ctrl && a.ctrl->error.v != 0) return;  // (no control block: the form without a workspace)
    // perm was not written if an expert is over its capacity (padded layout) or if the histogram does not account
    // for every slot (an expert id outside [0, E)): nothing is gathered then
    __shared__ int s_rows;
    if (threadIdx.x == 0) s_rows = 0;
    __syncthreads();
    int over = 0, mine = 0;
    for (int e = threadIdx.x; e < a.E; e += kThreads) {
        const int c = a.counts[e];
        mine += c;
        over |= (a.capacity > 0 && c > a.capacity) ? 1 : 0;
    }
    if (mine) atomicAdd(&s_rows, mine);
    if (__syncthreads_or(over)) return;
    if (s_rows != a.N) return;
    const int wave = (blockIdx.x * kThreads + threadIdx.x) >> 6;
    gather_rows(a, wave, (gridDim.x * kThreads) >> 6, row_bytes);
}

// Measurement aid (moe_probe_mfma): nothing but independent bf16 matrix-core instructions, one wavefront per SIMD,
// the 256 accumulator registers of the 256 x 256 GEMM tile (16 independent 32x32x16 products per round), operands
// read once from `frag` (128 bytes per lane of a wavefront, whatever the caller put there).  What this reaches is what
// the matrix cores deliver on this chip at the clock it holds under that load, with no LDS or memory traffic at all.
__global__ __launch_bounds__(kThreads, 1) void k_probe_mfma(const uint4 *frag, int iters, float *sink) {
    const int lane = threadIdx.x & 63;
    bf16x8_t fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        fa[i] = __builtin_bit_cast(bf16x8_t, frag[(size_t)(i * 64 + lane)]);
        fb[i] = __builtin_bit_cast(bf16x8_t, frag[(size_t)((4 + i) * 64 + lane)]);
    }
    f32x16_t acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][n][v] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[n], fa[m], acc[m][n], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) s += acc[m][n][v];
    sink[(size_t)blockIdx.x * kThreads + threadIdx.x] = s;
}

// Measurement aid (moe_probe_stream): nothing but loads.  Every workgroup of NT threads reads `bytes_per_wg` bytes
// that start at byte (workgroup * stride) % span of `buf` and wrap inside its first `span` bytes, 1 KB per wavefront
// and instruction (16 bytes per lane, consecutive), kStreamDepth instructions per wavefront issued back to back and
// half of them awaited before the next batch.  LDS form: global_load_lds_dwordx4 into a per-wavefront ring in LDS,
// the way the GEMM main loop loads its stages; register form: global_load_dwordx4, the values folded into one word.
// What this reaches is what a CU can pull in with that many wavefronts, from HBM (span far beyond the caches), from
// the memory-side cache or from L2 (small span, stride 0), whatever else the kernel that is compared with it does.
constexpr int kStreamDepth = 8;
template <int NT, bool TO_LDS>
__global__ __launch_bounds__(NT, 1) void k_probe_stream(const char *buf, size_t span, size_t stride, size_t bytes_per_wg, u32 *sink) {
    extern __shared__ __align__(1024) char stream_lds[];
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t n_instr = bytes_per_wg / ((size_t)NW * 1024);
    u32x4_t acc = u32x4_t{0u, 0u, 0u, 0u};
    // (one modulo here, none per load: a load's step, NW KB, is at most the span)
    size_t off = ((size_t)blockIdx.x * stride + (size_t)wave * 1024 + (size_t)lane * 16) % span;
    auto next = [&]() {
        const char *src = buf + off;
        off += (size_t)NW * 1024;
        off = off >= span ? off - span : off;
        return src;
    };
    if (TO_LDS) {
        const u32 ring = lds_offset(stream_lds) + (u32)wave * (kStreamDepth * 1024);
        for (size_t it = 0; it + kStreamDepth <= n_instr; it += kStreamDepth) {
#pragma unroll
            for (int u = 0; u < kStreamDepth; ++u) {
                const char *src = next();
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                             :
                             : "s"(__builtin_amdgcn_readfirstlane(ring + (u32)u * 1024)), "v"(src)
                             : "m0", "memory");
            }
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kStreamDepth / 2) : "memory");
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        acc = *(const u32x4_t *)(stream_lds + (size_t)tid * 16);
    } else {
        for (size_t it = 0; it + kStreamDepth <= n_instr; it += kStreamDepth) {
            u32x4_t r[kStreamDepth];
#pragma unroll
            for (int u = 0; u < kStreamDepth; ++u) r[u] = *(const u32x4_t *)next();
#pragma unroll
            for (int u = 0; u < kStreamDepth; ++u) acc ^= r[u];
        }
    }
    sink[(size_t)blockIdx.x * NT + tid] = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
}

// standalone dispatch as one launch (see dispatch_fused_task); and the row movement of the histogram form by
// token (ragged layout), which moves nothing unless the histogram accounts for every slot
template <int STORE>
__global__ __launch_bounds__(kThreads) void k_dispatch_fused(KArgs a, size_t row_bytes) {
    dispatch_fused_task<STORE>(a, blockIdx.x, row_bytes);
}
template <int STORE>
__global__ __launch_bounds__(kThreads) void k_scatter(KArgs a, size_t row_bytes) {
    if (a.ctrl && a.ctrl->error.v != 0) return;
    if (a.offsets[a.E] != a.N) return;  // an expert id outside [0, E): perm and inv_perm were not written
    scatter_task<STORE>(a, blockIdx.x, row_bytes);
}

// standalone dispatch leaves the control block clean for the next call
__global__ __launch_bounds__(kThreads) void k_dispatch_finish(KArgs a) {
    // (one workgroup: the status must be read before the control block is cleared)
    if (threadIdx.x == 0 && a.status_dev && a.ctrl->error.v != 0) *a.status_dev = -(int)a.ctrl->error.v;
    __syncthreads();
    u32 *z = (u32 *)a.ctrl;
    const size_t n = a.zero_bytes / 4;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        z[i] = 0u;
}

template <typename ET, bool STREAM, bool SHARE>
__global__ __launch_bounds__(kThreads) void k_combine(KArgs a) {
    combine_task<ET, false, STREAM, SHARE>(a, blockIdx.x);
}

// Front tasks of the megakernel from their counter, in this order: [gate-weight transposition tiles | gate tasks | plan |
// permutation blocks]; then the wait for all of them, and the decode tables in LDS.  Returns nonzero if a wait failed or the
// routing was found invalid; the numbers of row blocks are left in StageLds.  A real call, like the GEMM stages (see
// there), so that the gate's registers are its own.
template <typename ET, int V>
static __device__ __attribute__((noinline)) int front_stage(KArgsAddr args, u32 smem_off, volatile int *caller_local) {
    KArgs a = load_kernel_args(args);
    mark_global(a);
    char *smem = lds_at((u32)uniform((int)smem_off));
    const int tid = threadIdx.x;
    Ctrl *c = a.ctrl;
    StageLds *sl = (StageLds *)(smem + a.sched_lds_off);
    *caller_local = 5;  // (see the call sites of tile_stage)
    if (tid == 0) sl->next = (int)atomicAdd(&c->next_task.v, 1u);
    // (Before the direct gate too, unlike alone: without it, in two builds that differ in where the code lies, 8 tokens x 8 of 128 experts of 2048 x 768
    // level and 1.7 % slower, 128 x 8 of 128 0.9 % slower and 0.2 % faster, 128 x 8 of 32 of 7168 x 2048 0.2 and 0.4 % slower, 1001 x 6 of 48 level and 0.5 % slower.)
    if constexpr (V > 0) {
        gate_warm_l2(a, lds_offset(smem + kMaxExperts * 4), blockIdx.x, gridDim.x);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    int task = uniform(sl->next);
    auto draw_next = [&](int phase) __attribute__((always_inline)) {
        __syncthreads();
        if (tid == 0) {
            if (phase >= 0) mark_phase_end(sl, phase);
            sl->next = (int)atomicAdd(&c->next_task.v, 1u);
        }
        __syncthreads();
        task = uniform(sl->next);
    };
    auto wait_for = [&](const u32 *p, u32 target) __attribute__((always_inline)) {
        __syncthreads();
        if (tid == 0) sl->ok = !wait_ge(c, sl, p, target, a.wait_ticks) ? 0 : ld_relaxed_agent(&c->error.v) == 0 ? 1 : 2;
        __syncthreads();
        return uniform(sl->ok);  // 0: not reached, 1: reached, 2: reached, but an error is recorded
    };
    // (the tasks' results are atomics and written-through stores, which sync_stores() sees into memory: a release fence would write
    // back everything dirty in the XCD's L2, and that stalls the other workgroups' loads.  Only the single-workgroup plan and
    // its permutation blocks store their many tables in the ordinary way.)
    auto release_and_count = [&](u32 *counter, bool fence) __attribute__((always_inline)) {
        sync_stores();
        if (tid == 0) {
            if (fence) fence_release(0);
            atomicAdd(counter, 1u);
        }
    };
    // (the next task is only drawn when this one is done: there are about as many gate tasks
    // as workgroups, and drawing ahead would give the first workgroups two each)
    if constexpr (V > 0) {
        while (task < a.t_gate) {
            wgt_task(a, task, smem);
            release_and_count(&c->wgt_done.v, false);
            draw_next(-1);
        }
    }
    bool seen_wgt = false;
    while (task < a.t_plan) {
        route_task<ET, V, true, kThreads>(a, args, task - a.t_gate, smem, a.plan_from_idx == 0, &sl->pick, [&]() __attribute__((always_inline)) {
            if (!seen_wgt) seen_wgt = wait_for(&c->wgt_done.v, (u32)a.t_gate) != 0;  // the transposed gate weights are complete
            return seen_wgt;
        });
        release_and_count(&c->route_done.v, false);
        draw_next(0);
    }
    int n_rb = 0, n_rbs = 0;
    const int routed = wait_for(&c->route_done.v, (u32)a.nRT);
    bool bad = routed != 1;
    if (a.plan_all) {
        PlanAll p(a, smem);
        // (counts and offsets are reported also when an id was invalid or an expert is over its capacity, unless the error
        // cut the wait short)
        const int planned = routed != 0 ? plan_all_tables(a, p, &n_rb, &n_rbs) : MOE_OK;
        if (task == a.t_plan && routed != 0 && (routed == 2 || planned != MOE_OK)) {
            for (int e = tid; e <= a.E; e += kThreads) {
                a.offsets[e] = a.capacity > 0 ? e * a.capacity : p.off[e];
                if (e < a.E) a.counts[e] = p.cnt[e];
            }
            if (tid == 0 && planned != MOE_OK) set_error(c, planned);
        }
        bad = bad || planned != MOE_OK;
        if (!bad && a.perm_lds_off) plan_all_perm(a, p, smem);
        if (!bad && task < a.t_g1) plan_all_flags(a, p);
        while (task < a.t_g1) {
            const bool plan = task < a.t_perm;
            if (!bad) {
                if (plan)
                    plan_all_publish(a, p, n_rb, n_rbs);
                else
                    perm_block_lds(a, p, task - a.t_perm);
            }
            release_and_count(&c->perm_done.v, false);  // (the plan too: nobody waits for it alone)
            draw_next(plan ? 1 : 2);
        }
    } else {
        if (task == a.t_plan) {
            if (routed != 0) plan_task(a, smem);
            release_and_count(&c->plan_done.v, true);
            draw_next(1);
        }
        bad = wait_for(&c->plan_done.v, 1u) != 1 || bad;
        while (task < a.t_g1) {
            const int b = task - a.t_perm;
            if (!bad) perm_task<ET>(a, b, smem, a.blk_base + (size_t)b * a.E, a.counts);
            release_and_count(&c->perm_done.v, true);
            draw_next(2);
        }
        if (!bad) {
            n_rb = (int)c->n_rb;
            n_rbs = (int)c->n_rbs;
            if (a.tab_lds_off > 0) {  // [offsets | rb_base | rbs_base | counts | rb_expert | rbs_expert]
                int32_t *t_off = (int32_t *)(smem + a.tab_lds_off);
                int32_t *t_rbb = t_off + a.E + 1;
                int32_t *t_rsb = t_rbb + a.E + 1;
                int32_t *t_cnt = t_rsb + a.E + 1;
                int32_t *t_rbe = t_cnt + a.E + 1;
                int32_t *t_rse = t_rbe + n_rb;
                for (int i = tid; i <= a.E; i += kThreads) {
                    t_off[i] = a.offsets[i];
                    t_rbb[i] = a.rb_base[i];
                    t_rsb[i] = a.rbs_base[i];
                    t_cnt[i] = i < a.E ? a.counts[i] : 0;
                }
                for (int i = tid; i < n_rb; i += kThreads) t_rbe[i] = a.rb_expert[i];
                for (int i = tid; i < n_rbs; i += kThreads) t_rse[i] = a.rbs_expert[i];
            }
        }
    }
    // (with a copy of perm in LDS, GEMM1 needs nothing more: the wait comes behind it, see wait_for_perm)
    if (!a.perm_lds_off) bad = wait_for(&c->perm_done.v, (u32)(a.nPB + a.plan_all)) != 1 || bad;
    if (tid == 0) {
        sl->n_rb = n_rb;
        sl->n_rbs = n_rbs;
    }
    __syncthreads();
    return bad ? 1 : 0;
}

// The permutation and the flag ranges are in memory (before the first GEMM2 tile, where the front stage has not waited for them)
__device__ __forceinline__ bool wait_for_perm(const KArgs &a, StageLds *sl) {
    Ctrl *c = a.ctrl;
    __syncthreads();
    if (threadIdx.x == 0)
        sl->ok = wait_ge(c, sl, &c->perm_done.v, (u32)(a.nPB + a.plan_all), a.wait_ticks) && ld_relaxed_agent(&c->error.v) == 0;
    __syncthreads();
    return uniform(sl->ok) != 0;
}

// The statistics from the workgroups' reports: sums, and for the phases the time from the earliest start to the latest end.
__device__ __forceinline__ void sum_reports(const KArgs &a, char *smem, int error) {
    const int tid = threadIdx.x, w = tid & (kWgStats - 1), part = tid / kWgStats;
    constexpr int PARTS = kThreads / kWgStats, U = 32;  // (32 loads in flight per thread: the reports of 256 workgroups at once)
    const int n = (int)gridDim.x;
    const bool phase = w >= 8 && w <= 13, start = w == MOE_NUM_STATS;
    u64 v = start ? ~0ull : 0ull;
    for (int b = part; b < n; b += PARTS * U) {
        u64 r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = a.wg_stats[(size_t)min(b + u * PARTS, n - 1) * kWgStats + w];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b + u * PARTS < n) v = phase ? max(v, r[u]) : start ? min(v, r[u]) : v + r[u];
    }
    u64 *part_v = (u64 *)smem;  // [PARTS][kWgStats]
    part_v[tid] = v;
    __syncthreads();
    if (tid <= MOE_NUM_STATS) {
        for (int i = 1; i < PARTS; ++i) {
            const u64 r = part_v[i * kWgStats + w];
            v = phase ? max(v, r) : start ? min(v, r) : v + r;
        }
        part_v[tid] = v;
    }
    __syncthreads();
    if (tid < MOE_NUM_STATS) {
        const u64 t0 = part_v[MOE_NUM_STATS];
        if (tid == 7) v = (u64)(long long)(-error);
        if (phase) v = v > t0 ? (v - t0) * 10ull : 0ull;  // 100 MHz ticks -> ns
        if (tid == 14) v *= 10ull;
        if (tid == 15) v = (u64)n;
        a.stats[tid] = v;
    }
}

// The whole layer in one persistent kernel.  Every workgroup walks through three
// stages, drawing work from counters in the control block:
//   1. front tasks, one counter, in this order: [gate-weight transposition | gate tasks | plan | permutation blocks];
//   2. GEMM tiles, four kinds in turn (GEMM1 then GEMM2, big then small row blocks), each kind
//      from one list per XCD (see TileQueue): its own XCD's list first, then the others;
//   3. combine tasks, dealt out by workgroup number.
// No wait can deadlock, whatever the grid size: a task only waits for tasks of an
// earlier kind (permutation <- plan <- gate <- transposition, GEMM1 <- permutation, GEMM2 <- GEMM1,
// combine <- GEMM2), a workgroup only moves on to a later kind when every entry of the
// kinds before has been drawn, and whoever drew an entry is running it.  So the not yet finished entry of the earliest kind is always either
// running with everything it needs, or about to be drawn by a workgroup that is not
// waiting.  A workgroup draws its next entry while it works on the current one, which
// hides the counter's latency (tiles; front tasks are drawn one by one).  The kernel body itself only strings the stage
// functions together (see StageLds) and never hands out a reference to its argument
// block.
// P: tile policy (of the big tile when row blocks have two heights), PS: policy of the small tile
// (= P when there is one height).
template <class P, class PS>
__global__ __launch_bounds__(kThreads, P::MIN_WAVES) void k_megakernel(KArgs a) {
    using ET = typename P::ET;
    constexpr bool MIXED = !std::is_same<P, PS>::value;
    static_assert(P::MIN_WAVES == PS::MIN_WAVES, "one occupancy for both tile codes");
    extern __shared__ __align__(16) char smem[];
    __shared__ int s_last;
    Ctrl *c = a.ctrl;
    const int tid = threadIdx.x;
    const KArgsAddr kargs = kernel_args_address();
    StageLds *sl = (StageLds *)(smem + a.sched_lds_off);
    if (tid < MOE_NUM_STATS) sl->stat[tid] = 0ull;
    if (tid == 0) sl->t_start = now_ticks();
    __syncthreads();

    // The stage functions get the address of a local of this kernel.  That keeps the compiler from
    // marking the calls as tail calls, which is what lets it drop the saving and restoring of
    // callee-saved registers in these functions (they have one caller, which keeps nothing in them):
    // some 270 registers per lane through scratch memory, per call, otherwise.
    volatile int stage_mark = 0;
    const u32 lds = lds_offset_opaque(smem);

    // ---- stage 1: gate, plan, permutation
    int front = 0;
    if constexpr (sizeof(ET) == 2) {  // (one function per gate: each has registers of its own)
        switch (a.gate_direct ? kGateDirect : a.Wg ? gate_variant(a.E, a.d) : 0) {
            case kGateDirect: front = front_stage<ET, kGateDirect>(kargs, lds, &stage_mark); break;
            case 1: front = front_stage<ET, 1>(kargs, lds, &stage_mark); break;
            case 2: front = front_stage<ET, 2>(kargs, lds, &stage_mark); break;
            case 3: front = front_stage<ET, 3>(kargs, lds, &stage_mark); break;
            case 4: front = front_stage<ET, 4>(kargs, lds, &stage_mark); break;
            case 5: front = front_stage<ET, 5>(kargs, lds, &stage_mark); break;
            case 6: front = front_stage<ET, 6>(kargs, lds, &stage_mark); break;
            default: front = front_stage<ET, 0>(kargs, lds, &stage_mark); break;
        }
    } else {
        front = front_stage<ET, 0>(kargs, lds, &stage_mark);
    }
    const bool bad = uniform(front) != 0;
    const int n_rb = uniform(sl->n_rb), n_rbs = uniform(sl->n_rbs);

    if (!bad) {
        // ---- stage 2: GEMM tiles, one call per kind, this XCD's lists first
        const int home = xcd_id() % kTileQueues;
        if constexpr (P::FUSED) {
            // ---- stage 2, fused: row blocks through both GEMMs, then combine
            fused_stage<P>(kargs, lds, home, n_rb, &stage_mark);
            combine_stage<ET>(a, smem);
        } else if (a.scheduler == MOE_SCHED_READY_QUEUE) {
            // ---- stages 2 and 3 from the ready queues
            ready_queue_stage<P, PS, MIXED>(a, kargs, smem, home, n_rb, n_rbs, &stage_mark);
        } else {
            MOE_TT_BEGIN();
            if (!MIXED || n_rb > 0) tile_stage<P, true, false>(kargs, lds, home, n_rb, n_rbs, -1, -1, -1, &stage_mark);
            MOE_TT(c, 20);
            if (MIXED && n_rbs > 0) tile_stage<PS, true, true>(kargs, lds, home, n_rb, n_rbs, -1, -1, -1, &stage_mark);
            MOE_TT(c, 21);
            const bool permuted = !a.perm_lds_off || wait_for_perm(a, sl);
            if (permuted && (!MIXED || n_rb > 0)) tile_stage<P, false, false>(kargs, lds, home, n_rb, n_rbs, -1, -1, -1, &stage_mark);
            MOE_TT(c, 22);
            if (permuted && MIXED && n_rbs > 0) tile_stage<PS, false, true>(kargs, lds, home, n_rb, n_rbs, -1, -1, -1, &stage_mark);
            MOE_TT(c, 23);
            // ---- stage 3: combine
            if (permuted) combine_stage<ET>(a, smem);
        }
    }
    // Last workgroup out sums up the workgroups' reports and clears the control block.  (What it reads of the others' work are
    // atomics and the reports, which are written through.)
    __syncthreads();
    if (tid <= MOE_NUM_STATS) store_through(&a.wg_stats[(size_t)blockIdx.x * kWgStats + tid], tid < MOE_NUM_STATS ? sl->stat[tid] : sl->t_start);
    sync_stores();
    if (tid == 0) {
        const u32 g = blockIdx.x % kExitGroups, in_group = (gridDim.x - g + kExitGroups - 1) / kExitGroups;
        const u32 groups = min(gridDim.x, (u32)kExitGroups);
        s_last = 0;
        if (atomicAdd(&c->exit_group[g].v, 1u) == in_group - 1) s_last = atomicAdd(&c->exit_count.v, 1u) == groups - 1 ? 1 : 0;
        if (s_last) fence_acquire(0);
    }
    __syncthreads();
    if (s_last) {
        if (a.stats) sum_reports(a, smem, (int)c->error.v);
        __syncthreads();
#ifdef MOE_TILE_TIMING
        // development build: the per-part tick sums follow the statistics (the caller's array has room for them)
        if (a.stats && tid < 48) a.stats[MOE_NUM_STATS + tid] = c->dbg[tid];
        __syncthreads();
#endif
        u32 *z = (u32 *)c;
        for (size_t i = tid; i < a.zero_bytes / 4; i += kThreads) z[i] = 0u;
    }
}

// --------------------------------------------------------------- host side
// The standalone dispatch runs as one launch while (slots) x (workgroups of 16 tokens) is at most this: every
// workgroup counts every slot, which hides behind the row movement up to about this much.
constexpr long long kFusedDispatchWork = 64ll << 20;
constexpr size_t kLdsBudget = 160 * 1024 - 256;  // dynamic LDS a kernel may ask for: the CU's 160 KB less the kernels' few static words
constexpr int kCombineTasks = 256;  // of the megakernel, one per CU of the chip ...
constexpr int kCombineMaxTokens = 256;  // ... with at most so many tokens (their weights are kept in LDS)
constexpr int kGroupStride = 32;  // words: see KArgs::group_stride
constexpr int kMaxDevices = 16;  // devices the host-side launch memo covers (others ask the runtime on every call)

static inline size_t align_up(size_t v, size_t al) { return (v + al - 1) / al * al; }

static int elem_size(int dtype) { return dtype == MOE_DT_F32 ? 4 : 2; }

// The gate is split over its reduction when there are at most kGateSplitBlocks blocks of 16 tokens,
// into at most kGateSplitTasks tasks in all.
constexpr int kGateSplitBlocks = 64, kGateSplitTasks = 256, kGateSplitMax = 16;
constexpr int kGateParts = 128;  // blocks whose finished parts are counted, of either split
static_assert(kGateParts >= kGateSplitBlocks && kGateParts >= kDirectSplitTokens, "one counter per block");

// LM: 256-row tiles plus a 128-row tile for short tails; S: 32-row tiles; S2: 64-row tiles, and 32-row ones for experts of no
// more rows than that; FS / FM: row blocks of the fused FFN (32 / 64 rows)
enum TileKind { TK_F32 = 0, TK_LM = 1, TK_S2 = 2, TK_S = 3, TK_FS = 4, TK_FM = 5 };

// Parts of an fp32 GEMM2 tile (see g2_join) where `tiles` tiles are likely: as many as there are CUs for (256), and no more than pay for
// what a part costs, which is to be drawn, counted and added up.  A tile's length is its reduction times the 32-row blocks an expert
// is likely to have, half of one more than its average fills; the fewer tiles there are, the shorter a part may be.  At most 32, 64
// and more tiles, us, whole / this many parts / one more step: 128 tokens x 2 of 4 experts of 512 x 512 77.4 / 73.3 / 74.2, 4 x 2
// of 4 of 512 x 768 58.3 / 57.4 / 57.7, of 512 x 512 53.1 / - / 54.8; 256 x 2 of 8 of 512 x 512 82.4 / 81.6 / 83.5, 16 x 2 of 8 of
// 512 x 1024 66.9 / 66.1 / 66.2, of 512 x 768 63.5 / - / 64.7; 128 x 1 of 8 of 768 x 2048 92.7 / 86.0 / 94.5, of 768 x 768 72.1 / - / 72.9, 1 x 2 of 2
// of 4096 x 1024 99.6 / - / 101.4.  Parts of 128 indices wherever CUs were left took 16 x 2 of 8 of 512 x 512 from 58.5 to 63.8.
// (By the problem's shape alone: the sums, and so the results, are the same under both schedulers.)
static int g2_parts_of_tile(const moe_problem_t *p, int avg, long long tiles) {
    constexpr int kMinPart = 128;  // reduction indices
    const int rows = (avg < TileF32::BM ? avg : TileF32::BM) + 16;
    const long long length = (long long)p->f * (rows > 32 ? rows : 32) / 32;
    const int shortest = tiles <= 32 ? 256 : tiles <= 64 ? 512 : 768;
    if (length < 3 * 256) return 1;
    long long S = 256 / tiles;
    if (S > kG2MaxParts) S = kG2MaxParts;
    if (S > p->f / kMinPart) S = p->f / kMinPart;
    if (S > length / shortest) S = length / shortest;
    return S > 1 ? (int)S : 1;
}

struct Plan {
    moe_problem_t p;
    int tile_m, tile_n, N, NP, per_dest, ncb, nPB, nRT, nCT, comb_tokens, comb_span, comb_per_span, maxRB_layout;
    int kind;
    Tiling tl;
    // workspace byte offsets
    size_t o_ctrl, o_blk_hist, o_seg_cnt, o_group_counter, o_h_ready, o_dest_done, o_gate_parts, zero_bytes;
    size_t o_gate_partial;
    size_t o_rq_slots, init_zero_bytes;  // the ready queues empty themselves: zeroed by moe_workspace_init only
    int rq_cap;
    size_t o_blk_base, o_seg_begin, o_flag_base, o_dest_flag_begin, o_dest_group_begin, o_rb_base, o_rb_expert, o_rbs_base, o_rbs_expert, o_h, total;
    size_t o_wgt, o_wg_stats;
    int gate_tok;  // tokens per gate task
    int g2_split, g2_rows;  // see g2_join
    size_t o_g2_partial, o_g2_parts;
};

static int make_plan(const moe_problem_t *p, Plan *pl) {
    if (!p) return MOE_ERR_INVALID_ARG;
    if (p->T < 1 || p->d < 1 || p->E < 1 || p->k < 1 || p->f < 1 || p->R < 1) return MOE_ERR_INVALID_ARG;
    if (p->k > p->E || p->T % p->R != 0) return MOE_ERR_INVALID_ARG;
    if (p->dtype != MOE_DT_F32 && p->dtype != MOE_DT_BF16) return MOE_ERR_INVALID_ARG;
    if (p->signal_mode != MOE_SIGNAL_PER_TILE && p->signal_mode != MOE_SIGNAL_PER_DEST) return MOE_ERR_INVALID_ARG;
    if (p->fence_scope != MOE_SCOPE_AGENT && p->fence_scope != MOE_SCOPE_SYSTEM) return MOE_ERR_INVALID_ARG;
    if (p->tile_m < 0 || p->tile_n < 0) return MOE_ERR_INVALID_ARG;
    if (p->group_size < 0 || (p->group_size != 0 && p->signal_mode != MOE_SIGNAL_PER_DEST)) return MOE_ERR_INVALID_ARG;
    if (p->scheduler != MOE_SCHED_STATIC && p->scheduler != MOE_SCHED_READY_QUEUE) return MOE_ERR_INVALID_ARG;
    if (p->capacity < 0) return MOE_ERR_INVALID_ARG;
    if (p->fuse_ffn != 0 && p->fuse_ffn != 1) return MOE_ERR_INVALID_ARG;
    if (p->fuse_ffn && p->scheduler != MOE_SCHED_STATIC) return MOE_ERR_INVALID_ARG;
    if ((long long)p->E * p->capacity > (1ll << 30)) return MOE_ERR_UNSUPPORTED;
    if (p->E > kMaxExperts || p->k > 32 || p->R > kMaxDest) return MOE_ERR_UNSUPPORTED;
    if ((long long)p->T * p->k > (1ll << 30)) return MOE_ERR_UNSUPPORTED;
    const int tm = p->tile_m ? p->tile_m : 128, tn = p->tile_n ? p->tile_n : 64;
    if (tm != 32 && tm != 64 && tm != 128) return MOE_ERR_UNSUPPORTED;
    if (tn != 64 && tn != 128) return MOE_ERR_UNSUPPORTED;
    // 16-byte pieces everywhere; the MFMA main loop steps K by 64, the fp32 one by 16
    const int kstep = (p->dtype == MOE_DT_BF16) ? 64 : 16;
    if (p->d % kstep != 0 || p->f % kstep != 0) return MOE_ERR_UNSUPPORTED;
    pl->p = *p;
    pl->tile_m = tm;
    pl->tile_n = tn;
    pl->N = p->T * p->k;
    pl->NP = p->capacity > 0 ? p->E * p->capacity : pl->N;  // rows of the sorted order (h, x_perm, perm)
    pl->per_dest = p->T / p->R;
    pl->ncb = (p->d + tn - 1) / tn;
    pl->nPB = (p->T + kPermBlock - 1) / kPermBlock;
    pl->gate_tok = p->dtype == MOE_DT_BF16 ? gate_tokens(p->T) : kRouteTokens;
    pl->nRT = (p->T + pl->gate_tok - 1) / pl->gate_tok;
    // Combine tasks of the megakernel: one per workgroup.  A task is a chain of trips to memory (flag numbers, flags, weights, rows),
    // and all become ready together with the last tiles.  (The standalone combine has a rule of its own: standalone_combine_tokens.)
    pl->comb_tokens = (p->T + kCombineTasks - 1) / kCombineTasks;
    if (pl->comb_tokens > kCombineMaxTokens) pl->comb_tokens = kCombineMaxTokens;
    // The ready-queue scheduler enqueues combine tasks per destination: none may span two.
    pl->comb_span = p->scheduler == MOE_SCHED_READY_QUEUE ? pl->per_dest : p->T;
    pl->comb_per_span = (pl->comb_span + pl->comb_tokens - 1) / pl->comb_tokens;
    if (p->scheduler == MOE_SCHED_READY_QUEUE) {  // equal shares of a destination where up to twice as many tasks make them equal
        const int want = pl->comb_per_span;
        for (int n = want; n <= 2 * want && n <= pl->per_dest; ++n)
            if (pl->per_dest % n == 0) {
                pl->comb_per_span = n;
                pl->comb_tokens = pl->per_dest / n;
                break;
            }
    }
    pl->nCT = p->T / pl->comb_span * pl->comb_per_span;
    // tile shape: the smallest row block that holds an average expert, never
    // smaller than the publish tile (a publish tile must not span two compute tiles)
    const int avg = pl->N / p->E;
    int bm;
    if (p->dtype == MOE_DT_F32) {
        pl->kind = TK_F32;
        bm = TileF32::BM;
        // GEMM1 takes 32-column tiles when 64-column ones would not give every CU of the chip a tile
        const long long blocks = (long long)(pl->N < p->E ? pl->N : p->E) * (avg / bm + 1);
        pl->tl.BN1 = blocks * ((p->f + TileF32::BN - 1) / TileF32::BN) < 256 ? TileF32::BN_NARROW : TileF32::BN;
        pl->tl.BN2 = TileF32::BN;
    } else if (p->fuse_ffn) {
        // the fused FFN: row blocks of 32 rows for decode-sized experts, else 64; the block's h must fit the LDS
        // beside the stage buffers (checked at launch: MOE_ERR_UNSUPPORTED if it does not)
        pl->kind = (avg < 96 && tm == 32) ? TK_FS : TK_FM;
        bm = pl->kind == TK_FS ? CfgFS::BM : CfgFM::BM;
        pl->tl.BN1 = 128;
        pl->tl.BN2 = 256;
    } else {
        // Experts of 32 rows and more on average: an expert of 33 to 64 rows in two 32-row blocks has its weights streamed, and its tiles
        // run, twice; below that most have one block and the second tile code costs more than it saves.  32 / 64 rows, us:
        // 128 tokens x 8 of 32 experts of 7168 x 2048 603 / 578, 2313 x 1 of 32 of 704 x 14272 897 / 691, 240 x 1 of 7 of 2304 x 11392 345 / 310;
        // 76 x 8 of 22 (28 rows) of 3328 x 1152 167 / 174, 128 x 8 of 128 (8 rows) of 2048 x 768 249 / 255.
        pl->kind = (avg >= 96 || tm > 32) ? TK_LM : avg >= 32 ? TK_S2 : TK_S;
        bm = pl->kind == TK_LM ? CfgL::BM : pl->kind == TK_S2 ? CfgS2::BM : CfgS::BM;
        pl->tl.BN1 = 128;
        pl->tl.BN2 = 256;
    }
    if (p->fuse_ffn && p->dtype != MOE_DT_BF16) return MOE_ERR_UNSUPPORTED;
    // fp32 layers of few GEMM2 tiles cut them along the reduction (kG2SplitTiles bounds the tiles there can be)
    pl->g2_split = 1;
    pl->g2_rows = pl->N < TileF32::BM ? pl->N : TileF32::BM;
    long long g2_tiles = 0;  // at most
    if (p->dtype == MOE_DT_F32) {
        const long long nt2 = (p->d + TileF32::BN - 1) / TileF32::BN, experts = pl->N < p->E ? pl->N : p->E;
        g2_tiles = (pl->N / bm + experts) * nt2;
        if (g2_tiles <= kG2SplitTiles) pl->g2_split = g2_parts_of_tile(p, avg, experts * (avg / bm + 1) * nt2);
    }
    if (pl->g2_split == 1) g2_tiles = 0;
    pl->tl.BMS = pl->kind == TK_LM ? CfgM::BM : pl->kind == TK_S2 ? CfgS::BM : 0;
    // few rows per expert: the layer streams weights (measured: about -1 % on cfg2; +2 to 4 % on cfg3 and cfg4,
    // which have thousands of rows per expert and are bound by the matrix cores, if it were applied there)
    pl->tl.tail_with_big = avg < 512 ? 1 : 0;
    // a publish tile must lie inside one compute tile, in both directions (the fp32 tile is 64 columns wide)
    if (pl->tl.BN2 % tn != 0) return MOE_ERR_UNSUPPORTED;
    if (pl->tl.BMS % tm != 0) return MOE_ERR_UNSUPPORTED;
    if (bm % tm != 0) return MOE_ERR_UNSUPPORTED;
    pl->tl.BM = bm;
    pl->tl.NT1 = (p->f + pl->tl.BN1 - 1) / pl->tl.BN1;
    pl->tl.NT2 = (p->d + pl->tl.BN2 - 1) / pl->tl.BN2;
    pl->tl.maxRB = pl->N / bm + p->E;
    pl->maxRB_layout = pl->N / 32 + 2 * p->E;  // big plus small row blocks; the layout does not depend on the tile choice
    if ((long long)(pl->tl.maxRB + p->E) * (pl->tl.NT1 + pl->tl.NT2) > (1ll << 30)) return MOE_ERR_UNSUPPORTED;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    pl->o_ctrl = take(sizeof(Ctrl));
    pl->o_blk_hist = take((size_t)pl->nPB * p->E * 4);
    pl->o_seg_cnt = take((size_t)p->E * p->R * 4);
    pl->o_h_ready = take((size_t)pl->maxRB_layout * 4);
    pl->o_dest_done = take((size_t)p->R * 4);
    pl->o_gate_parts = take((size_t)kGateParts * 4);
    pl->o_g2_parts = take((size_t)g2_tiles * sizeof(Counter));
    pl->zero_bytes = o;
    // What follows is zero between calls because its users leave it so (moe_workspace_init zeroes it
    // once).  Sizes are the largest any signal mode, group size or scheduler needs, so that the
    // layout depends on the shape of the problem only and these may change from call to call.
    // Fence groups: one counter per group, at most one group per flag (group_size 1) plus R.
    const size_t max_flags = ((size_t)(pl->N + tm - 1) / tm + (size_t)p->E * p->R) * pl->ncb;
    const size_t spread = (size_t)p->R * kGroupStride;  // (a counter per destination has a cache line to itself)
    pl->o_group_counter = take((max_flags + p->R > spread ? max_flags + p->R : spread) * 4);
    // One ready queue per XCD, each able to hold every GEMM2 tile (or part of one) and every combine task (at most
    // one per token).
    pl->rq_cap = (pl->tl.maxRB + p->E) * pl->tl.NT2 * pl->g2_split + p->T;
    pl->o_rq_slots = take((size_t)kTileQueues * pl->rq_cap * 4);
    pl->init_zero_bytes = o;
    pl->o_blk_base = take((size_t)pl->nPB * p->E * 4);
    pl->o_seg_begin = take((size_t)p->E * p->R * 4);
    pl->o_flag_base = take((size_t)p->E * p->R * 4);
    pl->o_dest_flag_begin = take((size_t)(p->R + 1) * 4);
    pl->o_dest_group_begin = take((size_t)(p->R + 1) * 4);
    pl->o_wg_stats = take((size_t)kMaxWorkgroups * kWgStats * 8);
    pl->o_rb_base = take((size_t)(p->E + 1) * 4);
    pl->o_rb_expert = take((size_t)pl->maxRB_layout * 4);
    pl->o_rbs_base = take((size_t)(p->E + 1) * 4);
    pl->o_rbs_expert = take((size_t)p->E * 4);
    pl->o_h = take((size_t)pl->NP * p->f * elem_size(p->dtype));
    // partial logits of a gate split over its reduction (fp32 problems of few tokens): at most kGateSplitTasks tasks
    // (and the logits of one split by experts: bf16 problems of few tokens)
    pl->o_gate_partial = take(p->dtype == MOE_DT_F32 ? (size_t)kGateSplitTasks * kRouteTokens * p->E * 8
                                                     : (size_t)(p->T < kDirectSplitTokens ? p->T : kDirectSplitTokens) * p->E * 8);
    pl->o_g2_partial = take((size_t)g2_tiles * pl->g2_split * pl->g2_rows * TileF32::BN * 4);
    // transposed gate weights (bf16 problems; unused when the routing is an input)
    pl->o_wgt = take(p->dtype == MOE_DT_BF16 ? (size_t)p->E * p->d * 2 : 0);
    pl->total = o;
    return MOE_OK;
}

static void fill_args(const Plan &pl, void *workspace, KArgs *a) {
    const moe_problem_t &p = pl.p;
    memset(a, 0, sizeof(*a));
    a->T = p.T; a->d = p.d; a->E = p.E; a->k = p.k; a->f = p.f; a->R = p.R;
    a->dtype = p.dtype; a->tile_m = pl.tile_m; a->tile_n = pl.tile_n;
    a->signal_mode = p.signal_mode; a->fence_scope = p.fence_scope; a->epoch = p.epoch;
    a->group_size = p.group_size;
    a->group_stride = p.group_size > 0 ? 1 : kGroupStride;
    a->wait_ticks = p.wait_ticks ? (u64)p.wait_ticks : kWaitTicks;
    a->scheduler = p.scheduler;
    a->N = pl.N; a->NP = pl.NP; a->capacity = p.capacity; a->per_dest = pl.per_dest; a->ncb = pl.ncb;
    a->nPB = pl.nPB; a->nRT = pl.nRT; a->nCT = pl.nCT; a->comb_tokens = pl.comb_tokens;
    a->comb_span = pl.comb_span; a->comb_per_span = pl.comb_per_span;
    a->seg_from_blocks = (pl.per_dest % kPermBlock == 0) ? 1 : 0;
    a->disp_tokens = scatter_tokens(p.T);
    a->tl = pl.tl;
    a->g2_split = 1;  // (the megakernel splits: see there)
    a->gate_tok = pl.gate_tok;
    a->t_gate = 0;  // the megakernel adds the transposition tasks when it has a bf16 gate to compute
    a->t_plan = pl.nRT;
    a->t_perm = a->t_plan + 1;
    a->t_g1 = a->t_perm + pl.nPB;
    a->t_end = a->t_g1 + (pl.tl.maxRB + p.E) * (pl.tl.NT1 + pl.tl.NT2) + pl.nCT;
    char *ws = (char *)workspace;
    if (ws) {
        a->ctrl = (Ctrl *)(ws + pl.o_ctrl);
        a->blk_hist = (int32_t *)(ws + pl.o_blk_hist);
        a->seg_cnt = (int32_t *)(ws + pl.o_seg_cnt);
        a->group_counter = (u32 *)(ws + pl.o_group_counter);
        a->h_ready = (u32 *)(ws + pl.o_h_ready);
        a->wg_stats = (u64 *)(ws + pl.o_wg_stats);
        if (p.scheduler == MOE_SCHED_READY_QUEUE) {
            a->dest_done = (u32 *)(ws + pl.o_dest_done);
            a->rq_slots = (u32 *)(ws + pl.o_rq_slots);
            a->rq_cap = pl.rq_cap;
        }
        a->blk_base = (int32_t *)(ws + pl.o_blk_base);
        a->seg_begin = (int32_t *)(ws + pl.o_seg_begin);
        a->flag_base = (int32_t *)(ws + pl.o_flag_base);
        a->dest_flag_begin = (int32_t *)(ws + pl.o_dest_flag_begin);
        a->dest_group_begin = (int32_t *)(ws + pl.o_dest_group_begin);
        a->rb_base = (int32_t *)(ws + pl.o_rb_base);
        a->rb_expert = (int32_t *)(ws + pl.o_rb_expert);
        a->rbs_base = (int32_t *)(ws + pl.o_rbs_base);
        a->rbs_expert = (int32_t *)(ws + pl.o_rbs_expert);
        a->h = ws + pl.o_h;
        a->zero_bytes = pl.zero_bytes;
    }
}

// Tokens per task of the standalone combine.  A CU holds three of its workgroups: up to 768 tasks run at once, and as long as
// that many are enough, fewer tokens per task, whose rows more wavefronts share, are faster; from there on a wavefront per
// token.  A row must have enough 16-byte pieces for the lanes that share it.  Rows not in the L2, 1 / 2 / 4 tokens per task, us:
// 513 tokens x 8 rows of 2048 5.4 / 5.9 / 8.2; 768 6.6 / 7.2 / 8.6; 900 8.5 / 7.7 / 9.2; 1536 11.7 / 10.6 / 12.8; 1800 14.2 / 13.8 /
// 14.0; 2048 15.2 / 14.6 / 13.8; 1024 x 2 of 4096 7.0 / 6.2 / 6.7; 1024 x 6 of 1024 6.3 / 4.8 / 5.3; 513 x 4 of 512 3.2 / 3.0 / 2.9.
static int standalone_combine_tokens(int T, size_t row_bytes) {
    const size_t pieces = row_bytes / 16;
    return T >= 16384 ? 16 : T >= 8192 ? 8 : T > 1536 || pieces < 128 ? 4 : T > 768 || pieces < 256 ? 2 : 1;
}

// What the gate's screen may assume of x and Wg, decided here because a task would wait for it.  Direct global->LDS loads of
// 16 bytes are only issued from 16-byte aligned addresses.  Unaligned rows of Wg (E is no multiple of 8, or a view that starts
// between 16-byte boundaries, which is legal: elements are 2 bytes) go through registers; an unaligned x (standalone only: the
// experts' products ask for aligned rows) takes exact logits of all experts, whose ordinary loads accept any address.  So do
// gate weights of 4 GB and more and rows of x longer than 2^26: the screen addresses the weights (and a piece past their end)
// with 32 bits, the 16 rows of a task with 31.
static void set_gate(KArgs *a, const void *x, const void *Wg, const float *bias, bool alone) {
    a->x = x; a->Wg = Wg; a->bias = bias;
    a->gate_screens = ((uintptr_t)x & 15) == 0 && a->d <= 1 << 26 && (long long)a->d * a->E * 2 <= 0xffffff00ll;
    a->gate_rows_aligned = (a->E & 7) == 0 && ((uintptr_t)Wg & 15) == 0;
    // few tokens: see gate_direct.hpp; its tasks have other sizes than the screen's
    if (Wg && a->dtype == MOE_DT_BF16 && gate_is_direct(a->T, a->E, a->d, alone)) {
        a->gate_direct = direct_threads(a->E, 1, alone ? direct_threads_alone(a->E, a->d) : kThreads);
        a->gate_tok = direct_tokens(a->T);
        a->nRT = (a->T + a->gate_tok - 1) / a->gate_tok;
    }
}

static size_t plan_smem(const Plan &pl) { return plan_smem_bytes(pl.p.E, pl.p.R, pl.nPB); }

static int check_ws(const void *ws) {
    if (!ws || ((uintptr_t)ws & 255u)) return MOE_ERR_WORKSPACE;
    return MOE_OK;
}

static int hip_ok(hipError_t e) { return e == hipSuccess ? MOE_OK : MOE_ERR_HIP; }

// Allow `kernel` `bytes` of dynamic LDS on the current device.  The limit of a kernel is only ever raised, and
// what it was raised to is remembered per (device, kernel), so that a call which needs no more than an earlier
// one asks the runtime nothing (a host-side memo: no device state, nothing a call can observe).
static int set_smem_raw(const void *kernel, size_t bytes) {
    if (bytes > 160 * 1024) return MOE_ERR_UNSUPPORTED;
    if (bytes <= 48 * 1024) return MOE_OK;
    struct Entry {
        int dev;
        const void *kernel;
        size_t limit;
    };
    static std::mutex lock;
    static Entry table[64];
    static int n = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MOE_ERR_HIP;
    std::lock_guard<std::mutex> g(lock);
    Entry *hit = nullptr;
    for (int i = 0; i < n; ++i)
        if (table[i].dev == dev && table[i].kernel == kernel) hit = &table[i];
    if (hit && hit->limit >= bytes) return MOE_OK;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return MOE_ERR_HIP;
    if (hit)
        hit->limit = bytes;
    else if (n < 64)
        table[n++] = Entry{dev, kernel, bytes};
    return MOE_OK;
}
template <class K>
static int set_smem(K kernel, size_t bytes) {
    return set_smem_raw((const void *)kernel, bytes);
}

template <class P, class PS>
static int launch_mega(const Plan &pl, const KArgs &a_in, hipStream_t st) {
    size_t smem = tile_smem_bytes<P>();
    if (tile_smem_bytes<PS>() > smem) smem = tile_smem_bytes<PS>();
    KArgs a = a_in;
    if (P::FUSED) {  // the row block's h, behind the GEMM region and the publish bookkeeping (the gate's LDS is free by then)
        a.fused = 1;
        a.fused_h_off = (int)align_up(smem, 16);
        smem = a.fused_h_off + (size_t)P::BM * pl.p.f * elem_size(pl.p.dtype);
        if (smem + sizeof(StageLds) + 16 > kLdsBudget) return MOE_ERR_UNSUPPORTED;
    }
    const size_t rsm = gate_task_smem_bytes(pl.p.E, pl.p.d, elem_size(pl.p.dtype));
    if (a_in.Wg && rsm > smem) smem = rsm;
    if (plan_smem(pl) > smem) smem = plan_smem(pl);
    // The decode tables live behind everything else, for the life of the workgroup, where they are small (6 KB: up to 255
    // experts and not very many row blocks); only with them there every workgroup can derive the plan by itself.
    const size_t tab_bytes = (size_t)(4 * (pl.p.E + 1) + pl.tl.maxRB + pl.p.E) * 4;
    auto tables_fit = [&](size_t before) { return tab_bytes <= 6 * 1024 && before + tab_bytes + sizeof(StageLds) + 16 <= kLdsBudget; };
    size_t with_plan = plan_all_smem_bytes(pl.p.E, pl.p.R, pl.nPB);
    // the whole permutation's masks and bases, in the place of one block's, where they fit the GEMM region
    const size_t perm_scratch = perm_all_bytes(pl.p.E, pl.nPB);
    const bool perm_fits = perm_scratch <= kPermScratch && with_plan + perm_scratch <= smem;
    if (with_plan < smem) with_plan = smem;
    a.plan_all = plan_all_fits(pl.p.E, pl.p.R, pl.nPB) && tables_fit(with_plan) ? 1 : 0;
    if (a.plan_all) smem = with_plan;
    if (a.plan_all && pl.N <= kPlanSlots) {
        a.plan_from_idx = 1;
        if (!a.Wg) {  // nothing is left for gate tasks to do
            a.t_plan -= a.nRT, a.t_perm -= a.nRT, a.t_g1 -= a.nRT, a.t_end -= a.nRT;
            a.nRT = 0;
        }
    }
    a.tab_lds_off = 0;
    if (tables_fit(smem)) {
        a.tab_lds_off = (int)align_up(smem, 16);
        smem = a.tab_lds_off + tab_bytes;
    }
    // perm in LDS too (kPermSlots): the static order without padding, whose GEMM1 stage is the only early reader of perm
    if (a.plan_from_idx && perm_fits && !P::FUSED && a.scheduler == MOE_SCHED_STATIC && a.capacity == 0 && pl.N <= kPermSlots &&
        align_up(smem, 16) + (size_t)pl.N * 2 + sizeof(StageLds) + 32 <= kLdsBudget) {
        a.perm_lds_off = (int)align_up(smem, 16);
        smem = a.perm_lds_off + (size_t)pl.N * 2;
    }
    a.sched_lds_off = (int)align_up(smem, 16);
    smem = a.sched_lds_off + sizeof(StageLds);
    auto kern = k_megakernel<P, PS>;
    int rc = set_smem(kern, smem);
    if (rc) return rc;
    // The CU count and the occupancy of this kernel are asked for once per device and LDS size (a host-side memo
    // of what the runtime answered, like the one in set_smem_raw).  A program whose batches need more than four sizes asks again on
    // some calls, which its host hardly sees: 10.4 us per call with one size, 10.7 with 16 of them in turn.
    struct Memo {
        size_t smem;
        int cus, per_cu;
    };
    static std::mutex memo_lock;
    static Memo memo[kMaxDevices][4];
    static int memo_n[kMaxDevices];
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MOE_ERR_HIP;
    const bool memoised = dev >= 0 && dev < kMaxDevices;
    bool found = false;
    if (memoised) {
        std::lock_guard<std::mutex> g(memo_lock);
        for (int i = 0; i < memo_n[dev]; ++i)
            if (memo[dev][i].smem == smem) cus = memo[dev][i].cus, per_cu = memo[dev][i].per_cu, found = true;
    }
    if (!found) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return MOE_ERR_HIP;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kThreads, smem) != hipSuccess) return MOE_ERR_HIP;
        std::lock_guard<std::mutex> g(memo_lock);
        if (memoised && memo_n[dev] < 4) memo[dev][memo_n[dev]++] = Memo{smem, cus, per_cu};
    }
    if (per_cu < 1) return MOE_ERR_UNSUPPORTED;
    if (per_cu > 2) per_cu = 2;
    long long grid = (long long)cus * per_cu;
    if (grid > a.t_end) grid = a.t_end;
    if (grid > kMaxWorkgroups) grid = kMaxWorkgroups;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), smem, st, a);
    return hip_ok(hipGetLastError());
}

}  // namespace moe

using namespace moe;

// ---- scratch for callers that cannot allocate (see moe_dispatch_noalloc): one array per GPU the library runs on,
// held until the process ends.  In host code the array's name is only a handle: the device address comes from
// hipGetSymbolAddress, once per device with that device current, and only that address is handed to kernels.
constexpr size_t kStaticScratchBytes = 64 * 1024;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static int static_scratch_address(unsigned char **out) {
    static std::mutex lock;
    static unsigned char *addr[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MOE_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return MOE_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> g(lock);
    if (!addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MOE_ERR_HIP;
        addr[dev] = (unsigned char *)ptr;
    }
    *out = addr[dev];
    return MOE_OK;
}

extern "C" {

const char *moe_status_string(int s) {
    switch (s) {
        case MOE_OK: return "ok";
        case MOE_ERR_INVALID_ARG: return "invalid argument";
        case MOE_ERR_UNSUPPORTED: return "unsupported problem";
        case MOE_ERR_WORKSPACE: return "workspace missing or misaligned";
        case MOE_ERR_NOT_READY: return "a ready flag was not at the expected epoch";
        case MOE_ERR_HIP: return "HIP runtime error";
        case MOE_ERR_TIMEOUT: return "a bounded in-kernel wait expired";
        case MOE_ERR_BAD_ROUTING: return "expert id outside [0, E)";
        case MOE_ERR_CAPACITY: return "an expert received more rows than the capacity";
        default: return "unknown status";
    }
}

size_t moe_workspace_bytes(const moe_problem_t *p) {
    Plan pl;
    if (make_plan(p, &pl) != MOE_OK) return 0;
    return pl.total;
}

size_t moe_num_flags(const moe_problem_t *p) {
    Plan pl;
    if (make_plan(p, &pl) != MOE_OK) return 0;
    // a segment of c rows touches at most c/tile_m + 1 row blocks; there are E*R segments
    return ((size_t)(pl.N + pl.tile_m - 1) / pl.tile_m + (size_t)p->E * p->R) * pl.ncb;  // (make_plan sizes the group counters with the same bound)
}

int moe_workspace_init(const moe_problem_t *p, void *workspace, void *stream) {
    Plan pl;
    int rc = make_plan(p, &pl);
    if (rc) return rc;
    if ((rc = check_ws(workspace))) return rc;
    hipLaunchKernelGGL(k_zero, dim3(64), dim3(kThreads), 0, (hipStream_t)stream, (u32 *)workspace, pl.init_zero_bytes / 4);
    return hip_ok(hipGetLastError());
}

int moe_route(const moe_problem_t *p, const void *x, const void *Wg, const float *gate_bias, int32_t *topk_idx,
              float *topk_w, void *stream) {
    Plan pl;
    int rc = make_plan(p, &pl);
    if (rc) return rc;
    if (!x || !Wg || !topk_idx || !topk_w) return MOE_ERR_INVALID_ARG;
    KArgs a;
    fill_args(pl, nullptr, &a);
    set_gate(&a, x, Wg, gate_bias, true);
    a.idx = topk_idx; a.w = topk_w;
    size_t smem = gate_task_smem_bytes(p->E, p->d, elem_size(p->dtype));
    hipStream_t st = (hipStream_t)stream;
    auto launch = [&](auto kern, int threads = kThreads) {
        const int rc2 = set_smem(kern, smem);
        if (rc2) return rc2;
        hipLaunchKernelGGL(kern, dim3(a.nRT), dim3(threads), smem, st, a, 0);
        return hip_ok(hipGetLastError());
    };
    if (p->dtype == MOE_DT_F32) return launch(k_route<float, 0, kThreads>);
    if (a.gate_direct) {
        const int threads = direct_threads_alone(p->E, p->d);
        smem = direct_lds_bytes(p->E, p->d, threads);
        return threads == 512 ? launch(k_route<bf16_t, kGateDirect, 512>, 512) : launch(k_route<bf16_t, kGateDirect, kThreads>);
    }
    if (route_exact(p->T, p->E, p->d)) return launch(k_route<bf16_t, 0, kThreads>);
    switch (gate_variant(p->E, p->d)) {
        case 1: return launch(k_route<bf16_t, 1, kThreads>);
        case 2: return launch(k_route<bf16_t, 2, kThreads>);
        case 3: return launch(k_route<bf16_t, 3, kThreads>);
        case 4: return launch(k_route<bf16_t, 4, kThreads>);
        case 6: return launch(k_route<bf16_t, 6, kThreads>);
        default: return launch(k_route<bf16_t, 5, kThreads>);
    }
}

// The launches of a dispatch, shared by moe_dispatch (scratch in the caller's workspace) and
// moe_dispatch_noalloc (scratch in this library's static device array).  `short_only`: the form that needs the
// control block and the plan's tables is not available.
static int dispatch_launches(const Plan &pl, const KArgs &a, bool short_only, hipStream_t st) {
    const moe_problem_t *p = &pl.p;
    int rc;
    const size_t row_bytes = (size_t)p->d * elem_size(p->dtype);
    int ggrid = (pl.NP + 3) / 4;  // gather: one wavefront per row while rows last
    if (ggrid > 8192) ggrid = 8192;
    // rows that do not fit the 256 MB memory-side cache are stored past it; others are written through
    const bool past_cache = (size_t)pl.NP * row_bytes > ((size_t)192 << 20);
    const int sgrid = (p->T + a.disp_tokens - 1) / a.disp_tokens;
    // rows by token (read once, stored k times): ragged layout; the padded layout's histogram form keeps the gather
    // by sorted position, which also zeroes the unused rows
    auto move_rows = [&]() {
        if (!a.x_perm) return;
        if (p->capacity > 0)
            hipLaunchKernelGGL(k_gather, dim3(ggrid), dim3(kThreads), 0, st, a, row_bytes);
        else if (past_cache)
            hipLaunchKernelGGL(k_scatter<1>, dim3(sgrid), dim3(kThreads), 0, st, a, row_bytes);
        else
            hipLaunchKernelGGL(k_scatter<0>, dim3(sgrid), dim3(kThreads), 0, st, a, row_bytes);
    };
    if ((long long)pl.N * sgrid <= kFusedDispatchWork) {
        // one launch: every workgroup counts all N slots itself (no scratch at all)
        if (past_cache)
            hipLaunchKernelGGL(k_dispatch_fused<1>, dim3(sgrid), dim3(kThreads), 0, st, a, row_bytes);
        else
            hipLaunchKernelGGL(k_dispatch_fused<0>, dim3(sgrid), dim3(kThreads), 0, st, a, row_bytes);
        return hip_ok(hipGetLastError());
    }
    const size_t bsmem = block_perm_smem_bytes(p->E, pl.nPB);
    if (bsmem <= 64 * 1024) {
        // short form: per-block histograms, then every block derives its own base positions from all of
        // them (no single-workgroup plan, whose tile and flag tables a dispatch alone does not need)
        hipLaunchKernelGGL(k_block_hist, dim3(pl.nPB), dim3(kThreads), (size_t)p->E * 8, st, a);
        if (p->dtype == MOE_DT_F32) {
            if ((rc = set_smem(k_block_perm<float>, bsmem))) return rc;
            hipLaunchKernelGGL(k_block_perm<float>, dim3(pl.nPB), dim3(kThreads), bsmem, st, a);
        } else {
            if ((rc = set_smem(k_block_perm<bf16_t>, bsmem))) return rc;
            hipLaunchKernelGGL(k_block_perm<bf16_t>, dim3(pl.nPB), dim3(kThreads), bsmem, st, a);
        }
        move_rows();
        return hip_ok(hipGetLastError());
    }
    if (short_only) return MOE_ERR_UNSUPPORTED;
    const size_t psmem = plan_smem(pl);
    if ((rc = set_smem(k_plan, psmem))) return rc;
    // histogram (gate task without the gate), plan, permutation, row gather, clean-up
    if (p->dtype == MOE_DT_F32) {
        hipLaunchKernelGGL((k_route<float, 0, kThreads>), dim3(pl.nPB), dim3(kThreads), kMaxExperts * 4, st, a, 1);
        hipLaunchKernelGGL(k_plan, dim3(1), dim3(kThreads), psmem, st, a);
        hipLaunchKernelGGL(k_perm<float>, dim3(pl.nPB), dim3(kThreads), (size_t)p->E * 8, st, a);
    } else {
        hipLaunchKernelGGL((k_route<float, 0, kThreads>), dim3(pl.nPB), dim3(kThreads), kMaxExperts * 4, st, a, 1);
        hipLaunchKernelGGL(k_plan, dim3(1), dim3(kThreads), psmem, st, a);
        hipLaunchKernelGGL(k_perm<bf16_t>, dim3(pl.nPB), dim3(kThreads), (size_t)p->E * 8, st, a);
    }
    move_rows();
    hipLaunchKernelGGL(k_dispatch_finish, dim3(1), dim3(kThreads), 0, st, a);
    return hip_ok(hipGetLastError());
}

int moe_dispatch(const moe_problem_t *p, const void *x, const int32_t *topk_idx, int32_t *counts, int32_t *offsets,
                 int32_t *perm, int32_t *inv_perm, void *x_perm, int32_t *status_dev, void *workspace, void *stream) {
    Plan pl;
    int rc = make_plan(p, &pl);
    if (rc) return rc;
    if (!topk_idx || !counts || !offsets || !perm || !inv_perm) return MOE_ERR_INVALID_ARG;
    if (x_perm && !x) return MOE_ERR_INVALID_ARG;
    if ((rc = check_ws(workspace))) return rc;
    KArgs a;
    fill_args(pl, workspace, &a);
    a.x = x; a.idx = const_cast<int32_t *>(topk_idx);
    a.counts = counts; a.offsets = offsets; a.perm = perm; a.inv_perm = inv_perm; a.x_perm = x_perm;
    a.status_dev = status_dev;
    return dispatch_launches(pl, a, false, (hipStream_t)stream);
}

int moe_dispatch_noalloc(const moe_problem_t *p, const void *x, const int32_t *topk_idx, int32_t *counts,
                         int32_t *offsets, int32_t *perm, int32_t *inv_perm, void *x_perm, int32_t *status_dev,
                         void *stream) {
    Plan pl;
    int rc = make_plan(p, &pl);
    if (rc) return rc;
    if (!topk_idx || !counts || !offsets || !perm || !inv_perm) return MOE_ERR_INVALID_ARG;
    if (x_perm && !x) return MOE_ERR_INVALID_ARG;
    // the block histograms, the only scratch of the short form, must fit the static array
    if ((size_t)pl.nPB * p->E * 4 > kStaticScratchBytes) return MOE_ERR_UNSUPPORTED;
    unsigned char *scratch_dev = nullptr;
    if ((rc = static_scratch_address(&scratch_dev))) return rc;
    KArgs a;
    fill_args(pl, nullptr, &a);  // no workspace: no control block, no plan tables
    a.blk_base = (int32_t *)scratch_dev;
    a.x = x; a.idx = const_cast<int32_t *>(topk_idx);
    a.counts = counts; a.offsets = offsets; a.perm = perm; a.inv_perm = inv_perm; a.x_perm = x_perm;
    a.status_dev = status_dev;
    return dispatch_launches(pl, a, true, (hipStream_t)stream);
}

int moe_megakernel_forward(const moe_problem_t *p, const void *x, const void *Wg, const float *gate_bias,
                           const void *W1, const void *W3, const void *W2, int32_t *topk_idx, float *topk_w,
                           int32_t *counts, int32_t *offsets, int32_t *perm, int32_t *inv_perm, int32_t *slot_flag,
                           void *staging, uint32_t *flags, void *out, uint64_t *stats, void *workspace,
                           void *stream) {
    Plan pl;
    int rc = make_plan(p, &pl);
    if (rc) return rc;
    if (!x || !W1 || !W3 || !W2 || !topk_idx || !topk_w || !counts || !offsets || !perm || !inv_perm || !slot_flag ||
        !staging || !flags || !out)
        return MOE_ERR_INVALID_ARG;
    if (p->epoch == 0) return MOE_ERR_INVALID_ARG;
    if ((rc = check_ws(workspace))) return rc;
    KArgs a;
    fill_args(pl, workspace, &a);
    set_gate(&a, x, Wg, gate_bias, false);
    a.W1 = W1; a.W3 = W3; a.W2 = W2;
    a.idx = topk_idx; a.w = topk_w; a.counts = counts; a.offsets = offsets; a.perm = perm; a.inv_perm = inv_perm;
    a.slot_flag = slot_flag; a.staging = staging; a.flags = flags; a.out = out;
    a.stats = (u64 *)stats;
    // gate tasks: whole permutation blocks when the routing is an input; fp32 problems of few tokens (at most
    // kGateSplitBlocks blocks of 16) split every gate task over the reduction, so that the gate runs on all workgroups
    // instead of a handful
    int gate_tasks = Wg ? a.nRT : pl.nPB;
    if (Wg && p->dtype == MOE_DT_F32 && pl.nRT <= kGateSplitBlocks) {
        int S = kGateSplitTasks / pl.nRT;
        if (S > kGateSplitMax) S = kGateSplitMax;
        if (S > route_max_slices(p->d)) S = route_max_slices(p->d);
        if (S > 1) {
            a.gate_split = S;
            gate_tasks = pl.nRT * S;
            a.gate_partial = (double *)((char *)workspace + pl.o_gate_partial);
            a.gate_parts = (u32 *)((char *)workspace + pl.o_gate_parts);
        }
    }
    if (a.gate_direct && direct_parts(p->T, p->E, p->d) > 1) {
        a.gate_split = direct_parts(p->T, p->E, p->d);
        a.gate_direct = direct_threads(p->E, a.gate_split, kThreads);
        gate_tasks = a.nRT * a.gate_split;
        a.gate_partial = (double *)((char *)workspace + pl.o_gate_partial);
        a.gate_parts = (u32 *)((char *)workspace + pl.o_gate_parts);
    }
    if (Wg && p->dtype == MOE_DT_BF16 && !a.gate_direct) {
        a.WgT = (char *)workspace + pl.o_wgt;
        a.t_gate = wgt_tasks(p->d, p->E);
    }
    const int extra = gate_tasks - pl.nRT + a.t_gate;
    a.nRT = gate_tasks;
    a.t_plan += extra; a.t_perm += extra; a.t_g1 += extra; a.t_end += extra;
    if (pl.g2_split > 1) {
        a.g2_split = pl.g2_split;
        a.g2_rows = pl.g2_rows;
        a.g2_partial = (float *)((char *)workspace + pl.o_g2_partial);
        a.g2_parts = (Counter *)((char *)workspace + pl.o_g2_parts);
        a.t_end += (pl.tl.maxRB + p->E) * pl.tl.NT2 * (pl.g2_split - 1);
    }
    hipStream_t st = (hipStream_t)stream;
    // (Instantiated, and laid out in the library, in this order.  It decides where the code of a call lies, which it fetches cold, and no more:
    // the 32-row kernel in front of the 64-row one -> this, mean of four seeds, 8 tokens x 8 of 128 experts 120.2 -> 119.6 us, 128 x 8 of 128 251.7 ->
    // 250.8, 1001 x 6 of 48 181.4 -> 180.8, others level; 8 tokens take 0.7 % more with the 256-row code in front of both, 1.4 % more with the fp32 code.)
    switch (pl.kind) {
        case TK_S2: return launch_mega<Bf16Policy<CfgS2>, Bf16Policy<CfgS>>(pl, a, st);
        case TK_S: return launch_mega<Bf16Policy<CfgS>, Bf16Policy<CfgS>>(pl, a, st);
        case TK_LM: return launch_mega<Bf16Policy<CfgL>, Bf16Policy<CfgM>>(pl, a, st);
        case TK_FS: return launch_mega<FusedPolicy<CfgFS>, FusedPolicy<CfgFS>>(pl, a, st);
        case TK_FM: return launch_mega<FusedPolicy<CfgFM>, FusedPolicy<CfgFM>>(pl, a, st);
        case TK_F32: return launch_mega<F32Policy, F32Policy>(pl, a, st);
        default: return MOE_ERR_UNSUPPORTED;  // (no such kind)
    }
}

int moe_probe_stream(const void *buf, size_t span_bytes, size_t stride_bytes, size_t bytes_per_workgroup, int32_t workgroups,
                     int32_t wavefronts, int32_t to_lds, uint32_t *sink, void *stream) {
    if (!buf || !sink || workgroups < 1 || workgroups > 65536) return MOE_ERR_INVALID_ARG;
    if (wavefronts != 4 && wavefronts != 8 && wavefronts != 16) return MOE_ERR_INVALID_ARG;
    if (to_lds != 0 && to_lds != 1) return MOE_ERR_INVALID_ARG;
    // every piece is 16 bytes at a multiple of 16 below span_bytes
    if (span_bytes < 16 * 1024 || span_bytes % 16 != 0 || stride_bytes % 16 != 0 || bytes_per_workgroup < 1) return MOE_ERR_INVALID_ARG;
    // the whole LDS of a CU minus a margin: one workgroup per CU, whatever its size
    const size_t smem = 128 * 1024;
    hipStream_t st = (hipStream_t)stream;
    const char *b = (const char *)buf;
    int rc;
#define MOE_STREAM_CASE(NT, L)                                                                                          \
    if (wavefronts * 64 == NT && to_lds == L) {                                                                         \
        if ((rc = set_smem(k_probe_stream<NT, L != 0>, smem))) return rc;                                               \
        hipLaunchKernelGGL((k_probe_stream<NT, L != 0>), dim3(workgroups), dim3(NT), smem, st, b, span_bytes, stride_bytes, \
                           bytes_per_workgroup, sink);                                                                  \
    }
    MOE_STREAM_CASE(256, 0) MOE_STREAM_CASE(256, 1) MOE_STREAM_CASE(512, 0) MOE_STREAM_CASE(512, 1)
    MOE_STREAM_CASE(1024, 0) MOE_STREAM_CASE(1024, 1)
#undef MOE_STREAM_CASE
    return hip_ok(hipGetLastError());
}

int moe_probe_mfma(const void *frag, int32_t iters, int32_t workgroups, float *sink, void *stream) {
    if (!frag || !sink || iters < 1 || workgroups < 1 || workgroups > 65536) return MOE_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_probe_mfma, dim3(workgroups), dim3(kThreads), 0, (hipStream_t)stream, (const uint4 *)frag, iters, sink);
    return hip_ok(hipGetLastError());
}

int moe_combine(const moe_problem_t *p, const void *staging, const uint32_t *flags, const int32_t *slot_flag,
                const float *topk_w, void *out, int32_t *status_dev, void *stream) {
    Plan pl;
    int rc = make_plan(p, &pl);
    if (rc) return rc;
    if (!staging || !topk_w || !out) return MOE_ERR_INVALID_ARG;
    if ((slot_flag != nullptr) != (flags != nullptr)) return MOE_ERR_INVALID_ARG;
    KArgs a;
    fill_args(pl, nullptr, &a);
    a.staging = const_cast<void *>(staging);
    a.flags = const_cast<uint32_t *>(flags);
    a.slot_flag = const_cast<int32_t *>(slot_flag);
    a.w = const_cast<float *>(topk_w);
    a.out = out;
    a.status_dev = status_dev;
    hipStream_t st = (hipStream_t)stream;
    // rows that do not fit the 256 MB last-level cache are streamed past it
    const size_t row_bytes = (size_t)p->d * elem_size(p->dtype);
    const bool past_cache = (size_t)pl.N * row_bytes > ((size_t)192 << 20);
    a.comb_tokens = standalone_combine_tokens(p->T, row_bytes);
    a.nCT = (p->T + a.comb_tokens - 1) / a.comb_tokens;
    a.comb_span = p->T; a.comb_per_span = a.nCT;
    auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(a.nCT), dim3(kThreads), 0, st, a); };
    auto pick = [&](auto et) {
        using ET = decltype(et);
        if (a.comb_tokens < 4)
            past_cache ? launch(k_combine<ET, true, true>) : launch(k_combine<ET, false, true>);
        else
            past_cache ? launch(k_combine<ET, true, false>) : launch(k_combine<ET, false, false>);
    };
    if (p->dtype == MOE_DT_F32)
        pick(float{});
    else
        pick(bf16_t{});
    return hip_ok(hipGetLastError());
}

}  // extern "C"
