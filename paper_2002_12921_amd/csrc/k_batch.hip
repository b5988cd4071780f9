// Batched Vegas iterations: many independent problems (own dimension, grid,
// event count and integrand parameters) in one persistent launch.
//
// The event kernel's blocks take work items -- a range of one problem's
// events -- from an atomic counter until none is left.  Items are ordered by
// cost (larger dimension first), so the tail of the launch is made of cheap
// items.  When a block moves to another problem it reloads that problem's
// grid table into LDS; each item leaves one partial row (S1, S2, H[d][N]).
// The finish kernel then reduces each problem's rows (one block per problem
// and column group), records the iteration and refines the grid, as the
// single-problem reduction does.
#include "grid_ops.hpp"

namespace vegas {

// Fewest waves per SIMD the register allocation must allow: 4, i.e. up to
// 128 registers.  The FP32-mixed kernel of the d <= 16 bucket needs about
// 100; capped at 80 (6 waves) it spilled 30 registers to scratch, which
// moved about 9 GB per launch through HBM for the 256-problem batch (its
// histogram launches took 22 ms per run against 18 ms without the spills).
template <class P, int DMAX>
struct BatchMinWaves {
    static constexpr int value = 4;
};

// The events of one work item into the block's LDS histogram and the item's
// (S1, S2) row.  DE > 0: compiled for exactly DE dimensions (the problem's
// d), with no per-dimension guards, so the whole event runs as one block of
// straight-line code; DE = 0: each dimension is guarded against d <= DMAX.
// ltab, lhist: LDS addresses of the table and the histogram.
template <class P, int KIND, int DMAX, int DE, bool HIST>
__device__ __forceinline__ void batch_item_events(const BatchArgs& a, const BatchItem& it, const BatchProblem& pr,
                                                  uint32_t ltab, uint32_t lhist, int rl2, int d, int N,
                                                  double* red)
{
    constexpr int DM = DE > 0 ? DE : DMAX;
    EvalConsts<P, KIND, DM> cst;
    cst.load(pr.cst, pr.thr, d, N, ltab);
    const HistAdder<TabLog2<P, KIND>::value> hadd(ltab, lhist, rl2);
    const uint32_t key0 = pr.key0, key1 = pr.key1, ctr3 = pr.ctr3;
    double s1 = 0.0, c1 = 0.0, s2 = 0.0, c2 = 0.0, g1 = 0.0, g2 = 0.0;
    int ng = 0;
    const uint64_t end = it.e0 + it.n;
    for (uint64_t e = it.e0 + threadIdx.x; e < end; e += blockDim.x) {
        EventEval<P, KIND, DM, (DE > 0)> ev;
        ev.run(cst, ltab, e, a.t, ctr3, key0, key1, d, N);
        double v, v2;
        {
            // rounded as written in every variant (with or without histograms)
#pragma clang fp contract(off)
            v = ev.value(cst);
            v2 = v * v;
            g1 += v;
            g2 += v2;
        }
        if (++ng == kGroup) {
            kahan_add(s1, c1, g1);
            kahan_add(s2, c2, g2);
            g1 = g2 = 0.0;
            ng = 0;
        }
        if constexpr (HIST) hadd.template add<DM, (DE > 0)>(ev.off, d, v2);
    }
    kahan_add(s1, c1, g1);
    kahan_add(s2, c2, g2);
    // block_sums synchronises, which also completes every histogram atomic
    const double v12[2] = {s1 - c1, s2 - c2};
    const double S = block_sums(v12, red);
    if (threadIdx.x < 2) a.partials[it.row_off + threadIdx.x] = S;
}

// The exact-d variant for d in [LO, DE] (an if-chain from DE down), the
// guarded one below LO.
template <class P, int KIND, int DMAX, int DE, int LO, bool HIST>
__device__ __forceinline__ void batch_item_dispatch(const BatchArgs& a, const BatchItem& it, const BatchProblem& pr,
                                                    uint32_t ltab, uint32_t lhist, int rl2, int d, int N,
                                                    double* red)
{
    if constexpr (DE < LO) {
        batch_item_events<P, KIND, DMAX, 0, HIST>(a, it, pr, ltab, lhist, rl2, d, N, red);
    } else {
        if (d == DE)
            batch_item_events<P, KIND, DMAX, DE, HIST>(a, it, pr, ltab, lhist, rl2, d, N, red);
        else
            batch_item_dispatch<P, KIND, DMAX, DE - 1, LO, HIST>(a, it, pr, ltab, lhist, rl2, d, N, red);
    }
}

// The buckets up to d = 16 run each item with the loop compiled for the
// problem's exact d (items are sorted by d, so a block seldom changes
// variant); larger buckets guard each dimension.
template <class P, int KIND, int DMAX, bool HIST>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(BatchMinWaves<P, DMAX>::value, 8))) void k_batch_sample(
    BatchArgs a)
{
    // the bucket's d range: (DMAX/2, DMAX], and 1..4 for the smallest
    constexpr int kLo = DMAX <= 4 ? 1 : DMAX / 2 + 1;
    constexpr bool kExact = DMAX <= 16;
    using tab_t = typename TabEntry<P, KIND>::type;
    extern __shared__ __align__(128) unsigned char smem[];
    // the block's wave partials; between items, the item taken (256 bytes in
    // all: the host leaves that much of the LDS)
    __shared__ double red[2 * kBlock / 64];
    int& s_item = *reinterpret_cast<int*>(red);
    // table, then the histogram [dim][bin][replica], lane l adding into replica l mod rep
    const int rl2 = a.hrep_log2;
    int cur = -1;
    int d = 0, N = 0, dN = 0;
    uint32_t hoff = 0;
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    for (;;) {
        if (threadIdx.x == 0) s_item = a.item_lo + int(atomicAdd(a.queue, 1u));
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= a.item_hi) break;  // every block leaves once the queue is empty
        const BatchItem it = a.items[item];
        const BatchProblem& pr = a.probs[it.prob];
        if (it.prob != cur) {
            cur = it.prob;
            d = pr.d;
            N = pr.N;
            dN = d * N;
            const tab_t* gtab = P::is64 ? reinterpret_cast<const tab_t*>(pr.tab64)
                                        : reinterpret_cast<const tab_t*>(pr.tab32);
            for (int k = threadIdx.x; k < dN; k += blockDim.x) tab[k] = gtab[k];
            hoff = (uint32_t(dN) * uint32_t(sizeof(tab_t)) + 127u) & ~127u;
        }
        double* hist = reinterpret_cast<double*>(smem + hoff);
        const uint32_t ltab = lds_address(smem);
        if constexpr (HIST)
            for (int k = threadIdx.x; k < dN << rl2; k += blockDim.x) hist[k] = 0.0;
        __syncthreads();

        if constexpr (kExact)
            batch_item_dispatch<P, KIND, DMAX, DMAX, kLo, HIST>(a, it, pr, ltab, ltab + hoff, rl2, d, N, red);
        else
            batch_item_events<P, KIND, DMAX, 0, HIST>(a, it, pr, ltab, ltab + hoff, rl2, d, N, red);

        if constexpr (HIST) {
            double* row = a.partials + it.row_off;
            for (int k = threadIdx.x; k < dN; k += blockDim.x) row[2 + k] = replica_sum(hist, k, rl2);
        }
        __syncthreads();
    }
}

#ifdef VEGAS_BATCH_PREC

// The event kernels of one precision and integrand are one compilation of
// this file each (VEGAS_BATCH_PREC, VEGAS_BATCH_KIND).
template <class P, int KIND, bool HIST>
static const void* batch_fn(int dmax)
{
    switch (dmax) {
    case 4: return reinterpret_cast<const void*>(&k_batch_sample<P, KIND, 4, HIST>);
    case 8: return reinterpret_cast<const void*>(&k_batch_sample<P, KIND, 8, HIST>);
    case 16: return reinterpret_cast<const void*>(&k_batch_sample<P, KIND, 16, HIST>);
    case 32: return reinterpret_cast<const void*>(&k_batch_sample<P, KIND, 32, HIST>);
    default: return reinterpret_cast<const void*>(&k_batch_sample<P, KIND, 64, HIST>);
    }
}

#define VEGAS_PART_NAME2(p, k) batch_fn_##p##_##k
#define VEGAS_PART_NAME(p, k) VEGAS_PART_NAME2(p, k)
const void* VEGAS_PART_NAME(VEGAS_BATCH_PREC, VEGAS_BATCH_KIND)(int dmax, bool hist)
{
    using P = pick_type<VEGAS_BATCH_PREC == 64, P64, P32>::type;
    return hist ? batch_fn<P, VEGAS_BATCH_KIND, true>(dmax) : batch_fn<P, VEGAS_BATCH_KIND, false>(dmax);
}

#else

// Per problem and column group: reduce the problem's item rows, record the
// iteration, refine (adaptation iterations).  Also resets the work queue for
// the next event launch on the stream.
template <int T>
__global__ __launch_bounds__(T) void k_batch_finish(BatchArgs a, int kind, int rec_idx, int flags)
{
    const int g = blockIdx.x, p = blockIdx.y;
    if (p == 0 && g == 0 && threadIdx.x < kMaxBuckets) a.queue[threadIdx.x] = 0u;
    const BatchProblem pr = a.probs[p];
    if (g > pr.d) return;
    MergeArgs m{};
    m.partials = a.partials + pr.row0;
    m.last = pr.last;
    m.edges = pr.edges;
    m.tab64 = pr.tab64;
    m.tab32 = pr.tab32;
    m.thr = pr.thr;
    m.cst = pr.cst;
    m.records = pr.records;
    m.rec_flag = pr.rec_flag;
    m.result = pr.result;
    m.alpha = pr.alpha;
    m.M = pr.M;
    m.rows = pr.n_items;
    m.d = pr.d;
    m.N = pr.N;
    m.pstride = pr.pstride;
    m.rstride = pr.pstride;  // batch rows carry S1, S2 and H
    m.kind = kind;
    m.flags = MERGE_BEGIN | MERGE_END | flags;
    m.rec_idx = rec_idx;
    merge_group<T>(m, g);
}

// Restart every problem: uniform grid and tables, no recorded iterations.
__global__ __launch_bounds__(kMergeThreads) void k_batch_reset(BatchArgs a, int n_rec, int kind)
{
    const int g = blockIdx.x, p = blockIdx.y;
    if (p == 0 && g == 0 && threadIdx.x < kMaxBuckets) a.queue[threadIdx.x] = 0u;
    const BatchProblem pr = a.probs[p];
    if (g < pr.d) {
        double* E = pr.edges + size_t(g) * (pr.N + 1);
        for (int k = threadIdx.x; k <= pr.N; k += blockDim.x) E[k] = double(k) / double(pr.N);
        __syncthreads();
        write_tables(g, E, pr.cst, kind, pr.N, pr.tab64, pr.tab32, pr.thr);
    } else if (g == pr.d) {
        for (int k = threadIdx.x; k < pr.pstride; k += blockDim.x) pr.last[k] = 0.0;
        for (int k = threadIdx.x; k < 2 * n_rec; k += blockDim.x) pr.records[k] = 0.0;
        for (int k = threadIdx.x; k < n_rec; k += blockDim.x) pr.rec_flag[k] = 0;
        if (threadIdx.x == 0) {
            const double nan = __builtin_nan("");
            DevResult* R = pr.result;
            R->integral = R->sigma = R->chi2_dof = R->last_integral = R->last_var = nan;
            R->n_iter = R->n_combined = R->n_events = R->n_nonfinite = 0;
        }
    }
}

__global__ void k_batch_combine(BatchArgs a, int n_rec)
{
    const BatchProblem pr = a.probs[blockIdx.x];
    const int n = pr.result->n_iter < n_rec ? int(pr.result->n_iter) : n_rec;
    combine_records(pr.records, pr.rec_flag, n, pr.result, HostPost{});
}

hipError_t launch_batch_combine(const BatchArgs& a, int n_rec, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_combine, dim3(a.n_probs), dim3(64), 0, s, a, n_rec);
    return hipGetLastError();
}

// groups: column groups over all problems. Where they fit the chip at once as
// blocks of 1024 threads (two on a CU, by their 67 KiB of LDS), those finish
// first, a wave's chain of rows being a quarter as long. With more of them,
// blocks of 256 threads, of which a CU holds eight: the 256-problem batch
// (2600 groups, 24 MB of rows) took 51 us with the one and 19 with the other.
hipError_t launch_batch_finish(const BatchArgs& a, int dmax, int groups, int kind, int rec_idx, int flags,
                               hipStream_t s)
{
    const bool wide = groups <= 512;
    hipLaunchKernelGGL(wide ? k_batch_finish<kMergeThreads> : k_batch_finish<256>, dim3(dmax + 1, a.n_probs),
                       dim3(wide ? kMergeThreads : 256), 0, s, a, kind, rec_idx, flags);
    return hipGetLastError();
}

hipError_t launch_batch_reset(const BatchArgs& a, int dmax, int n_rec, int kind, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_reset, dim3(dmax + 1, a.n_probs), dim3(256), 0, s, a, n_rec, kind);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------

// Parts defined by the other compilations.
const void* batch_fn_64_0(int dmax, bool hist);
const void* batch_fn_64_1(int dmax, bool hist);
const void* batch_fn_64_2(int dmax, bool hist);
const void* batch_fn_64_3(int dmax, bool hist);
const void* batch_fn_32_0(int dmax, bool hist);
const void* batch_fn_32_1(int dmax, bool hist);
const void* batch_fn_32_2(int dmax, bool hist);
const void* batch_fn_32_3(int dmax, bool hist);

static const void* batch_kernel(int prec, int kind, int dmax, bool hist)
{
    using Fn = const void* (*)(int, bool);
    static const Fn f64[] = {batch_fn_64_0, batch_fn_64_1, batch_fn_64_2, batch_fn_64_3};
    static const Fn f32[] = {batch_fn_32_0, batch_fn_32_1, batch_fn_32_2, batch_fn_32_3};
    return (prec == FP64 ? f64 : f32)[kind](dmax, hist);
}

// Without histograms the launch keeps the same grid (and LDS size): it is a
// work queue, so residency only sets how many blocks share the items.
hipError_t launch_batch_sample(int prec, int kind, int dmax, size_t lds, const BatchArgs& a, int blocks,
                               int threads, bool hist, hipStream_t s)
{
    void* args[] = {const_cast<BatchArgs*>(&a)};
    return hipLaunchKernel(batch_kernel(prec, kind, dmax, hist), dim3(blocks), dim3(threads), args, lds, s);
}

int batch_max_blocks_per_cu(int prec, int kind, int dmax, size_t lds, int threads)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel(prec, kind, dmax, true), threads, lds) !=
        hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

#endif  // VEGAS_BATCH_PREC

}  // namespace vegas
