// Event kernel of one Vegas iteration: points -> map -> integrand -> block
// partials of S1 = sum f w, S2 = sum (f w)^2 and H[i][b] = sum (f w)^2 over
// events in bin b of dimension i (the accumulators of Lepage's method that
// the paper's per-event stage fills, sec. 2.2).
//
// Layout: the grid's (lower edge, width) table [d][N] and the block's
// histogram [d][N] (FP64) live in LDS; events never touch memory.  Each
// thread strides over the launch's events; S1/S2 are Kahan-summed per thread,
// reduced across the block and written as the block's row (S1, S2) of the
// partial table (summed later in a fixed order); the block's histogram is
// added into one of kHistSlots accumulators with FP64 atomics (its sums come
// from LDS atomics in no fixed order anyway).
#include "device_common.hpp"

namespace vegas {

// Histogram modes of the event kernel: none (an iteration whose grid is not
// refined), or LDS replicas behind the table with the dimensions in sets of
// one (HistAdder), two or four (HistSets).
constexpr int kHistNone = 0, kHistSets1 = 1, kHistSets2 = 2, kHistSets4 = 3;

// Waves per SIMD the register allocation allows, at least and at most.
//   FP64 up to d = 8, all but the discontinuous integrand: 6 (80 VGPRs).  They
//     fit without spills, and the launch runs two 768-thread blocks per CU.  At
//     8 waves (64 VGPRs, two 1024-thread blocks) the d = 8 Gaussian spilled 15
//     registers and took 62.2-63.0 us per 1e7 events, at 7 (896-thread blocks)
//     it still spilled 8 and took 70.0-70.8 us, at 6: 57.9-58.5 us (all with an
//     earlier form of the loop; today's takes 51).
//   FP32-mixed up to d = 8: 8, two 1024-thread blocks per CU (without the
//     bound, the sums at the kernel's end took some past 64 VGPRs).
//   FP64 discontinuous integrand, d = 14 to 24: 3, one 768-thread block per CU.
//     Its FP64 c_i and thresholds leave too few scalar registers, and at 128
//     VGPRs (4 waves) the d = 16 kernel spilled 18 of them: 132.1-132.3 against
//     123.4-123.6 us per 1e7 events; d = 20 with N = 100: 232 against 172 us.
//     FP32-mixed likewise at d = 17 to 19 (FP64 c_i beside 20 bins; N = 100, d =
//     19: 211 against 134 us).
//   Beyond d = 8 with histograms: at most 4.  From d N of about 600 on the LDS
//     holds one 1024-thread block's table and replicated histogram, which the
//     compiler cannot know from the dynamic LDS size: told so, it may use up to
//     128 registers and keep an event's table reads in flight together instead
//     of waiting on each (the d = 20 bimodal kernel waited on every one).  Below,
//     smaller blocks share a CU, or two of 1024 where 64 registers do (the
//     FP32-mixed Gaussian at d = 12 and 16); a variant compiled for more waves
//     has not been measured there.
//   4 to 8 elsewhere.
template <class P, int KIND, int DMAX, bool EXACT, int HM>
struct Waves {
    static constexpr bool three =
        KIND == GENZ_DISC && EXACT && (P::is64 ? DMAX >= 14 && DMAX <= 24 : DMAX >= 17 && DMAX <= 19);
    static constexpr bool six = P::is64 && KIND != GENZ_DISC && DMAX <= 8;
    static constexpr bool eight = !P::is64 && DMAX <= 8;
    static constexpr int min = three ? 3 : six ? 6 : eight ? 8 : 4;
    static constexpr int max = three ? 3 : (DMAX > 8 && HM != 0) ? 4 : six ? 6 : 8;
};

template <class P, int KIND, int DMAX, bool EXACT, int HM>
struct MaxThreads {
    static constexpr int value = Waves<P, KIND, DMAX, EXACT, HM>::three ? 768 : kBlock;
};

template <class P, int KIND, int DMAX, bool EXACT, int HM>
__global__ __attribute__((amdgpu_flat_work_group_size(1, MaxThreads<P, KIND, DMAX, EXACT, HM>::value),
                          amdgpu_waves_per_eu(Waves<P, KIND, DMAX, EXACT, HM>::min,
                                              Waves<P, KIND, DMAX, EXACT, HM>::max))) void k_sample(
    SampleArgs a)
{
    using tab_t = typename TabEntry<P, KIND>::type;
    constexpr int GL = HM == kHistNone ? 0 : HM - 1;  // log2 of the dimensions in a set
    extern __shared__ __align__(128) unsigned char smem[];
    const int dN = a.d * a.N;
    const size_t tab_bytes = (size_t(dN) * sizeof(tab_t) + 127) & ~size_t(127);
    const int rl2 = GL > 0 ? 4 - GL : a.hrep_log2;
    // counters of the histogram: whole sets
    const int nh = GL > 0 ? ((DMAX + (1 << GL) - 1) >> GL << GL) * a.N : dN;
    const size_t hist_bytes = HM == kHistNone ? 0 : size_t(nh) * sizeof(double) << rl2;
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    double* hist = reinterpret_cast<double*>(smem + tab_bytes);
    double* red = reinterpret_cast<double*>(smem + tab_bytes + hist_bytes);
    const uint32_t ltab = lds_address(smem);
    static_assert(GL == 0 || EXACT, "sets of dimensions: kernels without guards only");
    const HistAdder<TabLog2<P, KIND>::value> hadd(ltab, ltab + uint32_t(tab_bytes), rl2);
    constexpr bool kHoldRows = DMAX <= 24 && !(KIND == GENZ_DISC && DMAX > 12);
    const HistSets<GL, DMAX, kHoldRows> hsets(ltab + uint32_t(tab_bytes), a.N);

    // the table's first entries and the constants are on their way while the
    // histogram is cleared
    const tab_t* gtab = static_cast<const tab_t*>(a.tab);
    const tab_t first = gtab[min(int(threadIdx.x), dN - 1)];
    EvalConsts<P, KIND, DMAX> cst;
    cst.load(a.cst, a.thr, a.d, a.N, ltab);
    if constexpr (HM != kHistNone) {   // 16 bytes per store (hist is 128-byte aligned), then an odd last double
        double2* h2 = reinterpret_cast<double2*>(hist);
        for (int k = threadIdx.x; k < int(hist_bytes / sizeof(double2)); k += blockDim.x)
            h2[k] = make_double2(0.0, 0.0);
        if ((hist_bytes & 8) && threadIdx.x == 0) hist[hist_bytes / sizeof(double) - 1] = 0.0;
    }
    if (int(threadIdx.x) < dN) tab[threadIdx.x] = first;
    for (int k = threadIdx.x + blockDim.x; k < dN; k += blockDim.x) tab[k] = gtab[k];
    __syncthreads();

    const int d = EXACT ? DMAX : a.d;
    double s1 = 0.0, c1 = 0.0, s2 = 0.0, c2 = 0.0;
    double g1 = 0.0, g2 = 0.0;
    int ng = 0;
    // event k = j * stride + threadIdx.x * gridDim.x + blockIdx.x in pass j:
    // the last, partial pass is spread over every block rather than a few
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    const uint64_t end = a.e0 + a.n;
    for (uint64_t e = a.e0 + uint64_t(threadIdx.x) * gridDim.x + blockIdx.x; e < end; e += stride) {
        EventEval<P, KIND, DMAX, EXACT> ev;
        ev.run(cst, ltab, e, a.t, a.ctr3, a.key0, a.key1, d, a.N);
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
        if constexpr (GL > 0)
            hsets.add(ev.bin, v2);
        else if constexpr (HM != kHistNone)
            hadd.template add<DMAX, EXACT>(ev.off, d, v2);
    }
    kahan_add(s1, c1, g1);
    kahan_add(s2, c2, g2);

    // block_sums synchronises, which also completes every histogram atomic
    const double v12[2] = {s1 - c1, s2 - c2};
    const double S = block_sums(v12, red);
    if (threadIdx.x < 2) a.partials[size_t(blockIdx.x) * 2 + threadIdx.x] = S;
    // the block's histogram (replicas summed) goes into slot
    // (blockIdx / 8) mod kHistSlots with device-scope FP64 atomics: no
    // histogram row to write and read back, and 8 slots keep the atomics on
    // one address few.  Workgroups go to the 8 XCDs round-robin, so each XCD's
    // blocks spread over all the slots (blockIdx mod 8 gave each XCD one slot
    // and ran about 1 % slower)
    double* slot = a.hslots + size_t((blockIdx.x >> 3) % kHistSlots) * dN;
    if constexpr (HM != kHistNone) {
        for (int k = threadIdx.x; k < nh; k += blockDim.x) {
            if constexpr (GL == 0) {
                atomicAdd(&slot[k], replica_sum(hist, k, rl2));
            } else {
                // counter k: bin b of dimension i of its set
                const int s = k / (a.N << GL), r = k - s * (a.N << GL);
                const int i = (s << GL) + (r & ((1 << GL) - 1)), b = r >> GL;
                if (i < DMAX) atomicAdd(&slot[i * a.N + b], replica_sum<4 - GL>(hist, k));
            }
        }
    }
}

#ifndef VEGAS_SAMPLE_PREC

// Per-event records for parity checks: b, delta, x, w, f of each event.
template <class P, int KIND, int DMAX>
__global__ __launch_bounds__(kBlock) void k_dump(DumpArgs a)
{
    using tab_t = typename TabEntry<P, KIND>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t ltab = lds_address(smem);
    const int dN = a.d * a.N;
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    const tab_t* gtab = static_cast<const tab_t*>(a.tab);
    for (int k = threadIdx.x; k < dN; k += blockDim.x) tab[k] = gtab[k];
    __syncthreads();
    EvalConsts<P, KIND, DMAX> cst;
    cst.load(a.cst, a.thr, a.d, a.N, ltab);
    cst.leave_out_constant(a.d);
    const uint64_t stride = uint64_t(gridDim.x) * kBlock;
    for (uint64_t k = uint64_t(blockIdx.x) * kBlock + threadIdx.x; k < a.n; k += stride) {
        EventEval<P, KIND, DMAX> ev;
        ev.run(cst, ltab, a.e0 + k, a.t, a.ctr3, a.key0, a.key1, a.d, a.N);
        double* row = a.out + k * size_t(3 * a.d + 2);
        // x = centre + u; delta as the kernel represents it (FP32: (RN32(lo) +
        // h)/2^32, and u carries the factor S); w and f with their exponents
        const double ds = P::is64 ? 1.0 : double(cst.dscale);
#pragma unroll
        for (int i = 0; i < DMAX; ++i) {
            if (i < a.d) {
                row[i] = double(ev.bin[i]);
                row[a.d + i] = double(ev.del[i]) * 0x1p-32 + cst.bc.h64;
                row[2 * a.d + i] = double(ev.u[i]) * ds + a.cst->cA64[i];
            }
        }
        row[3 * a.d] = ldexp(double(ev.wp), ev.ew) * cst.Cw;
        row[3 * a.d + 1] = ldexp(double(ev.F), ev.fe) * cst.Cf;
    }
}

// Adjoint at fixed samples (Gaussian): per-thread FP64 sums of
// v * d ln f / d theta_j, theta = (mu_0..mu_{d-1}, a):
//   d ln f / d mu_j = 2 (x_j - mu_j) / a^2,  d ln f / d a = (2 s / a^2 - d) / a.
// Block rows go to a partial table; k_adjoint_merge adds them in a fixed
// order and writes gout * sum / M.  EXACT: d == DMAX, so the per-dimension
// guards fold away and the table reads of an event can all be in flight.
template <class P, int DMAX, bool EXACT>
__global__ __launch_bounds__(kBlock) void k_adjoint(AdjointArgs a)
{
    using tab_t = typename TabEntry<P, GAUSS>::type;
    using real = typename P::real;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t ltab = lds_address(smem);
    const int dN = a.d * a.N;
    const size_t tab_bytes = (size_t(dN) * sizeof(tab_t) + 15) & ~size_t(15);
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    double* red = reinterpret_cast<double*>(smem + tab_bytes);
    const tab_t* gtab = static_cast<const tab_t*>(a.tab);
    for (int k = threadIdx.x; k < dN; k += blockDim.x) tab[k] = gtab[k];
    __syncthreads();

    const DevConst* c = a.cst;
    EvalConsts<P, GAUSS, DMAX> cst;
    cst.load(c, nullptr, a.d, a.N, ltab);
    // the FP32 path's u carries the factor S = 2^(ws + 32): its constants take S^-1, S^-2 (exact)
    const double ds = P::is64 ? 1.0 : double(c->dscale32) * 0x1p-32;
    const real ka = P::is64 ? real(c->kexp64) : real(double(c->ka32) * ds);
    // d ln f / d mu_j = 2 ka u_j: the events' sum of v u_j, then one product
    // with 2 ka per block row (the factor 2 is exact)
    const real ka2 = real(2) * ka;
    const double inv_a = c->inv_a;
    const int d = EXACT ? DMAX : a.d;
    const double ka64 = c->kexp64 * ds * ds;
    double g[DMAX + 1];
#pragma unroll
    for (int j = 0; j <= DMAX; ++j) g[j] = 0.0;

    const uint64_t stride = uint64_t(gridDim.x) * kBlock;
    for (uint64_t k = uint64_t(blockIdx.x) * kBlock + threadIdx.x; k < a.n; k += stride) {
        EventEval<P, GAUSS, DMAX, EXACT> ev;
        ev.run(cst, ltab, k, a.t, a.ctr3, a.key0, a.key1, d, a.N);
        const double v = ev.value(cst);
#pragma unroll
        for (int j = 0; j < DMAX; ++j)
            if (j < d) g[j] += v * double(ev.u[j]);  // times 2 ka once per block
        const double da = 2.0 * ev.s64 * ka64 - double(d);
        g[DMAX] += v * (da * inv_a);
    }

    // sums over the block, column j in thread j: d components of mu, then a
    const double t = block_sums(g, red);
    double* row = a.partials + size_t(blockIdx.x) * (d + 1);
    const int j = int(threadIdx.x);
    if (j < d) row[j] = t * double(ka2);
    if (j == DMAX) row[d] = t;
}

// Final step of the adjoint: the rows' fixed-order sums scaled by gout/M,
// stored in FP64 or rounded once to FP32 (grad_fp32).
// One wave per component.
__global__ __launch_bounds__(64) void k_adjoint_merge(AdjointArgs a, int rows)
{
    adjoint_merge_column(a.partials, rows, a.d, blockIdx.x, *a.gout / double(a.n), a.grad, a.grad_fp32);
}

// Forward pass with the gradient (Gaussian, frozen grid, no histograms):
// the event kernel without histograms -- same events per thread, same
// grouped Kahan S1, S2, so the estimate is bitwise that of k_sample -- that
// also sums each event's v d ln f / d theta_j, as k_adjoint does, into
// per-block rows gpart[block][d + 1] (merged by k_merge's gradient block).
// It launches like the event kernel (two 1024-thread blocks per CU, 8 waves
// per SIMD), so FP32 up to d = 8 is compiled for 8 waves: at its natural
// 70 registers (d = 8) only one block fitted per CU and the grid ran in two
// rounds of 4 waves per SIMD (at 64, d = 8 spills 28 bytes a lane).
template <class P, int DMAX, bool EXACT>
struct GradMinWaves {
    static constexpr int value = (!P::is64 && DMAX <= 8 && EXACT) ? 8 : 1;
};

template <class P, int DMAX, bool EXACT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(GradMinWaves<P, DMAX, EXACT>::value))) void
k_sample_grad(SampleArgs a, double* gpart)
{
    using tab_t = typename TabEntry<P, GAUSS>::type;
    using real = typename P::real;
    extern __shared__ __align__(128) unsigned char smem[];
    const uint32_t ltab = lds_address(smem);
    const int dN = a.d * a.N;
    const size_t tab_bytes = (size_t(dN) * sizeof(tab_t) + 127) & ~size_t(127);
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    double* red = reinterpret_cast<double*>(smem + tab_bytes);
    const tab_t* gtab = static_cast<const tab_t*>(a.tab);
    for (int k = threadIdx.x; k < dN; k += blockDim.x) tab[k] = gtab[k];
    __syncthreads();

    const DevConst* c = a.cst;
    EvalConsts<P, GAUSS, DMAX> cst;
    cst.load(c, nullptr, a.d, a.N, ltab);
    const double ds = P::is64 ? 1.0 : double(c->dscale32) * 0x1p-32;
    const real ka = P::is64 ? real(c->kexp64) : real(double(c->ka32) * ds);
    const real ka2 = real(2) * ka;
    const double inv_a = c->inv_a;
    const int d = EXACT ? DMAX : a.d;
    const double ka64 = c->kexp64 * ds * ds;
    double s1 = 0.0, c1 = 0.0, s2 = 0.0, c2 = 0.0;
    double g1 = 0.0, g2 = 0.0;
    int ng = 0;
    double g[DMAX + 1];
#pragma unroll
    for (int j = 0; j <= DMAX; ++j) g[j] = 0.0;
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    const uint64_t end = a.e0 + a.n;
    for (uint64_t e = a.e0 + uint64_t(threadIdx.x) * gridDim.x + blockIdx.x; e < end; e += stride) {
        EventEval<P, GAUSS, DMAX, EXACT> ev;
        ev.run(cst, ltab, e, a.t, a.ctr3, a.key0, a.key1, d, a.N);
        double v, v2;
        {
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
#pragma unroll
        for (int j = 0; j < DMAX; ++j)
            if (j < d) g[j] += v * double(ev.u[j]);  // times 2 ka once per block
        const double da = 2.0 * ev.s64 * ka64 - double(d);
        g[DMAX] += v * (da * inv_a);
    }
    kahan_add(s1, c1, g1);
    kahan_add(s2, c2, g2);
    // the same sums in the same order as the event kernel's, then the components'
    const double v12[2] = {s1 - c1, s2 - c2};
    const double S = block_sums(v12, red);
    if (threadIdx.x < 2) a.partials[size_t(blockIdx.x) * 2 + threadIdx.x] = S;
    const double t = block_sums(g, red + 2 * (blockDim.x >> 6));
    double* grow = gpart + size_t(blockIdx.x) * (d + 1);
    const int j = int(threadIdx.x);
    if (j < d) grow[j] = t * double(ka2);
    if (j == DMAX) grow[d] = t;
}

#endif  // !VEGAS_SAMPLE_PREC

// ---------------------------------------------------------------------------
// Dispatch.  The event kernels are compiled for every d up to kExactDim and
// for the buckets' own dimensions beyond; other d run guarded in the next
// larger bucket.  Guards split an event into a block per dimension and keep
// its table reads from being in flight together: per 1e7 events, d = 13
// FP32-mixed with N = 37, 144 us guarded and 78 us exact with histograms (93
// and 66 us without), and d = 5 product peak FP64 with N = 100, 71 and 46 us.
// (The event kernels of one precision and integrand are one
// compilation of this file each: VEGAS_SAMPLE_PREC, VEGAS_SAMPLE_KIND.)

constexpr int kExactDim = 20;

// Largest d whose kernels take the dimensions in sets: beyond, their bins and
// constants do not fit the registers (d = 64, FP32-mixed Gaussian: 183 us per
// 3e6 events with 4 conflicting replicas, 312 us with sets and spills; d = 32
// discontinuous: 118 and 145 us).
constexpr int sets_dim(int kind) { return kind == GENZ_DISC ? 20 : kind == GENZ_PEAK ? 24 : 32; }

static int dim_bucket(int d)
{
    if (d <= kExactDim) return d;
    if (d <= 24) return 24;
    if (d <= 32) return 32;
    if (d <= 48) return 48;
    return 64;
}

// Parts defined by the other compilations: the kernel for (d, histogram mode).
using SampleFn = const void* (*)(int d, int hm);
const void* sample_fn_64_0(int d, int hm);
const void* sample_fn_64_1(int d, int hm);
const void* sample_fn_64_2(int d, int hm);
const void* sample_fn_64_3(int d, int hm);
const void* sample_fn_32_0(int d, int hm);
const void* sample_fn_32_1(int d, int hm);
const void* sample_fn_32_2(int d, int hm);
const void* sample_fn_32_3(int d, int hm);

#ifdef VEGAS_SAMPLE_PREC

template <class P, int KIND, int HM, int... D>
static const void* exact_fn(int d, IntSeq<D...>)
{
    static const void* const fn[] = {reinterpret_cast<const void*>(&k_sample<P, KIND, D + 1, true, HM>)...};
    return fn[d - 1];
}

template <int KIND>
constexpr int kSetsDim = sets_dim(KIND);

// d in (kExactDim, 64] but for the buckets' own: guarded, sets of one only
template <class P, int KIND, int HM, int DMAX>
static const void* guarded_fn()
{
    return reinterpret_cast<const void*>(&k_sample<P, KIND, DMAX, false, (HM > kHistSets1 ? kHistSets1 : HM)>);
}

template <class P, int KIND, int HM, int DMAX>
static const void* whole_fn()
{
    // the FP64 discontinuous integrand's constants do not fit the registers
    // beyond d = 24: without guards, the kernels spilled them in the loop
    if constexpr (P::is64 && KIND == GENZ_DISC && DMAX > 24)
        return guarded_fn<P, KIND, HM, DMAX>();
    else
        return reinterpret_cast<const void*>(&k_sample<P, KIND, DMAX, true, (DMAX > kSetsDim<KIND> && HM > kHistSets1 ? kHistSets1 : HM)>);
}

template <class P, int KIND, int HM>
static const void* sample_fn(int d)
{
    if (d <= kExactDim) return exact_fn<P, KIND, HM>(d, typename MakeIntSeq<kExactDim>::type());
    switch (dim_bucket(d)) {
    case 24: return d == 24 ? whole_fn<P, KIND, HM, 24>() : guarded_fn<P, KIND, HM, 24>();
    case 32: return d == 32 ? whole_fn<P, KIND, HM, 32>() : guarded_fn<P, KIND, HM, 32>();
    case 48: return d == 48 ? whole_fn<P, KIND, HM, 48>() : guarded_fn<P, KIND, HM, 48>();
    default: return d == 64 ? whole_fn<P, KIND, HM, 64>() : guarded_fn<P, KIND, HM, 64>();
    }
}

#define VEGAS_PART_NAME2(p, k) sample_fn_##p##_##k
#define VEGAS_PART_NAME(p, k) VEGAS_PART_NAME2(p, k)
const void* VEGAS_PART_NAME(VEGAS_SAMPLE_PREC, VEGAS_SAMPLE_KIND)(int d, int hm)
{
    using P = pick_type<VEGAS_SAMPLE_PREC == 64, P64, P32>::type;
    switch (hm) {
    case kHistNone: return sample_fn<P, VEGAS_SAMPLE_KIND, kHistNone>(d);
    case kHistSets1: return sample_fn<P, VEGAS_SAMPLE_KIND, kHistSets1>(d);
    case kHistSets2: return sample_fn<P, VEGAS_SAMPLE_KIND, kHistSets2>(d);
    default: return sample_fn<P, VEGAS_SAMPLE_KIND, kHistSets4>(d);
    }
}

#else

// The histogram mode of a launch.  Sets of two or four take the place of
// conflicting replicas where 8 or 4 of them are used (in practice where 16
// exceed the LDS, d N > 1150 or so), the kernel is one of those that can, and
// the last set's padding fits.
static int hist_mode(int prec, int kind, int d, int N, int rep, bool hist)
{
    if (!hist) return kHistNone;
    const bool whole = d == dim_bucket(d) && d <= sets_dim(kind);
    const int gl = !whole ? 0 : rep == 8 && d >= 2 ? 1 : rep == 4 && d >= 4 ? 2 : 0;
    return gl > 0 && lds_bytes(prec, kind, d, N, rep, gl) + red_bytes(2) <= kLdsLimit ? 1 + gl : kHistSets1;
}

static const void* sample_kernel(int prec, int kind, int d, int hm)
{
    static const SampleFn f64[] = {sample_fn_64_0, sample_fn_64_1, sample_fn_64_2, sample_fn_64_3};
    static const SampleFn f32[] = {sample_fn_32_0, sample_fn_32_1, sample_fn_32_2, sample_fn_32_3};
    return (prec == FP64 ? f64 : f32)[kind](d, hm);
}

#define VEGAS_DMAX_SWITCH(DM, CALL)            \
    switch (DM) {                              \
    case 4: { constexpr int D_ = 4; CALL; }    \
    case 8: { constexpr int D_ = 8; CALL; }    \
    case 16: { constexpr int D_ = 16; CALL; }  \
    case 32: { constexpr int D_ = 32; CALL; }  \
    default: { constexpr int D_ = 64; CALL; }  \
    }

// The records' kernel guards every dimension.
static int dump_bucket(int d)
{
    return d <= 4 ? 4 : d <= 8 ? 8 : d <= 16 ? 16 : d <= 32 ? 32 : 64;
}

template <class P, int KIND>
static const void* dump_fn(int d)
{
    VEGAS_DMAX_SWITCH(dump_bucket(d), return reinterpret_cast<const void*>(&k_dump<P, KIND, D_>))
}

template <class P>
static const void* dump_fn_kind(int kind, int d)
{
    switch (kind) {
    case GAUSS: return dump_fn<P, GAUSS>(d);
    case BIMODAL: return dump_fn<P, BIMODAL>(d);
    case GENZ_DISC: return dump_fn<P, GENZ_DISC>(d);
    default: return dump_fn<P, GENZ_PEAK>(d);
    }
}

template <class P, int... D>
static const void* adjoint_exact(int d, IntSeq<D...>)
{
    static const void* const fn[] = {reinterpret_cast<const void*>(&k_adjoint<P, D + 1, true>)...};
    return fn[d - 1];
}

template <class P, int... D>
static const void* grad_exact(int d, IntSeq<D...>)
{
    static const void* const fn[] = {reinterpret_cast<const void*>(&k_sample_grad<P, D + 1, true>)...};
    return fn[d - 1];
}

template <class P>
static const void* adjoint_fn(int d)
{
    switch (dim_bucket(d)) {
    case 24:
        return d == 24 ? reinterpret_cast<const void*>(&k_adjoint<P, 24, true>)
                       : reinterpret_cast<const void*>(&k_adjoint<P, 24, false>);
    case 32:
        return d == 32 ? reinterpret_cast<const void*>(&k_adjoint<P, 32, true>)
                       : reinterpret_cast<const void*>(&k_adjoint<P, 32, false>);
    case 48:
        return d == 48 ? reinterpret_cast<const void*>(&k_adjoint<P, 48, true>)
                       : reinterpret_cast<const void*>(&k_adjoint<P, 48, false>);
    case 64:
        return d == 64 ? reinterpret_cast<const void*>(&k_adjoint<P, 64, true>)
                       : reinterpret_cast<const void*>(&k_adjoint<P, 64, false>);
    default: return adjoint_exact<P>(d, typename MakeIntSeq<kExactDim>::type());
    }
}

template <class P>
static const void* sample_grad_fn(int d)
{
    switch (dim_bucket(d)) {
    case 24:
        return d == 24 ? reinterpret_cast<const void*>(&k_sample_grad<P, 24, true>)
                       : reinterpret_cast<const void*>(&k_sample_grad<P, 24, false>);
    case 32:
        return d == 32 ? reinterpret_cast<const void*>(&k_sample_grad<P, 32, true>)
                       : reinterpret_cast<const void*>(&k_sample_grad<P, 32, false>);
    case 48:
        return d == 48 ? reinterpret_cast<const void*>(&k_sample_grad<P, 48, true>)
                       : reinterpret_cast<const void*>(&k_sample_grad<P, 48, false>);
    case 64:
        return d == 64 ? reinterpret_cast<const void*>(&k_sample_grad<P, 64, true>)
                       : reinterpret_cast<const void*>(&k_sample_grad<P, 64, false>);
    default: return grad_exact<P>(d, typename MakeIntSeq<kExactDim>::type());
    }
}

hipError_t launch_sample_grad(int prec, const SampleArgs& a, double* gpart, int blocks, int threads, hipStream_t s)
{
    const void* fn = prec == FP64 ? sample_grad_fn<P64>(a.d) : sample_grad_fn<P32>(a.d);
    const size_t tab = size_t(a.d) * a.N * tab_entry_bytes(prec, GAUSS);
    const size_t lds = ((tab + 127) & ~size_t(127)) + red_bytes(2 + dim_bucket(a.d) + 1);
    void* args[] = {const_cast<SampleArgs*>(&a), &gpart};
    return hipLaunchKernel(fn, dim3(blocks), dim3(threads), args, lds, s);
}

size_t sample_data(int prec, int kind, int d, int N, int rep, bool hist)
{
    const int hm = hist_mode(prec, kind, d, N, rep, hist);
    return lds_bytes(prec, kind, d, N, hist ? rep : 0, hm > kHistSets1 ? hm - 1 : 0);
}

bool sample_in_sets(int prec, int kind, int d, int N, int rep)
{
    return hist_mode(prec, kind, d, N, rep, true) > kHistSets1;
}

hipError_t launch_sample(int prec, int kind, const SampleArgs& a, int blocks, int threads, hipStream_t s)
{
    const bool hist = a.hist != 0;
    const int rep = 1 << a.hrep_log2;
    const void* fn = sample_kernel(prec, kind, a.d, hist_mode(prec, kind, a.d, a.N, rep, hist));
    void* args[] = {const_cast<SampleArgs*>(&a)};
    const size_t lds = with_sums(sample_data(prec, kind, a.d, a.N, rep, hist));
    return hipLaunchKernel(fn, dim3(blocks), dim3(threads), args, lds, s);
}

hipError_t launch_dump(int prec, int kind, const DumpArgs& a, hipStream_t s)
{
    const void* fn = prec == FP64 ? dump_fn_kind<P64>(kind, a.d) : dump_fn_kind<P32>(kind, a.d);
    const size_t tab = size_t(a.d) * a.N * tab_entry_bytes(prec, kind);
    const size_t lds = tab;
    uint64_t blocks = (a.n + kBlock - 1) / kBlock;
    if (blocks > 1024) blocks = 1024;
    if (blocks == 0) blocks = 1;
    void* args[] = {const_cast<DumpArgs*>(&a)};
    return hipLaunchKernel(fn, dim3(unsigned(blocks)), dim3(kBlock), args, lds, s);
}

hipError_t launch_adjoint(int prec, const AdjointArgs& a, int blocks, hipStream_t s)
{
    const void* fn = prec == FP64 ? adjoint_fn<P64>(a.d) : adjoint_fn<P32>(a.d);
    const size_t tab = size_t(a.d) * a.N * tab_entry_bytes(prec, GAUSS);
    const size_t lds = ((tab + 15) & ~size_t(15)) + red_bytes(dim_bucket(a.d) + 1);
    void* args[] = {const_cast<AdjointArgs*>(&a)};
    hipError_t e = hipLaunchKernel(fn, dim3(blocks), dim3(kBlock), args, lds, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_adjoint_merge, dim3(a.d + 1), dim3(64), 0, s, a, blocks);
    return hipGetLastError();
}

int sample_max_blocks_per_cu(int prec, int kind, int d, int N, int threads, int rep)
{
    int n = 0;
    const void* fn = sample_kernel(prec, kind, d, hist_mode(prec, kind, d, N, rep, true));
    hipFuncAttributes at;
    if (hipFuncGetAttributes(&at, fn) == hipSuccess && threads > at.maxThreadsPerBlock) return 0;  // not launchable
    const size_t lds = with_sums(sample_data(prec, kind, d, N, rep, true));
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, threads, lds) != hipSuccess) return 1;
    return n > 0 ? n : 1;
}

#endif  // VEGAS_SAMPLE_PREC

}  // namespace vegas
