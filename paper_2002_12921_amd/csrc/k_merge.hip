// Reduction, statistics and refinement kernels of one Vegas iteration.
//
// k_merge reduces what the event kernel left: the per-block rows (S1, S2), in a
// fixed order, and the kHistSlots histogram accumulators.  Block 0 adds the
// rows, folds them into the iteration's double-double accumulator (several
// chunks form one iteration) and, at its end, records the statistics; at the
// end block 1+i adds dimension i's slots in order, clears them, records the row
// and, when asked, refines the dimension's grid; with MERGE_GRAD, block
// d+1+j sums column j of the gradient rows.  No block waits for another and no
// device-wide fence is needed: the next kernel on the stream sees the result.
//
// What bounds it is latency: a launch, a round trip to memory, the sums'
// dependent steps.  So everything a block needs is read at its start, in one
// round; sums and scans across a wave go through DPP (an exchange through the
// LDS crossbar waits some 130 cycles, and a refinement made 30 of them, a
// statistics block 14); and blocks are 256 threads, as many as N <= 255 bins
// need.  (Behind a finished kernel even an empty one takes 4 us; alone, the d = 8
// reduction with refinement takes 2.0 us, 3.2 with crossbar exchanges and
// 1024-thread blocks; 3 iterations of 2000 events with a wait: 37 -> 31 us.)
// It stays a kernel of its own: counting the event kernel's blocks to let the
// last one reduce takes a release, an acquire and an atomic on one address in
// every block, which alone made that kernel 4 us longer at 1e5 events, 7 at 1e6.
#include <cstring>

#include "grid_ops.hpp"

namespace vegas {

constexpr int kSlotThreads = 256;

// S1, S2: waves 0 and 2 take the rows' S1, waves 1 and 3 their S2, half of the
// rows each.
__device__ static void merge_sums(const MergeArgs& a)
{
    __shared__ double ps[4], pc[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool begin = a.flags & MERGE_BEGIN, end = a.flags & MERGE_END;
    // the accumulator and the counts, read while the rows are
    PriorCounts prior{};
    double hi0 = 0.0, lo0 = 0.0;
    if (wave == 0) {
        if (end && !(a.flags & MERGE_NO_RECORD)) prior = {a.result->n_events, a.result->n_nonfinite};
        if (!begin && lane < 2) {
            hi0 = a.acc[lane];
            lo0 = a.acc[a.pstride + lane];
        }
    }
    double s = 0.0, c = 0.0;
    for (int r0 = (wave >> 1) * 64 + lane; r0 < a.rows; r0 += 128 * 4) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = r0 + 128 * u < a.rows ? a.partials[size_t(r0 + 128 * u) * 2 + (wave & 1)] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) twosum_add(s, c, v[u]);
    }
    wave_pair_sum_last(s, c);
    if (lane == 63) {
        ps[wave] = s;
        pc[wave] = c;
    }
    __syncthreads();
    if (wave != 0) return;
    double v = 0.0;
    if (lane < 2) {
        double t = ps[lane], e = pc[lane];
        twosum_add(t, e, ps[lane + 2]);
        e += pc[lane + 2];
        const double val = t + e;
        double hi = val, lo = 0.0;
        if (!begin) {  // double-double accumulation across chunks
            hi = hi0;
            lo = lo0;
            twosum_add(hi, lo, val);
        }
        a.acc[lane] = hi;
        a.acc[a.pstride + lane] = lo;
        v = hi + lo;
        if (end) a.last[lane] = v;
    }
    if (!end) return;
    const double S2 = lane_value(v, 1);
    if (lane == 0) finish_iteration(a, v, S2, prior);
}

// Dimension i at the end of an iteration: its slots' sum, and the refinement.
__device__ static void merge_slots(const MergeArgs& a, int i)
{
    const int t = threadIdx.x, N = a.N;
    double* last = a.last + 2 + size_t(i) * N;
    if (a.flags & MERGE_NO_HIST) {  // an iteration without histograms: its row reads zero
        if (t < N) last[t] = 0.0;
        return;
    }
    __shared__ double fin[kMaxBins + 1], Eo[kMaxBins + 1];
    const bool refine = a.flags & MERGE_REFINE;
    if (N <= 64 && t >= 64) return;  // one wave does it all
    const double* E = a.edges + size_t(i) * (N + 1);
    const double Eb = refine && t <= N ? E[t] : 0.0;
    const double Eb1 = refine && t < N ? E[t + 1] : 0.0;
    double mine = 0.0;
    if (t < N) {
        const size_t dN = size_t(a.d) * N;
        double* h = a.hslots + size_t(i) * N + t;
        double v[kHistSlots];
#pragma unroll
        for (int q = 0; q < kHistSlots; ++q) v[q] = h[q * dN];
#pragma unroll
        for (int q = 0; q < kHistSlots; ++q) {
            mine += v[q];
            h[q * dN] = 0.0;
        }
        last[t] = mine;
    }
    if (!refine) return;
    if (N <= 64) {
        refine_dim_wave(a, i, mine, Eb, Eb1);
        return;
    }
    fin[t] = mine;
    Eo[t] = Eb;
    __syncthreads();
    refine_dim(a, i, fin, Eo);
}

__global__ __launch_bounds__(kSlotThreads) void k_merge(MergeArgs a)
{
    const int g = blockIdx.x;
    if (g == 0)
        merge_sums(a);
    else if (g <= a.d)
        merge_slots(a, g - 1);
    else if (threadIdx.x < 64)  // MERGE_GRAD: a column of the gradient rows, scaled by 1/M
        adjoint_merge_column(a.gpart, a.rows, a.d, g - a.d - 1, 1.0 / a.M, a.grad_out, 0);
}

// grad = gout * G, rounded once to the output's precision.
__global__ void k_grad_scale(const double* G, const double* gout, void* grad, int n, int grad_fp32)
{
    const double s = *gout;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const double g = s * G[j];
        if (grad_fp32)
            static_cast<float*>(grad)[j] = float(g);
        else
            static_cast<double*>(grad)[j] = g;
    }
}

// Stand-alone refinement from the stored histograms of the last iteration.
__global__ __launch_bounds__(kSlotThreads) void k_refine(MergeArgs a)
{
    __shared__ double h[kMaxBins], Eo[kMaxBins + 1];
    const int i = blockIdx.x;
    for (int b = threadIdx.x; b < a.N; b += blockDim.x) h[b] = a.last[2 + size_t(i) * a.N + b];
    for (int b = threadIdx.x; b <= a.N; b += blockDim.x) Eo[b] = a.edges[size_t(i) * (a.N + 1) + b];
    __syncthreads();
    refine_any(a, i, h, Eo);
}

// Derived constants of the integrand (see DevConst), by a block of at least 64
// threads: thread i < kMaxDim those of dimension i, and its factor of the
// normalisation; thread 0 then the product over the dimensions, in order.  (By
// one thread the stores of the 64 dimensions and the functions of each
// dimension followed one another: k_set_params at d = 8 took 5.4 us, now 3.1.)
__device__ static void prepare_consts(int prec, int kind, int d, int N, const double* __restrict__ q,
                                      DevConst* __restrict__ c)
{
    __shared__ double factor[kMaxDim];
    const double log2e = 1.4426950408889634074;
    const int i = threadIdx.x;
    bool no_exponent = false;
    if (i < kMaxDim) {
        double p1 = 0.0, p2 = 0.0, cA = 0.0, cB = 0.0, f = 1.0;
        float p1f = 0.0f;
        if (i < d) {
            table_centres(kind, d, i, q, cA, cB);
            if (kind == GAUSS || kind == BIMODAL) {
                p1 = q[1 + i];
                if (kind == BIMODAL) p2 = q[1 + d + i] - q[1 + i];  // FP64 map: u_B = u_A - (muB - muA)
            } else if (kind == GENZ_DISC) {
                // nu exp(sum c x) = [nu e^{sum c a}] exp(sum c (x - a)); per dimension
                // nu e^{c a} = c / (e^{c (1 - a)} - 1)
                const double cc = q[i], aa = q[d + i];
                f = cc / expm1(cc * (1.0 - aa));
                p1 = cc;
                p2 = aa;
            } else if (kind == GENZ_PEAK) {
                // nu prod 1/(c^-2 + u^2) = [nu prod c^2] prod 1/(1 + c^2 u^2)
                const double cc = q[i], aa = q[d + i];
                f = cc / (atan(cc * (1.0 - aa)) + atan(cc * aa));
                p1 = cc * cc;
                p2 = aa;
                p1f = float(cc * cc);
            }
        }
        c->p1_64[i] = p1;
        c->p2_64[i] = p2;
        c->cA64[i] = cA;
        c->cB64[i] = cB;
        c->p1_32[i] = p1f;
        factor[i] = f;
        // an exponent that is not a number, which the exponential's cut would
        // hide: a parameter is not, infinity less infinity (u_B = u_A - (muB -
        // muA)), or a square beyond the range over an infinite width
        no_exponent = p1 != p1 || p2 != p2 || (kind == BIMODAL && isinf(p1));
        if ((kind == GAUSS || kind == BIMODAL) && i < d) {
            const double ka = 1.0 / (q[0] * q[0]), A = cA * cA * d * ka, B = cB * cB * d * ka;
            no_exponent = no_exponent || A != A || B != B;
        }
        // (e^(c (1 - a)) is beyond the range from 710 on, and the constant 0: infinity times 0)
        if (kind == GENZ_DISC && i < d) no_exponent = no_exponent || p1 * (1.0 - p2) > 1e6;
    }
    const bool bad = __syncthreads_or(no_exponent);
    if (threadIdx.x != 0) return;
    c->n_bins = N;
    c->pad1 = 0;
    c->dscale32 = width_scale32(N);
    const int ws = int(rint(log2(double(N))));
    // the constants every event is multiplied by, as sums of two (an error here
    // does not average out): N^d and the normalisation
    const auto times = [](double& hi, double& lo, double f) {
        const double p = hi * f;
        lo = fma(lo, f, fma(hi, f, -p));
        hi = p;
    };
    double nd = 1.0, nd_lo = 0.0, Cf = 1.0, Cf_lo = 0.0;
    for (int k = 0; k < d; ++k) times(nd, nd_lo, double(N));
    const int shift = prec == FP64 ? 0 : -ws * d;
    const double Cw = ldexp(nd, shift), Cw_lo = ldexp(nd_lo, shift);
    double kexp64 = 0.0, kexp2_64 = 0.0, inv_a = 0.0;
    float ka32 = 0.0f;
    if (kind == GAUSS || kind == BIMODAL) {
        const double a = q[0], sqrt_pi = 0x1.c5bf891b4ef6bp+0, sqrt_pi_lo = -0x1.618f13eb7ca89p-54;
        const double x = a * sqrt_pi, r = fma(a, sqrt_pi, -x) + a * sqrt_pi_lo;
        Cf = pow(x, double(-d));
        if (kind == BIMODAL) Cf = 0.5 * Cf;
        Cf_lo = Cf * (double(-d) * (r / x));
        kexp64 = 1.0 / (a * a);
        kexp2_64 = log2e / (a * a);
        inv_a = 1.0 / a;
        ka32 = float(1.0 / (a * a));
    } else {
        if (kind == GENZ_DISC) kexp2_64 = log2e;
        // (a user integrand carries its own normalisation: C = N^d)
        if (kind != USER)
            for (int k = 0; k < d; ++k) times(Cf, Cf_lo, factor[k]);
    }
    double C = Cf * Cw;
    const double rest = fma(Cf, Cw, -C) + (Cf * Cw_lo + Cf_lo * Cw);
    if (fabs(rest) < fabs(C)) C += rest;  // (not beyond the range of the parts)
    if (fabs(Cf_lo) < fabs(Cf)) Cf += Cf_lo;
    c->Cw = Cw;
    c->kexp64 = kexp64;
    c->kexp2_64 = kexp2_64;
    c->inv_a = inv_a;
    c->pad2 = 0.0f;
    c->ka32 = ka32;
    c->pad0 = 0.0f;
    c->Cf = Cf;
    c->C = C;
    int e = 0;
    double m = frexp(C, &e);
    if (e > 1021) {
        m = ldexp(m, e - 1021);
        e = 1021;
    }
    c->mant = m;
    c->magic = bad ? __builtin_nan("") : 0x1.8p52 + double(e);
}

__global__ void k_prepare(int prec, int kind, int d, int N, const double* __restrict__ q,
                          DevConst* __restrict__ c)
{
    prepare_consts(prec, kind, d, N, q, c);
}

// New integrand parameters in one launch (block i: dimension i): every block
// reads the caller's n values (FP64, or FP32 widened exactly), block 0 stores
// them and the derived constants, and each block rebuilds its dimension's
// tables (whose FP32 entries are offsets from the parameters' centres) with
// the centres taken from the parameters themselves, so no block waits for
// another.
__global__ __launch_bounds__(256) void k_set_params(int prec, int kind, int d, int N, const void* __restrict__ src,
                                                    const void* __restrict__ rest, int n, int is_fp32, ProblemPtrs p)
{
    __shared__ double q[kMaxParams];
    const int i = blockIdx.x, b = threadIdx.x;
    // the block's edges, read beside the parameters (N <= 255: a bin per thread)
    const double* E = p.edges + size_t(i) * (N + 1);
    const double lo = E[min(b, N)], hi = E[min(b + 1, N)];
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        // value k: src[k], or with rest given, src[0] and rest[k - 1]
        const void* a = rest && k > 0 ? rest : src;
        const int j = rest && k > 0 ? k - 1 : k;
        q[k] = is_fp32 ? double(static_cast<const float*>(a)[j]) : static_cast<const double*>(a)[j];
    }
    __syncthreads();
    if (i == 0) {
        for (int k = threadIdx.x; k < n; k += blockDim.x) p.params[k] = q[k];
    }
    double cA, cB;
    table_centres(kind, d, i, q, cA, cB);
    const float ds = width_scale32(N);
    if (b < N) write_table_entry(i, b, lo, hi, cA, cB, ds, kind, N, p.tab64, p.tab32);
    if (kind == GENZ_DISC && threadIdx.x < 64) {
        const uint64_t T = disc_threshold_wave(E, N, cA);
        if (threadIdx.x == 0) p.thr[i] = T;
    }
    if (i == 0) prepare_consts(prec, kind, d, N, q, p.cst);
}

// Uniform grid E_k = k/N and a clean state (tables: k_build_tables).
__global__ void k_init_state(ProblemPtrs p, int d, int N, int pstride)
{
    const int i = blockIdx.x;
    if (i < d) {
        double* E = p.edges + size_t(i) * (N + 1);
        for (int k = threadIdx.x; k <= N; k += blockDim.x) E[k] = double(k) / double(N);
        return;
    }
    for (int k = threadIdx.x; k < 2 * pstride; k += blockDim.x) p.acc[k] = 0.0;
    for (int k = threadIdx.x; k < pstride; k += blockDim.x) p.last[k] = 0.0;
    for (int k = threadIdx.x; k < kHistSlots * (pstride - 2); k += blockDim.x) p.hslots[k] = 0.0;
    for (int k = threadIdx.x; k < 2 * kMaxRecords; k += blockDim.x) p.records[k] = 0.0;
    for (int k = threadIdx.x; k < kMaxRecords; k += blockDim.x) p.rec_flag[k] = 0;
    if (threadIdx.x == 0) {
        const double nan = __builtin_nan("");
        DevResult* R = p.result;
        R->integral = R->sigma = R->chi2_dof = R->last_integral = R->last_var = nan;
        R->n_iter = R->n_combined = R->n_events = R->n_nonfinite = 0;
    }
}

__global__ void k_zero(double* x, size_t n)
{
    for (size_t k = size_t(blockIdx.x) * blockDim.x + threadIdx.x; k < n; k += size_t(gridDim.x) * blockDim.x)
        x[k] = 0.0;
}

__global__ void k_build_tables(ProblemPtrs p, int kind, int N)
{
    const int i = blockIdx.x;
    write_tables(i, p.edges + size_t(i) * (N + 1), p.cst, kind, N, p.tab64, p.tab32, p.thr);
}

// host.to (may be null): pinned host memory the result block is written to as
// well, which saves the copy behind this kernel (a kernel's gap and a call).
__global__ __launch_bounds__(64) void k_combine(const double* records, const int32_t* rec_flag, int n_rec, DevResult* R,
                                                HostPost host)
{
    combine_records(records, rec_flag, n_rec, R, host);
}

// n values to pinned host memory, by one block, which then posts the mark. Every
// wave waits for its own writes to reach the host, so few are faster: edges of
// 404, 808 and 2020 values read from an idle context in 10.6, 11.0 and 11.9 us
// with 256 threads, 13.3, 14.9 and 16.4 with 1024; by a copy call 13.7, 13.9, 14.1.
__global__ __launch_bounds__(256) void k_copy_out(const double* __restrict__ src, int n, HostPost host)
{
    double* dst = static_cast<double*>(host.to);
    for (int k = threadIdx.x; k < n; k += blockDim.x) dst[k] = src[k];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) host_post(host);
}

// New edges of dimensions i0, i0 + 1, ... (block i: dimension i0 + i), carried
// by the launch itself: the edges, the tables and the threshold.
__global__ __launch_bounds__(256) void k_set_edges(EdgeValues v, int i0, ProblemPtrs p, int kind, int N)
{
    const int i = i0 + blockIdx.x;
    const double* E = v.e + size_t(blockIdx.x) * (N + 1);
    for (int k = threadIdx.x; k <= N; k += blockDim.x) p.edges[size_t(i) * (N + 1) + k] = E[k];
    write_tables(i, E, p.cst, kind, N, p.tab64, p.tab32, p.thr);
}

__global__ void k_reset_results(double* records, int32_t* rec_flag, DevResult* R)
{
    for (int k = threadIdx.x; k < 2 * kMaxRecords; k += blockDim.x) records[k] = 0.0;
    for (int k = threadIdx.x; k < kMaxRecords; k += blockDim.x) rec_flag[k] = 0;
    if (threadIdx.x == 0) {
        const double nan = __builtin_nan("");
        R->integral = R->sigma = R->chi2_dof = R->last_integral = R->last_var = nan;
        R->n_iter = R->n_combined = R->n_events = R->n_nonfinite = 0;
    }
}

__global__ void k_copy_last(const DevResult* R, double* out)
{
    if (threadIdx.x == 0) {
        out[0] = R->last_integral;
        out[1] = sqrt(R->last_var);
    }
}

// ---------------------------------------------------------------------------

hipError_t launch_merge(const MergeArgs& a, hipStream_t s)
{
    // blocks 1..d have work at the end of an iteration only
    const int blocks = (a.flags & MERGE_END) ? a.d + 1 + ((a.flags & MERGE_GRAD) ? a.d + 1 : 0) : 1;
    hipLaunchKernelGGL(k_merge, dim3(blocks), dim3(kSlotThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_grad_scale(const double* G, const double* gout, void* grad, int n, int grad_fp32, hipStream_t s)
{
    hipLaunchKernelGGL(k_grad_scale, dim3(1), dim3(128), 0, s, G, gout, grad, n, grad_fp32);
    return hipGetLastError();
}

hipError_t launch_refine(const MergeArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(k_refine, dim3(a.d), dim3(kSlotThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_prepare(int prec, int kind, int d, int N, const double* params, DevConst* cst,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_prepare, dim3(1), dim3(64), 0, s, prec, kind, d, N, params, cst);
    return hipGetLastError();
}

hipError_t launch_init_state(const ProblemPtrs& p, int d, int N, int pstride, hipStream_t s)
{
    hipLaunchKernelGGL(k_init_state, dim3(d + 1), dim3(256), 0, s, p, d, N, pstride);
    return hipGetLastError();
}

hipError_t launch_zero(double* x, size_t n, hipStream_t s)
{
    const unsigned blocks = unsigned(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024);
    hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, x, n);
    return hipGetLastError();
}

hipError_t launch_build_tables(const ProblemPtrs& p, int kind, int d, int N, hipStream_t s)
{
    hipLaunchKernelGGL(k_build_tables, dim3(d), dim3(256), 0, s, p, kind, N);
    return hipGetLastError();
}

hipError_t launch_combine(const double* records, const int32_t* rec_flag, int n_rec, DevResult* result,
                          const HostPost& host, hipStream_t s)
{
    hipLaunchKernelGGL(k_combine, dim3(1), dim3(64), 0, s, records, rec_flag, n_rec, result, host);
    return hipGetLastError();
}

hipError_t launch_copy_out(const double* src, int n, const HostPost& host, hipStream_t s)
{
    hipLaunchKernelGGL(k_copy_out, dim3(1), dim3(256), 0, s, src, n, host);
    return hipGetLastError();
}

static_assert(sizeof(EdgeValues) + sizeof(ProblemPtrs) + 64 <= 4096, "a launch's arguments");
hipError_t launch_set_edges(const double* host_edges, const ProblemPtrs& p, int kind, int d, int N, hipStream_t s)
{
    const int per = kEdgeValues / (N + 1);  // dimensions a launch carries
    for (int i0 = 0; i0 < d; i0 += per) {
        EdgeValues v;
        const int n = d - i0 < per ? d - i0 : per;
        std::memcpy(v.e, host_edges + size_t(i0) * (N + 1), sizeof(double) * size_t(n) * (N + 1));
        hipLaunchKernelGGL(k_set_edges, dim3(n), dim3(256), 0, s, v, i0, p, kind, N);
        const hipError_t he = hipGetLastError();
        if (he != hipSuccess) return he;
    }
    return hipSuccess;
}

hipError_t launch_set_params(int prec, int kind, int d, int N, const void* src, int n, int is_fp32,
                             const ProblemPtrs& p, hipStream_t s, const void* rest)
{
    hipLaunchKernelGGL(k_set_params, dim3(d), dim3(256), 0, s, prec, kind, d, N, src, rest, n, is_fp32, p);
    return hipGetLastError();
}

hipError_t launch_reset_results(double* records, int32_t* rec_flag, DevResult* result,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_reset_results, dim3(1), dim3(256), 0, s, records, rec_flag, result);
    return hipGetLastError();
}

hipError_t launch_copy_last(const DevResult* result, double* out2, hipStream_t s)
{
    hipLaunchKernelGGL(k_copy_last, dim3(1), dim3(64), 0, s, result, out2);
    return hipGetLastError();
}

}  // namespace vegas
