// Event and dump kernels for an integrand compiled at run time from the
// caller's source (the paper's route for integrands written in C, C++ or GPU
// code and linked into the integrator, sec. 2.3).  This header is not built
// with the library: the host hands it, with vegas_internal.hpp and
// device_common.hpp, to the runtime compiler once per context, after the
// caller's source, with
//   VEGAS_DIM      the dimension d (a compile-time constant, so the point
//                  stays in registers and the caller's loops unroll),
//   VEGAS_THREADS  the largest block the event kernel is launched with,
//   VEGAS_FP32     defined for an FP32-mixed context,
// and vegas_real typedef'd to float (FP32-mixed) or double (FP64).  The
// caller's source defines
//   __device__ vegas_real vegas_integrand(const vegas_real* x, int dim, const double* params)
// evaluated at the mapped point x[0..d-1] in [0,1)^d; params is the context's
// parameter array in device memory.
//
// Everything but the integrand is the built-in event kernel's path in the
// context's precision: the same Philox words, exact bins, map and Jacobian
// N^d prod W_b, the same grouped-Kahan FP64 sums of v = f w and v^2, and the
// same per-dimension, per-bin FP64 histograms of v^2 (LDS replicas, then the
// block's histogram added into slot (blockIdx / 8) mod kHistSlots), so the
// reduction, refinement and combination kernels of the library serve it
// unchanged.
#pragma once

#include "device_common.hpp"

namespace vegas {
namespace user {

constexpr int D = VEGAS_DIM;
static_assert(D >= 1 && D <= kMaxDim, "VEGAS_DIM out of range");

// Binning constants and the LDS address of each dimension's table (scalars the
// compiler cannot split, as in the built-in kernels).
struct MapConsts {
    BinConsts bc;
    uint32_t base[D];

    __device__ __forceinline__ MapConsts(int N, uint32_t tab, int entry_log2)
    {
        bc.mul = uint32_t(N);
        bc.add = uint32_t(N) >> 1;
        bc.h64 = (N & 1) ? 0x1p-33 : 0.0;
#pragma unroll
        for (int i = 0; i < D; ++i) base[i] = __builtin_amdgcn_readfirstlane(tab + (uint32_t(i * N) << entry_log2));
    }
};

#ifdef VEGAS_FP32
// FP32-mixed context.  The table is the built-in FP32 one with centre 0:
// entry (RN32((E_b + h W / 2^32) S), RN32(W) 2^ws), S = 2^(ws + 32), so
// x S = fma(RN32(lo), W 2^ws, first entry) in FP32 and x = (x S) / S exactly;
// the width product is kept in FP32 with its binary exponent moved out every
// 8 dimensions, and the value f w = 2^ew (f wp) C is formed in FP64.
using tab_t = float2;
using map_real = float;
constexpr int kEntryLog2 = 3;
#else
// FP64 context: x_i = fma(lo, W, E_b + h W), W the bin's width times 2^-32, the
// built-in FP64 map with centre 0; the width product takes 2^32 per dimension,
// ahead of its width.
using tab_t = double2;
using map_real = double;
constexpr int kEntryLog2 = 4;
#endif

struct Event {
    uint32_t off[D];   // LDS address of each dimension's table entry
    map_real del[D];   // lo (FP32: RN32(lo))
    map_real x[D];
    map_real wp;
    int ew;            // FP32: binary exponent moved out of wp

    __device__ __forceinline__ void run(const MapConsts& mc, uint64_t e, uint32_t t, uint32_t ctr3, uint32_t key0,
                                        uint32_t key1, float ds)
    {
#pragma clang fp contract(off)
        const uint32_t elo = uint32_t(e), ehi = uint32_t(e >> 32);
#ifdef VEGAS_FP32
        float w = 1.0f;
#else
        double w = 1.0;
#pragma unroll
        for (int i = 0; i < width_start(D <= 24, D); i += 32) w *= 0x1p32;
#endif
        int ewl = 0;
#pragma unroll
        for (int g = 0; g < (D + 3) / 4; ++g) {
            const U4 k = philox4x32_10(elo, ehi, t, ctr3 + uint32_t(g), key0, key1);
#ifndef VEGAS_FP32
            if (D > 24 && g >= kWidthGroups && 4 * g + 4 <= D) w *= 0x1p128;
#endif
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * g + q;
                if (i < D) {
                    int bi;
                    uint32_t lo;
                    bin_words(k.w[q], mc.bc, bi, lo);
                    const lds_ptr<const tab_t> p = entry_of<tab_t>(bi, mc.base[i]);
                    off[i] = uint32_t(uint64_t(p));
                    const tab_t tb = *(const tab_t*)p;
                    del[i] = map_real(lo);
#ifdef VEGAS_FP32
                    x[i] = fmaf(del[i], tb.y, tb.x) * ds;
#else
                    x[i] = fma(del[i], tb.y, tb.x);
#endif
                    w *= tb.y;
                }
            }
#ifdef VEGAS_FP32
            if ((g & 1) == 1 && 4 * g + 4 < D) {
                int e2;
                w = frexpf(w, &e2);
                ewl += e2;
            }
#endif
        }
        wp = w;
        ew = ewl;
    }
    __device__ __forceinline__ int bin(int i, const MapConsts& mc) const { return int((off[i] - mc.base[i]) >> kEntryLog2); }
    __device__ __forceinline__ double delta(int i, const MapConsts& mc) const { return double(del[i]) * 0x1p-32 + mc.bc.h64; }
#ifdef VEGAS_FP32
    __device__ __forceinline__ double weight(double Cw) const { return ldexp(double(wp), ew) * Cw; }
    __device__ __forceinline__ double value(float f, double C) const
    {
#pragma clang fp contract(off)
        return ldexp(double(f) * double(wp), ew) * C;  // the product of two floats is exact in FP64
    }
#else
    __device__ __forceinline__ double weight(double Cw) const { return wp * Cw; }
    __device__ __forceinline__ double value(double f, double C) const
    {
#pragma clang fp contract(off)
        return f * wp * C;
    }
#endif
};

// 2^-(ws + 32): the FP32 map's scale back to x (unused in FP64)
__device__ __forceinline__ float map_scale(const DevConst* c) { return ldexpf(c->dscale32, -32); }

// LDS: table [d][N] (128-byte aligned), histogram [d][N][rep] (HIST only),
// then the block reduction's wave partials.
template <bool HIST>
__device__ __forceinline__ void sample(const SampleArgs& a, const double* __restrict__ params)
{
    extern __shared__ __align__(128) unsigned char smem[];
    const int N = a.N;
    const int dN = D * N;
    const size_t tab_bytes = (size_t(dN) * sizeof(tab_t) + 127) & ~size_t(127);
    const int rl2 = a.hrep_log2, rep = 1 << rl2;
    const size_t hist_bytes = HIST ? size_t(dN) * rep * sizeof(double) : 0;
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    double* hist = reinterpret_cast<double*>(smem + tab_bytes);
    double* red = reinterpret_cast<double*>(smem + tab_bytes + hist_bytes);
    const uint32_t ltab = lds_address(smem);
    const HistAdder<kEntryLog2> hadd(ltab, ltab + uint32_t(tab_bytes), rl2);
    const MapConsts mc(N, ltab, kEntryLog2);

    const tab_t* gtab = static_cast<const tab_t*>(a.tab);
    for (int k = threadIdx.x; k < dN; k += blockDim.x) tab[k] = gtab[k];
    if constexpr (HIST)
        for (int k = threadIdx.x; k < dN * rep; k += blockDim.x) hist[k] = 0.0;
    const double C = a.cst->C;  // N^d (scaled, see DevConst)
    const float ds = map_scale(a.cst);
    __syncthreads();

    double s1 = 0.0, c1 = 0.0, s2 = 0.0, c2 = 0.0;
    double g1 = 0.0, g2 = 0.0;
    int ng = 0;
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    const uint64_t end = a.e0 + a.n;
    for (uint64_t e = a.e0 + uint64_t(threadIdx.x) * gridDim.x + blockIdx.x; e < end; e += stride) {
        Event ev;
        ev.run(mc, e, a.t, a.ctr3, a.key0, a.key1, ds);
        const vegas_real f = vegas_integrand(ev.x, D, params);
        double v, v2;
        {
#pragma clang fp contract(off)
            v = ev.value(f, C);
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
        if constexpr (HIST) hadd.template add<D, true>(ev.off, D, v2);
    }
    kahan_add(s1, c1, g1);
    kahan_add(s2, c2, g2);

    // block_sums synchronises, which also completes every histogram atomic
    const double v12[2] = {s1 - c1, s2 - c2};
    const double S = block_sums(v12, red);
    if (threadIdx.x < 2) a.partials[size_t(blockIdx.x) * 2 + threadIdx.x] = S;
    if constexpr (HIST) {
        double* slot = a.hslots + size_t((blockIdx.x >> 3) % kHistSlots) * dN;
        for (int k = threadIdx.x; k < dN; k += blockDim.x) atomicAdd(&slot[k], replica_sum(hist, k, rl2));
    }
}

}  // namespace user
}  // namespace vegas

extern "C" __global__ __launch_bounds__(VEGAS_THREADS) void vegas_user_sample(vegas::SampleArgs a,
                                                                              const double* __restrict__ params)
{
    vegas::user::sample<true>(a, params);
}

extern "C" __global__ __launch_bounds__(VEGAS_THREADS) void vegas_user_sample_nohist(vegas::SampleArgs a,
                                                                                     const double* __restrict__ params)
{
    vegas::user::sample<false>(a, params);
}

// Per-event records b[d], delta[d], x[d], w, f (w = N^d prod W_b), widened
// to FP64, one event per thread; LDS holds the table.
extern "C" __global__ __launch_bounds__(256) void vegas_user_dump(vegas::DumpArgs a, const double* __restrict__ params)
{
    using namespace vegas;
    constexpr int D = user::D;
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = a.N;
    using tab_t = user::tab_t;
    tab_t* tab = reinterpret_cast<tab_t*>(smem);
    const tab_t* gtab = static_cast<const tab_t*>(a.tab);
    for (int k = threadIdx.x; k < D * N; k += blockDim.x) tab[k] = gtab[k];
    __syncthreads();
    const user::MapConsts mc(N, lds_address(smem), user::kEntryLog2);
    const double Cw = a.cst->Cw;
    const float ds = user::map_scale(a.cst);
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < a.n; k += stride) {
        user::Event ev;
        ev.run(mc, a.e0 + k, a.t, a.ctr3, a.key0, a.key1, ds);
        double* row = a.out + k * size_t(3 * D + 2);
#pragma unroll
        for (int i = 0; i < D; ++i) {
            row[i] = double(ev.bin(i, mc));
            row[D + i] = ev.delta(i, mc);
            row[2 * D + i] = double(ev.x[i]);
        }
        row[3 * D] = ev.weight(Cw);
        row[3 * D + 1] = double(vegas_integrand(ev.x, D, params));
    }
}
