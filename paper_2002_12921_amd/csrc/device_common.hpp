// Device building blocks of the Vegas event kernels: Philox4x32-10, exact
// binning, the piecewise-linear map, the integrands and block reductions.
#pragma once

#include "vegas_internal.hpp"

namespace vegas {

// Type selection (std::conditional, which the runtime compiler lacks).
template <bool B, class T, class F>
struct pick_type {
    using type = T;
};
template <class T, class F>
struct pick_type<false, T, F> {
    using type = F;
};

// The integers 0..N-1 as a type (std::integer_sequence, likewise).
template <int... I>
struct IntSeq {};
template <int N, int... I>
struct MakeIntSeq {
    using type = typename MakeIntSeq<N - 1, N - 1, I...>::type;
};
template <int... I>
struct MakeIntSeq<0, I...> {
    using type = IntSeq<I...>;
};

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11, sec. 3.2): ten rounds of
// two 32x32->64 multiplies whose halves are XOR-mixed with the other words
// and the key; the key advances by the Weyl constants between rounds.  The
// key and counter words 2..3 are uniform across a wave, so the key schedule
// stays in scalar registers.  Each 64-bit product is one v_mad_u64_u32 and
// each three-way XOR one v_bitop3_b32 (truth table 0x96 = a ^ b ^ c).
struct U4 {
    uint32_t w[4];
};

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                            uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = uint64_t(c0) * 0xD2511F53u;
        const uint64_t p1 = uint64_t(c2) * 0xCD9E8D57u;
        const uint32_t n0 = xor3(uint32_t(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3(uint32_t(p0 >> 32), c3, k1);
        c1 = uint32_t(p1);
        c3 = uint32_t(p0);
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    U4 o;
    o.w[0] = c0;
    o.w[1] = c1;
    o.w[2] = c2;
    o.w[3] = c3;
    return o;
}

// ---------------------------------------------------------------------------
// Precision policies and grid-table entry types.
//
// FP64: delta = (lo + h)/2^32 (see bin_words) is never formed.  With the width
//   scaled, W = (E_{b+1} - E_b) 2^-32, the table entry is (E_b - c + h W, W) for
//   the integrand's centre c, so u = x - c = fma(lo, W, first entry) is one
//   convert and one fma (x itself is not formed; the centre is 0 for user
//   integrands).  The width product takes the factors 2^-32 back ahead of them: it
//   starts at 2^(32 d), or beyond d = 24, where that overflows, at 2^32 for each
//   dimension of the first groups of four and of a last, partial one, and each other
//   group multiplies by 2^128; so it never falls below the product of the widths
//   and ends as that.  (Forming delta took an fma per dimension and,
//   where 2^-32 and h sat in scalar registers, a copy of h.)
// FP32: the map works on u' = (x - c) S with S = 2^(ws + 32).  With
//   delta = (lo + h)/2^32 (see bin_words) and W = RN32(width), the table entry is
//     (RN32((E_b - c + h W / 2^32) S), W 2^ws),
//   so u' = RN32(lo) (W 2^ws) + first entry is one int-to-float convert and one
//   FP32 fma: the convert rounds lo exactly as RN32(delta) would (delta itself
//   is never formed), the offset from the integrand's centre c makes u carry
//   rounding relative to u rather than to x, the factor 2^ws keeps the width
//   product near one, and the integrand's constants absorb S^-1, S^-2 exactly.
//   The bimodal integrand has two centres: (cA entry, cB entry, W 2^ws, 0).
struct P64 {
    using real = double;
    static constexpr bool is64 = true;
};
struct P32 {
    using real = float;
    static constexpr bool is64 = false;
};

template <class P, int KIND>
struct TabEntry {
    using type = float2;
};
template <int KIND>
struct TabEntry<P64, KIND> {
    using type = double2;
};
template <>
struct TabEntry<P32, BIMODAL> {
    using type = float4;
};
// log2 of an entry's bytes
template <class P, int KIND>
struct TabLog2 {
    static constexpr int value = sizeof(typename TabEntry<P, KIND>::type) == 16 ? 4 : 3;
};

// e^x 2^e, magic = 1.5 2^52 + e: n = round(x log2 e) is read off the sum with magic
// (its low word is e + n), the rest f = x log2 e - n in [-1/2, 1/2] is formed with
// one rounding (log2 e as a sum of two), and 2^f is a polynomial of degree 11
// (minimax for the relative error with the constant 1 and the linear coefficient
// RN(ln 2) held: 9e-18). x is cut at -4000 ln 2, where the result is 0 for every e
// of a finite C; above, x log2 e stays below 10^8 (the discontinuous integrand's c
// (1 - a) is at most 10^6 there), and the sum's low word holds any such n. (magic is
// not a number where x is not, which the cut hides, or where it may be larger: the
// parameters are looked at instead, once.) Against exp(x) times C: 17 instructions
// for 23 (the loop is bound by their issue). Per 1e7 events, N = 50, without
// histograms: the d = 8 Gaussian 45.1 -> 43.4 us, d = 4 28.9 -> 27.0, the bimodal
// integrand (two of them) d = 8 55.8 -> 52.2. held: the coefficients of f^10 to
// f^6, see EvalConsts.
constexpr double kExpCut = 2772.0;  // 4000 ln 2
__device__ __forceinline__ double exp_scaled(double x, double magic, const double (&held)[5])
{
#pragma clang fp contract(off)
    const double log2e = 0x1.71547652b82fep+0, log2e_lo = 0x1.777d0ffda0d24p-56;
    const double t = fma(x, log2e, magic), n = t - magic;
    const double f = fma(x, log2e_lo, fma(x, log2e, -n));
    double p = 0x1.e8112113876cbp-32;
    p = fma(p, f, held[0]);
    p = fma(p, f, held[1]);
    p = fma(p, f, held[2]);
    p = fma(p, f, held[3]);
    p = fma(p, f, held[4]);
    p = fma(p, f, 0x1.5d87fe78b3b99p-10);
    p = fma(p, f, 0x1.3b2ab6fba110cp-7);
    p = fma(p, f, 0x1.c6b08d704a0d4p-5);
    p = fma(p, f, 0x1.ebfbdff82c59cp-3);
    p = fma(p, f, 0x1.62e42fefa39efp-1);
    p = fma(p, f, 1.0);
    return ldexp(p, __double2loint(t));
}
__device__ __forceinline__ float exp2_unit(float z) { return __builtin_amdgcn_exp2f(z); }

// The word k stands for y = (k + 1/2)/2^32, so yN = (kN + N/2) / 2^32.  With
// P = kN + floor(N/2), one 32x32+32 -> 64-bit multiply-add, yN = (P + h)/2^32
// where h = 1/2 for odd N and 0 for even N; since P + h never reaches the next
// multiple of 2^32, the bin b = floor(yN) is the high word of P and
// delta = yN - b = (lo + h) / 2^32, lo the low word.  The bin is exact in
// every precision and FP64 gets delta exactly; the FP32 map carries RN32(lo).
struct BinConsts {
    uint32_t mul, add;  // N, floor(N/2)
    double h64;         // h / 2^32 (per-event records)
};

// LDS as 32-bit addresses: a pointer formed from the sum of a dynamic LDS
// array's start and an offset costs an addition of its own per access, because
// the start is known only after instruction selection; as an integer it is
// part of the scalar each offset is formed with.
template <class T>
using lds_ptr = __attribute__((address_space(3))) T*;

__device__ __forceinline__ uint32_t lds_address(unsigned char* p)
{
    return uint32_t(reinterpret_cast<uint64_t>((lds_ptr<unsigned char>)p));
}

// Entry b of a table of T at LDS address `base`.  Indexed as a pointer: as a
// shift and a sum, the compiler merges the shift with the extraction of the
// bin from its 64-bit product into an alignbit, a mask and an addition, where
// one shift-add does.
template <class T>
__device__ __forceinline__ lds_ptr<const T> entry_of(int b, uint32_t base)
{
    return (lds_ptr<const T>)(uint64_t(base)) + b;
}

__device__ __forceinline__ void bin_words(uint32_t k, const BinConsts& bc, int& b, uint32_t& lo)
{
    const uint64_t P = uint64_t(k) * bc.mul + bc.add;
    b = int(uint32_t(P >> 32));
    lo = uint32_t(P);
}

// Binary exponent the FP64 width product starts at: all 2^32 of it (whole), or
// those of the first kWidthGroups groups of four (d >= 17 there) and of a partial
// one. (Choosing the last group's factor in the loop instead made the d = 40
// discontinuous kernel without histograms 157 -> 190 us per 4e6 events: a scalar
// register more, of which it spills hundreds; a factor at the end the bimodal one
// with histograms 228 -> 240.)
constexpr int kWidthGroups = 2;
__device__ __forceinline__ constexpr int width_start(bool whole, int d)
{
    return whole ? 32 * d : 128 * kWidthGroups + 32 * (d % 4);
}

// Integrand constants of one problem, read once per thread into registers
// (they are uniform, so they normally live in scalar registers).
template <class P, int KIND, int DMAX>
struct EvalConsts {
    using real = typename P::real;
    // the FP64 discontinuous and bimodal integrands' constants per dimension
    // take two scalar registers each
    static constexpr bool kFewScalars = P::is64 && (KIND == GENZ_DISC || KIND == BIMODAL) && DMAX > 8 && DMAX <= 20;
    real p1[DMAX], p2[DMAX];
    double c64[DMAX];   // FP32 path, DISC: c_i / S (exponent summed in FP64, d > 8)
    float c32[DMAX];    // FP32 path, DISC: RN32(c_i / S) (exponent summed in FP32, d <= 8)
    // FP64 path: the exponential of GAUSS, BIMODAL and DISC (DevConst), and the
    // width product's start: the constant's mantissa (PEAK: 1) times the power of
    // two of width_start
    static constexpr bool kExp = P::is64 && KIND != GENZ_PEAK, kWhole = DMAX <= 24;
    double kexp, magic, w0;  // kexp: GAUSS, BIMODAL: -1/a^2
    // coefficients of exp_scaled, in scalar registers where those are free
    // (GAUSS): the compiler holds all in vector registers, and the d = 18
    // kernel (N = 100) spilled 28 instead of 24 (136 against 131 us)
    double held[5];
    real dscale;        // FP32 path, 1/S = 2^-(ws + 32)
    double k2;          // FP32 path: log2(e)/(a S)^2 (GAUSS, BIMODAL), log2(e) (DISC)
    BinConsts bc;
    // LDS address of each dimension's table, as a scalar the compiler cannot
    // split (it otherwise regroups the sums: one more addition per dimension);
    // formed one after another with many dimensions and where kFewScalars
    static constexpr bool kHoldBase = DMAX <= 24 && !kFewScalars;
    uint32_t base[kHoldBase ? DMAX : 1];
    double C, Cf, Cw;
    // DISC: x_i > a_i exactly when the event's binning word k_i >= K_i; lane
    // l holds K_l (l < d), read with v_readlane (which ignores EXEC, so it is
    // safe in the partial last pass); never: some K_i = 2^32, no event is
    // inside
    uint32_t kv;
    bool never;

    // For records of w and f: both without C (magic stays what it is where the
    // exponent is not a number).
    __device__ __forceinline__ void leave_out_constant(int d)
    {
        w0 = ldexp(1.0, width_start(kWhole, d));
        magic = magic == magic ? 0x1.8p52 : magic;
    }

    // thr_g: the d thresholds T_i of the discontinuous integrand in
    // P = b 2^32 + lo (disc_threshold; other kinds: unused, may be null).
    // tab: LDS address of the table [d][n_bins].
    // Called by every thread of the wave (it takes a ballot).
    __device__ __forceinline__ void load(const DevConst* __restrict__ c, const uint64_t* __restrict__ thr_g, int d,
                                         int n_bins, uint32_t tab)
    {
        if constexpr (kHoldBase) {
#pragma unroll
            for (int i = 0; i < DMAX; ++i)
                base[i] = __builtin_amdgcn_readfirstlane(tab + (uint32_t(i * n_bins) << TabLog2<P, KIND>::value));
        }
        // only what the kernel's precision and integrand read (scalar registers
        // are scarce); the FP32 path works on u S, S = 2^(ws + 32), so its
        // constants take the matching powers of 1/S (exact)
        const double ds = double(c->dscale32) * 0x1p-32, ds2 = ds * ds;
#pragma unroll
        for (int i = 0; i < DMAX; ++i) {
            p1[i] = real(0);
            p2[i] = real(0);
            c64[i] = 0.0;
            c32[i] = 0.0f;
            if constexpr (P::is64) {
                // the centres are in the table: GENZ c (DISC) or c^2 (PEAK),
                // BIMODAL muB - muA
                if constexpr (KIND == GENZ_DISC || KIND == GENZ_PEAK) p1[i] = c->p1_64[i];
                if constexpr (KIND == BIMODAL) p2[i] = c->p2_64[i];
            } else {
                if constexpr (KIND == GENZ_PEAK) p1[i] = real(sqrt(c->p1_64[i]) * ds);  // c_i / S
                if constexpr (KIND == GENZ_DISC) {
                    c64[i] = c->p1_64[i] * ds;
                    c32[i] = float(c64[i]);
                }
            }
        }
        constexpr double coef[5] = {0x1.e61229bbb383ap-28, 0x1.b5260c8388969p-24, 0x1.62bfcd861ec29p-20, 0x1.ffcbfbf914474p-17, 0x1.4309130c28fc2p-13};
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            held[k] = coef[k];
            if constexpr (kExp && KIND == GAUSS) asm("" : "+s"(held[k]));
        }
        kexp = -c->kexp64;
        magic = c->magic;
        w0 = ldexp(kExp ? c->mant : 1.0, width_start(kWhole, d));
        k2 = (P::is64 || KIND == GENZ_DISC) ? c->kexp2_64 : c->kexp2_64 * ds2;
        dscale = real(ds);
        const uint32_t N = uint32_t(c->n_bins);
        bc.mul = N;
        bc.add = N >> 1;
        bc.h64 = (N & 1u) ? 0x1p-33 : 0.0;
        C = c->C;
        Cf = c->Cf;
        Cw = c->Cw;
        kv = 0;
        never = false;
        if constexpr (KIND == GENZ_DISC) {
            // P = k N + floor(N/2) grows with k, so P >= T exactly when
            // k >= K = ceil((T - floor(N/2)) / N) (0 when T <= floor(N/2))
            const int lane = int(threadIdx.x & 63u);
            uint64_t K = 0;
            if (lane < d) {
                const uint64_t T = thr_g[lane], off = N >> 1;
                K = T <= off ? 0 : (T - off + N - 1) / N;
            }
            never = __ballot(K > 0xffffffffull) != 0;
            kv = uint32_t(K);
        }
    }
};

// Per-event evaluation shared by the sampling, dump and adjoint kernels.
// Computes, for the event's d uniforms, the bins, the offsets u_i = x_i - c_i
// from the integrand's centres, the width product wp and the integrand's
// significand F; the event value is v = ldexp(F * wp, ew + fe) * C
// (FP64: ew = fe = 0, and C is in F and wp where the integrand has an
// exponential).  EXACT: d == DMAX, so no per-dimension guards are needed.
template <class P, int KIND, int DMAX, bool EXACT = false>
struct EventEval {
    using real = typename P::real;
    using tab_t = typename TabEntry<P, KIND>::type;

    int bin[DMAX];       // bin of each dimension
    uint32_t off[DMAX];  // LDS address of its table entry
    real u[DMAX];     // x_i - centre_i (GAUSS, BIMODAL: mu / muA; DISC, PEAK: a_i); FP32: times S
    real del[DMAX];   // lo (FP32: RN32(lo))
    real wp;          // width product (scaled, see Cw; FP32: and ew)
    real F;           // integrand significand
    real s;           // GAUSS: sum u_i^2
    double s64;       // GAUSS: sum u_i^2 as accumulated (FP64 in both paths; FP32: of u S)
    int ew;           // FP32: binary exponent taken out of the width product
    int fe;           // FP32: binary exponent of the integrand (f ~ 2^fe F)

    // tab: LDS address of the table [d][N]
    __device__ __forceinline__ void run(const EvalConsts<P, KIND, DMAX>& c, uint32_t tab,
                                        uint64_t e, uint32_t t,
                                        uint32_t ctr3, uint32_t key0, uint32_t key1, int d_rt, int N)
    {
        // every fused multiply-add here is an explicit fma(): nothing else is
        // contracted, so all kernel variants round the same way
#pragma clang fp contract(off)
        const int d = EXACT ? DMAX : d_rt;
        // the FP32 path sums the exponent in FP32 up to d = 8 (error <= d 2^-24
        // of the exponent) and in FP64 beyond, where that grows past the
        // method's tolerance
        constexpr bool kQ32 = !P::is64 && DMAX <= 8;
        using q_t = typename pick_type<kQ32, float, double>::type;
        real w = P::is64 ? real(c.w0) : real(1);
        real sa = real(0), sb = real(0);  // FP64 path: GAUSS/BIMODAL sums of squares; DISC: sum c u
        q_t qa = q_t(0), qb = q_t(0);     // FP32 path: the same sums
        real den = real(1);               // PEAK: product of denominators
        bool inside = true;               // DISC: all x_i > a_i
        int ewl = 0;                      // FP32: exponent taken out of w
        const uint32_t elo = uint32_t(e), ehi = uint32_t(e >> 32);
        uint32_t next = tab;              // table of the next dimension, where EvalConsts does not hold them
        // one Philox call per group of four dimensions (the last group may be
        // partial: DMAX need not be a multiple of 4)
#pragma unroll
        for (int g = 0; g < (DMAX + 3) / 4; ++g) {
            if (4 * g < d) {
                const U4 k = philox4x32_10(elo, ehi, t, ctr3 + uint32_t(g), key0, key1);
                // the group's four bins and table entries first, so that its
                // LDS reads are in flight together before any is used
                int bq[4];
                uint32_t oq[4], loq[4];
                tab_t tq[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 4 * g + q;
                    if (i < d) {
                        if constexpr (P::is64 && !EvalConsts<P, KIND, DMAX>::kWhole)
                            if (g >= kWidthGroups && q == 3) w *= real(0x1p128);
                        bin_words(k.w[q], c.bc, bq[q], loq[q]);
                        constexpr int L = TabLog2<P, KIND>::value;
                        lds_ptr<const tab_t> pq;
                        if constexpr (EvalConsts<P, KIND, DMAX>::kHoldBase) {
                            pq = entry_of<tab_t>(bq[q], c.base[i]);
                        } else {
                            pq = entry_of<tab_t>(bq[q], next);
                            next += uint32_t(N) << L;
                            asm volatile("" : "+s"(next));
                        }
                        oq[q] = uint32_t(uint64_t(pq));
                        tq[q] = *(const tab_t*)pq;
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 4 * g + q;
                    if (i < d) {
                        const uint32_t lo = loq[q];
                        off[i] = oq[q];
                        bin[i] = bq[q];
                        const tab_t tb = tq[q];
                        real ui, ubi = real(0), width;
                        real dl;
                        if constexpr (P::is64) {
                            dl = double(lo);
                            width = tb.y;
                            ui = fma(dl, tb.y, tb.x);
                            if constexpr (KIND == BIMODAL) ubi = ui - c.p2[i];  // p2 = muB - muA
                        } else if constexpr (KIND == BIMODAL) {
                            dl = float(lo);
                            width = tb.z;
                            ui = fma(dl, tb.z, tb.x);
                            ubi = fma(dl, tb.z, tb.y);
                        } else {
                            dl = float(lo);
                            width = tb.y;
                            ui = fma(dl, tb.y, tb.x);
                        }
                        del[i] = dl;
                        u[i] = ui;
                        w *= width;
                        if constexpr (KIND == GAUSS) {
                            if constexpr (P::is64)
                                sa = fma(ui, ui, sa);
                            else  // (u^2 of an FP32 u is exact in FP64)
                                qa = fma(q_t(ui), q_t(ui), qa);
                        } else if constexpr (KIND == BIMODAL) {
                            if constexpr (P::is64) {
                                sa = fma(ui, ui, sa);
                                sb = fma(ubi, ubi, sb);
                            } else {
                                qa = fma(q_t(ui), q_t(ui), qa);
                                qb = fma(q_t(ubi), q_t(ubi), qb);
                            }
                        } else if constexpr (KIND == GENZ_DISC) {
                            // x_i > a_i as the FP64 x decides it: one integer
                            // comparison of the binning word with K_i, in both
                            // precisions
                            inside = inside & (k.w[q] >= uint32_t(__builtin_amdgcn_readlane(int(c.kv), i)));
                            if constexpr (P::is64)
                                sa = fma(c.p1[i], ui, sa);
                            else if constexpr (kQ32)
                                qa = fma(c.c32[i], ui, qa);
                            else
                                qa = fma(c.c64[i], double(ui), qa);
                        } else {  // GENZ_PEAK: (c u)^2 + 1
                            if constexpr (P::is64) {
                                den *= fma(c.p1[i] * ui, ui, real(1));  // p1 = c^2
                            } else {
                                const real cu = c.p1[i] * ui;  // p1 = c / S, ui = u S
                                den *= fma(cu, cu, real(1));
                            }
                        }
                    }
                }
                if constexpr (!P::is64) {
                    // every 8 dimensions move w's exponent into ew (no FP32 under/overflow)
                    if ((g & 1) == 1 && 4 * g + 4 < d) {
                        int e2;
                        w = frexpf(w, &e2);
                        ewl += e2;
                    }
                }
            }
        }
        if constexpr (KIND == GENZ_DISC) inside = inside && !c.never;
        wp = w;
        s = sa;
        s64 = P::is64 ? double(sa) : double(qa);
        ew = ewl;
        if constexpr (P::is64) {
            fe = 0;
            if constexpr (KIND == GAUSS)
                F = exp_scaled(fmax(sa * c.kexp, -kExpCut), c.magic, c.held);
            else if constexpr (KIND == BIMODAL)
                F = exp_scaled(fmax(sa * c.kexp, -kExpCut), c.magic, c.held) +
                    exp_scaled(fmax(sb * c.kexp, -kExpCut), c.magic, c.held);
            else if constexpr (KIND == GENZ_DISC)
                F = inside ? exp_scaled(fmax(sa, -kExpCut), c.magic, c.held) : 0.0;  // sa = sum c (x - a)
            else
                F = real(1) / den;
        } else {
            // FP32 significand, FP64 exponent: with the exponent A (base 2)
            // formed in FP64, m = floor(A) and F = 2^(m - A) in (1/2, 1] in
            // FP32, so f = 2^-m F Cf keeps FP64 range
            s = float(qa);
            if constexpr (KIND == GAUSS) {
                const double arg = double(qa) * c.k2;
                const double m = floor(arg);
                F = exp2_unit(float(m - arg));
                fe = -int(m);
            } else if constexpr (KIND == BIMODAL) {
                const double aa = double(qa) * c.k2, ab = double(qb) * c.k2;
                const double m = floor(fmin(aa, ab));
                F = exp2_unit(float(fmax(m - aa, -200.0))) + exp2_unit(float(fmax(m - ab, -200.0)));
                fe = -int(m);
            } else if constexpr (KIND == GENZ_DISC) {
                const double arg = -double(qa) * c.k2;  // qa = sum c (x - a) >= 0 inside
                const double m = floor(arg);
                F = inside ? exp2_unit(float(m - arg)) : 0.0f;
                fe = -int(m);
            } else {
                F = 1.0f / den;
                fe = 0;
            }
        }
    }

    // The product is rounded as written (no fusion into a following add), so
    // every kernel variant accumulates the same rounded v.
    __device__ __forceinline__ double value(const EvalConsts<P, KIND, DMAX>& c) const
    {
#pragma clang fp contract(off)
        if constexpr (EvalConsts<P, KIND, DMAX>::kExp)
            return F * wp;  // (C is in both)
        else if constexpr (P::is64)
            return F * wp * c.C;
        else
            return ldexp(double(F * wp), ew + fe) * c.C;
    }
};

// ---------------------------------------------------------------------------
// Reductions.
// Event kernels add kGroup events per thread in plain FP64, then fold the
// group's sums into Kahan-compensated S1, S2.
constexpr int kGroup = 8;

// Kahan step: s + (-c) tracks the running sum.
__device__ __forceinline__ void kahan_add(double& s, double& c, double v)
{
    const double y = v - c;
    const double t = s + y;
    c = (t - s) - y;
    s = t;
}

// Branch-free compensated step (Knuth's TwoSum): the sum is s + c.
__device__ __forceinline__ void twosum_add(double& s, double& c, double v)
{
    const double t = s + v;
    const double bp = t - s;
    c += (s - (t - bp)) + (v - bp);
    s = t;
}

// The value a DPP control takes from another lane (0 where it takes none).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Sum over the wave's 64 lanes, valid in lane 63 (all lanes must be active):
// prefix sums within the rows of 16 lanes, then row totals passed on.  The
// exchanges stay in the vector unit; through the LDS crossbar each step waits
// for a round trip.
__device__ __forceinline__ double wave_sum_last(double v)
{
    v += dpp_move<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
    v += dpp_move<0x112, 0xf>(v);
    v += dpp_move<0x114, 0xf>(v);
    v += dpp_move<0x118, 0xf>(v);
    v += dpp_move<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
    return v;
}

// Block sums of n doubles: every wave leaves its sums of its lanes' v[0..n-1]
// in red (n x blockDim.x/64 doubles of LDS), and after one barrier thread j
// adds column j over the waves in order; returned in threads 0..n-1.
template <int n>
__device__ __forceinline__ double block_sums(const double (&v)[n], double* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < n; ++j) {
        const double s = wave_sum_last(v[j]);
        if (lane == 63) red[wave * n + j] = s;
    }
    __syncthreads();
    double t = 0.0;
    if (int(threadIdx.x) < n) {
        const int nw = int(blockDim.x) >> 6;
        for (int k = 0; k < nw; ++k) t += red[k * n + int(threadIdx.x)];
    }
    return t;
}

// Inclusive prefix sum over the 64 lanes of a wave: the steps of wave_sum_last
// leave in every lane the sum of the lanes up to it.
__device__ __forceinline__ double wave_inclusive_scan(double v) { return wave_sum_last(v); }

// Running maximum over the 64 lanes of a wave (lane order) of values >= 0.
__device__ __forceinline__ double wave_inclusive_max(double v)
{
    v = fmax(v, dpp_move<0x111, 0xf>(v));
    v = fmax(v, dpp_move<0x112, 0xf>(v));
    v = fmax(v, dpp_move<0x114, 0xf>(v));
    v = fmax(v, dpp_move<0x118, 0xf>(v));
    v = fmax(v, dpp_move<0x142, 0xa>(v));
    v = fmax(v, dpp_move<0x143, 0xc>(v));
    return v;
}

// The pair sums (s + c) over the 64 lanes of a wave by exact two-sums, the
// total in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void dpp_pair_add(double& s, double& c)
{
    const double s2 = dpp_move<CTRL, ROW_MASK>(s), c2 = dpp_move<CTRL, ROW_MASK>(c);
    twosum_add(s, c, s2);
    c += c2;
}

__device__ __forceinline__ void wave_pair_sum_last(double& s, double& c)
{
    dpp_pair_add<0x111, 0xf>(s, c);
    dpp_pair_add<0x112, 0xf>(s, c);
    dpp_pair_add<0x114, 0xf>(s, c);
    dpp_pair_add<0x118, 0xf>(s, c);
    dpp_pair_add<0x142, 0xa>(s, c);
    dpp_pair_add<0x143, 0xc>(s, c);
}

// Fixed-order sum of column j of the rows part[rows][d + 1] of an adjoint by
// one wave: lane l adds rows l, l + 64, ... in order with two-sums (eight loads
// in flight), then the lanes' pairs are added.  The column times `scale` goes
// to out[j], in FP64 or rounded once to FP32 (out_fp32).
__device__ __forceinline__ void adjoint_merge_column(const double* part, int rows, int d, int j, double scale,
                                                     void* out, int out_fp32)
{
    const int lane = threadIdx.x & 63;
    double s = 0.0, c = 0.0;
    for (int r0 = lane; r0 < rows; r0 += 64 * 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = r0 + 64 * u < rows ? part[size_t(r0 + 64 * u) * (d + 1) + j] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) twosum_add(s, c, v[u]);
    }
    wave_pair_sum_last(s, c);
    if (lane == 63) {
        const double g = (s + c) * scale;
        if (out_fp32)
            static_cast<float*>(out)[j] = float(g);
        else
            static_cast<double*>(out)[j] = g;
    }
}

// Value of lane l, the same l in every lane.
__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

__device__ __forceinline__ void lds_atomic_add(double* p, double v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Adds into the block's histogram in LDS.
//
// What bounds an atomic is that the 16 lanes the LDS serves together (lanes
// 16 q .. 16 q + 15 of a wave) hit 16 different bank pairs: 9.4 cycles per wave
// then, 17 where two of them can meet, 31 at random.

// [dimension][bin][replica], 2^rl2 replicas: 16 of them give every lane a bank
// pair of its own.  The table [dimension][bin] and the histogram share their
// indexing, so a histogram address is the entry's table address shifted onto
// the bin's replicas, plus the lane's own start: one shift-add per dimension
// with the shift in a scalar register, for every N, d and replica count.  (A
// layout with a compile-time stride of 64 bins per dimension reached the same
// count for d in {4, 8, 12, 16} and 16 replicas only, and padded the bins to 64.)
template <int TL2>  // log2 of a table entry's bytes
struct HistAdder {
    int sh;          // a table address to a histogram address
    uint32_t start;  // histogram's start and the lane's replica, less the shifted table start

    // tab, hist: LDS addresses of the table and the histogram
    __device__ __forceinline__ HistAdder(uint32_t tab, uint32_t hist, int rl2)
    {
        sh = rl2 + 3 - TL2;
        start = hist + ((threadIdx.x & ((1u << rl2) - 1u)) << 3) - (sh >= 0 ? tab << sh : tab >> 1);
    }

    template <int D, bool EXACT>
    __device__ __forceinline__ void add(const uint32_t (&off)[D], int d, double v2) const
    {
        if (TL2 == 4 && sh < 0) {  // one replica of 8 bytes beside 16-byte entries: the shift is to the right
#pragma unroll
            for (int i = 0; i < D; ++i)
                if (EXACT || i < d)
                    lds_atomic_add((double*)(lds_ptr<double>)(uint64_t((off[i] >> 1) + start)), v2);
            return;
        }
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (EXACT || i < d)
                lds_atomic_add((double*)(lds_ptr<double>)(uint64_t((off[i] << sh) + start)), v2);
    }
};

// [set][bin][dimension of the set][replica], for fewer than 16 replicas: the
// dimensions are taken in sets of G = 2^GL with R = 16 / G replicas, so that a
// bin's counters of a whole set fill one row of 128 bytes, and the lanes of
// each G-th part of 16 go through the set's dimensions in an order of their own
// (dimension k xor part in step k): the 16 lanes then add into the 16 places
// of their rows, as with 16 replicas, for G / 16 of the LDS.  It costs GL
// selects per dimension.  Per 1e7 events, conflicting replicas -> sets: d = 20, N
// = 100 bimodal FP32-mixed (8 replicas) 194 -> 156 us, d = 16, N = 100 Gaussian
// 108 -> 91 us FP32-mixed and 123 -> 104 us FP64, d = 8, N = 200 (4 replicas)
// FP32-mixed 66 -> 46 us.  (Interleaving the table the same way would make the
// address the plain layout's, but left a dimension's entries on every G-th
// bank: 191 us for that bimodal.)
template <int GL, int D, bool HOLD>
struct HistSets {
    static constexpr int G = 1 << GL, R = 16 >> GL;
    // the row's start and the lane's place in step i, held where registers
    // allow (HOLD), else the place in each step of a whole and of the last set
    static constexpr bool kHold = HOLD;
    uint32_t at[kHold ? D : G], last[G], set_bytes;

    // the dimension of its set that the lane takes in step k of a set of m
    static __device__ __forceinline__ uint32_t order(int k, int m)
    {
        const uint32_t part = (threadIdx.x & 15u) / R;
        if (GL == 2 && m == 4) return uint32_t(k) ^ part;
        if (m >= 2 && k < 2) return uint32_t(k) ^ (part & 1u);
        return uint32_t(k);
    }

    __device__ __forceinline__ HistSets(uint32_t hist, int N)
    {
        set_bytes = uint32_t(N) * 128u;
        auto place = [&](int k, int m) { return (order(k, m) * R + (threadIdx.x & uint32_t(R - 1))) << 3; };
        if constexpr (kHold) {
#pragma unroll
            for (int i = 0; i < D; ++i)
                at[i] = hist + uint32_t(i / G) * set_bytes + place(i % G, D - i / G * G < G ? D % G : G);
        } else {
#pragma unroll
            for (int k = 0; k < G; ++k) {
                at[k] = hist + place(k, G);
                last[k] = hist + place(k, D % G);
            }
        }
    }

    // Exchanges x and y in the lanes whose part has bit BIT.
    template <int BIT>
    static __device__ __forceinline__ void exchange(int& x, int& y)
    {
        const bool other = ((threadIdx.x & 15u) / R) & (1u << BIT);
        const int a = x, b = y;
        x = other ? b : a;
        y = other ? a : b;
    }

    __device__ __forceinline__ void add(const int (&bin)[D], double v2) const
    {
        int b[D];
#pragma unroll
        for (int i = 0; i < D; ++i) b[i] = bin[i];
#pragma unroll
        for (int s = 0; s < D; s += G) {
            if (s + 1 < D) exchange<0>(b[s], b[s + 1]);
            if constexpr (GL == 2) {
                if (s + 3 < D) {
                    exchange<0>(b[s + 2], b[s + 3]);
                    exchange<1>(b[s], b[s + 2]);
                    exchange<1>(b[s + 1], b[s + 3]);
                }
            }
        }
        struct Row {
            double r[16];
        };
#pragma unroll
        for (int i = 0; i < D; ++i) {
            uint32_t row;
            if constexpr (kHold)
                row = at[i];
            else
                row = (D - i / G * G < G ? last[i % G] : at[i % G]) + uint32_t(i / G) * set_bytes;
            lds_atomic_add((double*)(lds_ptr<double>)((lds_ptr<Row>)(uint64_t(row)) + b[i]), v2);
        }
    }
};

// Sum of bin k's replicas (hist in LDS, [bin][replica], 2^rl2 of them).  Lane
// k starts at replica k: the lanes of a wave then read different banks, where
// reading replica 0 of every bin first would have all of them on the same one
// (16 replicas are 128 bytes, half of the 64 banks).
template <int RL2>
__device__ __forceinline__ double replica_sum(const double* hist, int k)
{
    const double* h = hist + (k << RL2);
    constexpr int R = 1 << RL2, Q = R < 8 ? R : 8;  // Q reads in flight
    double s = 0.0;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += Q) {
        double v[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) v[r] = h[(r0 + r + k) & (R - 1)];
#pragma unroll
        for (int r = 0; r < Q; ++r) s += v[r];
    }
    return s;
}

__device__ __forceinline__ double replica_sum(const double* hist, int k, int rl2)
{
    switch (rl2) {
    case 4: return replica_sum<4>(hist, k);
    case 3: return replica_sum<3>(hist, k);
    case 2: return replica_sum<2>(hist, k);
    case 1: return replica_sum<1>(hist, k);
    default: return hist[k];
    }
}

}  // namespace vegas
