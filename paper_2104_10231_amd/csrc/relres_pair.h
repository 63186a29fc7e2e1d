// relres_pair.h -- the per-pair terms of Eq. 20 on the device, shared by the
// force, adjoint and molecular-dynamics kernels.  Not part of the public ABI.
#pragma once

#include "relres_internal.h"

namespace relres {

// Reciprocal and square root of the pair terms.  FP32: hardware estimates.
// FP64: the FP32 estimate refined by NR Newton steps in FP64, each of which
// squares the relative error (2^-22 -> ~2^-44 -> rounding level); one step is
// ample for FP64 energy/virial sums of FP32-force runs, two give full FP64.
struct MathF32 {
    using T = float;
    static __device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
    // r = sqrt(x) and ir = 1/r from one reciprocal-square-root estimate
    static __device__ __forceinline__ void root(float x, float& r, float& ir)
    {
        ir = __builtin_amdgcn_rsqf(x);
        r = x * ir;
    }
};

template <int NR>
struct MathF64 {
    using T = double;
    static __device__ __forceinline__ double recip(double x)
    {
        double y = (double)__builtin_amdgcn_rcpf((float)x);
#pragma unroll
        for (int k = 0; k < NR; ++k) y = fma(y, fma(-x, y, 1.0), y);
        return y;
    }
    static __device__ __forceinline__ void root(double x, double& r, double& ir)
    {
        double y = (double)__builtin_amdgcn_rsqf((float)x);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const double e = fma(-(x * y), y, 1.0);   // 1 - x y^2
            y = fma(0.5 * y, e, y);
        }
        ir = y;
        r = x * y;
        r = fma(0.5 * y, fma(-r, r, x), r);          // one more step on r itself
    }
};

// A quartic zone of Eq. 20 at d = r - r_-: g = gamma_0 .. gamma_4 and the shift
// taken off.  (Energy and derivative from one Horner scheme save three
// multiplications, but the derivative's rounding error grows by a quarter; the
// multiples kept in the table take more LDS than they save.)
template <typename T>
__device__ __forceinline__ void zone_term(const T* g, T shift, T d, T ir, T& fpair, T& en)
{
    const T dp = g[1] + d * (T(2) * g[2] + d * (T(3) * g[3] + d * (T(4) * g[4])));
    fpair = -dp * ir;
    en = g[0] + d * (g[1] + d * (g[2] + d * (g[3] + d * g[4]))) - shift;
}

// Pair terms of the FG part of Eq. 20 (r < r_s+): fpair = -u~'(r)/r and the
// energy.  Called only for r2 < r_s+^2.
template <typename M, typename T = typename M::T>
__device__ __forceinline__ void fg_term(const PairCoef<T>& c, const Cutoffs<T>& cut, T r2,
                                        T& fpair, T& en)
{
    if (r2 < cut.rsi2) {
        const T r2i = M::recip(r2);
        const T r6i = r2i * r2i * r2i;
        fpair = r6i * (c.fg_c12 * r6i - c.fg_c6) * r2i;
        en = r6i * (c.fg_e12 * r6i - c.fg_e6) - c.fg_shift;
    } else {
        T r, ir;
        M::root(r2, r, ir);
        zone_term(c.fg_g, c.fg_shift, r - cut.rsi, ir, fpair, en);
    }
}

// Pair terms of the CG part of Eq. 20 (hybrid pairs, r < r_c+).  A wave's
// entries lie in all four of its distance ranges, so every branch there is
// costs every wave: the two quartic zones are one (the pair's own coefficients
// by address), and the constant inside r_s- is the inner zone at d = 0.  Launches
// with energy and virial, also with the sums halved only at the end: 20480 atoms
// at 14 A 16.8 to 16.4 us, 98304-atom copolymer 19.2 to 18.8, 80000 atoms at 14 A
// 49.1 to 47.8, 1500 propane atoms (FP64) 7.14 to 7.02; forces only the same.
template <typename M, typename T = typename M::T>
__device__ __forceinline__ void cg_term(const PairCoef<T>& c, const Cutoffs<T>& cut, T r2,
                                        T& fpair, T& en)
{
    const bool inner = r2 < cut.rso2;
    if (!inner && r2 < cut.rci2) {
        const T r2i = M::recip(r2);
        const T r6i = r2i * r2i * r2i;
        fpair = r6i * (c.cg_c12 * r6i - c.cg_c6) * r2i;
        en = r6i * (c.cg_e12 * r6i - c.cg_e6) - c.cm[5];
    } else {
        const bool flat = r2 < cut.rsi2;
        T r, ir;
        M::root(flat ? cut.rsi2 : r2, r, ir);      // no root of a vanishing distance
        const T d = flat ? T(0) : r - (inner ? cut.rsi : cut.rci);
        const T* g = inner ? c.sp : c.cm;
        zone_term(g, g[5], d, ir, fpair, en);
    }
}

}  // namespace relres
