// FP64 1/sqrt, sin/cos and decay factor of the pair kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace bem {

// Phases of the FP64 kernels are counted in 256ths of a revolution.
constexpr double PHASE64 = 256.0;
constexpr double PHASE64_NARROW = 2147483648.0;   // sincos_256<false>: below it
template <class R> constexpr double phase_unit() { return 1.0; }
template <> constexpr double phase_unit<double>() { return PHASE64; }

// e^{2 pi i n / 256}, n < 256 (LDS), by the workgroup's threads
__device__ __forceinline__ void phase_table(double2 *tab) {
    for (int n = threadIdx.x; n < 256; n += blockDim.x) {
        double sn, cs;
        ::sincos(n * (6.283185307179586476925286766559 / 256.0), &sn, &cs);
        tab[n] = make_double2(cs, sn);
    }
}

// sin and cos of 2 pi u / 256: u = n + f, |f| <= 1/2, the table entry n times
// the series of the remainder c f, c = 2 pi / 256 (|c f| <= 0.0123: terms beyond
// (c f)^6 are below 4e-18), cos - 1 and sin added to the entry last.  The entry is
// taken from the low bits of n + 1.5 2^52, right while |u| < 2^51 (k r of 5e13).
// WIDE = false converts n to 32 bits, which saturates from |u| = 2^31 on (k r of
// 5e7), and is for the one kernel that has no register left for the addition.
template <bool WIDE = true>
__device__ __forceinline__ void sincos_256(double u, double &s, double &c,
                                           const double2 *__restrict__ tab) {
    constexpr double k = 6.283185307179586476925286766559 / 256.0, k2 = k * k;
    constexpr double s1 = k, s3 = -k * k2 / 6.0, s5 = k * k2 * k2 / 120.0;
    constexpr double c2 = -k2 / 2.0, c4 = k2 * k2 / 24.0, c6 = -k2 * k2 * k2 / 720.0;
    const double n = __builtin_rint(u);
    const double f = u - n, f2 = f * f;
    const double sn = __builtin_fma(__builtin_fma(f2, s5, s3), f2, s1) * f;
    const double cm = __builtin_fma(__builtin_fma(f2, c6, c4), f2, c2) * f2;   // cos - 1
    const int i = WIDE ? (int)__builtin_bit_cast(long long, n + 6755399441055744.0) : (int)n;
    const double2 e = tab[i & 255];
    c = __builtin_fma(e.x, cm, __builtin_fma(-e.y, sn, e.x));
    s = __builtin_fma(e.y, cm, __builtin_fma(e.x, sn, e.y));
}

// 1/sqrt(x): hardware estimate y (2^-24 or better) and one third-order step,
// y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2 (remainder 2^-70).
__device__ __forceinline__ double rsqrt64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-(x * y), y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

// 2^x for x <= 0: x = n / 64 + f, a table of 2^(k / 64) (LDS) and the series of
// 2^f, |f ln 2| <= 0.0055 (remainder 4e-17).
constexpr int DECAY_TAB = 64;
__device__ __forceinline__ void decay_table(double *tab) {
    for (int n = threadIdx.x; n < DECAY_TAB; n += blockDim.x) tab[n] = ::exp2(n * (1.0 / DECAY_TAB));
}
__device__ __forceinline__ double decay64(double x, const double *__restrict__ tab) {
    x = fmax(x, -1100.0);   // (below the smallest number: 0)
    const double n = __builtin_rint(64.0 * x);
    const double f = __builtin_fma(-0.015625, n, x) * 0.69314718055994530941723212145818;
    double p = __builtin_fma(f, 1.0 / 120.0, 1.0 / 24.0);
    p = __builtin_fma(p, f, 1.0 / 6.0);
    p = __builtin_fma(p, f, 0.5);
    p = __builtin_fma(p, f, 1.0);
    p = __builtin_fma(p, f, 1.0);
    const int k = (int)n;
    return __builtin_ldexp(p * tab[k & (DECAY_TAB - 1)], k >> 6);
}

}   // namespace bem
