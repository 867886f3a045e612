// Complex arithmetic and Bessel/Hankel sequences for the gfx950 kernels.
//
// Hankel functions H_n^{(1)}(x) = J_n(x) + i Y_n(x) of real argument: H_0 and
// H_1 from polynomial fits in two ranges (hankel01), higher orders by the
// upward three-term recurrence H_{n+1} = (2n/x) H_n - H_{n-1}, which is
// stable because Y_n dominates.  J_n by Miller's backward recurrence,
// normalised against whichever of J_0(x), J_1(x) is larger in magnitude.
#pragma once

#include <hip/hip_runtime.h>

#include "hankelcoef.hpp"

namespace qbx {

struct cd {
    double x, y;
};

// complex float, for the translation tables of the FP32 far field
struct cf {
    float x, y;
};

__host__ __device__ __forceinline__ cd mk(double a, double b) { return {a, b}; }
__host__ __device__ __forceinline__ cd operator+(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
__host__ __device__ __forceinline__ cd operator-(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
// Complex product with explicit fused multiply-adds: the library is built
// without automatic contraction, so every rounding is written in the source
// and results do not depend on how the compiler schedules a kernel.
__host__ __device__ __forceinline__ cd operator*(cd a, cd b)
{
    return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
__host__ __device__ __forceinline__ cd operator*(double s, cd a) { return {s * a.x, s * a.y}; }
__host__ __device__ __forceinline__ cd operator*(cd a, double s) { return {s * a.x, s * a.y}; }
__host__ __device__ __forceinline__ cd conj(cd a) { return {a.x, -a.y}; }
__host__ __device__ __forceinline__ cd neg(cd a) { return {-a.x, -a.y}; }
// acc += a * b
__host__ __device__ __forceinline__ void cfma(cd &acc, cd a, cd b)
{
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(-a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(a.y, b.x, acc.y);
}
__host__ __device__ __forceinline__ cd cdiv(cd a, cd b)
{
    double d = b.x * b.x + b.y * b.y;
    return {(a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d};
}

// Miller start index M for J_0..J_N at argument x (the recurrence starts
// from f_{M+1} = 0).  Starting there leaves a relative error of about
// ((M+1)/n) (J_{M+1}/J_n)^2 in J_n.  For orders k + 1 >= x the ratios obey
// J_{k+1}/J_k = x / (2(k+1) - x J_{k+2}/J_{k+1}) <= x / (2(k+1) - x), so
// from k0 = max(N, ceil x) their product bounds J_M / J_k0; M is the first
// order where it falls below 1e-10.  For small x that is a few orders above
// N, which keeps the recurrence short and its dynamic range small.  M never
// exceeds the classical max(x, N) + 24 + 4 cbrt(max(x, N) + 1), which is
// what governs when x is near or above N (there the bound decays slowly).
__host__ __device__ __forceinline__ int miller_start(double x, int N)
{
    double m = x > (double)N ? x : (double)N;
    int cap = (int)m + 24 + (int)(4.0 * cbrt(m + 1.0));
    int k = (int)ceil(m);
    double bound = 1.0;
    while (k < cap && bound > 1e-10) {
        bound *= x / (2.0 * (k + 1) - x);
        ++k;
    }
    return k;
}

// The start where all values up to M are summed: the same product down to
// 1e-18 and no cap, as what is left out counts by itself and not squared.
__host__ __device__ __forceinline__ int miller_start_sum(double x, int N)
{
    int k = (int)ceil(x > (double)N ? x : (double)N);
    double bound = 1.0;
    while (bound > 1e-18) {
        bound *= x / (2.0 * (k + 1.0) - x);
        ++k;
    }
    return k;
}

// J_n(x), n = 0..N, written to out[n * stride].  x >= 0.
__device__ inline void besselj_seq(double x, int N, double *out, long long stride)
{
    if (x == 0.0) {
        out[0] = 1.0;
        for (int n = 1; n <= N; ++n) out[n * stride] = 0.0;
        return;
    }
    int M = miller_start(x, N);
    double inv = 2.0 / x;
    double fp1 = 0.0, f = 1e-280, f1 = 0.0;
    for (int n = M; n > 0; --n) {
        if (n <= N) out[n * stride] = f;
        if (n == 1) f1 = f;
        double fm = fma(n * inv, f, -fp1);
        fp1 = f;
        f = fm;
        if (fabs(f) > 1e250) {
            f *= 1e-250;
            fp1 *= 1e-250;
            f1 *= 1e-250;
            for (int m = n; m <= N; ++m) out[m * stride] *= 1e-250;
        }
    }
    double jz = j0(x), jo = j1(x);
    double s = fabs(jz) >= fabs(jo) ? jz / f : jo / f1;
    out[0] = jz;
    for (int n = 1; n <= N; ++n) out[n * stride] *= s;
}

// 1/sqrt(d) to about an ulp: the hardware estimate and one third-order step.
__device__ __forceinline__ double fast_rsqrt(double d)
{
    double y = __builtin_amdgcn_rsq(d);
    double e = fma(-(d * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// r = sqrt(r2) and 1/r: one estimate for both where r2 is far from the ends of
// the range, the plain operations there.
__device__ __forceinline__ void dist_and_inverse(double r2, double &r, double &ir)
{
    if (r2 > 1e-290 && r2 < 1e290) {
        ir = fast_rsqrt(r2);
        double r0 = r2 * ir;
        r = fma(fma(-r0, r0, r2), 0.5 * ir, r0);
        ir = fma(ir, fma(-r, ir, 1.0), ir);
    } else {
        r = sqrt(r2);
        ir = 1.0 / r;
    }
}

// 1/x from an estimate a few ulps off (orders up to 40 raise its error to
// their power).
__device__ __forceinline__ double refine_inverse(double x, double est)
{
    double e = fma(-x, est, 1.0);
    return fabs(e) < 0.5 ? fma(est, e, est) : est;    // 0, infinity stay
}

// Coefficient tables are read through the constant address space, as scalar
// loads, and the polynomial steps take them as scalar operands: a
// double-precision instruction has no 64-bit literal, and the compiler's own
// choice (constants moved into vector registers, the rest spilled) costs two
// moves a step.  coef_after gives an opaque pointer that is there only once
// `v` is, so that a loop neither keeps a hundred coefficients in registers
// nor loads them all ahead.
#ifdef __HIP_DEVICE_COMPILE__
typedef const __attribute__((address_space(4))) double *CoefPtr;
__device__ __forceinline__ CoefPtr coef_after(const double *t, double v)
{
    CoefPtr c = (CoefPtr)t;
    asm volatile("" : "+s"(c) : "v"(v));
    return c;
}
__device__ __forceinline__ double fma_s(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}
#else
typedef const double *CoefPtr;
__device__ __forceinline__ CoefPtr coef_after(const double *t, double) { return t; }
__device__ __forceinline__ double fma_s(double a, double b, double c) { return fma(a, b, c); }
#endif

// Four polynomials of ROWS coefficients each (in turn, highest first) at s.
// The coefficients of two rows are one load, two loads ahead of their use.
template <int ROWS>
__device__ __forceinline__ void poly4(const double *t, double s, double (&p)[4])
{
    static_assert(ROWS % 2 == 0, "rows are loaded in pairs");
    constexpr int G = ROWS / 2, AHEAD = 2;
    double c[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g < AHEAD) {
            CoefPtr q = coef_after(t + 8 * g, s);
#pragma unroll
            for (int i = 0; i < 8; ++i) c[g][i] = q[i];
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g + AHEAD < G) {
            CoefPtr q = coef_after(t + 8 * (g + AHEAD), g ? p[0] : s);
#pragma unroll
            for (int i = 0; i < 8; ++i) c[g + AHEAD][i] = q[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = g ? fma_s(p[i], s, c[g][i]) : c[g][i];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = fma_s(p[i], s, c[g][4 + i]);
    }
}

// (1/pi) ln z, z > 0: z = 2^e m, m in [sqrt(1/2), sqrt(2)),
// ln m = 2 atanh((m - 1)/(m + 1)).  (Not (2/pi) ln z: 2/pi is a constant of the
// callers, 4/pi one more for the scalar registers, and the smooth rule took 13.7
// instead of 12.8 us for 1024 targets and 512 sources.)
__device__ __forceinline__ double log_over_pi(double z)
{
    double m = __builtin_amdgcn_frexp_mant(z);
    int e = __builtin_amdgcn_frexp_exp(z);
    bool low = m < 0.70710678118654752;
    m = low ? m + m : m;
    e -= low;
    double num = m - 1.0, den = m + 1.0;
    double r = __builtin_amdgcn_rcp(den);
    r = fma(fma(-den, r, 1.0), r, r);
    double t = num * r;
    t = fma(fma(-t, den, num), r, t);
    double t2 = t * t;
    CoefPtr c = coef_after(kLogPoly, t2);
    double q = c[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) q = fma_s(q, t2, c[k]);
    double lm = fma(t * t2, q, t);
    // ln 2 / pi in two parts, 2/pi times the rest
    double de = (double)e;
    return fma(de, 0.2206356001526516, fma(de, -7.461721539413406e-18, 0.63661977236758134308 * lm));
}

// sin x and cos x, 0 <= x <= kPhaseMax: reduction by multiples k of pi/2 in two
// parts, of which the first is exact and the second off by k 1e-33.
constexpr double kPhaseMax = 1e14;
__device__ __forceinline__ void fast_sincos(double x, double &s, double &c)
{
    double k = rint(x * 0.63661977236758134308);
    double r = fma(-k, 1.5707963267948965580, x);
    r = fma(-k, 6.1232339957367658860e-17, r);
    double z = r * r;
    CoefPtr p = coef_after(kSinCosPoly, z);
    double a = p[10], b = p[11];
#pragma unroll
    for (int i = 4; i >= 0; --i) {
        a = fma_s(a, z, p[2 * i]);
        b = fma_s(b, z, p[2 * i + 1]);
    }
    double sr = fma(r * z, a, r), cr = fma(z * z, b, fma(z, -0.5, 1.0));
    int q = (int)fma(-4.0, floor(0.25 * k), k);
    double u = (q & 1) ? cr : sr, v = (q & 1) ? sr : cr;
    s = (q & 2) ? -u : u;
    c = ((q + 1) & 2) ? -v : v;
}

// sin x, cos x and 1/sqrt(pi x) beyond kPhaseMax: the device library's
// reduction, for geometries with such distances only (FAR: their near field,
// direct sums and smooth rule have kernels of their own, as a call or 34 more
// VGPRs slow the common ones).  Bases of boxes need no such arguments: their
// order is at most 1024.
__device__ __attribute__((noinline)) void far_phase(double x, double &s, double &c, double &f)
{
    f = 0.56418958354775628695 / sqrt(x);
    if (x < __builtin_huge_val()) sincos(x, &s, &c);
    else s = c = 0.0;                        // H_n vanishes at infinity
}

// H_0(x) and H_1(x), x > 0, with ix = 1/x, in two ranges: up to 4 polynomials
// in x^2 beside the logarithm (about 90 double-precision instructions), above
// it modulus-and-phase form with polynomials in 1/x^2 (about 130); see
// hankelcoef.hpp.  Measured per wave (64 arguments, 1/x included): 670 cycles
// of a SIMD up to 4 and 1000 above, against 1450-1750 for the ascending series
// and 3500 for the device library's j0, y0, j1, y1; a wave with both, 1050.
// The error is that of those within rounding: 1e-16 of |H_n| on average, 5e-16
// at most, and 3e-16 and 1.3e-15 between 2 and 4 (9000 arguments, 1e-6 to 3000,
// against 30-digit values).  A lower bound makes the upper range's polynomials longer, a
// higher one costs the lower range its last bits (at 6, 3e-16 of |H| against
// the 1e-16 of the upper form).
constexpr double kHankelSmallX = 4.0;

template <bool FAR>
__device__ __forceinline__ void hankel01(double x, double ix, cd &h0, cd &h1)
{
    const double two_over_pi = 0.63661977236758134308;
    double p[4];
    if (x <= kHankelSmallX) {
        double t = x * x;
        poly4<kHankelSmallRows>(kHankelSmall, fma(t, 0.125, -1.0), p);
        // (2/pi) (ln(x/2) + gamma), from x itself: x^2 may underflow
        double l0 = log_over_pi(x * 0.89053620899509899), L = l0 + l0;
        double j0 = fma(t, p[0], 1.0), j1 = x * fma(t, p[2], 0.5);
        h0 = mk(j0, fma(L, j0, t * p[1]));
        h1 = mk(j1, fma(-two_over_pi, ix, fma(L, j1, x * fma(t, p[3], -0.15915494309189533577))));
        return;
    }
    poly4<kHankelLargeRows>(kHankelLarge, fma(ix * ix, 32.0, -1.0), p);
    // e = sqrt(2/(pi x)) e^{i (x - pi/4)}; H_1 has a further -i
    double sn, cs, f;
    if (!FAR || x <= kPhaseMax) {
        fast_sincos(x, sn, cs);
        f = fast_rsqrt(3.14159265358979323846 * x);
    } else {
        far_phase(x, sn, cs, f);
    }
    cd e = mk(f * (cs + sn), f * (sn - cs));
    double q0 = p[1] * ix, q1 = p[3] * ix;
    h0 = mk(fma(p[0], e.x, fma(-q0, e.y, e.x)), fma(p[0], e.y, fma(q0, e.x, e.y)));
    h1 = mk(fma(p[2], e.y, fma(q1, e.x, e.y)), -fma(p[2], e.x, fma(-q1, e.y, e.x)));
}

// A_n = tau^n H_n(x), n = 0..N, written to out[n * stride].  With
// tau = min(1, x/2) the sequence stays below (n-1)! in magnitude.
__device__ inline void scaled_hankel_seq(double x, double tau, int N, cd *out, long long stride)
{
    cd h0, h1;
    hankel01<false>(x, 1.0 / x, h0, h1);
    cd a0 = h0, a1 = tau * h1;
    out[0] = a0;
    if (N >= 1) out[stride] = a1;
    double t2 = tau * tau;
    double c = 2.0 * tau / x;                 // one division, outside the recurrence
    for (int n = 1; n < N; ++n) {
        double nc = (double)n * c;
        cd a2 = mk(fma(nc, a1.x, -(t2 * a0.x)), fma(nc, a1.y, -(t2 * a0.y)));
        out[(n + 1) * stride] = a2;
        a0 = a1;
        a1 = a2;
    }
}

}  // namespace qbx
