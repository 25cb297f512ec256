// FP64 logarithm, exponential, square root, reciprocal and sine/cosine of the
// row pass's modes, from small tables in LDS: the n_corr draw needs two
// logarithms, two square roots and two sine/cosine pairs a mode besides
// P_k's power, and the library's forms (special cases, long polynomials)
// were 700 of the 1100 instructions a mode took.
//
// Table-driven forms as in Tang, ACM TOMS 15 (1989) and 16 (1990): the
// argument is split into a table point and a small rest, on which a Taylor
// polynomial is exact to below 2^-54 of the result.  Largest errors, in units
// of 2^-53 of the result over 10^7 arguments each: log_t of an integer 1.0, of
// the draws' uniform numbers 1.9, exp_t 1.0 for |x| < 40, sqrt_t 1.0, rcp_t 1.0;
// cis_t, absolute, 1.0.  Against 80-bit
// references n_corr is 3.9e-16 off and the chi^2 gradients 4e-14, as they were
// with the library.
#pragma once
#include <cmath>

#include "common.h"

namespace c3d {

// table layout (complex entries): 64 of the logarithm {1/c_i, ln c_i}, 128
// {cos, sin} of 2 pi i / 128, 32 {2^(i/32), its
// rounding error}
constexpr int kLog = 0, kCis = 64, kExp = 192, kTab = 224;

// The logarithm's mantissa m in [1, 2) falls into interval i = floor(64 (m - 1));
// those from kHalf on count as m/2 with the exponent one higher, so that the
// result's terms do not cancel around m = 1: there c = 1 exactly.
constexpr int kHalf = 27;

// 1/c_i of the logarithm's table: any number near 1/m will do, and of 65 of them 2^-40
// apart it is the one whose ln c_i is closest to a double (Gal and Bachelis, ACM TOMS 17
// (1991)), so that the tabled logarithm has no error of its own.  c = 1 where the
// result's terms would cancel.
struct LogTab {
    double inv[64];
    LogTab() {
        for (int i = 0; i < 64; ++i) {
            const long double m = 1.0L + (i + 0.5L) / 64;
            inv[i] = i == 0 ? 1.0 : 0.5;
            long double off = 1.0L;
            for (int j = -32; j <= 32 && i != 0 && i != 63; ++j) {
                const double v = (double)(1.0L / m) * (1 + j * 0x1p-40);
                const long double l = ln(i, v);
                if (fabsl(l - (double)l) < off) off = fabsl(l - (double)l), inv[i] = v;
            }
        }
    }
    // x = 2^(e + 1) (m/2): ln x = (e + 1) ln 2 + ln(m inv) - ln(2 inv)
    static long double ln(int i, double v) { return -logl(i >= kHalf ? 2.0L * v : (long double)v); }
};

// the tables' entries in order (host)
template <typename F>
inline void table(F &&put) {
    static const LogTab t;
    for (int i = 0; i < 64; ++i) put((long double)t.inv[i], LogTab::ln(i, t.inv[i]));
    for (int i = 0; i < 128; ++i) {
        const long double a = 3.14159265358979323846264338327950288L * i / 64;
        put(i % 128 == 32 || i == 96 ? 0.0L : cosl(a), i % 64 == 0 ? 0.0L : sinl(a));
    }
    for (int i = 0; i < 32; ++i) {
        const long double v = exp2l(i / 32.0L);
        put((long double)(double)v, v - (double)v);
    }
}

// ln(2^sh x) for normal x > 0 (no zero, infinity or NaN: the callers' are
// k + 0 >= 1 and w + 1/2)
template <bool Comp = true>
__device__ __forceinline__ double log_t(const cx<double> *tab, double x, int sh) {
    const uint64_t b = __double_as_longlong(x);
    const uint32_t hi = (uint32_t)(b >> 32);
    const cx<double> t = tab[kLog + ((hi >> 14) & 63)];
    const int e = (int)((hi + ((64u - kHalf) << 14)) >> 20) - 1023 + sh;
    const double m = __longlong_as_double((int64_t)((b & 0x000FFFFFFFFFFFFFull) | 0x3FF0000000000000ull));
    const double r = fma(m, t.x, -1.0);  // |r| < 2^-6
    double p = fma(r, 1.0 / 9, -1.0 / 8);
    p = fma(r, p, 1.0 / 7);
    p = fma(r, p, -1.0 / 6);
    p = fma(r, p, 1.0 / 5);
    p = fma(r, p, -1.0 / 4);
    p = fma(r, p, 1.0 / 3);
    p = fma(r, p, -1.0 / 2);
    // ln 2 in two parts, the first with 42 significant bits: e times one rounded
    // constant would bias every logarithm of an octave by the same amount
    p = fma((double)e, 5.497923018708371e-14, fma(r * r, p, r));
    const double s = fma((double)e, 0.6931471805598903, t.y);
    if constexpr (!Comp) return s + p;
    // The sum's rounding error (Fast2Sum: e ln 2 >= ln c unless e = 0) counts: q's
    // exponent has alpha times the logarithm's error.  Without it q was 7.2 units of
    // 2^-53 off (rms over the draws' alpha, f_knee and k), with it and with the library 5.5.
    const double ds = fma((double)e, 0.6931471805598903, -s) + t.y;
    return s + (p + ds);
}

// e^x, x held to +-Lim (of 800: 0 and infinity); NaN stays NaN
template <int Lim = 800>
__device__ __forceinline__ double exp_t(const cx<double> *tab, double x) {
    x = x < -Lim ? -Lim : (x > Lim ? Lim : x);
    const double n = __builtin_rint(x * 46.16624130844683);  // 32 / ln 2
    const int j = (int)n;
    // ln 2 / 32 in two parts, the first with 32 significant bits: n times it is exact
    double r = fma(n, -0.02166084938653512, x);
    r = fma(n, -5.9631716539705866e-12, r);
    double p = fma(r, 1.0 / 720, 1.0 / 120);
    p = fma(r, p, 1.0 / 24);
    p = fma(r, p, 1.0 / 6);
    p = fma(r, p, 0.5);
    p = fma(r * r, p, r);
    const cx<double> t = tab[kExp + (j & 31)];
    return __builtin_ldexp(t.x + fma(t.x, p, t.y), j >> 5);
}

// cos and sin of 2 pi (w + 1/2) / 2^32
__device__ __forceinline__ cx<double> cis_t(const cx<double> *tab, uint32_t w) {
    const cx<double> t = tab[kCis + ((w + (1u << 24)) >> 25 & 127)];
    const int d = (int)(w << 7) >> 7;  // the rest, in [-2^24, 2^24)
    const double a = ((double)d + 0.5) * 1.4629180792671596e-9;  // 2 pi / 2^32
    const double z = a * a;
    double s = fma(z, -1.0 / 5040, 1.0 / 120);
    s = fma(z, s, -1.0 / 6);
    s = fma(a * z, s, a);
    double c = fma(z, -1.0 / 720, 1.0 / 24);
    c = fma(z, c, -0.5) * z;  // cos - 1
    return {t.x + fma(t.x, c, -(t.y * s)), t.y + fma(t.y, c, t.x * s)};
}

// square root of a normal x > 0 far from the ends of the range: the coupled
// iteration for sqrt(x) and 1 / (2 sqrt(x)) (Goldschmidt) from the hardware's estimate of
// 1 / sqrt(x), and one residual step
__device__ __forceinline__ double sqrt_t(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}

// q = k^malpha e^(malpha lbase), k >= 1: one exponential (the square of its half has
// twice that one's error).  Lim = kRoot holds q to 1e-289 ... 1e289, where sqrt_t takes
// it: sqrt(q) / (1 + q) and (w1 + sqrt(q) w2) / (1 + q) are then within 1e-144 of their
// limits.
constexpr int kRoot = 667;
template <int Lim = 800>
__device__ __forceinline__ double pow_t(const cx<double> *tab, uint32_t k, double malpha, double lbase) {
    return exp_t<Lim>(tab, malpha * (log_t(tab, (double)k, 0) + lbase));
}

// 1 / x for x >= 1 to DBL_MAX / 4, beyond which it is subnormal (0 at infinity
// alone; NaN stays NaN): Newton's iteration y (2 - x y) from the hardware's estimate
__device__ __forceinline__ double rcp_t(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    y = fma(fma(-x, y, 1.0), y, y);
    return x == (double)INFINITY ? 0.0 : y;
}

}  // namespace c3d
