// The FP64 mode functions (csrc/fp64fn.h) compiled for the host, against 80-bit
// references: largest and rms errors in units of 2^-53 of the result, one line each.
// The two hardware estimates are replaced by float ones (24 bits; the hardware's
// have at least as many).
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

static inline double as_double(int64_t v) {
    double d;
    memcpy(&d, &v, 8);
    return d;
}
static inline int64_t as_bits(double d) {
    int64_t v;
    memcpy(&v, &d, 8);
    return v;
}
static inline double float_rsq(double x) {
    int e;
    double m = frexp(x, &e);
    if (e & 1) m *= 0.5, ++e;
    return ldexp((double)(float)(1.0 / sqrt(m)), -e / 2);
}
static inline double float_rcp(double x) {
    if (!std::isfinite(x)) return 1.0 / x;
    int e;
    const double m = frexp(x, &e);
    return ldexp((double)(float)(1.0 / m), -e);
}
#define __builtin_amdgcn_rsq float_rsq
#define __builtin_amdgcn_rcp float_rcp
#define __longlong_as_double as_double
#define __double_as_longlong as_bits
using std::fma;
#include "../paper_2201_03509_amd/csrc/fp64fn.h"

struct Err {
    double most = 0, sum = 0;
    long n = 0;
    void add(long double got, long double want) {
        const double e = (double)(fabsl(got - want) / fabsl(want)) * 0x1p53;
        if (!(e <= most)) most = e;  // NaN too
        sum += e * e;
        ++n;
    }
    void print(const char *name) const { printf("%s %.4f %.4f\n", name, most, sqrt(sum / n)); }
};

int main() {
    std::vector<cx<double>> tab;
    c3d::table([&](long double x, long double y) { tab.push_back({(double)x, (double)y}); });
    std::mt19937_64 g(2);
    auto u = [&] { return (double)(g() >> 11) * 0x1p-53; };
    Err log_k, log_u, ex, rt, rc, q, q_lib, inv, inv_lib, sq, sq_lib;
    for (int i = 0; i < 2000000; ++i) {
        const uint32_t k = i < 4096 ? i + 2 : 2 + (uint32_t)(1e6 * exp(-12.0 * u()));
        const uint32_t w = i < 100 ? 0xFFFFFFFFu - i : i < 200 ? i - 100 : (uint32_t)g();
        log_k.add(c3d::log_t(tab.data(), (double)k, 0), logl((long double)k));
        const double lu = c3d::log_t<false>(tab.data(), (double)w + 0.5, -32);
        log_u.add(lu, logl(((long double)w + 0.5L) * 0x1p-32L));
        const double y = 80 * u() - 40;
        ex.add(c3d::exp_t(tab.data(), y), expl((long double)y));
        rt.add(c3d::sqrt_t(-lu), sqrtl(-(long double)lu));
        rc.add(c3d::rcp_t(1.0 + exp(y)), 1.0L / (1.0 + exp(y)));
        // the draws' parameters: 3000 to 1e6 modes, f_knee 3 mHz to 0.3 Hz, alpha -0.5 to -2.5
        const double M = pow(10.0, 3.5 + 2.5 * u()), lbase = log(32.5 / (2 * M * pow(10.0, -2.5 + 2 * u())));
        const double malpha = 0.5 + 2 * u();
        const uint32_t km = 1 + (uint32_t)(pow(M, u()) - 1);
        const long double qx = expl((long double)malpha * (logl((long double)km) + (long double)lbase));
        const double ql = exp(malpha * (log((double)km) + lbase));
        const double qt = c3d::pow_t<c3d::kRoot>(tab.data(), km, malpha, lbase);
        q.add(qt, qx);
        q_lib.add(ql, qx);
        inv.add(c3d::rcp_t(1.0 + qt), 1 / (1 + qx));
        inv_lib.add(1.0 / (1.0 + ql), 1 / (1 + qx));
        sq.add(c3d::sqrt_t(qt), sqrtl(qx));
        sq_lib.add(sqrt(ql), sqrtl(qx));
    }
    log_k.print("log_k");
    log_u.print("log_u");
    ex.print("exp");
    rt.print("sqrt");
    rc.print("rcp");
    q.print("q");
    q_lib.print("q_lib");
    inv.print("inv");
    inv_lib.print("inv_lib");
    sq.print("sq");
    sq_lib.print("sq_lib");
    const double inf = (double)INFINITY, big = 0x1.fffffffffffffp1021;  // DBL_MAX / 4
    const bool ends = c3d::exp_t(tab.data(), 900) == inf && c3d::exp_t(tab.data(), -900) == 0 &&
                      c3d::exp_t(tab.data(), inf) == inf && c3d::exp_t(tab.data(), -inf) == 0 &&
                      std::isnan(c3d::exp_t(tab.data(), (double)NAN)) && c3d::rcp_t(inf) == 0 &&
                      std::isnan(c3d::rcp_t((double)NAN)) && fabs(c3d::rcp_t(1e305) * 1e305 - 1) < 1e-15 &&
                      fabs(c3d::rcp_t(big) * big - 1) < 1e-15 && c3d::log_t(tab.data(), 1.0, 0) == 0 &&
                      c3d::pow_t(tab.data(), 2, 1e4, 0.0) == inf && c3d::pow_t(tab.data(), 2, -1e4, 0.0) == 0 &&
                      std::isnan(c3d::pow_t<c3d::kRoot>(tab.data(), 2, (double)NAN, 0.0)) &&
                      c3d::sqrt_t(c3d::pow_t<c3d::kRoot>(tab.data(), 2, -inf, 0.0)) < 1e-144 &&
                      c3d::sqrt_t(c3d::pow_t<c3d::kRoot>(tab.data(), 2, inf, 0.0)) > 1e144;
    printf("ends %d 0\n", ends);
    return 0;
}
