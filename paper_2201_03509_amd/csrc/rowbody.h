// Body of the row pass compiled per row length L (rowc.hip: FP32, rowd.hip and
// rows.hip: FP64): the rows k1 and M1 - k1 of one segment (0 < k1 < M1/2, the
// rows holding each other's mirror modes) in one block of C3_ROW_NT threads.
//
// Everything the generic row kernel (fft.hip) decides at run time is fixed
// here at compile time: the three stage radices (rowc.h), each thread's
// butterflies, the LDS strides and the index arithmetic; the stage
// twiddles are loaded whole from a per-length table (one base address per
// butterfly) instead of being built by chained products, and the mode loop
// takes w_N^k = w_N^k1 w_2L^k2 from a block constant and a table of L values.
// The first forward stage reads the two rows from memory and the last inverse
// stage writes them back.  Modes: 0 (n_corr constrained realisation), 1 (the
// chi^2's Whittle sums) and 4 (the periodogram of the noise-parameter draw):
// forward stages only, nothing written back; 2 (Fourier-diagonal filters).
// Mode 3 runs on the generic kernel.  The
// rows k1 = 0 and k1 = M1/2, each holding its own mirror modes, come two to a
// task (of one segment or two).
#pragma once
#include "fftmode.h"
#include "fp64fn.h"
#include "rowc.h"

namespace {
using c3::FftArgs;
using namespace c3fft;
using namespace c3rowc;

constexpr int NT = C3_ROW_NT;  // set by the including file

extern __shared__ __attribute__((aligned(16))) unsigned char c3_rowc_lds[];

template <typename T>
constexpr bool F64 = sizeof(T) == 8;

// one Stockham stage of the two interleaved rows (row b's element i at LDS
// index 2 i + b).  IO 1: inputs from the rows in memory (first forward
// stage); IO 2: outputs to the rows in memory (last inverse stage).
template <typename T, int L, int S, int DIR, int IO>
__device__ __forceinline__ void rstage(cx<T> *buf, const cx<T> *g0, const cx<T> *g1, cx<T> *o0,
                                       cx<T> *o1, const cx<T> *__restrict__ tw) {
    constexpr c3rowc::Plan P = plan(L, F64<T>);
    constexpr int R = P.r[S];
    constexpr int NS = row_ns(L, S, F64<T>);
    constexpr int LR = L / R;
    constexpr int NB = 2 * LR;  // butterflies of both rows
    constexpr int KB = (NB + NT - 1) / NT;
    constexpr long TOFF = S > 0 ? stage_off(L, S, F64<T>) : 0;
    cx<T> v[KB][R];
    int ob[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int q = (int)threadIdx.x + kb * NT;
        ob[kb] = -1;
        if (NB % NT == 0 || q < NB) {
            const int b = q & 1, j = q >> 1;
            if constexpr (IO == 1) {
                const cx<T> *g = b ? g1 : g0;
#pragma unroll
                for (int t = 0; t < R; ++t) v[kb][t] = g[j + t * LR];
            } else {
#pragma unroll
                for (int t = 0; t < R; ++t) v[kb][t] = buf[2 * (j + t * LR) + b];
            }
            const int jd = j / NS, k = j - jd * NS;
            if constexpr (S > 0) {
                const cx<T> *w = tw + TOFF + k * (R - 1);
#pragma unroll
                for (int t = 1; t < R; ++t) {
                    const cx<T> wt = w[t - 1];
                    v[kb][t] = DIR < 0 ? cmul(v[kb][t], wt) : cmulc(v[kb][t], wt);
                }
            }
            dft_any<R, DIR>(v[kb]);
            if constexpr (IO == 2) {
                cx<T> *o = b ? o1 : o0;  // last stage: jd = 0
#pragma unroll
                for (int t = 0; t < R; ++t) o[k + t * NS] = v[kb][t];
            } else {
                ob[kb] = 2 * (jd * NS * R + k) + b;
            }
        }
    }
    if constexpr (IO == 2) return;
    if constexpr (IO == 0) __syncthreads();  // in place: every read before any write
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
        if (ob[kb] >= 0) {
#pragma unroll
            for (int t = 0; t < R; ++t) buf[ob[kb] + 2 * t * NS] = v[kb][t];
        }
    __syncthreads();
}

// nhat_k of the n_corr draw (the same value as cr_mode) with the draw's
// constants folded: s0 W1 = sqrt(c log2 u0) (cos 2 pi u1, sin 2 pi u1) with
// c = -sigma0^2 ln 2 (Box-Muller radius sqrt(-2 ln u0) times 1/sqrt 2 and
// sigma0), and s0 sqrt(q) W2 = sqrt(c q log2 u2) (cos 2 pi u3, sin 2 pi u3).
// k > 0 and k < M here, so both draws are complex.
template <typename T>
struct FastCtx;
template <>
struct FastCtx<float> {
    float c;        // -sigma0^2 ln 2
    float isq;      // 1 / sqrt(N), times the 1/2 of the real-spectrum split
    float oscale;   // the output scale sqrt(N)/M, times the 1/2 of the re-pack
    float malpha, lbase2;
};

__device__ __forceinline__ cx<float> cr_fast(const ModeCtx &mc, const FastCtx<float> &fc, uint32_t k, cx<float> E) {
    const float x = fc.malpha * (__builtin_amdgcn_logf((float)k) + fc.lbase2);
    const float q = __builtin_amdgcn_exp2f(x);  // (f_k / f_knee)^-alpha = sigma0^2 / P_k
    const float inv = __builtin_amdgcn_rcpf(1.0f + q) * fc.oscale;
    cx<float> out = {E.x * fc.isq, E.y * fc.isq};
    if (!mc.mean_only) {
        const uint4 w = philox4x32_10(make_uint4(k, mc.it_lo, mc.it_hi, mc.seed_hi), mc.key);
        const float sc = 2.3283064365386963e-10f, off = 1.1641532182693481e-10f;  // (x + 1/2) 2^-32
        const float u0 = fmaf((float)w.x, sc, off), u1 = fmaf((float)w.y, sc, off);
        const float u2 = fmaf((float)w.z, sc, off), u3 = fmaf((float)w.w, sc, off);
        const float a0 = __builtin_amdgcn_sqrtf(fc.c * __builtin_amdgcn_logf(u0));
        const float a1 = __builtin_amdgcn_sqrtf(fc.c * q * __builtin_amdgcn_logf(u2));
        out.x = fmaf(a0, __builtin_amdgcn_cosf(u1), fmaf(a1, __builtin_amdgcn_cosf(u3), out.x));
        out.y = fmaf(a0, __builtin_amdgcn_sinf(u1), fmaf(a1, __builtin_amdgcn_sinf(u3), out.y));
    }
    return {out.x * inv, out.y * inv};
}

// The same in FP64 with the table functions of fp64fn.h: W1 = sqrt(-ln u0)
// (cos 2 pi u1, sin 2 pi u1), W2 likewise.
template <>
struct FastCtx<double> {
    const cx<double> *tab;  // the block's tables in LDS
    double s0;              // sigma0
    double isq, oscale;     // as above
    double malpha, lbase;   // -alpha, ln(fsamp / (N fknee))
    double is2;             // 1 / sigma0^2
};

// q_k (q_0 = 0), and its square root where that is drawn with (Lim = kRoot)
template <int Lim>
__device__ __forceinline__ double q_row(const FastCtx<double> &fc, int64_t k) {
    return k > 0 ? c3d::pow_t<Lim>(fc.tab, (uint32_t)k, fc.malpha, fc.lbase) : 0.0;
}
__device__ __forceinline__ double root_row(double q, int64_t k) { return k > 0 ? c3d::sqrt_t(q) : 0.0; }
// the draw (wa, wb) of a complex mode: sqrt(-ln u) (cos 2 pi v, sin 2 pi v)
__device__ __forceinline__ cx<double> draw_pair(const FastCtx<double> &fc, uint32_t wa, uint32_t wb) {
    const double r = c3d::sqrt_t(-c3d::log_t<false>(fc.tab, (double)wa + 0.5, -32));
    const cx<double> c = c3d::cis_t(fc.tab, wb);
    return {r * c.x, r * c.y};
}

__device__ __forceinline__ cx<double> cr_fast(const ModeCtx &mc, const FastCtx<double> &fc, uint32_t k,
                                              cx<double> E) {
    const double q = c3d::pow_t<c3d::kRoot>(fc.tab, k, fc.malpha, fc.lbase);
    const double inv = c3d::rcp_t(1.0 + q) * fc.oscale;
    cx<double> out = {E.x * fc.isq, E.y * fc.isq};
    if (!mc.mean_only) {
        const uint4 w = philox4x32_10(make_uint4(k, mc.it_lo, mc.it_hi, mc.seed_hi), mc.key);
        const cx<double> W1 = draw_pair(fc, w.x, w.y), W2 = draw_pair(fc, w.z, w.w);
        const double sq = c3d::sqrt_t(q);
        out.x = fma(fc.s0, fma(sq, W2.x, W1.x), out.x);
        out.y = fma(fc.s0, fma(sq, W2.y, W1.y), out.y);
    }
    return {out.x * inv, out.y * inv};
}

// the real modes k = 0 (q_0 = 0) and k = M: one normal each of W1, W2, no
// output scale
__device__ __forceinline__ cx<float> cr_real(const ModeCtx &mc, const FastCtx<float> &, int64_t k, cx<float> E) {
    return cr_mode<float>(mc, k, E);
}
__device__ __forceinline__ cx<double> cr_real(const ModeCtx &mc, const FastCtx<double> &fc, int64_t k,
                                              cx<double> E) {
    const double q = q_row<c3d::kRoot>(fc, k);
    double v = E.x * mc.invsqrtN;
    if (!mc.mean_only) {
        const uint4 w = philox4x32_10(make_uint4((uint32_t)k, mc.it_lo, mc.it_hi, mc.seed_hi), mc.key);
        const double W1 = draw_pair(fc, w.x, w.y).x, W2 = draw_pair(fc, w.z, w.w).x;
        v = fma(fc.s0 * 1.41421356237309504880, fma(root_row(q, k), W2, W1), v);
    }
    return {v * c3d::rcp_t(1.0 + q), 0.0};
}

// filt_mode, x0_mode and whittle_mode (fftmode.h): as they are in FP32, on the
// tables in FP64
__device__ __forceinline__ cx<float> filt_row(const ModeCtx &mc, const FastCtx<float> &, int64_t k, cx<float> E,
                                              int which) {
    return filt_mode(mc, k, E, which);
}
__device__ __forceinline__ cx<double> filt_row(const ModeCtx &mc, const FastCtx<double> &fc, int64_t k,
                                               cx<double> E, int which) {
    const double q = q_row<800>(fc, k);
    // 4 / (1 + q): the quarter of 1 + q has a normal reciprocal up to the largest q
    const double i1q = c3d::rcp_t(fma(q, 0.25, 0.25));
    const double h = which == 0   ? q * fc.is2
                     : which == 1 ? fc.s0 * fc.s0 * (0.25 * i1q)
                                  : 0.25 * q * i1q * fc.is2;
    return cscale(E, mc.invsqrtN * h);
}
__device__ __forceinline__ cx<float> x0_row(const ModeCtx &mc, const FastCtx<float> &, int64_t k, cx<float> E) {
    return x0_mode(mc, k, E);
}
__device__ __forceinline__ cx<double> x0_row(const ModeCtx &mc, const FastCtx<double> &fc, int64_t k,
                                             cx<double> E) {
    const double q = q_row<c3d::kRoot>(fc, k), i1q = c3d::rcp_t(1.0 + q);
    cx<double> v = cscale(E, mc.invsqrtN * (fc.s0 * fc.s0 * i1q));
    if (!mc.mean_only) {
        const uint4 w = philox4x32_10(make_uint4((uint32_t)k, mc.it_lo, mc.it_hi, mc.seed_hi), mc.key);
        const bool real = k == 0 || k == mc.M;
        const double h = fc.s0 * i1q * root_row(q, k) * (real ? 1.41421356237309504880 : 1.0);
        const cx<double> W = draw_pair(fc, w.z, w.w);
        v.x = fma(h, W.x, v.x);
        if (!real) v.y = fma(h, W.y, v.y);
    }
    return v;
}
__device__ __forceinline__ void whittle_row(const ModeCtx &mc, const FastCtx<float> &, int64_t k, cx<float> E,
                                            Wsum &s) {
    whittle_mode(mc, k, E, s);
}
__device__ __forceinline__ void whittle_row(const ModeCtx &mc, const FastCtx<double> &fc, int64_t k, cx<double> E,
                                            Wsum &s) {
    const double lr = c3d::log_t(fc.tab, (double)(uint32_t)k, 0) + fc.lbase;
    const double ip = (E.x * E.x + E.y * E.y) * mc.iscale * c3d::exp_t(fc.tab, mc.malpha * lr);
    s.a += ip + (mc.l2s0 - mc.malpha * lr);
    s.b += 1.0 - ip;
    s.c = fma(1.0 - ip, lr, s.c);
}

template <typename T>
__device__ __forceinline__ FastCtx<T> fast_ctx(const ModeCtx &mc, const cx<T> *tab) {
    FastCtx<T> fc;
    if constexpr (F64<T>) {
        fc.tab = tab;
        fc.s0 = mc.sigma0;
        fc.isq = 0.5 * mc.invsqrtN;
        fc.oscale = 0.5 * mc.outscale;
        fc.malpha = mc.malpha;
        fc.lbase = mc.lbase;
        fc.is2 = 1.0 / (mc.sigma0 * mc.sigma0);
    } else {
        fc.c = (float)(-mc.sigma0 * mc.sigma0 * 0.69314718055994530942);
        fc.isq = (float)(0.5 * mc.invsqrtN);
        fc.oscale = (float)(0.5 * mc.outscale);
        fc.malpha = (float)mc.malpha;
        fc.lbase2 = (float)mc.lbase2;
    }
    return fc;
}

// The real-spectrum split of a mirror pair: from Z_k (za) and Z_{M-k} (zb) of
// the packed transform and w = w_N^k, twice E_k and twice E_{M-k}:
// 2A = Zk + conj Zp, 2B = -i (Zk - conj Zp), 2 E_k = 2A + w_N^k 2B, and the
// partner from conj A, conj B and w_N^(M-k) = -conj(w_N^k).
template <typename T>
__device__ __forceinline__ void split_pair(cx<T> za, cx<T> zb, cx<T> w, cx<T> &ek,
                                           cx<T> &ep) {
    const cx<T> A = {za.x + zb.x, za.y - zb.y};
    const cx<T> D = {za.x - zb.x, za.y + zb.y};
    const cx<T> B = {D.y, -D.x};
    ek = cadd(A, cmul(w, B));
    const cx<T> wp = {-w.x, w.y};
    ep = cadd(cconj(A), cmul(wp, cconj(B)));
}

// The re-pack of a mirror pair: Z'_k = (nk + conj np)/2 + i (nk - conj np)
// conj(w_N^k)/2 and its partner (the factors 1/2 are in the modes' scales).
template <typename T>
__device__ __forceinline__ void repack_pair(cx<T> nk, cx<T> np, cx<T> w, cx<T> &zk,
                                            cx<T> &zq) {
    const cx<T> A = {nk.x + np.x, nk.y - np.y};
    const cx<T> D = {nk.x - np.x, nk.y + np.y};
    const cx<T> B = cmulc(D, w);
    zk = cx<T>{A.x - B.y, A.y + B.x};
    const cx<T> Bq = cmul(cconj(D), w);
    zq = cx<T>{A.x - Bq.y, -A.y + Bq.x};
}

// The modes of a row that holds its own mirror modes (modes 0 and 2), in LDS
// row b: k1 = 0 pairs k = M1 k2 with M - k at k2' = (L - k2) mod L and holds
// k = 0 and k = M (both real, from Z_0); k1 = M1/2 pairs k2 with
// L - 1 - k2.  A pair with k2' = k2 is the single mode k = M/2.
template <typename T, int MODE>
__device__ __forceinline__ void self_row_modes(const FftArgs &a, int L, cx<T> *buf, int seg, int k1, int b,
                                               const cx<T> *twh) {
    const SegInfo sg = a.segs[seg];
    const FftPlan &p = a.plans[sg.plan];
    const int M1 = p.M1, M = p.M;
    const ModeCtx mc = mode_ctx<MODE>(a, seg, sg.band, M);
    const FastCtx<T> fc = fast_ctx<T>(mc, buf + 2 * L);
    const T osc2 = (T)(0.5 * mc.outscale), osc4 = (T)(0.25 * mc.outscale);
    const cx<T> wa = twN((const cx<T> *)a.twpool, p, k1);
    const bool zero = k1 == 0;
    const int npair = zero ? L / 2 + 1 : (L + 1) / 2;
    for (int k2 = threadIdx.x; k2 < npair; k2 += NT) {
        const int e = 2 * k2 + b;
        if (zero && k2 == 0) {
            // E_0 = Re Z_0 + Im Z_0 and E_M = Re Z_0 - Im Z_0, real modes
            const cx<T> z = buf[e];
            const cx<T> E0 = {z.x + z.y, 0}, EM = {z.x - z.y, 0};
            cx<T> n0, nM;
            if constexpr (MODE == 0) {
                n0 = cr_real(mc, fc, 0, E0);
                nM = cr_real(mc, fc, M, EM);
            } else {
                n0 = a.which == 3 ? x0_row(mc, fc, 0, E0) : filt_row(mc, fc, 0, E0, a.which);
                nM = a.which == 3 ? x0_row(mc, fc, M, EM) : filt_row(mc, fc, M, EM, a.which);
            }
            const T h = (T)0.5 * (T)mc.outscale;
            buf[e] = cx<T>{h * (n0.x + nM.x), h * (n0.x - nM.x)};
            continue;
        }
        const int pk2 = zero ? L - k2 : L - 1 - k2;
        const int ep = 2 * pk2 + b;
        const cx<T> w = cmul(wa, twh[k2]);
        const int64_t k = k1 + (int64_t)M1 * k2, kp = (int64_t)M - k;
        cx<T> Ek, Ep;
        split_pair(buf[e], buf[ep], w, Ek, Ep);
        cx<T> nk, np;
        if constexpr (MODE == 0) {
            nk = cr_fast(mc, fc, (uint32_t)k, Ek);
            np = pk2 == k2 ? nk : cr_fast(mc, fc, (uint32_t)kp, Ep);
        } else if (a.which == 3) {  // not linear in E (its drawn term): E itself
            nk = cscale(x0_row(mc, fc, k, cscale(Ek, (T)0.5)), osc2);
            np = pk2 == k2 ? nk : cscale(x0_row(mc, fc, kp, cscale(Ep, (T)0.5)), osc2);
        } else {
            nk = cscale(filt_row(mc, fc, k, Ek, a.which), osc4);
            np = pk2 == k2 ? nk : cscale(filt_row(mc, fc, kp, Ep, a.which), osc4);
        }
        cx<T> zk, zq;
        repack_pair(nk, np, w, zk, zq);
        buf[e] = zk;
        if (pk2 != k2) buf[ep] = zq;
    }
}

// The modes of rows k1 and M1 - k1 (LDS rows 0 and 1), which hold each
// other's mirror modes: mode k = k1 + M1 k2 of row 0 pairs with M - k at
// k2' = L - 1 - k2 of row 1.
template <typename T, int MODE>
__device__ __forceinline__ void pair_row_modes(const FftArgs &a, int L, cx<T> *buf, int seg, const SegInfo &sg,
                                               const FftPlan &p, int ka, const cx<T> *twh) {
    const int M1 = p.M1, M = p.M;
    const cx<T> *pool = (const cx<T> *)a.twpool;
    const ModeCtx mc = mode_ctx<MODE>(a, seg, sg.band, M);
    const FastCtx<T> fc = fast_ctx<T>(mc, buf + 2 * L);
    const cx<T> wa = twN(pool, p, ka);  // w_N^k1; w_N^(k1 + M1 k2) = w_N^k1 w_2L^k2
    const T osc2 = (T)(0.5 * mc.outscale), osc4 = (T)(0.25 * mc.outscale);
    // The two factors 1/2 of the split and of the re-pack and the output
    // scale are applied once per mode: E below is twice the spectrum value
    // (halved in fc.isq or the mode scales) and nk, np come out already
    // times sqrt(N)/(2M).
    for (int k2 = threadIdx.x; k2 < L; k2 += NT) {
        const int pk2 = L - 1 - k2;  // the partner mode M - k sits in row 1
        const cx<T> Za = buf[2 * k2], Zb = buf[2 * pk2 + 1];
        const cx<T> w = cmul(wa, twh[k2]);
        const int64_t k = ka + (int64_t)M1 * k2, kp = (int64_t)M - k;
        cx<T> Ek, Ep;
        split_pair(Za, Zb, w, Ek, Ep);
        cx<T> nk, np;
        if constexpr (MODE == 0) {
            nk = cr_fast(mc, fc, (uint32_t)k, Ek);
            // one FP64 draw at a time: both at once spill
            if constexpr (F64<T>) __builtin_amdgcn_sched_barrier(0);
            np = cr_fast(mc, fc, (uint32_t)kp, Ep);
        } else {
            if (a.which == 3) {  // not linear in E (its drawn term): E itself
                nk = cscale(x0_row(mc, fc, k, cscale(Ek, (T)0.5)), osc2);
                np = cscale(x0_row(mc, fc, kp, cscale(Ep, (T)0.5)), osc2);
            } else {
                nk = cscale(filt_row(mc, fc, k, Ek, a.which), osc4);
                np = cscale(filt_row(mc, fc, kp, Ep, a.which), osc4);
            }
        }
        cx<T> zk, zq;
        repack_pair(nk, np, w, zk, zq);
        buf[2 * k2] = zk;
        buf[2 * pk2 + 1] = zq;
    }
}

// Whittle sums (the chi^2's noise term, mode 1) of rows k1 and M1 - k1: every
// mode k and its partner M - k, E_k from the split (halved: the split gives
// twice E)
template <typename T>
__device__ __forceinline__ Wsum pair_row_whittle(const FftArgs &a, int L, const cx<T> *buf, int seg,
                                                 const SegInfo &sg, const FftPlan &p, int ka,
                                                 const cx<T> *twh) {
    const ModeCtx mc = mode_ctx<1>(a, seg, sg.band, p.M);
    const FastCtx<T> fc = fast_ctx<T>(mc, buf + 2 * L);
    const cx<T> wa = twN((const cx<T> *)a.twpool, p, ka);
    Wsum ws = {0, 0, 0};
    for (int k2 = threadIdx.x; k2 < L; k2 += NT) {
        const int pk2 = L - 1 - k2;
        const cx<T> w = cmul(wa, twh[k2]);
        const int64_t k = ka + (int64_t)p.M1 * k2;
        cx<T> Ek, Ep;
        split_pair(buf[2 * k2], buf[2 * pk2 + 1], w, Ek, Ep);
        whittle_row(mc, fc, k, cscale(Ek, (T)0.5), ws);
        whittle_row(mc, fc, (int64_t)p.M - k, cscale(Ep, (T)0.5), ws);
    }
    return ws;
}

// the same for a row that holds its own mirror modes (pairs as in
// self_row_modes; row 0 adds the real mode k = M, E_M = Re Z_0 - Im Z_0, and
// leaves out the mean)
template <typename T>
__device__ __forceinline__ Wsum self_row_whittle(const FftArgs &a, int L, const cx<T> *buf, int seg, int k1, int b,
                                                 const cx<T> *twh) {
    const SegInfo sg = a.segs[seg];
    const FftPlan &p = a.plans[sg.plan];
    const int M1 = p.M1, M = p.M;
    const ModeCtx mc = mode_ctx<1>(a, seg, sg.band, M);
    const FastCtx<T> fc = fast_ctx<T>(mc, buf + 2 * L);
    const cx<T> wa = twN((const cx<T> *)a.twpool, p, k1);
    const bool zero = k1 == 0;
    const int npair = zero ? L / 2 + 1 : (L + 1) / 2;
    Wsum ws = {0, 0, 0};
    for (int k2 = threadIdx.x; k2 < npair; k2 += NT) {
        if (zero && k2 == 0) {
            const cx<T> z = buf[b];
            whittle_row(mc, fc, (int64_t)M, cx<T>{z.x - z.y, 0}, ws);
            continue;
        }
        const int pk2 = zero ? L - k2 : L - 1 - k2;
        const cx<T> w = cmul(wa, twh[k2]);
        const int64_t k = k1 + (int64_t)M1 * k2;
        cx<T> Ek, Ep;
        split_pair(buf[2 * k2 + b], buf[2 * pk2 + b], w, Ek, Ep);
        whittle_row(mc, fc, k, cscale(Ek, (T)0.5), ws);
        if (pk2 != k2) whittle_row(mc, fc, (int64_t)M - k, cscale(Ep, (T)0.5), ws);
    }
    return ws;
}

// Periodogram of a row pair's modes into the block's LDS bins (mode 4, the
// noise-parameter draw): |E_k|^2 / N for every mode k and its partner M - k
// of rows k1 and M1 - k1 (E from the split, halved).  Every lane of a wave
// walks the same number of steps (hist_add is a wave operation).
template <typename T>
__device__ __forceinline__ void pair_row_periodogram(const FftArgs &a, int L, const cx<T> *buf, int seg,
                                                     const SegInfo &sg, const FftPlan &p, int ka,
                                                     const cx<T> *twh, double *hist) {
    const ModeCtx mc = mode_ctx<4>(a, seg, sg.band, p.M);
    const double s2 = 0.25 * mc.invsqrtN * mc.invsqrtN;  // the split gives twice E
    const cx<T> wa = twN((const cx<T> *)a.twpool, p, ka);
    for (int base = 0; base < L; base += NT) {
        const int k2 = base + (int)threadIdx.x;
        int bk = -1, bp = -1;
        double vk = 0.0, vp = 0.0;
        if (k2 < L) {
            const int pk2 = L - 1 - k2;
            const cx<T> w = cmul(wa, twh[k2]);
            const int64_t k = ka + (int64_t)p.M1 * k2;
            cx<T> Ek, Ep;
            split_pair(buf[2 * k2], buf[2 * pk2 + 1], w, Ek, Ep);
            vk = ((double)Ek.x * Ek.x + (double)Ek.y * Ek.y) * s2;
            vp = ((double)Ep.x * Ep.x + (double)Ep.y * Ep.y) * s2;
            bk = xi_bin(k);
            bp = xi_bin((int64_t)p.M - k);
        }
        hist_add(hist, bk, vk);
        hist_add(hist, bp, vp);
    }
}

// the same for a row that holds its own mirror modes (pairs as in
// self_row_modes; row 0 adds the real mode k = M and leaves out the mean)
template <typename T>
__device__ __forceinline__ void self_row_periodogram(const FftArgs &a, int L, const cx<T> *buf, int seg, int k1,
                                                     int b, const cx<T> *twh, double *hist) {
    const SegInfo sg = a.segs[seg];
    const FftPlan &p = a.plans[sg.plan];
    const int M1 = p.M1, M = p.M;
    const ModeCtx mc = mode_ctx<4>(a, seg, sg.band, M);
    const double s1 = mc.invsqrtN * mc.invsqrtN, s2 = 0.25 * s1;
    const cx<T> wa = twN((const cx<T> *)a.twpool, p, k1);
    const bool zero = k1 == 0;
    const int npair = zero ? L / 2 + 1 : (L + 1) / 2;
    for (int base = 0; base < npair; base += NT) {
        const int k2 = base + (int)threadIdx.x;
        int bk = -1, bp = -1;
        double vk = 0.0, vp = 0.0;
        if (k2 < npair) {
            if (zero && k2 == 0) {
                const cx<T> z = buf[b];
                const double em = (double)(z.x - z.y);  // E_M, real
                vk = em * em * s1;
                bk = xi_bin(M);
            } else {
                const int pk2 = zero ? L - k2 : L - 1 - k2;
                const cx<T> w = cmul(wa, twh[k2]);
                const int64_t k = k1 + (int64_t)M1 * k2;
                cx<T> Ek, Ep;
                split_pair(buf[2 * k2 + b], buf[2 * pk2 + b], w, Ek, Ep);
                vk = ((double)Ek.x * Ek.x + (double)Ek.y * Ek.y) * s2;
                bk = xi_bin(k);
                if (pk2 != k2) {
                    vp = ((double)Ep.x * Ep.x + (double)Ep.y * Ep.y) * s2;
                    bp = xi_bin((int64_t)M - k);
                }
            }
        }
        hist_add(hist, bk, vk);
        hist_add(hist, bp, vp);
    }
}

// the block's bins added to the segment's (FP64 atomics), then cleared
__device__ __forceinline__ void hist_flush(const FftArgs &a, double *hist, int seg) {
    __syncthreads();
    for (int i = threadIdx.x; i < C3_XI_NBIN; i += NT)
        if (hist[i] != 0.0) {
            atomicAdd(&a.bins[(int64_t)seg * C3_XI_NBIN + i], hist[i]);
            hist[i] = 0.0;
        }
    __syncthreads();
}

// block sum of a thread's Whittle sums, added to the segment's; red: 3 NT/64
// doubles of LDS that no thread reads or writes otherwise
__device__ __forceinline__ void whittle_flush(const FftArgs &a, double *red, Wsum ws, int seg) {
    double v[3] = {ws.a, ws.b, ws.c};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        double x = v[j];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
        if ((threadIdx.x & 63) == 0) red[j * (NT / 64) + (threadIdx.x >> 6)] = x;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double x = 0;
        for (int w = 0; w < NT / 64; ++w) x += red[threadIdx.x * (NT / 64) + w];
        atomicAdd(&a.whittle[(int64_t)seg * 4 + threadIdx.x], x);
    }
    __syncthreads();
}

// the forward stages; the first reads the two rows from memory
template <typename T, int L>
__device__ __forceinline__ void row_load(cx<T> *buf, const cx<T> *ya, const cx<T> *yb) {
    static_assert(c3rowc::plan(L, F64<T>).r[0] > 0, "row length without a stage plan");
    rstage<T, L, 0, -1, 1>(buf, ya, yb, nullptr, nullptr, nullptr);
}
template <typename T, int L>
__device__ __forceinline__ void row_fwd(cx<T> *buf, const cx<T> *tws) {
    rstage<T, L, 1, -1, 0>(buf, nullptr, nullptr, nullptr, nullptr, tws);
    rstage<T, L, 2, -1, 0>(buf, nullptr, nullptr, nullptr, nullptr, tws);
    if constexpr (stages(L, F64<T>) == 4) rstage<T, L, 3, -1, 0>(buf, nullptr, nullptr, nullptr, nullptr, tws);
}
// the inverse stages; the last writes the two rows back
template <typename T, int L>
__device__ __forceinline__ void row_inv(cx<T> *buf, cx<T> *ya, cx<T> *yb, const cx<T> *tws) {
    constexpr int last = stages(L, F64<T>) - 1;
    rstage<T, L, 0, 1, 0>(buf, nullptr, nullptr, nullptr, nullptr, tws);
    rstage<T, L, 1, 1, 0>(buf, nullptr, nullptr, nullptr, nullptr, tws);
    if constexpr (last == 3) rstage<T, L, 2, 1, 0>(buf, nullptr, nullptr, nullptr, nullptr, tws);
    rstage<T, L, last, 1, 2>(buf, nullptr, nullptr, ya, yb, tws);
}

// converged segments (masked draw): no load.  A task of two segments runs
// while either is active; the workspace rows of a converged one are not
// read again (its column passes return before any load or store).
__device__ __forceinline__ bool row_idle(const FftArgs &a, const RowTask &task) {
    return a.active && !a.active[task.seg] && !(task.pad[0] > 0 && a.active[task.pad[0] - 1]);
}

// everything between the forward and the inverse stages
template <typename T, int MODE>
__device__ __forceinline__ void row_mid(const FftArgs &a, int L, cx<T> *buf, const RowTask &task, const SegInfo &sg,
                                        const FftPlan &p, double *hist) {
    // a task of two rows that each hold their own mirror modes (k1 = 0 or
    // M1/2): pad[0] = 1 + the second row's segment, kb = its k1
    const bool self = task.pad[0] > 0;
    const int kb = task.pad[1] & 0xFFFF;
    // FP64: an odd row out is paired with itself (both LDS rows the same, the
    // same values written twice); its sums count once
    const bool twice = F64<T> && self && task.pad[0] - 1 == task.seg && kb == task.k1;
    const int seg = task.seg;
    const int ka = task.k1;  // 0 < ka < M1 / 2 (rows ka and M1 - ka), or a row of a self task
    const cx<T> *twh = (const cx<T> *)a.twpool + p.twh;

    if constexpr (MODE == 4) {
        for (int i = threadIdx.x; i < C3_XI_NBIN; i += NT) hist[i] = 0.0;
        __syncthreads();
        if (self) {
            const int seg1 = task.pad[0] - 1;
            self_row_periodogram<T>(a, L, buf, seg, ka, 0, twh, hist);
            hist_flush(a, hist, seg);
            if (!twice) {
                self_row_periodogram<T>(a, L, buf, seg1, kb, 1, twh, hist);
                hist_flush(a, hist, seg1);
            }
        } else {
            pair_row_periodogram<T>(a, L, buf, seg, sg, p, ka, twh, hist);
            hist_flush(a, hist, seg);
        }
    } else if constexpr (MODE == 1) {
        // the rows' buffer is not written back: after the sums, it holds the
        // block's partial sums
        double *red = (double *)buf;
        if (self) {
            const int seg1 = task.pad[0] - 1;
            const Wsum w0 = self_row_whittle<T>(a, L, buf, seg, ka, 0, twh);
            Wsum w1 = self_row_whittle<T>(a, L, buf, seg1, kb, 1, twh);
            if (twice) w1 = Wsum{0, 0, 0};
            __syncthreads();
            whittle_flush(a, red, w0, seg);
            whittle_flush(a, red, w1, seg1);
        } else {
            const Wsum w = pair_row_whittle<T>(a, L, buf, seg, sg, p, ka, twh);
            __syncthreads();
            whittle_flush(a, red, w, seg);
        }
    } else {
        if (self) {
            // the stage and w_2L tables depend on L alone: the first row's serve both
            self_row_modes<T, MODE>(a, L, buf, seg, ka, 0, twh);
            self_row_modes<T, MODE>(a, L, buf, task.pad[0] - 1, kb, 1, twh);
        } else {
            pair_row_modes<T, MODE>(a, L, buf, seg, sg, p, ka, twh);
        }
        __syncthreads();
    }
}

}  // namespace
