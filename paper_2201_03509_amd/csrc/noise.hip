// Noise-parameter draw xi_n <- P(xi_n | d, g, n_corr, sky) per segment (Eq. 5;
// the correlated-noise PSD step, which needs only low-volume spectrum data).
//
// 1. White level: r = d - g t - n_corr; sigma0^2 = S / X, S = sum r^2 (FP64
//    tile partials here), X ~ chi^2_n by the Wilson-Hilferty transform.
// 2. The periodogram of n_corr on its mirrored extension, summed into integer
//    log-frequency bins J_b by the FFT row pass (mode 4).  Per bin the count
//    c_b and sum of ln k follow from its mode range [lo, hi] in closed form
//    (lgamma), f_b = (f_samp/N) exp(mean ln k).
// 3. alpha | f_knee, sigma0: binned Whittle ln L is strictly concave in alpha;
//    its maximiser by a bracketed, bisection-safeguarded Newton iteration,
//    alpha = alpha_hat + z1 / sqrt(-d2 lnL).
// 4. f_knee | alpha, sigma0: u = f_knee^alpha ~ Gamma(K, S_a / sigma0^2),
//    Wilson-Hilferty variate, f_knee = u^(1/alpha).
// z0, z1, z2: Box-Muller normals of the segment's Philox stream at counter
// word 2^32 - 2; mean_only: all zero.
#include "common.h"
#include "rng.h"

namespace {
using namespace c3;
using namespace c3rng;

// per sample tile: partial sum of (d - g t - n_corr)^2 (d of type TD, fixed at
// compile time so that the loads of several samples issue together)
template <typename T, typename TD>
__global__ __launch_bounds__(C3_NT) void k_xi_white(const int4 *__restrict__ tiles, const int64_t *__restrict__ seg_off,
                                                    const TD *__restrict__ d, const T *__restrict__ t,
                                                    const double *__restrict__ gain, const T *__restrict__ nc,
                                                    double *__restrict__ part) {
    const int4 tl = tiles[blockIdx.x];
    const int64_t base = seg_off[tl.x] + tl.y;
    const double g = gain[tl.x];
    double acc = 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < tl.z; i += C3_NT) {
        const double r = (double)d[base + i] - g * (double)t[base + i] - (double)nc[base + i];
        acc += r * r;
    }
    __shared__ double red[C3_NT / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0;
#pragma unroll
        for (int i = 0; i < C3_NT / 64; ++i) s += red[i];
        part[blockIdx.x] = s;
    }
}

// v of another lane of the wave, as the DPP control CTRL says
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((int64_t)((uint64_t)hi << 32 | lo));
}
// wave-wide sum, every lane gets the result (fixed order): between lanes 1 and 2
// apart, the halves of 8, the halves of 16 by DPP, rows and wave halves by
// swaps.  Six shuffles through LDS took most of a score evaluation's time.
__device__ __forceinline__ double wsum(double v) {
    v += dpp<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp<0x141>(v);  // row_half_mirror
    v += dpp<0x140>(v);  // row_mirror
#define C3_SWAP_SUM(SWAP)                                                                             \
    {                                                                                                 \
        const uint64_t b = (uint64_t)__double_as_longlong(v);                                         \
        const auto lo = SWAP((uint32_t)b, (uint32_t)b, false, false);                                 \
        const auto hi = SWAP((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);                 \
        v = __longlong_as_double((int64_t)((uint64_t)hi[0] << 32 | lo[0])) +                          \
            __longlong_as_double((int64_t)((uint64_t)hi[1] << 32 | lo[1]));                           \
    }
    C3_SWAP_SUM(__builtin_amdgcn_permlane16_swap)
    C3_SWAP_SUM(__builtin_amdgcn_permlane32_swap)
#undef C3_SWAP_SUM
    return v;
}

#define C3_XI_PER_LANE ((C3_XI_NBIN + 63) / 64)

// one wave per segment.  Bound by its own latency: about twelve evaluations of the
// score one after the other, and a ln Gamma per bin.  80 segments of 1e5 samples: 46
// us with 50 evaluations, LDS shuffles and two ln Gamma a bin, 17 now.
__global__ __launch_bounds__(C3_NT) void k_xi_sample(int nseg, const SegInfo *__restrict__ segs,
                                                     const FftPlan *__restrict__ plans,
                                                     const int32_t *__restrict__ seg_band,
                                                     const double *__restrict__ fsamp_band,
                                                     const int2 *__restrict__ seg_tiles,
                                                     const double *__restrict__ part,
                                                     const double *__restrict__ bins,
                                                     const double *__restrict__ fknee_in,
                                                     const uint64_t *__restrict__ seed_iter, int mean_only,
                                                     double *__restrict__ sigma0_out,
                                                     double *__restrict__ fknee_out,
                                                     double *__restrict__ alpha_out) {
    const int seg = blockIdx.x * (C3_NT / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (seg >= nseg) return;
    const SegInfo sg = segs[seg];
    if (sg.n <= 0 || sg.plan < 0) {
        if (lane == 0) sigma0_out[seg] = fknee_out[seg] = alpha_out[seg] = NAN;
        return;
    }
    const int64_t M = plans[sg.plan].M;
    const double N = 2.0 * (double)M;
    const double fs = fsamp_band[seg_band[seg]];
    const double fk_old = fknee_in[seg];

    double z[4] = {0, 0, 0, 0};
    if (!mean_only) {
        const uint64_t seed = seed_iter[0], it = seed_iter[1];
        normals4<double>(philox4x32_10(make_uint4(0xFFFFFFFEu, (uint32_t)it, (uint32_t)(it >> 32),
                                                  (uint32_t)(seed >> 32)),
                                       make_uint2((uint32_t)seed, (uint32_t)seg)),
                         z);
    }

    // 1. white level
    const int2 tr = seg_tiles[seg];
    double S = 0;
    for (int i = lane; i < tr.y; i += 64) S += part[tr.x + i];
    S = wsum(S);
    const double n = (double)sg.n;
    const double wh = 1.0 - 2.0 / (9.0 * n) + z[0] * sqrt(2.0 / (9.0 * n));
    const double s2 = S / (n * wh * wh * wh);

    // 2. bins of this segment: lane holds bins lane, lane + 64, ...
    const int nb = 1 + (M < 8 ? (int)M - 1 : 7 + 8 * ((63 - __builtin_clzll((unsigned long long)M)) - 3) +
                                             (int)(M >> ((63 - __builtin_clzll((unsigned long long)M)) - 3)) - 8);
    double Jb[C3_XI_PER_LANE], cb[C3_XI_PER_LANE], xb[C3_XI_PER_LANE], lf[C3_XI_PER_LANE];
    const double lscale = log(fs / N);
    // first mode of bin b, at most M + 1 (the first one past the spectrum), and
    // ln Gamma of it: bin b + 1's is the end of bin b, so one per bin does
    int64_t first[C3_XI_PER_LANE + 1];
    double lg[C3_XI_PER_LANE + 1];
#pragma unroll
    for (int j = 0; j < C3_XI_PER_LANE; ++j) {
        const int b = lane + 64 * j;
        const int e = (b - 7) / 8, m = (b - 7) % 8;
        first[j] = b < 7 ? b + 1 : e < 30 ? (int64_t)(8 + m) << e : M + 1;
        if (first[j] > M + 1) first[j] = M + 1;
        lg[j] = 0.0;
        if (b <= nb) lg[j] = lgamma((double)first[j]);
    }
    lg[C3_XI_PER_LANE] = 0.0;
    first[C3_XI_PER_LANE] = M + 1;
    double end_lg[C3_XI_PER_LANE];
    int64_t end[C3_XI_PER_LANE];
#pragma unroll
    for (int j = 0; j < C3_XI_PER_LANE; ++j) {  // bin b + 1 is the next lane's, or lane 0's next
        end_lg[j] = __shfl(lane == 0 ? lg[j + 1] : lg[j], (lane + 1) & 63, 64);
        end[j] = __shfl((long long)(lane == 0 ? first[j + 1] : first[j]), (lane + 1) & 63, 64);
    }
#pragma unroll
    for (int j = 0; j < C3_XI_PER_LANE; ++j) {
        const int b = lane + 64 * j;
        Jb[j] = cb[j] = xb[j] = lf[j] = 0;
        if (b >= nb || end[j] <= first[j]) continue;
        const double c = (double)(end[j] - first[j]);
        const double L = end_lg[j] - lg[j];  // sum of ln k over the bin
        Jb[j] = bins[(int64_t)seg * C3_XI_NBIN + b];
        cb[j] = c;
        lf[j] = lscale + L / c;                 // ln f_b
        xb[j] = lf[j] - log(fk_old);            // ln(f_b / f_knee)
    }

    // 3. alpha | f_knee: score(al) = sum a x e^(-al x) - sum c x, a = J / sigma0^2
    auto score = [&](double al, double *dscore) {
        double s = 0, ds = 0;
#pragma unroll
        for (int j = 0; j < C3_XI_PER_LANE; ++j) {
            if (cb[j] == 0.0) continue;
            const double ax = Jb[j] / s2 * xb[j] * exp(-al * xb[j]);
            s += ax - cb[j] * xb[j];
            ds -= ax * xb[j];
        }
        if (dscore) *dscore = wsum(ds);
        return wsum(s);
    };
    double lo = -1.0, hi = 1.0, flo = score(lo, nullptr), fhi = score(hi, nullptr);
    for (int i = 0; i < 60 && flo < 0.0; ++i) flo = score(lo *= 2.0, nullptr);
    for (int i = 0; i < 60 && fhi > 0.0; ++i) fhi = score(hi *= 2.0, nullptr);
    const bool ok = flo >= 0.0 && fhi <= 0.0;
    double al = 0.5 * (lo + hi), H = 0;
    if (ok) {
        for (int i = 0; i < 200; ++i) {
            double ds;
            const double f = score(al, &ds);
            if (f > 0.0) lo = al; else hi = al;
            double nx = al - f / ds;                   // Newton step
            // quadratic: what a step of 1e-9 leaves is below the rounding.  (Waiting
            // for steps of 1e-15 ran into the bracket's end at the root, which the
            // next step then left, and bisected the whole bracket again: 50
            // evaluations of the score for 8.)  A slope that overflows gives a step of 0.
            if (fabs(nx - al) <= 1e-9 * fmax(1.0, fabs(al)) && isfinite(ds)) {
                al = nx;
                break;
            }
            if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);  // bisection fallback
            const double step = fabs(nx - al);
            al = nx;
            if (step <= 1e-15 * fmax(1.0, fabs(al)) || hi - lo <= 1e-15 * fmax(1.0, fabs(al))) break;
        }
        score(al, &H);
        H = -H;
    }
    const double alpha = ok ? al + z[1] / sqrt(H) : NAN;

    // 4. f_knee | alpha: u = f_knee^alpha ~ Gamma(K, S_a / sigma0^2)
    double Sa = 0, K = 0;
#pragma unroll
    for (int j = 0; j < C3_XI_PER_LANE; ++j) {
        if (cb[j] == 0.0) continue;
        Sa += Jb[j] * exp(-alpha * lf[j]);
        K += cb[j];
    }
    Sa = wsum(Sa);
    K = wsum(K);
    const double gw = 1.0 - 1.0 / (9.0 * K) + z[2] / (3.0 * sqrt(K));
    const double u = K * gw * gw * gw * s2 / Sa;
    if (lane == 0) {
        sigma0_out[seg] = sqrt(s2);
        alpha_out[seg] = alpha;
        fknee_out[seg] = exp(log(u) / alpha);
    }
}

}  // namespace

namespace c3 {

hipError_t launch_xi_white(hipStream_t st, int mixed, const int4 *tiles, int ntile, const int64_t *seg_off,
                           const void *d, int d_f64, const void *t, const double *gain, const void *nc,
                           double *part) {
    if (ntile <= 0) return hipSuccess;
    const dim3 g((unsigned)ntile), b(C3_NT);
#define C3_XIW(T, TD)                                                                                    \
    hipLaunchKernelGGL((k_xi_white<T, TD>), g, b, 0, st, tiles, seg_off, (const TD *)d, (const T *)t, gain, \
                       (const T *)nc, part)
    if (mixed) {
        if (d_f64)
            C3_XIW(float, double);
        else
            C3_XIW(float, float);
    } else {
        if (d_f64)
            C3_XIW(double, double);
        else
            C3_XIW(double, float);
    }
#undef C3_XIW
    return hipGetLastError();
}

hipError_t launch_xi_sample(hipStream_t st, int nseg, const SegInfo *segs, const FftPlan *plans,
                            const int32_t *seg_band, const double *fsamp_band, const int2 *seg_tiles,
                            const double *part, const double *bins, const double *fknee_in,
                            const uint64_t *seed_iter, int mean_only, double *sigma0_out, double *fknee_out,
                            double *alpha_out) {
    if (nseg <= 0) return hipSuccess;
    const int per = C3_NT / 64;
    hipLaunchKernelGGL(k_xi_sample, dim3((unsigned)((nseg + per - 1) / per)), dim3(C3_NT), 0, st, nseg, segs,
                       plans, seg_band, fsamp_band, seg_tiles, part, bins, fknee_in, seed_iter, mean_only,
                       sigma0_out, fknee_out, alpha_out);
    return hipGetLastError();
}

}  // namespace c3
