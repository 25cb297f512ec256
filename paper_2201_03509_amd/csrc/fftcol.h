// Column passes of the four-step n_corr FFT (section 4.2) with the column
// length M1 fixed at compile time (fftcol.hip: FP32, fftcold.hip: FP64).
//
// One lane owns one column j2 of a segment: it loads the M1 elements
// z[M2 j1 + j2] (consecutive lanes read consecutive addresses), runs the whole
// FFT_M1 in registers as unrolled Stockham stages whose twiddles are folded to
// constants at compile time, applies the four-step twiddle w_M^(j2 k1) and
// writes Y[k1][j2].  No LDS and no barriers: every lane keeps its column's
// loads (one per element) in flight, which is what hides HBM
// latency in this pass.  The inverse kernel
// takes Y[k1][j2] times w_M^(-j2 k1), inverts the column and writes the first
// n real samples.  The LDS-tiled column kernels in fft.hip cover every other M1.
#pragma once
#include <utility>

#include "common.h"
#include "fftdev.h"

namespace {
using c3::FftArgs;
using namespace c3fft;

// word 3 of a raw buffer resource on gfx9-family chips (untyped dword access)
#define C3_BUF_WORD3 0x00020000

// Loads and stores below address a uniform (scalar) base plus a 32-bit lane
// offset, so the compiler needs no 64-bit address per element.
template <typename V>
__device__ __forceinline__ V ld_off(const void *base, uint32_t byte_off) {
    return *(const V *)((const char *)base + byte_off);
}
template <typename V>
__device__ __forceinline__ void st_off(void *base, uint32_t byte_off, V v) {
    *(V *)((char *)base + byte_off) = v;
}

__device__ __forceinline__ float ffma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double ffma(double a, double b, double c) { return __builtin_fma(a, b, c); }
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 bits2(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    return u32x2{(uint32_t)b, (uint32_t)(b >> 32)};
}

// reals t and t + 1 (t even) of the mirrored, padded extension of the n
// samples in the raw buffer rb (n values) as one complex value, from one
// load of two: adjacent samples below n, the mirror image of an adjacent pair
// (in reverse order) from n to 2n, the last sample twice at t = n - 1 (odd
// n), and the first sample twice in the pad beyond 2n (the pad repeats r_0).
// Needs n > 1: every load stays inside the n samples.
template <typename T>
__device__ __forceinline__ cx<T> ext_pair(__amdgpu_buffer_rsrc_t rb, uint32_t n, uint32_t t) {
    const uint32_t n2 = 2u * n;
    const bool lo = t + 1u < n, mir = t >= n, pad = t >= n2;
    const uint32_t b = lo ? t : (pad ? 0u : (mir ? n2 - 2u - t : n - 2u));
    T v0, v1;
    if constexpr (sizeof(T) == 4) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(rb, (int)(4u * b), 0, 0);
        v0 = __uint_as_float(v[0]), v1 = __uint_as_float(v[1]);
    } else {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rb, (int)(8u * b), 0, 0);
        v0 = __longlong_as_double((int64_t)((uint64_t)v[1] << 32 | v[0]));
        v1 = __longlong_as_double((int64_t)((uint64_t)v[3] << 32 | v[2]));
    }
    return cx<T>{lo || pad ? v0 : v1, mir ? v0 : v1};
}

// f(k1, w_M^(j2 k1)) for k1 < M1, with w_M^(j2 (a Q + b)) = w_M^(j2 Q a) w_M^(j2 b)
// from the two-level w_N table (N = 2M); each factor is used as soon as it is
// formed, so no table of M1 twiddles is held in registers
template <int M1, int Q, typename T, typename F>
__device__ __forceinline__ void col_twiddles(const cx<T> *pool, const FftPlan &p, int j2, F &&f) {
    cx<T> wb[Q];
#pragma unroll
    for (int b = 0; b < Q; ++b) wb[b] = twN(pool, p, 2 * (int64_t)j2 * b);
#pragma unroll
    for (int ai = 0; ai * Q < M1; ++ai) {
        const cx<T> wa = twN(pool, p, 2 * (int64_t)j2 * Q * ai);
#pragma unroll
        for (int b = 0; b < Q; ++b)
            if (ai * Q + b < M1) f(ai * Q + b, cmul(wa, wb[b]));
    }
}

// ------------------------------------------------------------- pass 1
template <typename T, int M1, int IN>
__device__ __forceinline__ void col_fwd(const FftArgs &a, const ColTask &sg) {
    // the column's loads need only the task: they are issued first, and the
    // segment's plan (twiddles) loads while they are in flight.  In the
    // masked draw a converged segment's block returns before any load.
    const int M2 = sg.M2;
    const int j2 = sg.c0 + (int)threadIdx.x;
    if (j2 >= M2) return;
    if (a.active && !a.active[sg.seg]) return;  // converged segment (whole block)
    const uint32_t n = (uint32_t)sg.n, n2 = 2u * (uint32_t)sg.n;
    constexpr uint32_t E = 2 * sizeof(T);  // bytes of a complex element
    cx<T> x[M1];
    if constexpr (IN == 0) {
        // a whole extended vector (N reals = M complex at the segment's offset)
        const cx<T> *v = (const cx<T> *)a.in_a + sg.ext_off;
        const uint32_t lo = E * (uint32_t)j2;
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) {
            x[j1] = ld_off<cx<T>>(v + (int64_t)j1 * M2, lo);
            if ((j1 & 15) == 15) __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (IN == 1) {
        // r = in_a (in T): the sweep's residual (n > 12 here: M >= M1 >= 16
        // is the next 5-smooth length >= n)
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((T *)a.in_a + sg.samp_off, 0, (int)sizeof(T) * sg.n, C3_BUF_WORD3);
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) {
            x[j1] = ext_pair<T>(r, n, 2u * (uint32_t)(M2 * j1 + j2));
            // keep the scheduler from computing every offset before the first
            // load: 16 rows in flight is plenty
            if ((j1 & 15) == 15) __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (IN == 2) {
        // r = in_a - in_b, both in T (d and s of a standalone draw): every
        // load of the column is issued before the first subtraction
        const __amdgpu_buffer_rsrc_t ra =
            __builtin_amdgcn_make_buffer_rsrc((T *)a.in_a + sg.samp_off, 0, (int)sizeof(T) * sg.n, C3_BUF_WORD3);
        const __amdgpu_buffer_rsrc_t rb =
            __builtin_amdgcn_make_buffer_rsrc((T *)a.in_b + sg.samp_off, 0, (int)sizeof(T) * sg.n, C3_BUF_WORD3);
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) {
            const uint32_t t = 2u * (uint32_t)(M2 * j1 + j2);
            x[j1] = csub(ext_pair<T>(ra, n, t), ext_pair<T>(rb, n, t));
            if ((j1 & 7) == 7) __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (IN == 5) {
        // r = in_a, FP32 data (FP64 transforms).  IN 3 branches on the type at each
        // element, which keeps its loads apart: 19 columns of 256 lanes took 11.8
        // us with it, 6 with the type compiled in.
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((float *)a.in_a + sg.samp_off, 0, 4 * sg.n, C3_BUF_WORD3);
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) {
            const cx<float> u = ext_pair<float>(r, n, 2u * (uint32_t)(M2 * j1 + j2));
            x[j1] = cx<T>{(T)u.x, (T)u.y};
            if ((j1 & 15) == 15) __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (IN == 4) {
        // r = in_a - in_b, FP32 data less an FP64 model (FP64 transforms)
        const __amdgpu_buffer_rsrc_t ra =
            __builtin_amdgcn_make_buffer_rsrc((float *)a.in_a + sg.samp_off, 0, 4 * sg.n, C3_BUF_WORD3);
        const __amdgpu_buffer_rsrc_t rb =
            __builtin_amdgcn_make_buffer_rsrc((T *)a.in_b + sg.samp_off, 0, (int)sizeof(T) * sg.n, C3_BUF_WORD3);
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) {
            const uint32_t t = 2u * (uint32_t)(M2 * j1 + j2);
            const cx<float> u = ext_pair<float>(ra, n, t);
            x[j1] = csub(cx<T>{(T)u.x, (T)u.y}, ext_pair<T>(rb, n, t));
            if ((j1 & 7) == 7) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // r = in_a - in_b in any input precision, converted to T
        const int64_t s0 = sg.samp_off;
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) {
            const uint32_t t = 2u * (uint32_t)(M2 * j1 + j2);
            T v[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t th = t + (uint32_t)h;
                const uint32_t u = th < n ? th : (th < n2 ? n2 - 1u - th : 0u);
                v[h] = load_as<T>(a.in_a, a.in_a_f64, s0 + u);
                if (a.in_b) v[h] -= load_as<T>(a.in_b, a.in_b_f64, s0 + u);
            }
            x[j1] = cx<T>{v[0], v[1]};
        }
    }
    const FftPlan &p = a.plans[a.segs[sg.seg].plan];
    reg_fft<M1, -1>(x);
    // the twiddle-table loads below must not be hoisted into the FFT, where
    // every register already holds column data
    __builtin_amdgcn_sched_barrier(0);
    cx<T> *Y = (cx<T> *)a.work + sg.scr_off;
    const uint32_t lo = E * (uint32_t)j2;
    // which of a product's two terms is rounded before their sum is written out:
    // left to the compiler it varies with the kernel around it
    col_twiddles<M1, tw_split(M1)>((const cx<T> *)a.twpool, p, j2, [&](int k1, cx<T> w) {
        const cx<T> v = x[k1];
        st_off(Y + (int64_t)k1 * M2, lo, cx<T>{ffma(v.x, w.x, -(v.y * w.y)), ffma(v.x, w.y, v.y * w.x)});
    });
}

// ------------------------------------------------------------- pass 3
template <typename T, int M1>
__device__ __forceinline__ void col_inv(const FftArgs &a, const ColTask &sg) {
    const int M2 = sg.M2;
    const int j2 = sg.c0 + (int)threadIdx.x;
    if (j2 >= M2) return;
    if (a.active && !a.active[sg.seg]) return;  // converged segment (whole block)
    const cx<T> *Y = (const cx<T> *)a.work + sg.scr_off;
    constexpr uint32_t E = 2 * sizeof(T);
    const uint32_t lo = E * (uint32_t)j2;
    cx<T> x[M1];
#pragma unroll
    for (int k1 = 0; k1 < M1; ++k1) x[k1] = ld_off<cx<T>>(Y + (int64_t)k1 * M2, lo);
    const FftPlan &p = a.plans[a.segs[sg.seg].plan];
    col_twiddles<M1, tw_split(M1)>((const cx<T> *)a.twpool, p, j2, [&](int k1, cx<T> w) {
        // times w_M^(-j2 k1), rounded as written (see the forward pass)
        const cx<T> v = x[k1];
        x[k1] = cx<T>{ffma(v.x, w.x, v.y * w.y), ffma(v.y, w.x, -(v.x * w.y))};
    });
    reg_fft<M1, 1>(x);
    if (a.full_io) {
        // the whole extended vector
        cx<T> *v = (cx<T> *)a.out + sg.ext_off;
#pragma unroll
        for (int j1 = 0; j1 < M1; ++j1) st_off(v + (int64_t)j1 * M2, lo, x[j1]);
        return;
    }
    // the first n real samples: a raw buffer of n values, whose hardware range
    // check drops the stores at t >= n (no per-element branch)
    const __amdgpu_buffer_rsrc_t out =
        __builtin_amdgcn_make_buffer_rsrc((T *)a.out + sg.samp_off, 0, (int)sizeof(T) * sg.n, C3_BUF_WORD3);
#pragma unroll
    for (int j1 = 0; j1 < M1; ++j1) {
        const uint32_t t = 2u * (uint32_t)(M2 * j1 + j2);
        if constexpr (sizeof(T) == 4) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[j1].x), out, (int)(4u * t), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[j1].y), out, (int)(4u * t + 4u), 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b64(bits2(x[j1].x), out, (int)(8u * t), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b64(bits2(x[j1].y), out, (int)(8u * t + 8u), 0, 0);
        }
    }
}

template <typename T, int M1, int PASS, int IN>
__device__ __forceinline__ void col_pass(const FftArgs &a, const ColTask &sg) {
    if constexpr (PASS == 0)
        col_fwd<T, M1, IN>(a, sg);
    else
        col_inv<T, M1>(a, sg);
}

// the input form of the forward pass (col_fwd's IN)
inline int col_input(const FftArgs &a, bool f64) {
    const bool own = !!a.in_a_f64 == f64 && (!a.in_b || !!a.in_b_f64 == f64);
    if (f64 && !a.full_io && !a.in_a_f64 && (!a.in_b || a.in_b_f64)) return a.in_b ? 4 : 5;
    return a.full_io ? 0 : !own ? 3 : a.in_b ? 2 : 1;
}

}  // namespace
