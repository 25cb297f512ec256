// FP64 kernel of the row pass compiled per row length: the including file sets
// C3_ROW_NT (threads) and C3_ROW_LIST (row lengths).
//
// Bound by FP64 and integer arithmetic (the mode draws, two Philox blocks a
// pair).  On 9.2e6 samples of 1e5 to 1.3e5 a segment the draw's rows took 450 us on
// the generic kernel, whose stages spilled and whose library functions were 700
// of 1100 instructions a mode, and 178 here; the chi^2's (mode 1) 174 and 90.
// Copying the rows in and out takes 60 us at 5.2 TB/s.
#pragma once
#include "rowbody.h"

namespace {
// Every row length of C3_ROW_LIST in one kernel, as in FP32, at four waves per
// SIMD (128 registers).  The mode loop is one for
// all lengths: compiled per length, its FP64 constants were hoisted together out
// of the switch and 82 registers spilled.
template <int MODE>
__global__ __launch_bounds__(NT, 4) void k_rowd(FftArgs a) {
    const RowTask task = a.row_tasks[blockIdx.x];
    if (task.seg < 0) return;  // an empty task (launch padding)
    if (row_idle(a, task)) return;
    double *hist = nullptr;  // mode 4: the block's periodogram bins
    cx<double> *buf = (cx<double> *)c3_rowc_lds;  // 2 L elements and the tables
    const int L = task.pad[1] >> 16;
    if constexpr (MODE == 4) {
        __shared__ double bins[C3_XI_NBIN];
        hist = bins;
    } else {
        // the tables of the mode arithmetic, behind the rows (read after the
        // stages' barriers)
        if (threadIdx.x < c3d::kTab) buf[2 * L + threadIdx.x] = ((const cx<double> *)a.twpool)[threadIdx.x];
    }
    cx<double> *ya = (cx<double> *)a.work + task.off_a, *yb = (cx<double> *)a.work + task.off_b;
    const SegInfo sg = a.segs[task.seg];
    const FftPlan &p = a.plans[sg.plan];
    const cx<double> *tws = (const cx<double> *)a.twpool + p.twr;
    switch (L) {
#define C3_ROW_CASE(LL)                   \
    case LL:                               \
        row_load<double, LL>(buf, ya, yb); \
        row_fwd<double, LL>(buf, tws);     \
        break;
        C3_ROW_LIST(C3_ROW_CASE)
#undef C3_ROW_CASE
    }
    row_mid<double, MODE>(a, L, buf, task, sg, p, hist);
    if constexpr (MODE == 0 || MODE == 2) {
        switch (L) {
#define C3_ROW_CASE(LL)                      \
    case LL:                                  \
        row_inv<double, LL>(buf, ya, yb, tws); \
        break;
            C3_ROW_LIST(C3_ROW_CASE)
#undef C3_ROW_CASE
        }
    }
}

inline hipError_t init_rows() {
    hipError_t e = hipSuccess;
    auto set = [&](const void *f) {
        hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, C3_LDS_MAX - 4096);
        if (r != hipSuccess) e = r;
    };
    set((const void *)k_rowd<0>);
    set((const void *)k_rowd<1>);
    set((const void *)k_rowd<2>);
    set((const void *)k_rowd<4>);
    return e;
}

inline hipError_t run_rows(hipStream_t st, const FftArgs &a) {
    if (a.nrow_tasks <= 0) return hipSuccess;
    const dim3 g(a.nrow_tasks), b(NT);
    const unsigned lds = (unsigned)a.row_lds;
    switch (a.mode) {
    case 0: hipLaunchKernelGGL((k_rowd<0>), g, b, lds, st, a); break;
    case 1: hipLaunchKernelGGL((k_rowd<1>), g, b, lds, st, a); break;
    case 2: hipLaunchKernelGGL((k_rowd<2>), g, b, lds, st, a); break;
    case 4: hipLaunchKernelGGL((k_rowd<4>), g, b, lds, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace
