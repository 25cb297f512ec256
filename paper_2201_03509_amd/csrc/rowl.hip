// FFT row pass compiled per row length, FP32, one kernel per length.
//
// The same code as a length's case in k_rowc (rowc.hip) runs 4 to 13 % faster as
// a kernel of its own (the 9.4e8-sample 70 GHz-like set, rows of 2430 to 4096
// points: 6.74 ms of row pass in the kernels of a register class, 6.02 so), but
// a launch costs a tail of one block's time, 15 us.  c3tune::own_rows weighs the two.  Us
// of row pass, shared and own: one length, 2000 points, 3000 tasks 87.5 and 82.7, 500
// tasks 30.0 and 28.2; two of 3700 points, 1280 tasks each 145 and 156, 2560 tasks 284 and
// 279; three of 2200 points, 2900 tasks 503 and 515 (a fourth beside them); six of
// 2150 points, 3500 tasks 590 and 603; some thirty of 4000 points, 700 tasks each, 754
// and 907.
#include "rowc_body.h"

namespace {
template <int L, int MODE>
__global__ __launch_bounds__(NT) void k_rowl(FftArgs a) {
    const RowTask task = a.row_tasks[blockIdx.x];
    if (task.seg < 0) return;  // an empty task (launch padding)
    double *hist = nullptr;    // mode 4: the block's periodogram bins
    if constexpr (MODE == 4) {
        __shared__ double bins[C3_XI_NBIN];
        hist = bins;
    }
    row_body<L, MODE>(a, task, hist);
}

template <int L>
void launch_length(dim3 g, dim3 b, unsigned lds, hipStream_t st, const FftArgs &a) {
    switch (a.mode) {
    case 0: hipLaunchKernelGGL((k_rowl<L, 0>), g, b, lds, st, a); break;
    case 1: hipLaunchKernelGGL((k_rowl<L, 1>), g, b, lds, st, a); break;
    case 2: hipLaunchKernelGGL((k_rowl<L, 2>), g, b, lds, st, a); break;
    default: hipLaunchKernelGGL((k_rowl<L, 4>), g, b, lds, st, a); break;
    }
}

}  // namespace

namespace c3 {

hipError_t rowl_init_attributes() {
    hipError_t e = hipSuccess;
    auto set = [&](const void *f) {
        hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, C3_LDS_MAX - 4096);
        if (r != hipSuccess) e = r;
    };
#define C3_ROWL_SET(L)                \
    set((const void *)k_rowl<L, 0>);  \
    set((const void *)k_rowl<L, 1>);  \
    set((const void *)k_rowl<L, 2>);  \
    set((const void *)k_rowl<L, 4>);
    C3_ROWC_LIST(C3_ROWL_SET)
#undef C3_ROWL_SET
    return e;
}

hipError_t launch_rowl(hipStream_t st, const FftArgs &a, int L) {
    if (a.nrow_tasks <= 0) return hipSuccess;
    const dim3 g(a.nrow_tasks), b(NT);
    const unsigned lds = (unsigned)a.row_lds;
    switch (L) {
#define C3_ROWL_CASE(LL) case LL: launch_length<LL>(g, b, lds, st, a); break;
        C3_ROWC_LIST(C3_ROWL_CASE)
#undef C3_ROWL_CASE
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace c3
