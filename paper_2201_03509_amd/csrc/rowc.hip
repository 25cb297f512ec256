// FFT row pass compiled per row length, FP32 (rowbody.h).
#include "rowc_body.h"

namespace {
// Every row length of a register class in one kernel: a set whose segments
// have several lengths would otherwise run its rows as that many launches one
// after the other, each with its own tail and, for few segments, on a part of
// the chip.  The block's length is in its task, so the choice is uniform.  The
// classes keep a short length's occupancy from falling to that of the lengths
// whose butterflies take twice the registers.
template <int MODE, bool WIDE>
__global__ __launch_bounds__(NT, WIDE ? 4 : 6) void k_rowc(FftArgs a) {
    const RowTask task = a.row_tasks[blockIdx.x];
    if (task.seg < 0) return;  // an empty task (launch padding)
    double *hist = nullptr;    // mode 4: the block's periodogram bins
    if constexpr (MODE == 4) {
        __shared__ double bins[C3_XI_NBIN];
        hist = bins;
    }
    switch (task.pad[1] >> 16) {
#define C3_ROWC_CASE(LL)                                                        \
    case LL:                                                                    \
        if constexpr (c3rowc::wide(LL) == WIDE) row_body<LL, MODE>(a, task, hist); \
        break;
        C3_ROWC_LIST(C3_ROWC_CASE)
#undef C3_ROWC_CASE
    }
}

}  // namespace

namespace c3 {

bool rowc_supported(int mode) { return mode == 0 || mode == 1 || mode == 2 || mode == 4; }

hipError_t rowc_init_attributes() {
    hipError_t e = hipSuccess;
    auto set = [&](const void *f) {
        hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, C3_LDS_MAX - 4096);
        if (r != hipSuccess) e = r;
    };
    set((const void *)k_rowc<0, false>);
    set((const void *)k_rowc<1, false>);
    set((const void *)k_rowc<2, false>);
    set((const void *)k_rowc<4, false>);
    set((const void *)k_rowc<0, true>);
    set((const void *)k_rowc<1, true>);
    set((const void *)k_rowc<2, true>);
    set((const void *)k_rowc<4, true>);
    return e;
}

hipError_t launch_rowc(hipStream_t st, const FftArgs &a, bool wide) {
    if (a.nrow_tasks <= 0) return hipSuccess;
    const dim3 g(a.nrow_tasks), b(NT);
    const unsigned lds = (unsigned)a.row_lds;
#define C3_ROWC_LAUNCH(MODE)                                                \
    case MODE:                                                              \
        if (wide)                                                           \
            hipLaunchKernelGGL((k_rowc<MODE, true>), g, b, lds, st, a);     \
        else                                                                \
            hipLaunchKernelGGL((k_rowc<MODE, false>), g, b, lds, st, a);    \
        break;
    switch (a.mode) {
        C3_ROWC_LAUNCH(0)
        C3_ROWC_LAUNCH(1)
        C3_ROWC_LAUNCH(2)
        C3_ROWC_LAUNCH(4)
    default:
        return hipErrorInvalidValue;
    }
#undef C3_ROWC_LAUNCH
    return hipGetLastError();
}

}  // namespace c3
