// Register column passes, FP32 (fftcol.h).
#include "fftcol.h"

namespace {
// Every column length of a register class in one kernel (one launch instead of
// one per length, as in the row pass); the block's length is in its task.
constexpr int col_class(int M1) { return M1 <= 36 ? 0 : M1 <= 64 ? 1 : 2; }
constexpr int col_waves(int cls) { return cls == 0 ? 4 : cls == 1 ? 3 : 2; }  // per SIMD

// PASS 0 reads its input as IN says (col_input), PASS 2 ignores it.
template <int CLS, int PASS, int IN>
__global__ __launch_bounds__(C3_COL_NT, col_waves(CLS)) void k_colr(FftArgs a) {
    const ColTask sg = a.col_tasks[blockIdx.x];
    switch (sg.pad[0]) {
#define C3_COL_CASE(M)                                                             \
    case M:                                                                        \
        if constexpr (col_class(M) == CLS) col_pass<float, M, PASS, IN>(a, sg);    \
        break;
        C3_COLREG_LIST(C3_COL_CASE)
#undef C3_COL_CASE
    }
}

}  // namespace

namespace c3 {

int fft_col_class(int mixed, int m1) { return mixed ? col_class(m1) : 0; }

hipError_t launch_fft_col_reg(hipStream_t st, int mixed, const FftArgs &a, int pass, int cls) {
    if (pass != 0 && pass != 2) return hipErrorInvalidValue;
    if (a.ncol_tasks <= 0) return hipSuccess;
    if (!mixed) return launch_fft_col_reg_f64(st, a, pass);
    const dim3 g(a.ncol_tasks), b(C3_COL_NT);
    const int in = col_input(a, false);
#define C3_COL_LAUNCH(CLS)                                              \
    case CLS:                                                           \
        if (pass == 2)                                                  \
            hipLaunchKernelGGL((k_colr<CLS, 2, 0>), g, b, 0, st, a);    \
        else if (in == 0)                                               \
            hipLaunchKernelGGL((k_colr<CLS, 0, 0>), g, b, 0, st, a);    \
        else if (in == 1)                                               \
            hipLaunchKernelGGL((k_colr<CLS, 0, 1>), g, b, 0, st, a);    \
        else if (in == 2)                                               \
            hipLaunchKernelGGL((k_colr<CLS, 0, 2>), g, b, 0, st, a);    \
        else                                                            \
            hipLaunchKernelGGL((k_colr<CLS, 0, 3>), g, b, 0, st, a);    \
        break;
    switch (cls) {
        C3_COL_LAUNCH(0)
        C3_COL_LAUNCH(1)
        C3_COL_LAUNCH(2)
    default:
        return hipErrorInvalidValue;
    }
#undef C3_COL_LAUNCH
    return hipGetLastError();
}

}  // namespace c3
