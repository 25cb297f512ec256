// Register column passes, FP32 (fftcol.h).
#include "fftcol.h"
#include "tune.h"

namespace {
// Every column length of a register class in one kernel (one launch instead of
// one per length, as in the row pass); the block's length is in its task.
constexpr int col_class(int M1) { return M1 <= 36 ? 0 : M1 <= 64 ? 1 : 2; }

// PASS 0 reads its input as IN says (col_input), PASS 2 ignores it.  WAVES per SIMD:
// the middle class is compiled for three (columns of 60 and 64 then spill ten
// registers) and for two.
template <int CLS, int WAVES, int PASS, int IN>
__global__ __launch_bounds__(C3_COL_NT, WAVES) void k_colr(FftArgs a) {
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

template <int CLS, int WAVES>
void launch_class(hipStream_t st, const FftArgs &a, int pass, int in) {
    const dim3 g(a.ncol_tasks), b(C3_COL_NT);
    if (pass == 2)
        hipLaunchKernelGGL((k_colr<CLS, WAVES, 2, 0>), g, b, 0, st, a);
    else if (in == 0)
        hipLaunchKernelGGL((k_colr<CLS, WAVES, 0, 0>), g, b, 0, st, a);
    else if (in == 1)
        hipLaunchKernelGGL((k_colr<CLS, WAVES, 0, 1>), g, b, 0, st, a);
    else if (in == 2)
        hipLaunchKernelGGL((k_colr<CLS, WAVES, 0, 2>), g, b, 0, st, a);
    else
        hipLaunchKernelGGL((k_colr<CLS, WAVES, 0, 3>), g, b, 0, st, a);
}

}  // namespace

namespace c3 {

int fft_col_class(int mixed, int m1) { return mixed ? col_class(m1) : 0; }

hipError_t launch_fft_col_reg(hipStream_t st, int mixed, const FftArgs &a, int pass, int cls) {
    if (pass != 0 && pass != 2) return hipErrorInvalidValue;
    if (a.ncol_tasks <= 0) return hipSuccess;
    if (!mixed) return launch_fft_col_reg_f64(st, a, pass);
    const int in = col_input(a, false);
    switch (cls) {
    case 0:
        launch_class<0, 4>(st, a, pass, in);
        break;
    case 1:
        if (c3tune::col_waves(a.ncol_tasks) == 2)
            launch_class<1, 2>(st, a, pass, in);
        else
            launch_class<1, 3>(st, a, pass, in);
        break;
    case 2:
        launch_class<2, 2>(st, a, pass, in);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace c3
