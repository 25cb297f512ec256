// Register column passes, FP64 (fftcol.h).
#include "fftcol.h"

namespace {
// Every column length in one kernel, at one wave per SIMD: a column takes 4 M1
// of its 512 registers, and the loads in flight (64 M1 x 16 bytes a wave) still
// cover the memory's latency several times.  9.2e6 samples of 1e5 to 1.3e5 a segment:
// forward 109 us on LDS tiles, 63 here (221 MB: 3.5 TB/s); inverse 90, 46 (221 MB:
// 4.8 TB/s).
template <int PASS, int IN>
__global__ __launch_bounds__(C3_COL_NT, 1) void k_cold(FftArgs a) {
    const ColTask sg = a.col_tasks[blockIdx.x];
    switch (sg.pad[0]) {
#define C3_COL_CASE(M)                            \
    case M:                                       \
        col_pass<double, M, PASS, IN>(a, sg);     \
        break;
        C3_COLREG_LIST_F64(C3_COL_CASE)
#undef C3_COL_CASE
    }
}

}  // namespace

namespace c3 {

hipError_t launch_fft_col_reg_f64(hipStream_t st, const FftArgs &a, int pass) {
    const dim3 g(a.ncol_tasks), b(C3_COL_NT);
    const int in = col_input(a, true);
    if (pass == 2) hipLaunchKernelGGL((k_cold<2, 0>), g, b, 0, st, a);
    else if (in == 0) hipLaunchKernelGGL((k_cold<0, 0>), g, b, 0, st, a);
    else if (in == 1) hipLaunchKernelGGL((k_cold<0, 1>), g, b, 0, st, a);
    else if (in == 2) hipLaunchKernelGGL((k_cold<0, 2>), g, b, 0, st, a);
    else if (in == 4) hipLaunchKernelGGL((k_cold<0, 4>), g, b, 0, st, a);
    else if (in == 5) hipLaunchKernelGGL((k_cold<0, 5>), g, b, 0, st, a);
    else hipLaunchKernelGGL((k_cold<0, 3>), g, b, 0, st, a);
    return hipGetLastError();
}

}  // namespace c3
