// FFT row pass compiled per row length, FP64: blocks of 512 threads and up to
// 80 KB, two to a CU.
#define C3_ROW_NT C3_ROWC_NT
#define C3_ROW_LIST C3_ROWD_LIST
#include "rowd.h"

namespace c3 {
hipError_t rowd_init_attributes() { return init_rows(); }
hipError_t launch_rowd(hipStream_t st, const FftArgs &a) { return run_rows(st, a); }
}  // namespace c3
