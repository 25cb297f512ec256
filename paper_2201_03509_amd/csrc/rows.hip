// FFT row pass compiled per row length, FP64, short rows: blocks of 256 threads,
// four to a CU.
#define C3_ROW_NT C3_ROWS_NT
#define C3_ROW_LIST C3_ROWS_LIST
#include "rowd.h"

namespace c3 {
hipError_t rows_init_attributes() { return init_rows(); }
hipError_t launch_rows(hipStream_t st, const FftArgs &a) { return run_rows(st, a); }
}  // namespace c3
