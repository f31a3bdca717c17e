// gemv_rows_kernel, GR_CROSS epilogue.
#include "gemm_rows.h"

namespace ssd {

hipError_t launch_rows_cross(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  return launch_rows_kind<GR_CROSS>(a, sh, blocks, s);
}

}  // namespace ssd
