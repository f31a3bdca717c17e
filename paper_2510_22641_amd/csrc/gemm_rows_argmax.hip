// gemv_rows_kernel, GR_ARGMAX epilogue.
#include "gemm_rows.h"

namespace ssd {

hipError_t launch_rows_argmax(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  return launch_rows_kind<GR_ARGMAX>(a, sh, blocks, s);
}

}  // namespace ssd
