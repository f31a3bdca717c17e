// gemv_rows_kernel, GR_GATED epilogue.
#include "gemm_rows.h"

namespace ssd {

hipError_t launch_rows_gated(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  return launch_rows_kind<GR_GATED>(a, sh, blocks, s);
}

}  // namespace ssd
