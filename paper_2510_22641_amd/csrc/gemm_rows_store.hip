// gemv_rows_kernel, GR_STORE epilogue.
#include "gemm_rows.h"

namespace ssd {

hipError_t launch_rows_store(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  return launch_rows_kind<GR_STORE>(a, sh, blocks, s);
}

}  // namespace ssd
