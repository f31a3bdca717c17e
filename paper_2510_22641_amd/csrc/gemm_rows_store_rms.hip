// gemv_rows_kernel, GR_STORE_RMS epilogue.
#include "gemm_rows.h"

namespace ssd {

hipError_t launch_rows_store_rms(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  return launch_rows_kind<GR_STORE_RMS>(a, sh, blocks, s);
}

}  // namespace ssd
