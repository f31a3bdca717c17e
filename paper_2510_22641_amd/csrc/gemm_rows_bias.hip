// gemv_rows_kernel, GR_BIAS epilogues (the imitation network's two layers).
#include "gemm_rows.h"

namespace ssd {

hipError_t launch_rows_bias(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  return launch_rows_kind<GR_BIAS>(a, sh, blocks, s);
}

}  // namespace ssd
