// Weight gradients C += dOut^T In, over one or several micro-batches: instances of gemm_mi16_kernel.
#include "gemm_tiles.hpp"

namespace gpts {

hipError_t launch_gemm_wgrad(Tile tile, const MfmaArgs& a, hipStream_t st) {
  return launch_tile<EPI_ACCUM, FORM_TN>(tile, a, st);
}

}  // namespace gpts
