// Weight gradients C += dOut^T In, over one or several micro-batches, up to four in a launch:
// instances of gemm_mi16_group_kernel.
#include "gemm_tiles.hpp"

namespace gpts {

hipError_t launch_gemm_wgrad(Tile tile, const MfmaArgs* a, int n, const ReduceSeg* sums, int n_sums, hipStream_t st) {
  return launch_wgrads(tile, a, n, sums, n_sums, st);
}

}  // namespace gpts
