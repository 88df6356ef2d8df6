// Data gradients C = dOut W on the raw weight: instances of gemm_mi16_kernel.
#include "gemm_tiles.hpp"

namespace gpts {

hipError_t launch_gemm_dgrad(Tile tile, int epi, const MfmaArgs& a, hipStream_t st) {
  switch (epi) {
    case EPI_PLAIN: return launch_tile<EPI_PLAIN, FORM_NN>(tile, a, st);
    case EPI_DGELU_TANH: return launch_tile<EPI_DGELU_TANH, FORM_NN>(tile, a, st);
    case EPI_DGELU_ERF: return launch_tile<EPI_DGELU_ERF, FORM_NN>(tile, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace gpts
