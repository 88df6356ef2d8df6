// Forward products C = A W^T (bf16), on raw weights or their images: instances of gemm_mi16_kernel.
#include "gemm_tiles.hpp"

namespace gpts {

hipError_t launch_gemm_fwd(Tile tile, int epi, const MfmaArgs& a, hipStream_t st) {
  switch (epi) {
    case EPI_BIAS: return launch_tile<EPI_BIAS, FORM_NT>(tile, a, st);
    case EPI_BIAS_RES: return launch_tile<EPI_BIAS_RES, FORM_NT>(tile, a, st);
    case EPI_BIAS_RES32_OUT32: return launch_tile<EPI_BIAS_RES32_OUT32, FORM_NT>(tile, a, st);
    case EPI_BIAS_RES32_OUT16: return launch_tile<EPI_BIAS_RES32_OUT16, FORM_NT>(tile, a, st);
    case EPI_GELU_TANH: return launch_tile<EPI_GELU_TANH, FORM_NT>(tile, a, st);
    case EPI_GELU_ERF: return launch_tile<EPI_GELU_ERF, FORM_NT>(tile, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace gpts
