// Instances of the large-row GEMM (gemm_tiled.hpp) for every epilogue.
#include "gemm_tiled.hpp"

namespace incvit {

hipError_t launch_gemm_tiled(int epi, const GemmArgs& a, int expected, int rows, hipStream_t s) {
  switch (epi) {
    case EPI_QKV: return launch_tiled_epi<EPI_QKV>(a, expected, rows, s);
    case EPI_FC1: return launch_tiled_epi<EPI_FC1>(a, expected, rows, s);
    case EPI_RES: return launch_tiled_epi<EPI_RES>(a, expected, rows, s);
    case EPI_ATT: return launch_tiled_epi<EPI_ATT>(a, expected, rows, s);
    case EPI_DOWN: return launch_tiled_epi<EPI_DOWN>(a, expected, rows, s);
    default: return launch_tiled_epi<EPI_PART>(a, expected, rows, s);
  }
}

}  // namespace incvit
