// Pairs of products in one launch, 64x64 tiles (gemm_mfma_pair.hpp).
#include "gemm_mfma_pair.hpp"

namespace optimus {

int launch_gemm_pair_64(bool deep, bool ragged, const PairLaunch& p) {
  if (ragged) return launch_pair<64, 64, 2, 2, 1, 1>(p);
  return deep ? launch_pair<64, 64, 2, 2, 3, 0>(p) : launch_pair<64, 64, 2, 2, 1, 0>(p);
}

}  // namespace optimus
