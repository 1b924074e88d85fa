// Pairs of products in one launch, 128x128 tiles (gemm_mfma_pair.hpp).
#include "gemm_mfma_pair.hpp"

namespace optimus {

int launch_gemm_pair_128(bool ragged, const PairLaunch& p) {
  return ragged ? launch_pair<128, 128, 2, 2, 1, 1>(p) : launch_pair<128, 128, 2, 2, 1, 0>(p);
}

}  // namespace optimus
