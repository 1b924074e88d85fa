// Two products in one launch: A B^T (the gradient of a linear layer's input) and A^T B (the gradient of its weight) of the same
// output gradient.  Neither reads what the other writes.
//
// What bounds the small ones is the launch, not the product: a dependent launch of one 64x64 tile per CU lasts 4 us before its
// first and after its last matrix instruction, and half the chip's LDS lies idle meanwhile.  In one grid the workgroups of both
// share the CUs.  The bodies are those of the single launches (gemm_mfma_tile), so the bits are too.
#pragma once
#include "gemm_mfma_kernel.hpp"

namespace optimus {

// The workgroups of the product that is named `first` come first in the grid, the other's behind them.
template <int BM, int BN, int WM, int WN, bool PLAIN_X, bool PLAIN_Y, int LOOP, int FORM>
__global__ __launch_bounds__(WM* WN * 64, (Occ<BM, BN, WM, WN>::value)) void gemm_pair_kernel(const KArgs x, const KArgs y,
                                                                                           const unsigned nx, const unsigned ny,
                                                                                           const int y_first) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds_all[lds_elems<BM, BN, LOOP>()];
  const unsigned w = blockIdx.x, n1 = y_first ? ny : nx;
  const bool second = w >= n1;
  const unsigned mine = second ? w - n1 : w;
  if (second != (y_first != 0)) gemm_mfma_tile<BM, BN, WM, WN, false, false, PLAIN_Y, false, LOOP, FORM>(y, mine, ny, lds_all);
  else gemm_mfma_tile<BM, BN, WM, WN, true, true, PLAIN_X, false, LOOP, FORM>(x, mine, nx, lds_all);
}

struct PairLaunch {
  const KArgs* x;
  const KArgs* y;
  unsigned nx, ny;
  int y_first;
  bool plain_x, plain_y;
  hipStream_t stream;
};
template <int BM, int BN, int WM, int WN, int LOOP, int FORM>
static int launch_pair(const PairLaunch& p) {
  const dim3 grid(p.nx + p.ny), block(WM * WN * 64);
#define OPTIMUS_PAIR(PX, PY) \
  hipLaunchKernelGGL((gemm_pair_kernel<BM, BN, WM, WN, PX, PY, LOOP, FORM>), grid, block, 0, p.stream, *p.x, *p.y, p.nx, p.ny, p.y_first)
  if constexpr (FORM == 0) {
    if (p.plain_x && p.plain_y) OPTIMUS_PAIR(true, true);
    else if (p.plain_x) OPTIMUS_PAIR(true, false);
    else if (p.plain_y) OPTIMUS_PAIR(false, true);
    else OPTIMUS_PAIR(false, false);
  } else {
    OPTIMUS_PAIR(false, false);
  }
#undef OPTIMUS_PAIR
  return hip_launch_status();
}

// 64x64 tiles: four stages of 64 k, or the four-slab ring, or its ragged form
int launch_gemm_pair_64(bool deep, bool ragged, const PairLaunch& p);
// 128x128 tiles: the ring, also ragged
int launch_gemm_pair_128(bool ragged, const PairLaunch& p);

}  // namespace optimus
