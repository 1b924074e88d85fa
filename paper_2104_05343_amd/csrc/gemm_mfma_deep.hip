// 64x64 tiles for launches that give a CU at most two workgroups: the loop with stages of 64 k, four of them in LDS (64 KiB).
//
// What bounds such a launch is the latency of the loads: a workgroup streams 128 rows of its panels through the four-slab ring
// with 32 KiB in flight, whatever the CU could fetch; twice as much here, and half the barriers.  Same sums in the same order as
// every other tile.  Eight stages (128 KiB) came out between the two: the first loads of 512 KiB across the chip's CUs arrive
// no faster, and every workgroup waits for its share of them before its first matrix instruction.
// Measured, us, ring / four stages / eight: A B [512 x 2048 x 2048] 15.7 / 11.6 / 12.6, [1024 x 1024 x 1024] 9.6 / 7.4 / 8.3, [2048 x
// 4096 x 1024] (512 workgroups) 31.0 / 29.0; A B^T [2048 x 2048 x 256] 16.3 / 10.8 / 11.4, [2048 x 4096 x 1024] 31.6 / 27.1; A^T B [512 x
// 2048 x 2048] 14.4 / 12.4 / 12.7; contractions of 256 and less the same within 0.3.
#include "gemm_mfma_kernel.hpp"

namespace optimus {

template <bool AKC, bool BKC>
static int launch_form(bool plain, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  const dim3 grid(nwg), block(256);
  if (plain) hipLaunchKernelGGL((gemm_mfma_kernel<64, 64, 2, 2, AKC, BKC, true, false, 3>), grid, block, 0, stream, ka);
  else hipLaunchKernelGGL((gemm_mfma_kernel<64, 64, 2, 2, AKC, BKC, false, false, 3>), grid, block, 0, stream, ka);
  return hip_launch_status();
}

int launch_gemm_mfma_deep(bool plain, int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  if (a_kcontig && !b_kcontig) return launch_form<true, false>(plain, ka, nwg, stream);
  if (a_kcontig && b_kcontig) return launch_form<true, true>(plain, ka, nwg, stream);
  if (!a_kcontig && !b_kcontig) return launch_form<false, false>(plain, ka, nwg, stream);
  return OPTIMUS_EINVAL;
}

}  // namespace optimus
