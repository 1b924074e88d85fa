// 64x64 tiles for launches that give a CU at most two workgroups, 128x64 and 128x128 tiles for those that give it one: the loop with stages
// of 64 k, four of them in LDS (64, 96 and 128 KiB).
//
// What bounds such a launch is the latency of the loads: a workgroup streams 128 rows of its panels through the four-slab ring
// with 32 KiB in flight, whatever the CU could fetch; twice as much here, and half the barriers.  Same sums in the same order as
// every other tile.  Eight stages (128 KiB) came out between the two: the first loads of 512 KiB across the chip's CUs arrive
// no faster, and every workgroup waits for its share of them before its first matrix instruction.
// Measured, us, ring / four stages / eight: A B [512 x 2048 x 2048] 15.7 / 11.6 / 12.6, [1024 x 1024 x 1024] 9.6 / 7.4 / 8.3, [2048 x
// 4096 x 1024] (512 workgroups) 31.0 / 29.0; A B^T [2048 x 2048 x 256] 16.3 / 10.8 / 11.4, [2048 x 4096 x 1024] 31.6 / 27.1; A^T B [512 x
// 2048 x 2048] 14.4 / 12.4 / 12.7; contractions of 256 and less the same within 0.3.
// The wider tiles, ring / four stages: 128x64 A B [2048 x 4096 x 1024] 33.3 / 25.1 (64x64 tiles, two a CU: 32), A B^T 36.7 / 25.3, A B [4096 x 4096 x
// 512] 32.8 / 24.5; 128x128 A B [2048 x 2048 x 2048] 22.6 / 20.8, A^T B [4096 x 8192 x 1024] 75.6 / 71.1, [1024 x 8192 x 3072] 64.6 / 58.4.
#include "gemm_mfma_kernel.hpp"

namespace optimus {

template <int BM, int BN, bool AKC, bool BKC>
static int launch_form(bool plain, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  const dim3 grid(nwg), block(256);
  if (plain) hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, 2, 2, AKC, BKC, true, false, 3>), grid, block, 0, stream, ka);
  else hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, 2, 2, AKC, BKC, false, false, 3>), grid, block, 0, stream, ka);
  return hip_launch_status();
}
template <int BM, int BN>
static int launch_tile(bool plain, int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  if (a_kcontig && !b_kcontig) return launch_form<BM, BN, true, false>(plain, ka, nwg, stream);
  if (a_kcontig && b_kcontig) return launch_form<BM, BN, true, true>(plain, ka, nwg, stream);
  if (!a_kcontig && !b_kcontig) return launch_form<BM, BN, false, false>(plain, ka, nwg, stream);
  return OPTIMUS_EINVAL;
}

int launch_gemm_mfma_deep(int variant, bool plain, int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  if (variant == 6) return launch_tile<128, 64>(plain, a_kcontig, b_kcontig, ka, nwg, stream);
  if (variant == 3) return launch_tile<128, 128>(plain, a_kcontig, b_kcontig, ka, nwg, stream);
  return launch_tile<64, 64>(plain, a_kcontig, b_kcontig, ka, nwg, stream);
}

}  // namespace optimus
