// The ragged forms of the bf16 matrix-core product kernel (see RAG and LONG in gemm_mfma_kernel.hpp): tiles that share a CU.
#include "gemm_mfma_kernel.hpp"

namespace optimus {

template <int BM, int BN, bool AKC, bool BKC, bool LONG>
static int launch_one(const KArgs& ka, unsigned nwg, hipStream_t stream) {
  if (ka.seq_splits > 1)
    hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, 2, 2, AKC, BKC, false, true, 1, LONG ? 2 : 1>), dim3(nwg), dim3(256), 0, stream, ka);
  else
    hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, 2, 2, AKC, BKC, false, false, 1, LONG ? 2 : 1>), dim3(nwg), dim3(256), 0, stream, ka);
  return hip_launch_status();
}
template <int BM, int BN, bool LONG = false>
static int launch_layout(int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  if (a_kcontig && !b_kcontig) return launch_one<BM, BN, true, false, LONG>(ka, nwg, stream);
  if (a_kcontig && b_kcontig) return LONG ? OPTIMUS_EINVAL : launch_one<BM, BN, true, true, false>(ka, nwg, stream);
  if (!a_kcontig && !b_kcontig) return launch_one<BM, BN, false, false, LONG>(ka, nwg, stream);
  return OPTIMUS_EINVAL;
}

int launch_gemm_mfma_ragged(int variant, bool long_panels, int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream) {
  if (long_panels) return variant == 3 ? launch_layout<128, 128, true>(a_kcontig, b_kcontig, ka, nwg, stream) : OPTIMUS_EINVAL;
  switch (variant) {
    case 3: return launch_layout<128, 128>(a_kcontig, b_kcontig, ka, nwg, stream);
    case 6: return launch_layout<128, 64>(a_kcontig, b_kcontig, ka, nwg, stream);
    case 7: return launch_layout<64, 64>(a_kcontig, b_kcontig, ka, nwg, stream);
    default: return OPTIMUS_EINVAL;
  }
}

}  // namespace optimus
