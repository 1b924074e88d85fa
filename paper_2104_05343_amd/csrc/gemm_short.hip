// Products with short panels in launches that fill the chip: the 64x64 tiles of gemm_generic.hip, but slabs of 64 bytes of k
// (16 of fp32, 32 of bf16; two of the eight parts), four wavefronts with the accumulators of all NACC parts of a 32x32 output
// each.  The bits of gemm_any_kernel: a k goes to the same part, the parts are added up the same way, and those past a panel's
// end are zeros there.
// What bounds gemm_any_kernel at such panels is work for the missing part of its slabs of 256 bytes; here it is the stores,
// which leave through LDS as whole rows (straight from the accumulators 17.8 us for a [2046 x 2046] output, this way 13.0).
#include "gemm_any.hpp"

namespace optimus {

template <typename T, bool AKC, bool BKC, int NACC, bool TINY>
__global__ __launch_bounds__(256, NACC == 8 ? 2 : NACC == 4 ? 3 : 4) void gemm_short_kernel(const GArgs a) {
  typedef Slab<T, 64, AKC, TINY, 64, 256> SA;
  typedef Slab<T, 64, BKC, TINY, 64, 256> SB;
  constexpr int KS = SA::KS, CH = SA::CHUNKS, STAGE = SA::BYTES + SB::BYTES;
  constexpr int PITCH = 68;   // floats per row of the finished tile, which leaves through LDS as whole rows
  constexpr int LDS = 2 * STAGE > 64 * PITCH * 4 ? 2 * STAGE : 64 * PITCH * 4;
  __shared__ __attribute__((aligned(16))) char lds[LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroups are dealt round-robin to the 8 XCDs: give each XCD a contiguous range of tiles, so that neighbours share
  // an L2 as they share operand rows
  long long wg = blockIdx.x;
  {
    const long long nwg = gridDim.x, per = nwg >> 3, rem = nwg & 7, xcd = wg & 7, slot = wg >> 3;
    wg = xcd * per + (xcd < rem ? xcd : rem) + slot;
  }
  const int tiles = a.tiles_m * a.tiles_n;
  const long long z = wg / tiles;
  const int t = (int)(wg % tiles);
  // column by column inside groups of four tile rows: the range of an XCD is then nearly square and reads the fewest bytes
  const int tg = t / (4 * a.tiles_n), gr = t - tg * 4 * a.tiles_n, rows_g = min(4, a.tiles_m - 4 * tg);
  const int m0 = (4 * tg + gr % rows_g) * 64, n0 = (gr / rows_g) * 64;
  if (a.skip_upper && n0 > m0 + 63) return;
  const int z1 = (int)(z / a.nz0), z0 = (int)(z % a.nz0);
  const int k_lo = a.k_lo_diag ? min(m0, a.Kp) : 0;
  const int k_hi = a.k_hi_diag ? min(a.Kp, m0 + 64) : a.Kp;
  const T* At = (const T*)a.A + z1 * a.sA1 + z0 * a.sA0 + (AKC ? (long long)m0 * a.lda : (long long)m0);
  const T* Bt = (const T*)a.B + z1 * a.sB1 + z0 * a.sB0 + (BKC ? (long long)n0 * a.ldb : (long long)n0);
  const int rows_a = a.Mb - m0, rows_b = a.Nb - n0;
  const int spp = (k_hi - k_lo + KS - 1) / KS;   // slabs per panel
  const int n = spp > 0 ? a.nl * spp : 0;
  const int rm = (wave >> 1) * 32, rn = (wave & 1) * 32;
  gf32x16 acc[NACC];
#pragma unroll
  for (int s = 0; s < NACC; ++s)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[s][e] = 0.f;
  const bool whole = rows_a >= 64 && rows_b >= 64 && a.lda < (1 << 22) && a.ldb < (1 << 22);
  unsigned off_a[CH], off_b[CH];
  SA::offsets(off_a, a.lda, tid);
  SB::offsets(off_b, a.ldb, tid);
  uint4 ra[CH], rb[CH];
  const T *oa = At, *ob = Bt;   // origin of the slab in ra, rb
  auto request = [&](int l, int k) {
    oa = At + l * a.sAl + (AKC ? (long long)k : (long long)k * a.lda);
    ob = Bt + l * a.sBl + (BKC ? (long long)k : (long long)k * a.ldb);
    if (whole && k_hi - k >= KS) {
      SA::load_full(ra, oa, off_a);
      SB::load_full(rb, ob, off_b);
    } else {
      SA::load(ra, oa, a.lda, rows_a, k_hi - k, tid);
      SB::load(rb, ob, a.ldb, rows_b, k_hi - k, tid);
    }
  };
  int l = 0, k = k_lo;
  if (n > 0) request(l, k);
  for (int i = 0; i < n; ++i) {
    char* la = lds + (i & 1) * STAGE;
    char* lb = la + SA::BYTES;
    SA::store(ra, la, oa, a.lda, rows_a, k_hi - k, tid);
    SB::store(rb, lb, ob, a.ldb, rows_b, k_hi - k, tid);
    const int at = k - k_lo;
    k += KS;
    if (k >= k_hi) { k = k_lo; ++l; }
    if (i + 1 < n) request(l, k);
    OPTIMUS_LDS_BARRIER();   // as in gemm_any_kernel: this slab is written, the one before it has been read
    auto two = [&](gf32x16& x, gf32x16& y) {
      eighth<SA, SB>(x, la, lb, rm, rn, 0, lane);
      eighth<SA, SB>(y, la, lb, rm, rn, 1, lane);
    };
    const int which = NACC == 2 ? 0 : (at / KS) & (NACC / 2 - 1);
    if (NACC == 2 || which == 0) two(acc[0], acc[1]);
    else if (NACC == 4 || which == 1) two(acc[2 < NACC ? 2 : 0], acc[3 < NACC ? 3 : 0]);
    else if (which == 2) two(acc[4 < NACC ? 4 : 0], acc[5 < NACC ? 5 : 0]);
    else two(acc[6 < NACC ? 6 : 0], acc[7 < NACC ? 7 : 0]);
  }
  EpiArgs e = a.epi;
  if (e.bias) e.bias += z0 * a.sBias0;
  const long long coff = z1 * a.sC1 + z0 * a.sC0;
  float* tile = (float*)lds;
  OPTIMUS_LDS_BARRIER();
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      auto part = [&](int s) { return s < NACC ? acc[s < NACC ? s : 0][g * 4 + c] : 0.f; };
      v[c] = ((part(0) + part(1)) + (part(2) + part(3))) + ((part(4) + part(5)) + (part(6) + part(7)));
    }
    *(float4*)(tile + (rm + (lane & 31)) * PITCH + rn + g * 8 + ((lane >> 5) << 2)) = make_float4(v[0], v[1], v[2], v[3]);
  }
  OPTIMUS_LDS_BARRIER();
  const int col = (tid & 15) * 4;
  if (n0 + col >= a.Nb) return;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = it * 16 + (tid >> 4);
    if (m0 + row >= a.Mb) return;
    const float4 w = *(const float4*)(tile + row * PITCH + col);
    const float v[4] = {w.x, w.y, w.z, w.w};
    epilogue_store4<false, true>(e, coff, m0 + row, n0 + col, v, min(4, a.Nb - n0 - col));
  }
}

template <typename T, int NACC, bool TINY = false>
static void launch_short(const GArgs& a, int a_kcontig, int b_kcontig, unsigned nwg, hipStream_t stream) {
  const dim3 grid(nwg), block(256);
  if (a_kcontig && b_kcontig) hipLaunchKernelGGL((gemm_short_kernel<T, true, true, NACC, TINY>), grid, block, 0, stream, a);
  else if (a_kcontig) hipLaunchKernelGGL((gemm_short_kernel<T, true, false, NACC, TINY>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((gemm_short_kernel<T, false, false, NACC, TINY>), grid, block, 0, stream, a);
}
template <typename T>
static void launch_type(const GArgs& a, const GemmDesc& d, bool tiny, unsigned nwg, hipStream_t stream) {
  constexpr int KS = 64 / (int)sizeof(T);   // k per slab
  if (tiny) launch_short<T, 2, true>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
  else if (d.Kp <= KS) launch_short<T, 2>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
  else if (d.Kp <= 2 * KS) launch_short<T, 4>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
  else launch_short<T, 8>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
}

int launch_gemm_short(const GArgs& a, const GemmDesc& d, bool tiny, unsigned nwg, hipStream_t stream) {
  if (d.dtype == OPTIMUS_BF16) launch_type<bf16_t>(a, d, tiny, nwg, stream);
  else launch_type<float>(a, d, tiny, nwg, stream);
  return hip_launch_status();
}

}  // namespace optimus
