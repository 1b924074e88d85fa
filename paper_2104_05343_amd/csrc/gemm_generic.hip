// Product kernel for everything the direct-to-LDS tiles of gemm_mfma.hip do not take: fp32 operands, and bf16 operands
// whose rows do not start on 16-byte boundaries.  Any shape, any stride, any alignment; fp32 accumulation.
//
// Products run on the matrix cores: v_mfma_f32_32x32x2_f32 for fp32 (fused multiply-adds of full fp32 operands, the
// precision of the scalar form at 157 TFLOP/s nominal) and v_mfma_f32_32x32x16_bf16 for bf16.
// Same panel loop as the other product kernel: the q SUMMA steps (Algorithms 1-3) are one k-loop.
//
// What bounds it: at the fp32 sizes of a layer's feed-forward half the matrix cores need 32 B/clk per CU from LDS and
// 16 (64x64 tile) or 32 (32x32 tile) from L2, so the loop is built around loads in flight: slabs of 256 bytes of k per
// row travel global -> registers (PF slabs ahead) -> LDS (two stages, one barrier per slab) -> fragments, with two
// wavefronts per SIMD so that one's matrix instructions cover the other's LDS traffic.
//   64x64 tile: eight wavefronts, 32x32 outputs each, wavefronts 0-3 on the first half of every slab, 4-7 on the second.
//   32x32 tile: the eight wavefronts share the output and take one eighth of every slab each; outputs too small to give
//   every CU a 64x64 tile then still use all CUs.
// All tiles keep the sums of the eight parts of the slabs apart and add them in the same order at the end, so the tile
// choice, and with it whole-grid against one-device launches, changes no bit.
// Short panels in launches that fill the chip: gemm_short.hip.
//
// Measured (fp32, 1024-wide layer on a 4 x 4 grid, one device): [1024 x 1024 x 1024] blocks 29 us (64x64 tiles, 74 TFLOP/s),
// [1024 x 4096 x 256] blocks 32 us (32x32 tiles, 67 TFLOP/s); scalar fused multiply-adds on 64x64 tiles took 180 and 733 us.
// With one wavefront per SIMD and slabs of 128 bytes 39 and 57 us; with bounds arithmetic in every slab 36 and 45 us.
#include "gemm_any.hpp"

namespace optimus {

template <typename T, int BT, bool AKC, bool BKC, bool TINY>
__global__ __launch_bounds__(GT_THREADS, 2) void gemm_any_kernel(const GArgs a) {
  typedef Slab<T, BT, AKC, TINY> SA;
  typedef Slab<T, BT, BKC, TINY> SB;
  constexpr int KS = SA::KS, CH = SA::CHUNKS;
  constexpr int PF = BT == 64 ? 2 : 4;     // slabs in flight per wavefront
  constexpr int PARTS = BT == 64 ? 4 : 1;  // parts of a slab per wavefront
  constexpr int STAGE = SA::BYTES + SB::BYTES;
  constexpr int LDS = 2 * STAGE > 32768 ? 2 * STAGE : 32768;
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
  const int m0 = (4 * tg + gr % rows_g) * BT, n0 = (gr / rows_g) * BT;
  if (a.skip_upper && n0 > m0 + BT - 1) return;
  const int z1 = (int)(z / a.nz0), z0 = (int)(z % a.nz0);
  // k range of a panel; the diagonal bounds are those of the 64-row tile, whichever tile runs (skipped terms are zeros,
  // but the slabs have to be cut alike)
  const int d0 = m0 & ~63;
  const int k_lo = a.k_lo_diag ? min(d0, a.Kp) : 0;
  const int k_hi = a.k_hi_diag ? min(a.Kp, d0 + 64) : a.Kp;
  const T* At = (const T*)a.A + z1 * a.sA1 + z0 * a.sA0 + (AKC ? (long long)m0 * a.lda : (long long)m0);
  const T* Bt = (const T*)a.B + z1 * a.sB1 + z0 * a.sB0 + (BKC ? (long long)n0 * a.ldb : (long long)n0);
  const int rows_a = a.Mb - m0, rows_b = a.Nb - n0;
  const int spp = (k_hi - k_lo + KS - 1) / KS;   // slabs per panel
  const int n = spp > 0 ? a.nl * spp : 0;
  const int rm = BT == 64 ? ((wave >> 1) & 1) * 32 : 0, rn = BT == 64 ? (wave & 1) * 32 : 0;
  const int part0 = BT == 64 ? (wave >> 2) * 4 : wave;   // first of this wavefront's parts

  gf32x16 acc[PARTS];
#pragma unroll
  for (int s = 0; s < PARTS; ++s)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[s][e] = 0.f;
  uint4 ra[PF][CH], rb[PF][CH];
  int l_ld = 0, k_ld = k_lo, l_st = 0, k_st = k_lo;   // the next slab to request, the next to store
  auto origin_a = [&](int l, int k) { return At + l * a.sAl + (AKC ? (long long)k : (long long)k * a.lda); };
  auto origin_b = [&](int l, int k) { return Bt + l * a.sBl + (BKC ? (long long)k : (long long)k * a.ldb); };
  auto next = [&](int& l, int& k) { k += KS; if (k >= k_hi) { k = k_lo; ++l; } };
  // Where no slab is cut the loop runs without any bounds arithmetic: the wavefronts of a workgroup do it at the same time,
  // between two barriers, so the matrix cores would wait for every instruction of it.
  const bool whole = rows_a >= BT && rows_b >= BT && (k_hi - k_lo) % KS == 0 && a.lda < (1 << 22) && a.ldb < (1 << 22);
  unsigned off_a[CH], off_b[CH];   // 32 bits: hence the limit on ld
  SA::offsets(off_a, a.lda, tid);
  SB::offsets(off_b, a.ldb, tid);
  auto sum_up = [&](auto whole_) {
    constexpr bool WHOLE = decltype(whole_)::value;
    auto request = [&](uint4 (&xa)[CH], uint4 (&xb)[CH]) {
      if constexpr (WHOLE) {
        const int l = l_ld < a.nl ? l_ld : 0;   // past the last slab: some slab, never used
        SA::load_full(xa, origin_a(l, k_ld), off_a);
        SB::load_full(xb, origin_b(l, k_ld), off_b);
      } else {
        const int k_left = l_ld < a.nl ? k_hi - k_ld : 0;
        SA::load(xa, origin_a(l_ld, k_ld), a.lda, rows_a, k_left, tid);
        SB::load(xb, origin_b(l_ld, k_ld), a.ldb, rows_b, k_left, tid);
      }
      next(l_ld, k_ld);
    };
    auto slab = [&](uint4 (&xa)[CH], uint4 (&xb)[CH], int stage, auto more) {
      char* la = lds + stage * STAGE;
      char* lb = la + SA::BYTES;
      if constexpr (WHOLE) {
        SA::store_full(xa, la, tid);
        SB::store_full(xb, lb, tid);
      } else {
        SA::store(xa, la, origin_a(l_st, k_st), a.lda, rows_a, k_hi - k_st, tid);
        SB::store(xb, lb, origin_b(l_st, k_st), a.ldb, rows_b, k_hi - k_st, tid);
        next(l_st, k_st);
      }
      if constexpr (decltype(more)::value) request(xa, xb);
      // every wavefront has written this slab, and has read the one before it, whose stage the next one overwrites
      OPTIMUS_LDS_BARRIER();
#pragma unroll
      for (int s = 0; s < PARTS; ++s) eighth<SA, SB>(acc[s], la, lb, rm, rn, part0 + s, lane);
    };
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      request(ra[u], rb[u]);
      __builtin_amdgcn_sched_barrier(0);   // in slab order, as in the loop: the waits there count back from the youngest load
    }
    // no way out between the slabs of a round: with one, the compiler no longer knows how many loads are in flight and
    // waits for all of them
    int i = 0;
    for (; i + PF <= n; i += PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) slab(ra[u], rb[u], (i + u) & 1, std::true_type{});
    }
#pragma unroll
    for (int u = 0; u < PF - 1; ++u)
      if (i + u < n) slab(ra[u], rb[u], (i + u) & 1, std::false_type{});
  };
  if (n > 0) {
    if (whole) sum_up(std::true_type{});
    else sum_up(std::false_type{});
  }
  EpiArgs e = a.epi;
  if (e.bias) e.bias += z0 * a.sBias0;
  const long long coff = z1 * a.sC1 + z0 * a.sC0;
  const int m = m0 + rm + (lane & 31), nc = n0 + rn + ((lane >> 5) << 2);
  float4* part = (float4*)lds;   // [wavefront][group of four columns][lane]
  OPTIMUS_LDS_BARRIER();
  auto sum4 = [](const float4& p, const float4& q, const float4& r, const float4& s) {
    return make_float4((p.x + q.x) + (r.x + s.x), (p.y + q.y) + (r.y + s.y), (p.z + q.z) + (r.z + s.z), (p.w + q.w) + (r.w + s.w));
  };
  auto group = [&](int s, int g) { return make_float4(acc[s][g * 4], acc[s][g * 4 + 1], acc[s][g * 4 + 2], acc[s][g * 4 + 3]); };
  auto put = [&](int g, const float4& lo, const float4& hi) {   // lo, hi: sums of parts 0-3 and 4-7
    const int col = nc + g * 8;
    if (m >= a.Mb || col >= a.Nb) return;
    const float v[4] = {lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w};
    epilogue_store4<false, true>(e, coff, m, col, v, min(4, a.Nb - col));
  };
  if constexpr (BT == 64) {
    // the two wavefronts of an output quarter swap halves: 0-3 store column groups 0 and 1, 4-7 groups 2 and 3
    const bool upper = wave >= 4;
    auto pick = [](bool c, const float4& x, const float4& y) { return make_float4(c ? x.x : y.x, c ? x.y : y.y, c ? x.z : y.z, c ? x.w : y.w); };
    float4 own[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) own[g] = sum4(group(0, g), group(1, g), group(2, g), group(3, g));
#pragma unroll
    for (int k = 0; k < 2; ++k) part[(wave * 2 + k) * 64 + lane] = pick(upper, own[k], own[2 + k]);
    OPTIMUS_LDS_BARRIER();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float4 other = part[((wave ^ 4) * 2 + k) * 64 + lane];
      const float4 mine = pick(upper, own[2 + k], own[k]);
      put(upper ? 2 + k : k, pick(upper, other, mine), pick(upper, mine, other));
    }
  } else {
#pragma unroll
    for (int g = 0; g < 4; ++g) part[(wave * 4 + g) * 64 + lane] = group(0, g);
    OPTIMUS_LDS_BARRIER();
    if (wave >= 4) return;
    float4 p[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) p[s] = part[(s * 4 + wave) * 64 + lane];
    put(wave, sum4(p[0], p[1], p[2], p[3]), sum4(p[4], p[5], p[6], p[7]));
  }
}

template <typename T, int BT, bool TINY = false>
static void launch_any(const GArgs& a, int a_kcontig, int b_kcontig, unsigned nwg, hipStream_t stream) {
  const dim3 grid(nwg), block(GT_THREADS);
  if (a_kcontig && b_kcontig) hipLaunchKernelGGL((gemm_any_kernel<T, BT, true, true, TINY>), grid, block, 0, stream, a);
  else if (a_kcontig) hipLaunchKernelGGL((gemm_any_kernel<T, BT, true, false, TINY>), grid, block, 0, stream, a);
  else if (b_kcontig) hipLaunchKernelGGL((gemm_any_kernel<T, BT, false, true, TINY>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((gemm_any_kernel<T, BT, false, false, TINY>), grid, block, 0, stream, a);
}
template <typename T>
static void launch_type(const GArgs& a, const GemmDesc& d, bool wide, bool tiny, unsigned nwg, hipStream_t stream) {
  if (tiny) launch_any<T, 32, true>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
  else if (wide) launch_any<T, 64>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
  else launch_any<T, 32>(a, d.a_kcontig, d.b_kcontig, nwg, stream);
}

int launch_gemm_generic(const GemmDesc& d, hipStream_t stream) {
  GArgs a;
  a.A = d.A; a.B = d.B;
  a.Mb = d.Mb; a.Nb = d.Nb; a.Kp = d.Kp; a.nl = d.nl;
  a.lda = d.lda; a.ldb = d.ldb; a.sAl = d.sAl; a.sBl = d.sBl;
  a.nz0 = d.nz0;
  a.sA0 = d.sA0; a.sA1 = d.sA1; a.sB0 = d.sB0; a.sB1 = d.sB1; a.sC0 = d.sC0; a.sC1 = d.sC1; a.sBias0 = d.sBias0;
  a.skip_upper = d.skip_upper; a.k_hi_diag = d.k_hi_diag; a.k_lo_diag = d.k_lo_diag;
  EpiArgs& e = a.epi;
  e.alpha = d.alpha; e.bias = d.bias; e.C = d.C; e.pre_act = d.pre_act; e.gelu_grad_of = d.gelu_grad_of;
  e.residual = d.residual; e.ldc = d.ldc; e.act = d.act; e.out_fp32 = d.out_fp32;
  e.in_bf16 = d.dtype == OPTIMUS_BF16;
  // four-element accesses of C and what is laid out like it (bias is read element by element)
  const auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  e.vec_ok = d.ldc % 4 == 0 && d.sC0 % 4 == 0 && d.sC1 % 4 == 0 && al16(d.C) && al16(d.pre_act) && al16(d.gelu_grad_of) && al16(d.residual);
  // 64x64 tiles where they give most CUs one; below that 32x32 tiles, four times the workgroups (64 workgroups of 64x64
  // tiles and 256 of 32x32 at [1024 x 4096 x 256]: the first leave three CUs of four idle)
  const long long nz = (long long)d.nz0 * d.nz1;
  const int chunk = d.dtype == OPTIMUS_BF16 ? 8 : 4;
  const bool tiny = (d.a_kcontig ? d.Kp : d.Mb) < chunk || (d.b_kcontig ? d.Kp : d.Nb) < chunk;   // rows shorter than a 16-byte load
  const bool wide = !tiny && (long long)((d.Mb + 63) / 64) * ((d.Nb + 63) / 64) * nz >= 192;
  // The short kernel where two of its slabs hold a panel and the launch has a tile for every CU, and, up to half of the other
  // kernel's slabs, where at most three of its slabs stand for one of those and CUs get several tiles.  Measured, us, fp32,
  // gemm_any_kernel / short.  [2046 x 2046] outputs, one panel: Kp = 16 27.4 / 13.0, 32 27.3 / 16.0, 48 27.2 / 19.0, 64 26.2 /
  // 21.1; 16 blocks of four panels each: 16 594 / 159, 32 595 / 286, 48 594 / 504, 64 540 / 647, 96 934 / 875.  16 blocks of
  // [256 x 256], four panels: 16 11.1 / 6.7, 32 11.2 / 9.8, 48 11.3 / 13.7.  (Scalar fused multiply-adds on 64x64 tiles, slabs
  // of 16: [2046 x 2046], one panel, 16 13.8; 16 blocks 16 230, 48 502.)
  const int ks = d.dtype == OPTIMUS_BF16 ? 32 : 16, slabs = (d.Kp + ks - 1) / ks;
  const long long tiles64 = (long long)((d.Mb + 63) / 64) * ((d.Nb + 63) / 64) * nz;
  const bool brief = (d.a_kcontig || !d.b_kcontig) &&
                     ((slabs <= (tiny ? 1 : 2) && tiles64 >= 256) ||
                      (!tiny && slabs <= 8 && slabs <= 3 * ((slabs + 3) / 4) && tiles64 >= 1024 && d.Mb >= 64 && d.Nb >= 64));
  const int bt = wide || brief ? 64 : 32;
  a.tiles_m = (d.Mb + bt - 1) / bt;
  a.tiles_n = (d.Nb + bt - 1) / bt;
  const long long nwg = (long long)a.tiles_m * a.tiles_n * nz;
  if (nwg <= 0 || nwg > 0x7fffffffLL) return OPTIMUS_ESHAPE;
  if (brief) return launch_gemm_short(a, d, tiny, (unsigned)nwg, stream);
  if (d.dtype == OPTIMUS_BF16) launch_type<bf16_t>(a, d, wide, tiny, (unsigned)nwg, stream);
  else launch_type<float>(a, d, wide, tiny, (unsigned)nwg, stream);
  return hip_launch_status();
}

int launch_gemm(const GemmDesc& d, hipStream_t stream) {
  if (gemm_mfma_supported(d)) return launch_gemm_mfma(d, stream);
  GemmDesc g = d;
  g.splits = 1;
  return launch_gemm_generic(g, stream);
}

}  // namespace optimus
