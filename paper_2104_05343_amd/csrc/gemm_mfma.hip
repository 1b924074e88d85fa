// Host side of the bf16 matrix-core product kernels (gemm_mfma_kernel.hpp): tile and split planner, launches, and the
// combine kernel of the panel split.
#include <string.h>

#include <atomic>

#include "combine.hpp"
#include "gemm_mfma_pair.hpp"

namespace optimus {

// Tuning hooks of the benchmark and the tests (process-wide; atomics, so that a hook set from one thread while
// another launches is a race on WHICH setting a launch sees, never on memory).  They select tiles and the k-loop, and
// a forced tile plans its own panel split; nothing else in the library is process-global state.
static std::atomic<int> g_variant{-1};
static std::atomic<int> g_loop{2};   // k-loop of the fast path where both exist (see gemm_mfma_kernel); 1 or 2
void gemm_set_variant(int v) {
  // v >= 1000: the older k-loop with variant v - 1000 (1000 + 255 = automatic tile); otherwise the default k-loop
  if (v >= 1000) { g_loop = 1; v -= 1000; if (v == 255) v = -1; } else g_loop = 2;
  g_variant = v;
}
int gemm_get_variant() { return g_variant; }
static std::atomic<int> g_corun_variant[2] = {{-1}, {-1}};
void gemm_set_corun_variants(int chain_v, int branch_v) { g_corun_variant[0] = chain_v; g_corun_variant[1] = branch_v; }
static std::atomic<int> g_last_plan{-1};
int gemm_last_plan() { return g_last_plan; }

// ---- fixed-order combine of panel-split partials + epilogue (combine.hpp) ----
__global__ __launch_bounds__(256) void gemm_combine_vec_kernel(const CombineJob j) {
  combine_quad_vec(j, blockIdx.x * 256u + threadIdx.x);
}
__global__ __launch_bounds__(256) void gemm_combine_jobs_kernel(const CombineJobs jobs) {
  unsigned wg = blockIdx.x;
  int k = 0;
  while (k + 1 < jobs.n && wg >= jobs.blocks[k]) wg -= jobs.blocks[k++];
  combine_quad_vec(jobs.j[k], wg * 256u + threadIdx.x);
}
// any width, alignment and number of quads
__global__ __launch_bounds__(256) void gemm_combine_kernel(const CombineJob j) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x, quads_per_row = (j.Nb + 3) / 4;
  const int n = (int)(idx % quads_per_row) * 4, nvalid = min(4, j.Nb - n);
  const long long r = idx / quads_per_row, z = r / j.Mb;
  const int m = (int)(r % j.Mb);
  if (z >= j.nz) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < j.splits; ++s) {
    const float* p = j.partials + (s * j.nz + z) * (long long)j.Mb * j.Nb + (long long)m * j.Nb + n;
    for (int c = 0; c < nvalid; ++c) v[c] += p[c];
  }
  const int z1 = (int)(z / j.nz0), z0 = (int)(z % j.nz0);
  EpiArgs e = j.epi;
  if (e.bias) e.bias += z0 * j.sBias0;
  epilogue_store4<false>(e, z1 * j.sC1 + z0 * j.sC0, m, n, v, nvalid);
}
int launch_gemm_combines(const CombineJobs& in, hipStream_t stream) {
  CombineJobs jobs = {};   // those of the short path
  long long blocks = 0;
  for (int k = 0; k < in.n; ++k) {
    const CombineJob& j = in.j[k];
    const long long b = (j.nz * j.Mb * ((j.Nb + 3) / 4) + 255) / 256;
    if (j.vec) {
      blocks += jobs.blocks[jobs.n] = (unsigned)b;
      jobs.j[jobs.n++] = j;
    } else {
      hipLaunchKernelGGL(gemm_combine_kernel, dim3((unsigned)b), dim3(256), 0, stream, j);
      const int rc = hip_launch_status();
      if (rc) return rc;
    }
  }
  if (jobs.n == 0) return OPTIMUS_OK;
  if (jobs.n == 1) hipLaunchKernelGGL(gemm_combine_vec_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, jobs.j[0]);
  else hipLaunchKernelGGL(gemm_combine_jobs_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, jobs);
  return hip_launch_status();
}

// ---- host side ----
struct Variant {
  int BM, BN, WM, WN;
};
// index = variant id used by gemm_set_variant
static const Variant kVariants[] = {
    {256, 256, 2, 4},   // 0: 8 waves, wave tile 128x64
    {256, 128, 4, 2},   // 1: 8 waves, wave tile 64x64
    {128, 256, 2, 4},   // 2: 8 waves, wave tile 64x64
    {128, 128, 2, 2},   // 3: 4 waves, wave tile 64x64, two workgroups per CU
    {256, 256, 2, 4},   // 4: same as 0 (kept so that variant ids stay stable)
    {64, 64, 2, 2},     // 5: the any-shape kernel (gemm_generic.hip)
    {128, 64, 2, 2},    // 6: 4 waves, wave tile 64x32: narrow outputs (attention with 64-wide heads)
    {64, 64, 2, 2},     // 7: 4 waves, wave tile 32x32: small blocks that need every CU (least bytes per CU)
    {256, 128, 2, 2},   // 8: 4 waves, wave tile 128x64 (a quarter fewer LDS bytes per flop than variant 1)
    {128, 256, 2, 2},   // 9: 4 waves, wave tile 64x128
};
constexpr int kAnyVariant = 5;

template <int BM, int BN, int WM, int WN, bool AKC, bool BKC>
static int launch_one(const KArgs& ka, long long nwg, hipStream_t stream) {
  const EpiArgs& e = ka.epi;
  if constexpr (BM * BN < 256 * 256) {  // (the 256x256 tile has no registers for a second accumulator)
    if (ka.seq_splits > 1) {
      if constexpr (BM + BN >= 384) {
        if (g_loop == 2) {
          hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, WM, WN, AKC, BKC, false, true, 2>), dim3((unsigned)nwg), dim3(WM * WN * 64),
                             0, stream, ka);
          return hip_launch_status();
        }
      }
      hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, WM, WN, AKC, BKC, false, true>), dim3((unsigned)nwg), dim3(WM * WN * 64), 0,
                         stream, ka);
      return hip_launch_status();
    }
  }
  if (ka.seq_splits > 1) return OPTIMUS_EINVAL;
  const bool plain = ka.splits == 1 && e.alpha == 1.0f && !e.bias && !e.pre_act && !e.act && !e.gelu_grad_of && !e.residual;
  // The 64-wide stages are measured 2-6 % faster than the four-slab ring on the tiles that own a CU (256x256, 256x128,
  // 128x256, 8 or 4 wavefronts) and, with two stages, slower or equal on the tiles that share one (128x128, 128x64, 64x64: several
  // workgroups per CU fill each other's gaps, and the finer ring refills sooner), so each keeps its own loop.  64x64 tiles in
  // launches of at most two workgroups per CU: launch_gemm_mfma.
  constexpr bool HAS_LOOP2 = BM + BN >= 384;
  if constexpr (HAS_LOOP2) {
    if (g_loop == 2) {
      if (plain)
        hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, WM, WN, AKC, BKC, true, false, 2>), dim3((unsigned)nwg), dim3(WM * WN * 64), 0, stream, ka);
      else
        hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, WM, WN, AKC, BKC, false, false, 2>), dim3((unsigned)nwg), dim3(WM * WN * 64), 0, stream, ka);
      return hip_launch_status();
    }
  }
  if (plain) {
    hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, WM, WN, AKC, BKC, true>), dim3((unsigned)nwg), dim3(WM * WN * 64), 0, stream, ka);
  } else {
    hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, WM, WN, AKC, BKC, false>), dim3((unsigned)nwg), dim3(WM * WN * 64), 0, stream, ka);
  }
  return hip_launch_status();
}

template <int BM, int BN, int WM, int WN>
static int launch_layout(const GemmDesc& d, const KArgs& ka, long long nwg, hipStream_t stream) {
  if (d.a_kcontig && !d.b_kcontig) return launch_one<BM, BN, WM, WN, true, false>(ka, nwg, stream);
  if (d.a_kcontig && d.b_kcontig) return launch_one<BM, BN, WM, WN, true, true>(ka, nwg, stream);
  if (!d.a_kcontig && !d.b_kcontig) return launch_one<BM, BN, WM, WN, false, false>(ka, nwg, stream);
  return OPTIMUS_EINVAL;  // [K][M] x [N][K] does not occur in the method
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

bool gemm_mfma_supported(const GemmDesc& d) {
  if (d.dtype != OPTIMUS_BF16) return false;
  if (!d.a_kcontig && d.b_kcontig) return false;
  if (!aligned16(d.A) || !aligned16(d.B)) return false;
  // every 16-byte chunk must be fully inside or fully outside the operand, and aligned
  if (d.lda % 8 || d.ldb % 8) return false;
  if (d.sAl % 8 || d.sBl % 8 || d.sA0 % 8 || d.sA1 % 8 || d.sB0 % 8 || d.sB1 % 8) return false;
  if (d.a_kcontig ? (d.Kp % 8) : (d.Mb % 8)) return false;
  if (d.b_kcontig ? (d.Kp % 8) : (d.Nb % 8)) return false;
  return true;
}

// Buffer addressing: a lane's byte offset plus the slab's inside the resource's 2 GiB window, which starts at the tile's
// corner of a panel.  k-contiguous operand: rows of the tile, ld apart, times the panel's length; k-strided: the panel's k
// rows, ld apart.
constexpr long long kWindow = 1LL << 31;
static bool panel_in_window(bool kcontig, int ld, long long k, int rows) {
  return 2 * (kcontig ? (long long)(rows - 1) * ld + k : (k - 1) * (long long)ld + rows) <= kWindow;
}
static bool panels_in_window(const GemmDesc& d) {   // as every form but the long one needs them; ragged blocks walk slabs in pairs
  const long long k = ((long long)d.Kp + 2 * BK - 1) / (2 * BK) * (2 * BK);
  return panel_in_window(d.a_kcontig, d.lda, k, 256) && panel_in_window(d.b_kcontig, d.ldb, k, 256);
}
// The long form starts a new window inside a panel of a k-strided operand: a slab of 32 k rows has to fit.  128x128 tiles.
static bool long_panels_ok(const GemmDesc& d) {
  const long long k = ((long long)d.Kp + 2 * BK - 1) / (2 * BK) * (2 * BK);
  return !d.b_kcontig && panel_in_window(d.a_kcontig, d.lda, d.a_kcontig ? k : BK, 128) && panel_in_window(false, d.ldb, BK, 128);
}
// Panels of over 1 GiB: the any-shape kernel, whose eight wavefronts share a 64x64 tile's k, or the tiles of this file.
// Measured, us, any-shape kernel / these.  A B, K = 32768: [512 x 1024] outputs 139 / 189, [1024 x 1024] 121 / 191,
// [1024 x 2048] 240 / 223, [2048 x 2048] 482 / 315, [2048 x 4096] 1085 / 445; K = 131072: [2048 x 1024] 1205 / 1405,
// [2048 x 2048] 2320 / 1433.  A^T B, second operand 2 GiB: 64 rows of output (256 tiles of 64x64) 428 / 571, 256 rows 2502 /
// 1350.  A k-contiguous operand whose rows are 2 MiB apart (A B^T, K = 1048576): [1024 x 1024] 5642 / 14585, [2048 x 2048]
// 23314 / 31273.
static bool any_shape_pays(const GemmDesc& d) {
  const long long ld = d.lda > d.ldb ? d.lda : d.ldb;
  if (512 * ld < (1LL << 30) && 2 * (long long)d.Kp * ld < (1LL << 30)) return false;
  const bool rows_far = (d.a_kcontig && d.lda > (1 << 18)) || (d.b_kcontig && d.ldb > (1 << 18));
  return rows_far || (long long)((d.Mb + 63) / 64) * ((d.Nb + 63) / 64) <= 512;
}
static bool variant_fits(const Variant& v, const GemmDesc& d) {
  if (d.Mb % v.BM || d.Nb % v.BN || d.Kp % (2 * BK)) return false;  // slabs are walked in pairs
  return panels_in_window(d);
}
// Blocks that no tile divides (64x64 is the smallest), or whose C allows no vector epilogue, take the ragged form of the
// tiles that share a CU: edges are cut at any size there, and a cut tile of 256 rows would be mostly edge.
static bool ragged_tile(int v) { return v == 3 || v == 6 || v == 7; }

// Tile shape and panel split for one product.  The split is chosen from ONE device's block only (never from the
// batch count), so that grid mode and device mode add the same slabs in the same order and give identical bits; the
// tile shape changes no bit and may be chosen for the whole launch (GemmDesc::plan_for_batch, see make_plan).
// Cost model (microseconds, calibrated on MI355X): fixed launch/prologue/epilogue cost, plus the slabs one
// workgroup walks times the measured time per slab of the variant, times the rounds needed to place all
// workgroups; a split adds the combine launch and the fp32 partial tiles written once and read once.
struct Plan {
  int variant;
  int splits;
  int ragged;  // 1: the tile's ragged form; 2: the same for long panels
  int seq;  // 1: the split is emulated inside each workgroup (KArgs::seq_splits): same bits, no partial tiles, no combine
  float us;  // the estimate it was chosen by
};

// have_ws: the caller's workspace holds the partial tiles of the planned split.  Without it the same split is
// emulated inside each workgroup (identical bits, see KArgs::seq_splits), so a result never depends on the workspace.
// compute units of the current device (the planner's unit of parallelism); 256 when there is no device to ask
int num_cus() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return 256; }
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) { (void)hipGetLastError(); n = 256; }
    cached[dev] = n;
  }
  return cached[dev];
}

// forced, forced_corun: the hooks as make_plan read them
static Plan compute_plan(const GemmDesc& d, bool vec_ok, bool have_ws, int forced, int forced_corun) {
  Plan best = {kAnyVariant, 1, 0, 0, 0.f};
  if (forced == kAnyVariant) return best;
  const bool long_panels = !panels_in_window(d);
  if (long_panels && !long_panels_ok(d)) return best;
  if (forced < 0 && any_shape_pays(d)) return best;
  const bool ragged = !vec_ok || !variant_fits(kVariants[7], d);
  const auto fits = [&](int v) { return long_panels ? v == 3 : ragged ? ragged_tile(v) : variant_fits(kVariants[v], d); };
  if (ragged) {   // a forced tile that has no such form is ignored
    best.ragged = long_panels ? 2 : 1;
    if (!fits(forced)) forced = -1;
    if (!fits(forced_corun)) forced_corun = -1;
  }
  const auto tiles_of = [&](int v) {
    return (long long)((d.Mb + kVariants[v].BM - 1) / kVariants[v].BM) * ((d.Nb + kVariants[v].BN - 1) / kVariants[v].BN);
  };
  // per candidate: variant id, workgroups resident per CU, fixed cost (launch, prologue, epilogue: us and us per MiB
  // of output), and the time per slab of one workgroup: alone on the chip (t_lone), with every CU holding one
  // workgroup (t_full: all CUs' loads share the L2 fabric; the rise is steep only near full occupancy, hence the
  // square), and the increment per further workgroup resident on the same CU (t_more).  Measured on MI355X with the
  // kernels as of the commit that last touched this table (one forced-variant sweep over the products of the
  // benchmark configurations 3-5); tests/test_gpu_planner.py fails when the kernels drift away from it.
  struct Cand { int v, per_cu; float fixed_us, out_us_per_mib, t_lone, t_full, t_more; };
  constexpr int kCands = 8;
  static const Cand cand[kCands] = {{0, 1, 12.0f, 0.15f, 0.54f, 0.64f, 0.00f},
                               {1, 1, 8.0f, 0.30f, 0.24f, 0.40f, 0.00f},
                               {2, 1, 8.0f, 0.30f, 0.24f, 0.405f, 0.00f},
                               {3, 2, 5.5f, 0.45f, 0.20f, 0.25f, 0.21f},
                               {6, 4, 4.5f, 0.50f, 0.19f, 0.21f, 0.133f},
                               {7, 5, 4.0f, 0.50f, 0.14f, 0.155f, 0.045f},
                               {8, 1, 8.0f, 0.30f, 0.24f, 0.41f, 0.00f},
                               {9, 1, 8.0f, 0.30f, 0.24f, 0.415f, 0.00f}};
  const long long slabs = (long long)d.nl * ((d.Kp + 2 * BK - 1) / (2 * BK)) * 2;
  const long long ncu = num_cus();
  const bool splittable = d.nl > 1 && !d.skip_upper && !d.k_hi_diag && !d.k_lo_diag;
  const float out_mib = (float)d.Mb * (float)d.Nb * 2.0f / 1048576.0f;
  float best_cost = 0.f;
  bool found = false;
  // Two passes.  The panel split changes the order in which a result is added up, so it is chosen from ONE block's
  // shape alone, as if the product ran by itself (pass 0): a product has the same bits wherever it is launched from.
  // The tile shape does not change them (every element walks the same slabs in the same order whatever tile it
  // lies in: the variants give identical bits, which the tests check), so a launch that covers several blocks
  // (the whole grid, the matrices of a batch of heads) or that shares the chip with a second product then picks
  // its tile, for that split, for the workgroups and the company it really has (pass 1).
  const long long batch = d.plan_for_batch ? (long long)(d.nz0 > 0 ? d.nz0 : 1) * (d.nz1 > 0 ? d.nz1 : 1) : 1;
  for (int pass = 0; pass < (batch > 1 || d.corun > 0 ? 2 : 1); ++pass) {
  const int fixed_sp = pass == 0 ? 0 : best.splits;
  if (pass == 1) found = false;
  for (int ci = 0; ci < kCands; ++ci) {
    const Cand& c = cand[ci];
    const int v = c.v;
    if (forced >= 0 && v != (forced == 4 ? 0 : forced)) continue;
    if (pass == 1 && forced_corun >= 0 && v != forced_corun) continue;
    if (!fits(v)) continue;
    const long long tiles = tiles_of(v) * (pass == 0 ? 1 : batch);
    for (int sp = fixed_sp ? fixed_sp : 1; sp <= (fixed_sp ? fixed_sp : 8); ++sp) {
      if (!fixed_sp && sp > 1 && (!splittable || slabs / sp < 8)) break;
      const long long wgs = tiles * sp;
      const long long cap = ncu * c.per_cu;
      const long long rounds = (wgs + cap - 1) / cap;
      const long long in_round = wgs < cap ? wgs : cap;
      const int resident = (int)((in_round + ncu - 1) / ncu);             // workgroups on the fullest CU
      const float busy = in_round >= ncu ? 1.0f : (float)in_round / (float)ncu;  // share of the CUs in use
      float t_slab = c.t_lone + (c.t_full - c.t_lone) * busy * busy + c.t_more * (float)(resident - 1);
      // One workgroup of 128x64 or 128x128 per CU has four stages (launch_gemm_mfma).  128x64 tiles, ring / four stages, us: [2048 x 4096 x 1024] A B 33.6 /
      // 25.5, A B^T 37.4 / 25.8, A^T B 28.2 / 26.3, [768 x 8192 x 2304] 60 / 44, 68 / 45, 50 / 46; 128x128: 42.4 / 40.3, 49.9 / 41.4, 43.5 / 40.9.  Contractions of more
      // than 6144 that can be split are better off so: operands from memory, split / one range of 128x64, A B^T [3072 x 8192 x 512] 43 / 54, A^T B [384 x
      // 8192 x 4096] 43 / 65, A B^T [2048 x 6144 x 1024] 41 / 34.  In one panel of 8192 and more the loads want 160 workgroups: A B [768 x 12288 x 1536],
      // 144 of them or 288 of 64x64, 90 / 70, [640 x 8192 x 2048], 160 or 320, 50 / 53.  Not counted: 128x128 tiles' gain where it is under 10 % (A B,
      // A^T B), and 128x64 in splits, which hardly occur in one workgroup per CU.  The split is the one of the product by itself; in company the
      // launch has the ring.
      const bool deep = !ragged && wgs <= ncu && (pass == 0 || d.corun == 0);
      // the 128x128 tile depends on the operand layouts: both k-contiguous (A B^T) is its slowest form, one of each its fastest
      if (v == 3) t_slab *= d.a_kcontig && d.b_kcontig ? (deep ? 1.0f : 1.14f) : (d.a_kcontig ? 0.92f : 1.04f);
      const bool few = d.a_kcontig && !splittable && slabs >= 256 && 8 * wgs < 5 * ncu;
      if (v == 6 && deep && sp == 1 && (!d.a_kcontig || !splittable || slabs <= 192) && !few) t_slab *= d.a_kcontig ? 0.7f : 0.9f;
      else if (v == 6 && d.a_kcontig && d.b_kcontig) t_slab *= 1.18f;
      if (v == 7 && !d.a_kcontig) t_slab *= 1.25f;   // both operands through the transposing LDS reads
      // The form with four stages (at most two workgroups per CU), for long contractions and all layouts alike (by itself, one workgroup
      // per CU: A B 0.74 of the ring's time, A B^T 0.66, A^T B 0.86, nothing at 256 k).  [1024 x 4096 x 256] in four ranges of it against
      // the ring's eight: A B 14.8 us to 12.3, A B^T 15.4 to 12.2, A^T B 13.5 to 12.0.
      if (v == 7 && !ragged && wgs <= 2 * ncu) t_slab *= resident == 1 ? 0.7f : 0.9f;
      const float per_wg = (float)((((slabs + sp - 1) / sp) + 1) & ~1LL) * t_slab;
      // split: the combine launch, and the fp32 partial tiles read back by it (their writes overlap the products)
      const float traffic_us =
          sp > 1 ? 4.0f + (float)sp * (float)d.Mb * (float)d.Nb * 4.0f / 3.0e6f * (pass == 0 ? 1.0f : (float)batch) : 0.f;
      float cost = c.fixed_us + c.out_us_per_mib * out_mib * (pass == 0 ? 1.0f : (float)batch) + (float)rounds * per_wg + traffic_us;
      // Two products that run side by side on two streams (the pairs of the layer's backward pass): the tiles of 8
      // wavefronts, which take a CU's LDS and registers alone, are the better partners, also where such a tile leaves
      // half the CUs idle when the product runs by itself (the other product's workgroups take those).  Measured on
      // the backward pass of the 4096-wide layers (one device of the q = 4 / q = 8 grids): 256x128 tiles for both
      // products 0.55 / 0.61 ms, 128x128 tiles for both 0.64 / 0.72 ms, 256x128 for the chain and 128x128 for the
      // branch 0.65 / 0.69 ms, the reverse 0.58 / 0.63 ms.  The factor, whole steps of one layer, 1 / 1.25 / 1.5: 4096-wide, q = 4, 897 /
      // 846 / 840 us, fused 877 / 842 / 836, q = 8 872 / 863 / 874; 1024-wide, q = 2, s = 1792, 705 / 680 / 676; q = 4 191 / 193 / 193.
      if (d.corun > 0 && c.per_cu >= 2 && pass == 1 && batch == 1) cost *= 1.25f;
      if (!found || cost < best_cost) {
        found = true;
        best_cost = cost;
        best = {v, sp, best.ragged, 0, cost};
      }
      // A launch with many blocks has workgroups enough without the split: one workgroup then walks all the slabs of
      // its tile and adds them up range by range as the split workgroups and their combine would (identical bits).
      if (pass == 1 && batch > 1 && sp > 1 && kVariants[v].BM * kVariants[v].BN < 256 * 256) {
        const long long rounds1 = (tiles + cap - 1) / cap;
        const long long in1 = tiles < cap ? tiles : cap;
        const int res1 = (int)((in1 + ncu - 1) / ncu);
        const float busy1 = in1 >= ncu ? 1.0f : (float)in1 / (float)ncu;
        const float t1 = c.t_lone + (c.t_full - c.t_lone) * busy1 * busy1 + c.t_more * (float)(res1 - 1);
        const float cost1 = c.fixed_us + c.out_us_per_mib * out_mib * (float)batch + (float)rounds1 * (float)slabs * t1;
        if (cost1 < best_cost) {
          best_cost = cost1;
          best = {v, sp, best.ragged, 1, cost1};
        }
      }
    }
  }
  }
  if (best.splits > 1 && !best.seq && !have_ws) {
    // No workspace: the same split, walked inside the workgroups (same bits).  One workgroup then owns all slabs of its
    // tile, so the tile is picked again for that walk: the tile with the least estimated time among those that have
    // registers for the second accumulator set (not 256x256).
    best.seq = 1;
    float seq_best = 0.f;
    int seq_v = -1;
    for (int ci = 0; ci < kCands; ++ci) {
      const Cand& c = cand[ci];
      if (kVariants[c.v].BM * kVariants[c.v].BN >= 256 * 256 || !fits(c.v)) continue;
      if (forced >= 0 && c.v != forced) continue;
      const long long tiles = tiles_of(c.v) * batch;
      const long long cap = ncu * c.per_cu;
      const long long rounds = (tiles + cap - 1) / cap;
      const long long in_round = tiles < cap ? tiles : cap;
      const int resident = (int)((in_round + ncu - 1) / ncu);
      const float busy = in_round >= ncu ? 1.0f : (float)in_round / (float)ncu;
      const float t = c.t_lone + (c.t_full - c.t_lone) * busy * busy + c.t_more * (float)(resident - 1);
      const float cost = c.fixed_us + c.out_us_per_mib * out_mib * (float)batch + (float)rounds * (float)slabs * t;
      if (seq_v < 0 || cost < seq_best) { seq_best = cost; seq_v = c.v; }
    }
    if (seq_v >= 0) best.variant = seq_v;
    else if (kVariants[best.variant].BM * kVariants[best.variant].BN >= 256 * 256) {
      static const int order[7] = {1, 2, 8, 9, 3, 6, 7};
      for (int k = 0; k < 7; ++k)
        if (fits(order[k])) { best.variant = order[k]; break; }
    }
  }
  return best;
}

// The plan is arithmetic on shapes, 1 us of host time for its sixty combinations of tile and split, and a layer's pass asked for it a
// hundred times (workspace sizes, every product): a thread keeps the last plans it computed, by everything a plan depends on.
// The hooks are read once, for the key and the plan: another thread may set them at any time.
// Host time of a pass before and now: two checkpointed layers of [128 x 128] blocks 266 / 232 us, one device of a 1024-wide
// layer 144 / 113.
struct PlanKey {
  int Mb, Nb, Kp, nl, lda, ldb, nz0, nz1, forced, forced_corun, flags, dev;
};
static Plan make_plan(const GemmDesc& d, bool vec_ok, bool have_ws) {
  struct Entry { PlanKey key; Plan plan; };
  constexpr unsigned kEntries = 256;
  static thread_local Entry table[kEntries] = {};   // (no product has a panel of length 0, so an empty entry matches none)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); dev = -1; }
  const int flags = (d.a_kcontig ? 1 : 0) | (d.b_kcontig ? 2 : 0) | (d.skip_upper ? 4 : 0) | (d.k_hi_diag ? 8 : 0) | (d.k_lo_diag ? 16 : 0) |
                    (d.plan_for_batch ? 32 : 0) | (vec_ok ? 64 : 0) | (have_ws ? 128 : 0) | (d.corun << 8);
  const PlanKey k = {d.Mb, d.Nb, d.Kp, d.nl, d.lda, d.ldb, d.nz0, d.nz1, g_variant.load(), d.corun > 0 ? g_corun_variant[d.corun - 1].load() : -1,
                     flags, dev};
  unsigned h = 0;
  const int* w = (const int*)&k;
  for (unsigned i = 0; i < sizeof(k) / sizeof(int); ++i) h = (h ^ (unsigned)w[i]) * 2654435761u;
  Entry& e = table[(h >> 16) % kEntries];
  if (memcmp(&e.key, &k, sizeof(k)) != 0) {
    e.plan = compute_plan(d, vec_ok, have_ws, k.forced, k.forced_corun);
    e.key = k;
  }
  return e.plan;
}

static bool epilogue_vec_ok(const GemmDesc& d) {
  return (d.ldc % 4 == 0) && (d.sC0 % 4 == 0) && (d.sC1 % 4 == 0) && aligned16(d.C) && (!d.pre_act || aligned16(d.pre_act)) &&
         (!d.gelu_grad_of || aligned16(d.gelu_grad_of)) && (!d.residual || aligned16(d.residual)) &&
         (!d.bias || (aligned16(d.bias) && d.sBias0 % 4 == 0));
}

size_t gemm_partials_bytes(const GemmDesc& d, int splits) {
  if (splits <= 1) return 0;
  return (size_t)splits * (size_t)d.nz0 * d.nz1 * (size_t)d.Mb * d.Nb * sizeof(float);
}

// Workspace the planned launch wants for its partial tiles: 0 when there is no split or when the split is emulated
// inside the workgroups anyway.
size_t gemm_plan_bytes(const GemmDesc& d) {
  if (!gemm_mfma_supported(d)) return 0;
  const Plan p = make_plan(d, epilogue_vec_ok(d), true);
  return p.seq ? 0 : gemm_partials_bytes(d, p.splits);
}

// The plan a launch of d would use (host arithmetic only; nothing is enqueued): {tile variant, panel split,
// 1 if the split is walked inside the workgroups}.  False when the matrix-core kernels do not take the product.
bool gemm_plan_of(const GemmDesc& d, bool have_ws, int out[3]) {
  if (!gemm_mfma_supported(d)) return false;
  const Plan p = make_plan(d, epilogue_vec_ok(d), have_ws);
  out[0] = p.variant; out[1] = p.splits; out[2] = p.seq;
  return true;
}

// The kernel's view of a product under a plan (not the library's hooks).
static KArgs kernel_args(const GemmDesc& d, const Plan& plan, bool vec_ok) {
  const Variant& v = kVariants[plan.variant];
  KArgs ka;
  ka.A = (const bf16_t*)d.A;
  ka.B = (const bf16_t*)d.B;
  ka.Mb = d.Mb; ka.Nb = d.Nb; ka.Kp = d.Kp; ka.nl = d.nl;
  ka.lda = d.lda; ka.ldb = d.ldb;
  ka.sAl = d.sAl; ka.sBl = d.sBl;
  ka.nz0 = d.nz0;
  ka.sA0 = d.sA0; ka.sA1 = d.sA1; ka.sB0 = d.sB0; ka.sB1 = d.sB1; ka.sC0 = d.sC0; ka.sC1 = d.sC1;
  ka.sBias0 = d.sBias0;
  ka.tiles_m = (d.Mb + v.BM - 1) / v.BM;
  ka.tiles_n = (d.Nb + v.BN - 1) / v.BN;
  // Order of a split product's workgroups by the bytes of one block's panels.  Operands outside the L2s, us, tile after tile / range after
  // range: A B [2048 x 16384 x 1024] (96 MiB) 82 / 80, A^T B [512 x 32768 x 1536] 78 / 72, [384 x 16384 x 384] (24 MiB) of A B 19.5 / 17.2,
  // of A^T B 20.0 / 18.1, [256 x 16384 x 512] 16.6 / 16.9, A B^T [320 x 12288 x 384] (16.5 MiB) 15.3 / 14.4; below, A^T B [1216 x 5632 x
  // 192] (15 MiB) 13.8 / 14.5, [512 x 8192 x 256] (12 MiB) 11.9 / 12.7, [1024 x 4096 x 256] (10 MiB) 12.3 / 13.1, A B [512 x 4096 x 512]
  // 11.8 / 12.7, [256 x 4096 x 256] 9.1 / 9.5: there an XCD's L2 (4 MiB) holds most of what its tiles need.
  ka.ranges_first = 2LL * d.nl * d.Kp * (d.Mb + d.Nb) > (16LL << 20);
  {
    const long long all = (long long)ka.tiles_m * ka.tiles_n;
    const long long mine = (all * (plan.seq || !ka.ranges_first ? 1 : plan.splits) + 7) / 8;
    const long long per_xcd = mine < all ? mine : all;
    int g = 1;
    while ((long long)(2 * g) * (2 * g) * v.BM <= per_xcd * v.BN * 2 && 2 * g <= 16) g *= 2;  // g ~ sqrt(per_xcd * BN / BM)
    ka.group = g;
  }
  ka.skip_upper = d.skip_upper; ka.k_hi_diag = d.k_hi_diag; ka.k_lo_diag = d.k_lo_diag;
  ka.splits = plan.seq ? 1 : plan.splits;
  ka.seq_splits = plan.seq ? plan.splits : 1;
  ka.partials = d.partials;
  ka.nz = (long long)d.nz0 * d.nz1;
  EpiArgs& e = ka.epi;
  e.alpha = d.alpha; e.bias = d.bias; e.C = d.C; e.pre_act = d.pre_act; e.gelu_grad_of = d.gelu_grad_of;
  e.residual = d.residual; e.ldc = d.ldc; e.act = d.act; e.out_fp32 = d.out_fp32; e.in_bf16 = 1;
  e.vec_ok = vec_ok ? 1 : 0;
  return ka;
}
static bool plain_store(const KArgs& ka) {
  const EpiArgs& e = ka.epi;
  return ka.splits == 1 && e.alpha == 1.0f && !e.bias && !e.pre_act && !e.act && !e.gelu_grad_of && !e.residual;
}
static long long workgroups(const KArgs& ka) { return (long long)ka.tiles_m * ka.tiles_n * ka.nz * ka.splits; }
static CombineJob combine_job(const GemmDesc& d, const KArgs& ka) {
  // rows of the partial tiles and of everything the epilogue touches in whole quads, counted in 32 bits
  const int vec = ka.epi.vec_ok && d.Nb % 4 == 0 && aligned16(d.partials) && ka.splits <= 8 && ka.nz * d.Mb * (d.Nb / 4) < (1LL << 31);
  return CombineJob{d.partials, ka.splits, ka.nz, d.Mb, d.Nb, d.nz0, d.sC0, d.sC1, d.sBias0, ka.epi, vec};
}

int launch_gemm_mfma(const GemmDesc& d, hipStream_t stream) {
  if (!gemm_mfma_supported(d)) return OPTIMUS_EINVAL;
  const bool vec_ok = epilogue_vec_ok(d);
  // d.partials: the workspace that the planned split asked for.  A hook that another thread has set since may ask for more: then
  // as without a workspace.
  Plan plan = make_plan(d, vec_ok, d.partials != nullptr);
  if (!plan.seq && gemm_partials_bytes(d, plan.splits) > d.partials_bytes) plan = make_plan(d, vec_ok, false);
  const int vi = plan.variant;
  if (vi == kAnyVariant) {
    g_last_plan = kAnyVariant | (1 << 8);
    return launch_gemm_generic(d, stream);
  }
  const KArgs ka = kernel_args(d, plan, vec_ok);
  if (ka.splits > 1 && gemm_partials_bytes(d, ka.splits) > d.partials_bytes) return OPTIMUS_EWORKSPACE;
  const long long nwg = workgroups(ka);
  if (nwg <= 0 || nwg > 0x7fffffffLL) return OPTIMUS_ESHAPE;
  int rc;
  // 64x64 tiles, at most two workgroups per CU, 128x64 and 128x128 tiles, one (all that the LDS of the four stages admits): twice the
  // loads in flight (figures: gemm_mfma_deep.hip).  Beside another product the wider tiles keep the ring, which can share a CU.
  const bool deep = !plan.ragged && !plan.seq && g_loop == 2 &&
                    (vi == 7 ? nwg <= 2LL * num_cus() : (vi == 6 || vi == 3) && nwg <= num_cus() && d.corun == 0);
  g_last_plan = plan.variant | (plan.splits << 8) | (plan.seq << 16) | (deep ? 1 << (vi == 7 ? 17 : 19) : 0);
  if (deep) {
    rc = launch_gemm_mfma_deep(vi, plain_store(ka), d.a_kcontig, d.b_kcontig, ka, (unsigned)nwg, stream);
  } else if (plan.ragged) rc = launch_gemm_mfma_ragged(vi, plan.ragged == 2, d.a_kcontig, d.b_kcontig, ka, (unsigned)nwg, stream);
  else switch (vi) {
    case 0: rc = launch_layout<256, 256, 2, 4>(d, ka, nwg, stream); break;
    case 1: rc = launch_layout<256, 128, 4, 2>(d, ka, nwg, stream); break;
    case 2: rc = launch_layout<128, 256, 2, 4>(d, ka, nwg, stream); break;
    case 3: rc = launch_layout<128, 128, 2, 2>(d, ka, nwg, stream); break;
    case 4: rc = launch_layout<256, 256, 2, 4>(d, ka, nwg, stream); break;
    case 6: rc = launch_layout<128, 64, 2, 2>(d, ka, nwg, stream); break;
    case 7: rc = launch_layout<64, 64, 2, 2>(d, ka, nwg, stream); break;
    case 8: rc = launch_layout<256, 128, 2, 2>(d, ka, nwg, stream); break;
    case 9: rc = launch_layout<128, 256, 2, 2>(d, ka, nwg, stream); break;
    default: rc = OPTIMUS_EINVAL; break;
  }
  if (rc != OPTIMUS_OK || ka.splits == 1) return rc;
  CombineJobs jobs = {};
  jobs.n = 1;
  jobs.j[0] = combine_job(d, ka);
  return launch_gemm_combines(jobs, stream);
}

// ---- two products in one launch (gemm_mfma_pair.hpp) ----
// Not for a split that is walked inside the workgroups (whole grids, callers without workspace), panels beyond a buffer resource and
// what the any-shape kernel takes, nor while a hook forces tile or loop, nor where the two single launches are the faster ones.  The splits
// are those of the single launches: same bits.
struct PairPlan {
  Plan x, y;
  long long sx, sy;   // slabs that a workgroup walks
};
static bool plan_pair(const GemmDesc& x, const GemmDesc& y, bool vec_x, bool vec_y, PairPlan* out) {
  if (!gemm_mfma_supported(x) || !gemm_mfma_supported(y) || g_loop != 2 || g_variant >= 0) return false;
  if (!x.a_kcontig || !x.b_kcontig || y.a_kcontig || y.b_kcontig) return false;
  Plan px = make_plan(x, vec_x, x.partials != nullptr), py = make_plan(y, vec_y, y.partials != nullptr);
  if (px.variant == kAnyVariant || py.variant == kAnyVariant || px.seq || py.seq || px.ragged == 2 || py.ragged == 2) return false;
  if (gemm_partials_bytes(x, px.splits) > x.partials_bytes || gemm_partials_bytes(y, py.splits) > y.partials_bytes) return false;
  const bool ragged = px.ragged || py.ragged;
  const long long ncu = num_cus();
  const auto slabs_of = [](const GemmDesc& d, int sp) {
    const long long slabs = (long long)d.nl * ((d.Kp + 2 * BK - 1) / (2 * BK)) * 2;
    return (((slabs + sp - 1) / sp) + 1) & ~1LL;
  };
  const long long sx = slabs_of(x, px.splits), sy = slabs_of(y, py.splits);
  const auto wgs_of = [](const GemmDesc& d, int v, int sp) {
    return (long long)((d.Mb + kVariants[v].BM - 1) / kVariants[v].BM) * ((d.Nb + kVariants[v].BN - 1) / kVariants[v].BN) *
           (d.nz0 * (long long)d.nz1) * sp;
  };
  // One tile for both, by the time of the longest workgroup on a CU of its own or of all of them over the CUs, whichever is more; time
  // per slab of one workgroup by how many share its CU as make_plan has it, with the factors of the two forms.
  const auto slab_us = [&](int v, long long res, bool is_y) {
    if (v == 3) return (0.25f + 0.21f * (float)(res - 1)) * (is_y ? 1.04f : 1.14f);
    const float t = ragged || res > 2 ? 0.155f + 0.045f * (float)(res - 1) : res == 1 ? 0.11f : 0.18f;
    return is_y ? 1.25f * t : t;
  };
  int best = -1;
  float best_cost = 0.f;
  for (const int v : {7, 3}) {
    if (!ragged && !(variant_fits(kVariants[v], x) && variant_fits(kVariants[v], y))) continue;
    const long long wx = wgs_of(x, v, px.splits), wy = wgs_of(y, v, py.splits), per_cu = v == 3 ? 2 : 5;
    const long long each = (wx + wy + ncu - 1) / ncu, res = each < per_cu ? each : per_cu;
    const float ux = (float)sx * slab_us(v, res, false), uy = (float)sy * slab_us(v, res, true);
    const float all = ((float)wx * ux + (float)wy * uy) / (float)(ncu * res);
    const float lx = (float)sx * slab_us(v, 1, false), ly = (float)sy * slab_us(v, 1, true), one = lx > ly ? lx : ly;
    const float cost = (v == 3 ? 5.5f : 4.0f) + (all > one ? all : one);
    if (best < 0 || cost < best_cost) { best = v; best_cost = cost; }
  }
  if (best < 0) return false;
  // The single launches, tiles of their own choice, where their estimates are less in sum.  A pair of 64x64 tiles, many to a CU, takes up to
  // 1.6 times its estimate, both products' panels being in the L2s at once: in large blocks that 128 does not divide.  Measured, us, pair / single
  // launches, rows x contraction x columns of the input's gradient, 64x64 tiles: [2048 x 3840 x 3840] 218 / 132, [4096 x 2688 x 5376] 383 / 271,
  // [8000 x 2048 x 2048] 233 / 165, but [8192 x 6912 x 576] 230 / 263; 128x128 tiles: [4096 x 2048 x 8192] 251 / 218, [4096 x 8192 x 2048] 240 /
  // 221, [4096 x 2048 x 2048] 65 / 70; cut: [2000 x 5120 x 5120] 225 / 272, [8008 x 8192 x 2048] 517 / 505.
  // And where the input's gradient is one long workgroup per CU at most, with four stages by itself and a slot of the ring among y's many short
  // ones: [2048 x 6144 x 384] 72 / 56, [2048 x 6144 x 512] 77 / 59, [1024 x 6144 x 1024] 66 / 50, but [2048 x 3072 x 384] 29 / 37.
  if (px.variant == 7 && px.splits == 1 && !px.ragged && wgs_of(x, 7, 1) <= ncu && sx >= 144 && sx >= 3 * sy) return false;
  if (best_cost * (best == 7 && !ragged && wgs_of(x, 7, px.splits) + wgs_of(y, 7, py.splits) >= 5 * ncu ? 1.25f : 1.0f) > px.us + py.us) return false;
  px.variant = py.variant = best;
  px.ragged = py.ragged = ragged ? 1 : 0;
  *out = {px, py, sx, sy};
  return true;
}

bool gemm_pair_planned(const GemmDesc& x, const GemmDesc& y) {
  PairPlan p;
  return plan_pair(x, y, epilogue_vec_ok(x), epilogue_vec_ok(y), &p);
}

bool launch_gemm_pair(const GemmDesc& x, const GemmDesc& y, CombineJobs* combines, hipStream_t stream, int* rc) {
  const bool vec_x = epilogue_vec_ok(x), vec_y = epilogue_vec_ok(y);
  PairPlan plan;
  if (!plan_pair(x, y, vec_x, vec_y, &plan)) return false;
  const Plan &px = plan.x, &py = plan.y;
  const int best = px.variant;
  const bool ragged = px.ragged != 0;
  const KArgs kx = kernel_args(x, px, vec_x), ky = kernel_args(y, py, vec_y);
  const long long nx = workgroups(kx), ny = workgroups(ky);
  if (nx <= 0 || ny <= 0 || nx + ny > 0x7fffffffLL) return false;
  PairLaunch p = {&kx, &ky, (unsigned)nx, (unsigned)ny, plan.sy > plan.sx ? 1 : 0, plain_store(kx), plain_store(ky), stream};
  const bool deep = best == 7 && !ragged && nx + ny <= 2LL * num_cus();
  g_last_plan = best | (py.splits << 8) | (deep ? 1 << 17 : 0) | (1 << 18);
  *rc = best == 7 ? launch_gemm_pair_64(deep, ragged, p) : launch_gemm_pair_128(ragged, p);
  if (*rc == OPTIMUS_OK && kx.splits > 1) combines->j[combines->n++] = combine_job(x, kx);
  if (*rc == OPTIMUS_OK && ky.splits > 1) combines->j[combines->n++] = combine_job(y, ky);
  return true;
}

}  // namespace optimus
