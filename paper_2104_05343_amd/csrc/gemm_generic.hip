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
// Both tiles keep the sums of the eight parts of the slabs apart and add them in the same order at the end, so the tile
// choice, and with it whole-grid against one-device launches, changes no bit.
//
// Measured (fp32, 1024-wide layer on a 4 x 4 grid, one device): [1024 x 1024 x 1024] blocks 29 us (64x64 tiles, 74 TFLOP/s),
// [1024 x 4096 x 256] blocks 32 us (32x32 tiles, 67 TFLOP/s); scalar fused multiply-adds on 64x64 tiles took 180 and 733 us.
// With one wavefront per SIMD and slabs of 128 bytes 39 and 57 us; with bounds arithmetic in every slab 36 and 45 us.
#include <type_traits>

#include "common.hpp"
#include "epilogue.hpp"

namespace optimus {

typedef __attribute__((ext_vector_type(8))) __bf16 gbf16x8;
typedef __attribute__((ext_vector_type(16))) float gf32x16;
typedef __attribute__((ext_vector_type(4))) short gs16x4;
typedef __attribute__((ext_vector_type(8))) short gs16x8;

struct GArgs {
  const void* A;
  const void* B;
  int Mb, Nb, Kp, nl;
  int lda, ldb;
  long long sAl, sBl;
  int nz0;
  long long sA0, sA1, sB0, sB1, sC0, sC1, sBias0;
  int tiles_m, tiles_n;
  int skip_upper, k_hi_diag, k_lo_diag;
  EpiArgs epi;
};

__device__ const uint4 g_zero_chunk[1] = {};
typedef unsigned gu32x4 __attribute__((ext_vector_type(4), aligned(2)));        // a chunk at any alignment of the element type
typedef __attribute__((address_space(1))) gu32x4 gchunk;

constexpr int GT_THREADS = 512;

// One operand's slab of ROWS rows (or columns) by 256 bytes of k, in LDS:
//   KC (k contiguous in memory): [ROWS][256 bytes + 16]; a fragment read is 16 bytes of one row, and 16 rows at a pitch of
//     68 banks cover the 64 banks once.
//   !KC, fp32: [64 k][ROWS + 8 floats]; a fragment read is one float per lane, the two half-waves four k-rows apart.
//   !KC, bf16: [128 k][ROWS], 16-column granules XOR 2 * (k & 3), read with the transposing ds_read_b64_tr_b16.
template <typename T, int ROWS, bool KC, bool TINY>
struct Slab {
  static constexpr int E = 16 / (int)sizeof(T);       // elements per 16-byte chunk
  static constexpr int KS = 256 / (int)sizeof(T);     // k per slab
  static constexpr int CHUNKS = ROWS * 16 / GT_THREADS;  // chunks per thread
  static constexpr int BYTES = KC ? ROWS * 272 : (sizeof(T) == 4 ? KS * (ROWS + 8) * 4 : KS * ROWS * 2);

  // element offset of the chunk from the slab's origin, and its place in the tile
  static __device__ __forceinline__ void place(int tid, int it, int& row, int& k) {
    const int c = tid + it * GT_THREADS;
    if (KC) { row = c >> 4; k = (c & 15) * E; }
    else { k = c / (ROWS / E); row = (c % (ROWS / E)) * E; }
  }
  static __device__ __forceinline__ int lds_off(int row, int k) {   // bytes
    if (KC) return row * 272 + k * (int)sizeof(T);
    if (sizeof(T) == 4) return (k * (ROWS + 8) + row) * 4;
    return (k * ROWS + ((((row >> 4) ^ (((k & 3) << 1) & (ROWS / 16 - 1)))) << 4) + (row & 15)) * 2;
  }
  static_assert(CHUNKS * GT_THREADS * E == ROWS * KS && KS * (int)sizeof(T) == 256, "the threads' chunks cover the slab once");

  // The chunks of a slab that exists in full: one per-lane offset (bytes) per chunk, computed once, behind a uniform base.
  static __device__ __forceinline__ void offsets(unsigned (&off)[CHUNKS], int ld, int tid) {
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
      int row, k;
      place(tid, it, row, k);
      off[it] = (unsigned)((KC ? row * ld + k : k * ld + row) * (int)sizeof(T));
    }
  }
  static __device__ __forceinline__ void load_full(uint4 (&r)[CHUNKS], const T* origin, const unsigned (&off)[CHUNKS]) {
    const __attribute__((address_space(1))) char* base = (const __attribute__((address_space(1))) char*)origin;
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
      const gu32x4 v = *(const gchunk*)(base + off[it]);
      r[it] = make_uint4(v[0], v[1], v[2], v[3]);
    }
  }
  static __device__ __forceinline__ void store_full(const uint4 (&r)[CHUNKS], char* lds, int tid) {
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
      int row, k;
      place(tid, it, row, k);
      *(uint4*)(lds + lds_off(row, k)) = r[it];
    }
  }
  // Requests the chunks of a slab of which rows_left rows and k_left k exist.  Every lane issues every load, so that the
  // compiler can count the loads in flight: chunks that do not exist come from a block of zeros, and a chunk that the end
  // of a row cuts is fetched so that it ends there (store() shifts it into place).  Where a row may be shorter than a chunk
  // (TINY) cut chunks are left to store() altogether.
  static __device__ __forceinline__ void load(uint4 (&r)[CHUNKS], const T* origin, int ld, int rows_left, int k_left, int tid) {
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
      int row, k;
      place(tid, it, row, k);
      const int run = KC ? k_left - k : rows_left - row;             // elements that exist along the chunk
      const bool across = KC ? row < rows_left : k < k_left;
      const int back = run < E ? E - run : 0;
      const T* p = origin + (KC ? (long long)row * ld + k : (long long)k * ld + row) - back;
      const bool there = across && run > 0 && !(TINY && back);
      const gchunk* src = there ? (const gchunk*)p : (const gchunk*)g_zero_chunk;
      const gu32x4 v = *src;
      r[it] = make_uint4(v[0], v[1], v[2], v[3]);
    }
  }
  static __device__ __forceinline__ void store(uint4 (&r)[CHUNKS], char* lds, const T* origin, int ld, int rows_left, int k_left, int tid) {
    const int len = KC ? k_left : rows_left;                         // uniform: does the end of the rows cut a chunk here?
    const bool cut = len < (KC ? KS : ROWS) && len % E != 0;
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
      int row, k;
      place(tid, it, row, k);
      if (cut) {
        const int run = KC ? k_left - k : rows_left - row;
        const bool across = KC ? row < rows_left : k < k_left;
        if (across && run > 0 && run < E) {
          if constexpr (TINY) {
            const T* p = origin + (KC ? (long long)row * ld + k : (long long)k * ld + row);
            T e[E];
#pragma unroll
            for (int c = 0; c < E; ++c) e[c] = c < run ? p[c] : (T)0;
            __builtin_memcpy(&r[it], e, 16);
          } else {
            const int bits = (E - run) * (int)sizeof(T) * 8;         // 16 .. 112
            const unsigned long long lo = r[it].x | ((unsigned long long)r[it].y << 32), hi = r[it].z | ((unsigned long long)r[it].w << 32);
            const unsigned long long nlo = bits >= 64 ? hi >> (bits - 64) : (lo >> bits) | (hi << (64 - bits)), nhi = bits >= 64 ? 0ull : hi >> bits;
            r[it] = make_uint4((unsigned)nlo, (unsigned)(nlo >> 32), (unsigned)nhi, (unsigned)(nhi >> 32));
          }
        }
      }
      *(uint4*)(lds + lds_off(row, k)) = r[it];
    }
  }
  // this lane's share of part s (0 .. 7) of the slab for the 32 rows from r0: eight k of an fp32 operand (lanes 0-31 take the
  // first four of them, lanes 32-63 the last four), or sixteen k of a bf16 operand (eight each)
  static __device__ __forceinline__ void frag(float (&f)[4], const char* lds, int r0, int s, int lane) {
    if (KC) {
      const float4 v = *(const float4*)(lds + lds_off(r0 + (lane & 31), s * 8 + (lane >> 5) * 4));
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) f[t] = *(const float*)(lds + lds_off(r0 + (lane & 31), s * 8 + (lane >> 5) * 4 + t));
    }
  }
  static __device__ __forceinline__ void frag(gbf16x8& f, const char* lds, int r0, int s, int lane) {
    if (KC) {
      f = *(const gbf16x8*)(lds + lds_off(r0 + (lane & 31), s * 16 + (lane >> 5) * 8));
    } else {
#if defined(__HIP_DEVICE_COMPILE__)
      const int lg = lane & 15;
      const char* p0 = lds + lds_off(r0 + (((lane >> 4) & 1) << 4) + ((lg & 3) << 2), s * 16 + ((lane >> 5) << 3) + (lg >> 2));
      const char* p1 = p0 + 4 * ROWS * 2;   // four k further: same swizzle term
      gs16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) gs16x4*)p0);
      gs16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) gs16x4*)p1);
      f = __builtin_bit_cast(gbf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#endif
    }
  }
};

// one eighth of a slab for a 32x32 output: operands swapped, so that a lane ends up with four consecutive columns of one row
template <typename SA, typename SB>
__device__ __forceinline__ void eighth(gf32x16& acc, const char* la, const char* lb, int rm, int rn, int s, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (SA::E == 4) {
    float fa[4], fb[4];
    SA::frag(fa, la, rm, s, lane);
    SB::frag(fb, lb, rn, s, lane);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[t], fa[t], acc, 0, 0, 0);
  } else {
    gbf16x8 fa, fb;
    SA::frag(fa, la, rm, s, lane);
    SB::frag(fb, lb, rn, s, lane);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa, acc, 0, 0, 0);
  }
#endif
}

// LDS traffic of this wavefront done, then the barrier: unlike __syncthreads() it leaves the slab loads in flight
#define OPTIMUS_LDS_BARRIER()                                        \
  do {                                                               \
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  \
  } while (0)

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
  const int bt = wide ? 64 : 32;
  a.tiles_m = (d.Mb + bt - 1) / bt;
  a.tiles_n = (d.Nb + bt - 1) / bt;
  const long long nwg = (long long)a.tiles_m * a.tiles_n * nz;
  if (nwg <= 0 || nwg > 0x7fffffffLL) return OPTIMUS_ESHAPE;
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
