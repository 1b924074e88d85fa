// bf16 matrix-core product kernels for gfx950 (CDNA4).
//
// Computes, per batch entry, C = alpha * sum_{l<nl} op(A_l) * op(B_l) with fp32 accumulation in
// v_mfma_f32_32x32x16_bf16 and applies the epilogue once.  The nl panels of a SUMMA product
// (Algorithms 1-3 of the paper: one panel per step l) are consumed by ONE k-loop that re-bases
// the operand pointers at panel boundaries, so the q steps cost nothing beyond pointer
// arithmetic and no partial C ever goes to HBM (unless the caller asked for a panel split).
//
// Tiling: a workgroup of WM*WN wavefronts owns a BM x BN output tile; k advances in slabs of
// BK = 32 through a ring of FOUR slabs per operand in LDS.
//   * Every wavefront issues buffer_load_dwordx4 ... lds, which moves 64 x 16
//     bytes from per-lane offsets straight into one contiguous KiB of LDS without passing
//     through registers.  The LDS swizzles below are therefore applied on the GLOBAL side:
//     lane p of a KiB fetches the 16 bytes that belong at LDS position p.  Buffer addressing
//     (SGPR resource + one 32-bit VGPR offset) is used because 64-bit per-lane addresses were
//     measured to stall the MFMA pipe twice as much.  Slab hand-over uses s_waitcnt vmcnt(N) and
//     a bare s_barrier: a fenced barrier would drain the loads in flight.
//     A k-strided operand moves one slab per step; a k-contiguous operand moves a PAIR of slabs
//     (64 k = one whole 128-byte line per row) every second step.  The pipeline runs over 16-wide
//     sub-steps with the fragments of the next sub-step requested between the MFMAs of the
//     current one, also across slab boundaries; the loads that refill a freed slab are spread one
//     by one between the MFMAs as well (see the comments at the loop).
//   * Ragged blocks (RAG): the same pipeline; what lies outside the operand (rows or columns past the block, k past the
//     end of a panel) gets a lane offset outside the buffer resource's range, which the hardware's range check turns
//     into zeros in LDS.  That costs a compare and a select per load where a second code path cost the pipeline: the
//     bounds-checked staging through registers that these blocks took before had one slab in flight and 128x128 tiles
//     only (one device of a 1280-wide layer on a 4 x 4 grid, [2000 x 1280 x 320] blocks: 97 to 215 us per product, now 14 to 26).
// LDS layouts (conflict free for their readers on the 64-bank, 256 B/clk LDS of this part):
//   * k-contiguous operand ([rows][k] in memory): pairs of slabs as rows of 8 sixteen-byte chunks, chunk index XOR
//     ((row >> 1) & 7); fragments are read with ds_read_b128.
//   * k-strided operand ([k][cols] in memory: B of A*B, both operands of A^T*B): kept as it is,
//     32-byte column granules XOR 2*(k & 3); fragments are fetched with the transposing read
//     ds_read_b64_tr_b16, which hands each lane four consecutive k of one column.
// The two MFMA operands are swapped (D^T = B^T A^T) so that every lane ends up with four
// consecutive columns of one output row; results leave through wavefront-private LDS chunks as
// whole rows of the tile (see ChunkBf16).
#pragma once
#include <type_traits>

#include "common.hpp"
#include "epilogue.hpp"

namespace optimus {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int BK = 32;
constexpr int NSTAGE = 4;
#ifndef OPTIMUS_LAB_DBG
#define OPTIMUS_LAB_DBG 0
#endif
// bit 32 (timing studies only): thread 0 of every workgroup stores the 100 MHz wall clock at four points of the kernel
// (entry, first matrix instruction, end of the k-loop, last store retired)
#if OPTIMUS_LAB_DBG & 32
__device__ unsigned long long g_lab_stamps[4 * 4096];
extern "C" int optimus_lab_read_stamps(unsigned long long* host) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(g_lab_stamps), sizeof(g_lab_stamps));
}
__device__ unsigned long long g_lab_stall[8 * 2048];
extern "C" int optimus_lab_read_stall(unsigned long long* host) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(g_lab_stall), sizeof(g_lab_stall));
}
#define OPTIMUS_LAB_STAMP(n)                                                                         \
  do {                                                                                               \
    if ((n) == 3) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                                   \
    if (threadIdx.x == 0 && blockIdx.x < 2048) {                                                      \
      g_lab_stamps[blockIdx.x * 8 + (n)] = wall_clock64();                                           \
      g_lab_stamps[blockIdx.x * 8 + 4 + (n)] = clock64();                                            \
    }                                                                                                \
  } while (0)
#else
#define OPTIMUS_LAB_STAMP(n) do {} while (0)
#endif

struct KArgs {
  const bf16_t* A;
  const bf16_t* B;
  int Mb, Nb, Kp, nl;
  int lda, ldb;
  long long sAl, sBl;
  int nz0;
  long long sA0, sA1, sB0, sB1, sC0, sC1;
  long long sBias0;
  int tiles_m, tiles_n;
  int group;  // tile rows walked together (see the tile walk in the kernel)
  int skip_upper, k_hi_diag, k_lo_diag;
  int splits;
  int ranges_first;  // order of a split product's workgroups: range after range, or tile after tile
  float* partials;
  // > 1 (with splits == 1): one workgroup walks all slabs but adds them up as `seq_splits` panel-split workgroups and
  // their fixed-order combine would -- a fresh accumulator per range, the ranges' sums added in range order
  int seq_splits;
  long long nz;  // total batch count
  EpiArgs epi;
};

// tile variants 3, 6, 7 with four stages of 64 k in LDS (gemm_mfma_deep.hip)
int launch_gemm_mfma_deep(int variant, bool plain, int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream);
// tile variants 3, 6, 7 in their ragged form, 3 also for long panels (gemm_mfma_ragged.hip)
int launch_gemm_mfma_ragged(int variant, bool long_panels, int a_kcontig, int b_kcontig, const KArgs& ka, unsigned nwg, hipStream_t stream);

// element offset inside an LDS tile
// The LDS of this part serves 256 bytes per clock (64 four-byte banks).  A ds_read_b128 is served 16 lanes at a
// time (16 consecutive rows, one chunk each): four 64-byte rows span the 64 banks, so the XOR term must take 4
// distinct values over the 4 rows of equal (row & 3) -> (row >> 2) & 3.  A ds_read_b64_tr_b16 is served 32 lanes at
// a time (4 k-rows x two adjacent 32-byte granules): rows start at bank 0, so the 8 (k, granule) pairs must fall in
// 8 distinct granule slots -> XOR with 2 * (k & 3) (masked to the row's granule count for 64-wide tiles).  Measured with a read-only microbenchmark: > 200 B/clk for
// these patterns against 128 B/clk for swizzles designed for 32 banks.
// k-contiguous operand: two slabs side by side, [row][64 k] = 128 bytes per row, so that one row
// of a load is a whole 128-byte cache line.  Two rows span the 64 banks: the XOR term takes 8 values over the 8 row
// pairs of a 16-lane group.
__device__ __forceinline__ int lds_off_kc2(int row, int chunk) { return row * (2 * BK) + ((chunk ^ ((row >> 1) & 7)) << 3); }
template <int ROWS>
__device__ __forceinline__ int lds_off_ks(int krow, int col) {
  return krow * ROWS + ((((col >> 4) ^ (((krow & 3) << 1) & (ROWS / 16 - 1)))) << 4) + (col & 15);
}

// ---- direct global -> LDS, one KiB per wavefront instruction ----
template <int ROWS, int NW>
struct DirectPlan {
  static constexpr int CHUNKS = ROWS * BK * 2 / 1024;  // KiB chunks in a [ROWS x BK] bf16 slab
  static constexpr int PER = CHUNKS / NW;
  static_assert(CHUNKS % NW == 0 && PER >= 1, "slab must divide over the wavefronts");
};

// Per-lane source offsets (BYTES, relative to the slab origin) of the KiB chunks this wavefront moves.
// k-contiguous operand: the unit is a PAIR of slabs (64 k): 8 rows of 128 bytes per instruction.
// k-strided operand: the unit is one slab of 32 k-rows.
template <int ROWS, bool KC, int NW, int PER>
__device__ __forceinline__ void direct_offsets(unsigned (&off)[PER], int ld, int wave, int lane) {
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int q = wave * PER + it;
    if (KC) {
      const int row = q * 8 + (lane >> 3);
      const int kc = (lane & 7) ^ ((row >> 1) & 7);  // inverse of lds_off_kc2 for LDS position (row, lane & 7)
      off[it] = (unsigned)(row * ld + kc * 8) * 2u;
    } else {
      constexpr int PPR = ROWS / 8;  // 16-byte pieces per k-row
      const int idx = q * 64 + lane;
      const int krow = idx / PPR, pp = idx % PPR;
      const int col = ((((pp >> 1) ^ (((krow & 3) << 1) & (ROWS / 16 - 1)))) << 4) + ((pp & 1) << 3);  // inverse of lds_off_ks
      off[it] = (unsigned)(krow * ld + col) * 2u;
    }
  }
}

typedef __attribute__((ext_vector_type(4))) int i32x4;

// Buffer resource (raw, stride 0) whose base is the current panel's tile origin, with a 2 GiB window: every offset
// used is below it (checked on the host).  Built by hand as four SGPR words.
__device__ __forceinline__ i32x4 make_rsrc(const bf16_t* base) {
  const unsigned long long p = (unsigned long long)base;
  return i32x4{(int)(unsigned)p, (int)(unsigned)((p >> 32) & 0xffffu), (int)0x80000000u, 0x00020000};
}

// The most k rows of a k-strided operand, in whole slabs, that one resource reaches: (rows - 1) * ld + 128 columns of a tile.
__device__ __forceinline__ int segment_rows(int ld) { return (int)(((1u << 30) - 128u) / (unsigned)ld + 1u) / BK * BK; }

// Ragged blocks.  A lane offset of 2 GiB fails the range check of the resource whatever the slab offset: the load writes
// zeros to LDS.  direct_cut gives it to the chunks of rows (columns) that do not exist, `left` of which do, and notes every
// chunk's k inside its unit; cut_off gives it to the chunks past the panel's end, k_left of which exist in this unit.
// Chunks are whole on both sides of a cut: panels and k-strided rows are multiples of 8 elements (checked on the host).
constexpr unsigned kOutside = 0x80000000u;
template <int ROWS, bool KC, int NW, int PER>
__device__ __forceinline__ void direct_cut(unsigned (&off)[PER], int (&kin)[PER], int left, int wave, int lane) {
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int q = wave * PER + it;
    int row;
    if (KC) {
      row = q * 8 + (lane >> 3);
      kin[it] = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
    } else {
      constexpr int PPR = ROWS / 8;
      const int idx = q * 64 + lane, pp = idx % PPR;
      kin[it] = idx / PPR;
      row = ((((pp >> 1) ^ (((kin[it] & 3) << 1) & (ROWS / 16 - 1)))) << 4) + ((pp & 1) << 3);
    }
    if (row >= left) off[it] = kOutside;
  }
}
template <bool RAG>
__device__ __forceinline__ unsigned cut_off(unsigned off, int kin, int k_left) {
  return !RAG || kin < k_left ? off : kOutside;
}

// rsrc: see make_rsrc; soff: byte offset of the slab inside the panel; off: per-lane byte offsets.
// The LDS load is written in assembly on purpose: issued through the compiler's builtin, every later LDS read is
// preceded by a compiler-inserted wait for ALL loads in flight (it cannot tell the stages apart), which collapses
// the four-stage pipeline to one slab.  Here the hand-over is explicit instead: s_waitcnt vmcnt(N) + barrier.
template <bool RAG, int PER, int KPER>
__device__ __forceinline__ void direct_issue(i32x4 rsrc, unsigned soff, const unsigned (&off)[PER], const int (&kin)[KPER], int k_left,
                                             bf16_t* lds_tile, int wave) {
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) bf16_t*)lds_tile;
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base + (unsigned)(wave * PER + it) * 1024u);
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(cut_off<RAG>(off[it], kin[RAG ? it : 0], k_left)),
                 "s"(rsrc), "s"(soff), "s"(m0v)
                 : "memory", "m0");
  }
}

// one KiB chunk (number c of the operand's issue unit) with this lane's offset
__device__ __forceinline__ void direct_issue_one(i32x4 rsrc, unsigned soff, unsigned off, bf16_t* lds_unit, int c) {
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) bf16_t*)lds_unit;
  const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base + (unsigned)c * 1024u);
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(off), "s"(rsrc), "s"(soff), "s"(m0v)
               : "memory", "m0");
}

// s_waitcnt vmcnt(n) only (expcnt / lgkmcnt left at their maxima), gfx9 encoding.  The builtin rather than inline
// assembly: the compiler's own wait-count pass then knows which LDS loads have landed and adds no full drain.
constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }  // + lgkmcnt(0)
#define OPTIMUS_WAIT_VMCNT_LGKM0(n)                      \
  do {                                                   \
    asm volatile("" ::: "memory");                       \
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(n));     \
    asm volatile("" ::: "memory");                       \
  } while (0)
#define OPTIMUS_WAIT_VMCNT(n)                      \
  do {                                             \
    asm volatile("" ::: "memory");                 \
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(n));     \
    asm volatile("" ::: "memory");                 \
  } while (0)
// barrier without the memory fence of __syncthreads(): loads of later slabs stay in flight across it
#define OPTIMUS_BARRIER()                  \
  do {                                     \
    asm volatile("" ::: "memory");         \
    __builtin_amdgcn_s_barrier();          \
    asm volatile("" ::: "memory");         \
  } while (0)

// fragment of 8 consecutive k of a k-strided slab for column rc0 + lane%32, k-group lane/32, sub-step ks
template <int ROWS>
__device__ __forceinline__ bf16x8 read_frag_ks(const bf16_t* lds, int rc0, int ks, int lane) {
  const int lg = lane & 15;
  const int col = rc0 + (((lane >> 4) & 1) << 4) + ((lg & 3) << 2);
  const int krow = ks * 16 + ((lane >> 5) << 3) + (lg >> 2);
  const bf16_t* p0 = lds + lds_off_ks<ROWS>(krow, col);
  const bf16_t* p1 = p0 + 4 * ROWS;  // krow + 4: same (k & 3), same swizzle term
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p0);
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p1);
  s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

template <int BM, int BN, int WM, int WN>
struct Tile {
  static constexpr int NW = WM * WN, THREADS = NW * 64;
  static constexpr int TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32;
  static constexpr int A_ELEMS = BM * BK, B_ELEMS = BN * BK;
};

// The operand's LDS ring holds four slabs.  A k-strided operand keeps four [32][ROWS] stages;
// a k-contiguous one keeps two [ROWS][64] pairs, slab s4 being half (s4 & 1) of pair (s4 >> 1).
template <int ROWS, bool KC>
__device__ __forceinline__ bf16x8 read_frag_ring(const bf16_t* ring, int s4, int rc0, int ks, int lane) {
  if (KC) {
    const bf16_t* pair = ring + (s4 >> 1) * (2 * ROWS * BK);
    return *(const bf16x8*)(pair + lds_off_kc2(rc0 + (lane & 31), (s4 & 1) * 4 + ks * 2 + (lane >> 5)));
  } else {
    return read_frag_ks<ROWS>(ring + s4 * (ROWS * BK), rc0, ks, lane);
  }
}
// Fragment set of one 16-wide sub-step (MI A-fragments, NI B-fragments) and the MFMAs that consume it.
template <int BM, int BN, int WM, int WN, bool AKC, bool BKC>
__device__ __forceinline__ void load_frags(bf16x8 (&fa)[BM / WM / 32], bf16x8 (&fb)[BN / WN / 32], const bf16_t* ringA,
                                           const bf16_t* ringB, int s4, int ks, int wm, int wn, int lane) {
  using T = Tile<BM, BN, WM, WN>;
#pragma unroll
  for (int mi = 0; mi < T::MI; ++mi) fa[mi] = read_frag_ring<BM, AKC>(ringA, s4, wm * T::TM + mi * 32, ks, lane);
#pragma unroll
  for (int ni = 0; ni < T::NI; ++ni) fb[ni] = read_frag_ring<BN, BKC>(ringB, s4, wn * T::TN + ni * 32, ks, lane);
}
// fragment R of a sub-step: R < MI -> A fragment R, else B fragment R - MI; nothing beyond MI + NI
template <int R, int BM, int BN, int WM, int WN, bool AKC, bool BKC>
__device__ __forceinline__ void load_frag_r(bf16x8 (&fa)[BM / WM / 32], bf16x8 (&fb)[BN / WN / 32], const bf16_t* ringA,
                                            const bf16_t* ringB, int s4, int ks, int wm, int wn, int lane) {
  using T = Tile<BM, BN, WM, WN>;
  if constexpr (R < T::MI) fa[R] = read_frag_ring<BM, AKC>(ringA, s4, wm * T::TM + R * 32, ks, lane);
  else if constexpr (R < T::MI + T::NI) fb[R - T::MI] = read_frag_ring<BN, BKC>(ringB, s4, wn * T::TN + (R - T::MI) * 32, ks, lane);
}
// MFMA number M of a sub-step (row-major over the MI x NI accumulators)
template <int M, int MI, int NI>
__device__ __forceinline__ void mfma_m(f32x16 (&acc)[MI][NI], const bf16x8 (&fa)[MI], const bf16x8 (&fb)[NI]) {
  constexpr int mi = M / NI, ni = M % NI;
  acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ni], fa[mi], acc[mi][ni], 0, 0, 0);
}
// slot (0 .. MF-1) in front of whose MFMA load G of GN is issued: spread evenly over the sub-step
constexpr int dma_slot(int g, int gn, int mf) { return ((2 * g + 1) * mf) / (2 * gn); }

// ---- coalesced tile stores ----
// The MFMA accumulator layout gives a lane 4 consecutive columns of one row: stored directly, a wavefront
// instruction writes 32 rows x 16 bytes, and every 128-byte line of C is completed by eight separate partial
// writes (measured: 8.5 us to store a 16 MiB block, 1.9 TB/s).  Instead a 32-row chunk of the wavefront's tile goes
// through a wavefront-private piece of LDS (free after the k-loop) and comes back as 16 bytes per lane with the
// lanes of a row side by side: whole rows of the tile (128 bytes for 64 bf16 columns) per store.
// LDS operations of one wavefront execute in order, so no barrier separates the write from the read-back.
template <int TN>
struct ChunkBf16 {
  static constexpr int PITCH = TN * 2 + 8;      // bytes per row: 34 (TN = 64) banks, conflict-free 8-byte writes
  static constexpr int BYTES = 32 * PITCH;
  static constexpr int LPR = TN / 8;            // lanes per row on the way out (16 bytes each)
  static constexpr int RPI = 64 / LPR;          // rows per store instruction
  static constexpr int NIT = 32 / RPI;
};
// write: v[g] = columns ni*32 + g*8 + 4*(lane/32) .. +3 of row (lane % 32) of the chunk, packed as 4 bf16
template <int TN>
__device__ __forceinline__ void chunk_write_bf16(char* lds_wave, int ni, const uint2 (&v)[4], int lane) {
  char* wr = lds_wave + (lane & 31) * ChunkBf16<TN>::PITCH + ((lane >> 5) << 3) + ni * 64;
#pragma unroll
  for (int g = 0; g < 4; ++g) *(uint2*)(wr + g * 16) = v[g];
}
// read back and store the whole 32 x TN chunk
template <int TN>
__device__ __forceinline__ void chunk_flush_bf16(const char* lds_wave, bf16_t* c_chunk, long long ldc, int lane) {
  using L = ChunkBf16<TN>;
  const int r0 = lane / L::LPR, c = lane % L::LPR;
#pragma unroll
  for (int it = 0; it < L::NIT; ++it) {
    const int row = it * L::RPI + r0;
    const char* rd = lds_wave + row * L::PITCH + c * 16;
    const uint2 lo = *(const uint2*)rd, hi = *(const uint2*)(rd + 8);
    *(uint4*)(c_chunk + (long long)row * ldc + c * 8) = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
}
template <int TN>
__device__ __forceinline__ void store_chunk_bf16(char* lds_wave, bf16_t* c_chunk, long long ldc, const uint2 (&v)[TN / 32][4],
                                                 int lane) {
#pragma unroll
  for (int ni = 0; ni < TN / 32; ++ni) chunk_write_bf16<TN>(lds_wave, ni, v[ni], lane);
  chunk_flush_bf16<TN>(lds_wave, c_chunk, ldc, lane);
}
// same for fp32 output: v[g] = the four floats; rows of TN floats leave as 16 bytes per lane
template <int TN>
struct ChunkF32 {
  static constexpr int PITCH = TN * 4 + 16;
  static constexpr int BYTES = 32 * PITCH;
  static constexpr int LPR = TN / 4;
  static constexpr int RPI = 64 / LPR;
  static constexpr int NIT = 32 / RPI;
};
template <int TN>
__device__ __forceinline__ void chunk_write_f32(char* lds_wave, int ni, const float4 (&v)[4], int lane) {
  char* wr = lds_wave + (lane & 31) * ChunkF32<TN>::PITCH + ((lane >> 5) << 4) + ni * 128;
#pragma unroll
  for (int g = 0; g < 4; ++g) *(float4*)(wr + g * 32) = v[g];
}
template <int TN>
__device__ __forceinline__ void chunk_flush_f32(const char* lds_wave, float* c_chunk, long long ldc, int lane) {
  using L = ChunkF32<TN>;
  const int r0 = lane / L::LPR, c = lane % L::LPR;
#pragma unroll
  for (int it = 0; it < L::NIT; ++it) {
    const int row = it * L::RPI + r0;
    *(float4*)(c_chunk + (long long)row * ldc + c * 4) = *(const float4*)(lds_wave + row * L::PITCH + c * 16);
  }
}
template <int TN>
__device__ __forceinline__ void store_chunk_f32(char* lds_wave, float* c_chunk, long long ldc, const float4 (&v)[TN / 32][4],
                                                int lane) {
#pragma unroll
  for (int ni = 0; ni < TN / 32; ++ni) chunk_write_f32<TN>(lds_wave, ni, v[ni], lane);
  chunk_flush_f32<TN>(lds_wave, c_chunk, ldc, lane);
}

// wavefronts per SIMD the kernel is compiled for: what two LDS stages of the tile allow on a 160 KiB CU
template <int BM, int BN, int WM, int WN>
struct Occ {
  static constexpr int lds_bytes = NSTAGE * (BM + BN) * BK * 2;
  static constexpr int wgs = (160 * 1024) / lds_bytes;
  static constexpr int waves_per_simd_raw = wgs * WM * WN / 4;
  static constexpr int value = waves_per_simd_raw < 1 ? 1 : (waves_per_simd_raw > 2 ? 2 : waves_per_simd_raw);
};

// FORM 0: full tiles.
// 1 (RAG) = the block is cut by the tiles, or its rows do not allow the vector epilogue everywhere: masked loads, and a
// bounds-checked epilogue for the wavefronts on the edge.
// 2 (RAG and LONG) = besides, a panel of a k-strided operand does not fit one buffer resource's window: see the load cursors.
// (One parameter: a longer kernel name moves the kernels in the code object, by 0x700 bytes here, and the three products of a
// 3072 -> 12288 layer on an 8 x 8 grid, the same instructions, took 132.4 us instead of 130.6.)
// PLAIN (not with RAG) = the epilogue is a bare store of the accumulator (alpha 1, no bias / activation / residual):
// a short, fully unrolled store sequence instead of the general epilogue, whose straight-line code costs
// microseconds per tile.
// LOOP selects the k-loop: 1 = ring of four 32-wide slabs, fragments read one sub-step ahead
// (the loop described above); 2 = stages of 64 k, the fragments of a whole stage read into registers while the
// matrix cores work on the registers of the stage before it (see the loop).
// 3 = the loop of 2 with four stages, for the smaller tiles in launches of few workgroups (gemm_mfma_deep.hip).
template <int BM, int BN, int LOOP = 2>
struct Loop2 {
  // three stages where one workgroup owns the CU anyway (the 384-row tiles: 144 KiB); two stages otherwise, which is the
  // LDS footprint of the four-slab ring, so that as many workgroups share a CU as with it
  static constexpr int NST = LOOP == 3 ? 4 : (BM + BN == 384) ? 3 : 2;
  static constexpr int RING32 = 2 * NST;                                        // the same space in 32-wide slabs
};

// elements of LDS that a workgroup of this tile and loop needs
template <int BM, int BN, int LOOP>
constexpr int lds_elems() { return (LOOP >= 2 ? Loop2<BM, BN, LOOP>::RING32 : NSTAGE) * (BM + BN) * BK; }

// One tile of a product: workgroup wg of the nwg that the product has.
template <int BM, int BN, int WM, int WN, bool AKC, bool BKC, bool PLAIN, bool SEQ = false, int LOOP = 1, int FORM = 0>
__device__ __forceinline__ void gemm_mfma_tile(const KArgs& a, unsigned wg, const unsigned nwg, bf16_t* const lds_all) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr bool RAG = FORM >= 1, LONG = FORM == 2;
  static_assert(!SEQ || !PLAIN, "the range-wise accumulation exists with the full epilogue");
  static_assert(!RAG || (LOOP == 1 && !PLAIN), "ragged blocks: the four-slab ring, the full epilogue");
  using T = Tile<BM, BN, WM, WN>;
  constexpr int THREADS = T::THREADS, NW = T::NW;
  constexpr int TM = T::TM, TN = T::TN, MI = T::MI, NI = T::NI;
  constexpr int RING = LOOP >= 2 ? Loop2<BM, BN, LOOP>::RING32 : NSTAGE;   // slabs per operand (see read_frag_ring)
  constexpr int LDS_BYTES = RING * (T::A_ELEMS + T::B_ELEMS) * 2;
  bf16_t* const ldsA = lds_all;
  bf16_t* const ldsB = lds_all + RING * T::A_ELEMS;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  OPTIMUS_LAB_STAMP(0);

  // ---- which tile: XCD-aware remap of the linear workgroup id ----
  // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of tiles so that
  // neighbours sharing A rows / B columns also share an L2.
  // 32 bits: a launch has fewer than 2^31 workgroups, and short ones feel 64-bit divisions (the products of an attention backward, 16
  // matrices, s = 1000, d = 80: 70.2 us with them, 66.0 without).
  {
    const unsigned per = nwg >> 3, rem = nwg & 7, xcd = wg & 7, slot = wg >> 3;
    const unsigned start = xcd * per + (xcd < rem ? xcd : rem);  // XCDs 0..rem-1 own per+1 workgroups
    wg = start + slot;
  }
  // Panel split: range after range where the panels are too much for the L2s (a.ranges_first; the line and both sides' times:
  // launch_gemm_mfma), otherwise tile after tile.  Range after range an XCD works on one range of k (or two) and many tiles, so the panels
  // it fetches are a part of k long: half the lines across the fabric that a few tiles with all of k need ([2048 x 16384 x 1024],
  // four ranges: 134 MiB instead of 268).
  const unsigned tiles = a.tiles_m * a.tiles_n;
  unsigned split, z;
  if (a.ranges_first) {
    z = wg / tiles;
    split = z / (unsigned)a.nz;
    z -= split * (unsigned)a.nz;
  } else {
    split = wg % a.splits;
    wg /= a.splits;
    z = wg / tiles;
  }
  int t = (int)(wg % tiles);
  int tm, tn;
  {  // column-major walk within groups of a.group tile rows: the contiguous tile range of an XCD is then a
     // block of a.group rows by (range / a.group) columns, sized on the host so that its A rows and B columns
     // weigh about the same (least bytes fetched per XCD)
    const int GROUP = a.group;
    int per_group = GROUP * a.tiles_n;
    int g = t / per_group;
    int first = g * GROUP;
    int gsz = min(GROUP, a.tiles_m - first);
    int r = t - g * per_group;
    tm = first + r % gsz;
    tn = r / gsz;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  if (a.skip_upper && n0 > m0 + BM - 1) return;

  const int z1 = (int)(z / a.nz0), z0 = (int)(z % a.nz0);
  const bf16_t* Az = a.A + z1 * a.sA1 + z0 * a.sA0;
  const bf16_t* Bz = a.B + z1 * a.sB1 + z0 * a.sB0;

  // ---- k range in slabs, over all panels ----
  // slabs are walked in pairs: a panel has Kw / BK of them (ragged blocks: the last pair may be cut, or half empty)
  const int Kw = RAG ? (a.Kp + 2 * BK - 1) & ~(2 * BK - 1) : a.Kp;
  const int tpp = Kw / BK;
  int t_lo = 0, t_hi = a.nl * tpp;
  if (a.k_lo_diag) t_lo = m0 / BK;
  if (a.k_hi_diag) t_hi = min(t_hi, RAG ? (min(a.Kp, m0 + BM) + 2 * BK - 1) / (2 * BK) * 2 : (min(a.Kp, m0 + BM) + BK - 1) / BK);
  if (a.splits > 1) {
    int total = t_hi - t_lo;
    int per = (total + a.splits - 1) / a.splits;
    per = (per + 1) & ~1;  // slabs are walked in pairs
    int lo = t_lo + (int)split * per;
    t_hi = min(t_hi, lo + per);
    t_lo = lo;
  }

  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0.f;
  // SEQ: `tot` holds the sum of the finished ranges, `acc` the running range (see KArgs::seq_splits); ranges are cut
  // exactly as the panel split cuts them
  f32x16 tot[SEQ ? MI : 1][SEQ ? NI : 1];
  int seq_per = 0, seq_next = 0;
  if constexpr (SEQ) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int e = 0; e < 16; ++e) tot[mi][ni][e] = 0.f;
    const int total = t_hi - t_lo;
    seq_per = (((total + a.seq_splits - 1) / a.seq_splits) + 1) & ~1;
    seq_next = seq_per;
  }

  const bf16_t* Atile = Az + (AKC ? (long long)m0 * a.lda : (long long)m0);
  const bf16_t* Btile = Bz + (BKC ? (long long)n0 * a.ldb : (long long)n0);

  if (t_lo < t_hi) {
    // slab index -> (panel l, offset k0 inside the panel); advanced incrementally
    int l = t_lo / tpp, k0 = (t_lo - l * tpp) * BK;
    if constexpr (LOOP >= 2) {
      // ---- stages of 64 k ----
      // LDS holds NST stages of [BM x 64] + [64 x BN].  An iteration (one stage, four 16-wide sub-steps) has two halves:
      //   first half:  matrix-core instructions of sub-steps 0, 1 (registers h0) | LDS reads of sub-steps 2, 3 (-> h1)
      //   wait + barrier: my reads of stage i are done (nobody reads it any more), my share of stage i+1 has landed
      //   second half: matrix-core instructions of sub-steps 2, 3 (h1) | LDS reads of sub-steps 0, 1 of stage i+1 (-> h0)
      //                | the loads of stage i+NST into the space stage i has left
      // One wait and one barrier per 64 k; the reads have had half an iteration to complete and the loads NST-1
      // iterations, so neither wait is normally exposed.  The memory instructions of a half are spread between its
      // matrix-core instructions: issued in one burst they fill the CU's LDS and memory-instruction queues, and a
      // wavefront that waits for queue space issues no matrix-core instruction either.
      constexpr int NST = Loop2<BM, BN, LOOP>::NST;
      constexpr int PA1 = DirectPlan<BM, NW>::PER, PB1 = DirectPlan<BN, NW>::PER;   // KiB chunks per wavefront per 32 k
      constexpr int NOA = AKC ? 2 * PA1 : PA1, NOB = BKC ? 2 * PB1 : PB1;             // distinct lane offsets
      constexpr int LP = 2 * PA1 + 2 * PB1;                                          // loads per wavefront per stage
      constexpr int A_ST = BM * 64, B_ST = BN * 64;                                  // elements per stage
      unsigned offA[NOA], offB[NOB];
      direct_offsets<BM, AKC, NW, NOA>(offA, a.lda, wave, lane);
      direct_offsets<BN, BKC, NW, NOB>(offB, a.ldb, wave, lane);
      bf16_t* const stA = lds_all;
      bf16_t* const stB = lds_all + NST * A_ST;
      const unsigned stepA = (unsigned)(AKC ? 64 : 64 * a.lda) * 2u, stepB = (unsigned)(BKC ? 64 : 64 * a.ldb) * 2u;
      const unsigned halfA = (unsigned)(32 * a.lda) * 2u, halfB = (unsigned)(32 * a.ldb) * 2u;   // 32 k-rows of a k-strided operand
      int lq = l, kq = k0;
      i32x4 ra = make_rsrc(Atile + lq * a.sAl), rb = make_rsrc(Btile + lq * a.sBl);
      unsigned sa = (unsigned)(AKC ? kq : kq * a.lda) * 2u, sb = (unsigned)(BKC ? kq : kq * a.ldb) * 2u;
      const int n64 = (t_hi - t_lo) >> 1;
      // load g (0 .. LP-1) of the stage that goes into LDS stage st: A's chunks first, then B's
      auto load_item = [&](int st, int g) {
        if (g < 2 * PA1) {
          if constexpr (AKC) direct_issue_one(ra, sa, offA[g], stA + st * A_ST, wave * NOA + g);
          else direct_issue_one(ra, sa + (unsigned)(g / PA1) * halfA, offA[g % PA1], stA + st * A_ST + (g / PA1) * 32 * BM, wave * PA1 + g % PA1);
        } else {
          const int h = g - 2 * PA1;
          if constexpr (BKC) direct_issue_one(rb, sb, offB[h], stB + st * B_ST, wave * NOB + h);
          else direct_issue_one(rb, sb + (unsigned)(h / PB1) * halfB, offB[h % PB1], stB + st * B_ST + (h / PB1) * 32 * BN, wave * PB1 + h % PB1);
        }
      };
      auto advance = [&]() {
        kq += 64;
        if (kq >= a.Kp) { kq = 0; ++lq; sa = 0; sb = 0; ra = make_rsrc(Atile + lq * a.sAl); rb = make_rsrc(Btile + lq * a.sBl); }
        else { sa += stepA; sb += stepB; }
      };
      auto issue_stage = [&](int st) {
#pragma unroll
        for (int g = 0; g < LP; ++g) load_item(st, g);
        advance();
      };
      // fragments of one whole stage: four 16-wide sub-steps; item r = fragment (r % NF) of sub-step (r / NF).
      // Every LDS address is a per-lane base computed once (the swizzles depend on the lane only) plus the stage's
      // offset plus a constant, so that a read costs no address arithmetic inside the loop:
      //   k-contiguous operand: one base per sub-step (chunk index XOR row term), fragment row blocks 32 * 128 bytes apart;
      //   k-strided operand:    one base per fragment (column granule XOR row term), sub-steps 16 k-rows apart.
      constexpr int NF = MI + NI, NRD = 4 * NF, NMF = 4 * MI * NI;
      typedef __attribute__((address_space(3))) char lds_char;
      lds_char* const lds3 = (lds_char*)lds_all;
      unsigned fbaseA[AKC ? 4 : MI], fbaseB[BKC ? 4 : NI];
      if constexpr (AKC) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) fbaseA[ks] = (unsigned)lds_off_kc2(wm * TM + (lane & 31), ks * 2 + (lane >> 5)) * 2u;
      } else {
        const int lg = lane & 15;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
          fbaseA[mi] = (unsigned)lds_off_ks<BM>(((lane >> 5) << 3) + (lg >> 2), wm * TM + mi * 32 + (((lane >> 4) & 1) << 4) + ((lg & 3) << 2)) * 2u;
      }
      if constexpr (BKC) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) fbaseB[ks] = (unsigned)(NST * A_ST + lds_off_kc2(wn * TN + (lane & 31), ks * 2 + (lane >> 5))) * 2u;
      } else {
        const int lg = lane & 15;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
          fbaseB[ni] = (unsigned)(NST * A_ST + lds_off_ks<BN>(((lane >> 5) << 3) + (lg >> 2), wn * TN + ni * 32 + (((lane >> 4) & 1) << 4) + ((lg & 3) << 2))) * 2u;
      }
      bf16x8 ha[4][MI], hb[4][NI];   // [sub-step][fragment]: sub-steps 0, 1 = h0, sub-steps 2, 3 = h1
      auto read_kc = [&](unsigned off) { return *(const __attribute__((address_space(3))) bf16x8*)(lds3 + off); };
      auto read_ks = [&](unsigned off, int rows) {   // two transposing reads: k-rows r .. r+3 and r+4 .. r+7 of the lane's column group
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(lds3 + off));
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(lds3 + off + 4 * rows * 2));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      auto read_item = [&](unsigned stoffA, unsigned stoffB, int ks, int f) {
        if (f < MI) {
          if constexpr (AKC) ha[ks][f] = read_kc(fbaseA[ks] + stoffA + (unsigned)(f * 32 * 128));
          else ha[ks][f] = read_ks(fbaseA[f] + stoffA + (unsigned)(ks * 16 * BM * 2), BM);
        } else {
          const int n = f - MI;
          if constexpr (BKC) hb[ks][n] = read_kc(fbaseB[ks] + stoffB + (unsigned)(n * 32 * 128));
          else hb[ks][n] = read_ks(fbaseB[n] + stoffB + (unsigned)(ks * 16 * BN * 2), BN);
        }
      };
      // one half of an iteration: the matrix-core instructions of sub-steps 2*HH, 2*HH+1; in front of each its share of
      // the reads of the other two sub-steps (of stage st_rd) and, in the second half, of the loads into stage st_ld
      constexpr int HM = 2 * MI * NI, HR = 2 * NF;
      auto half = [&](auto hh_, auto with_reads, auto with_loads, int st_rd, int st_ld) {
        constexpr int HH = decltype(hh_)::value;
        const unsigned offA_rd = (unsigned)(st_rd * A_ST * 2), offB_rd = (unsigned)(st_rd * B_ST * 2);
#pragma unroll
        for (int m = 0; m < HM; ++m) {
          if constexpr (decltype(with_reads)::value && !(OPTIMUS_LAB_DBG & 4)) {
            // all reads in front of the first half of the matrix-core instructions: the wait that follows the last
            // of them must not expose the latency of a read issued just before it
            constexpr int RS = HM / 2 > 0 ? HM / 2 : 1;
#pragma unroll
            for (int r = m * HR / RS; r < (m + 1) * HR / RS && r < HR; ++r) read_item(offA_rd, offB_rd, 2 * (1 - HH) + r / NF, r % NF);
          }
          if constexpr (decltype(with_loads)::value && !(OPTIMUS_LAB_DBG & 1)) {
#pragma unroll
            for (int g = m * LP / HM; g < (m + 1) * LP / HM; ++g) load_item(st_ld, g);
          }
          if constexpr (!(OPTIMUS_LAB_DBG & 8)) {
            const int ks = 2 * HH + m / (MI * NI), mi = (m / NI) % MI, ni = m % NI;
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hb[ks][ni], ha[ks][mi], acc[mi][ni], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (decltype(with_loads)::value) advance();
      };
      // prologue: the first NST stages, then the fragments of sub-steps 0, 1 of stage 0
      issue_stage(0);
      if (n64 > 1) issue_stage(1);
      if (NST > 2 && n64 > 2) issue_stage(2);
      if constexpr (NST > 3) {
        if (n64 > 3) issue_stage(3);
      }
      // all but the n youngest stages have landed, and this wavefront's reads are done
      [[maybe_unused]] auto wait_younger = [&](int n) {
        static_assert(NST <= 4 && (NST - 1) * LP <= 63, "the cases below; vmcnt has six bits");
        switch (n) {
          case 1: OPTIMUS_WAIT_VMCNT_LGKM0(LP); break;
          case 2: OPTIMUS_WAIT_VMCNT_LGKM0(NST > 2 ? 2 * LP : 0); break;
          case 3: OPTIMUS_WAIT_VMCNT_LGKM0(NST > 3 ? 3 * LP : 0); break;
          default: OPTIMUS_WAIT_VMCNT_LGKM0(0); break;
        }
      };
      {
        const int younger = (n64 > NST ? NST : n64) - 1;
        if constexpr (NST > 3) wait_younger(younger);
        else if (younger >= 2) OPTIMUS_WAIT_VMCNT(2 * LP);
        else if (younger == 1) OPTIMUS_WAIT_VMCNT(LP);
        else OPTIMUS_WAIT_VMCNT(0);
      }
      OPTIMUS_BARRIER();
      OPTIMUS_LAB_STAMP(1);
#pragma unroll
      for (int r = 0; r < HR; ++r) read_item(0u, 0u, r / NF, r % NF);
      int seq_next64 = seq_next >> 1;
      const int seq_per64 = seq_per >> 1;
      constexpr std::true_type yes{};
      constexpr std::false_type no{};
      constexpr std::integral_constant<int, 0> first{};
      constexpr std::integral_constant<int, 1> second{};
      int st_cur = 0, st_nxt = NST > 1 ? 1 : 0;
      auto range_end = [&](int i) {   // SEQ: a range of the emulated panel split ends in front of stage i
        if constexpr (SEQ) {
          if (i == seq_next64 && i > 0) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
              for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                  tot[mi][ni][e] += acc[mi][ni][e];
                  acc[mi][ni][e] = 0.f;
                }
            seq_next64 += seq_per64;
          }
        }
      };
      auto next_stage = [&]() {
        st_cur = st_nxt;
        st_nxt = st_nxt + 1 == NST ? 0 : st_nxt + 1;
      };
      // steady state: every iteration reads the next stage and refills the stage it leaves (straight-line body, constant
      // wait counts: with branches inside the loop the compiler copies the accumulators between the paths)
      int i = 0;
#if OPTIMUS_LAB_DBG & 64
      unsigned long long lab_sum_a = 0, lab_sum_b = 0, lab_tb = 0;
#endif
      for (; i + NST < n64; ++i) {
        range_end(i);
        half(first, yes, no, st_cur, 0);
#if OPTIMUS_LAB_DBG & 64
        const unsigned long long lab_ta = clock64();
#endif
        // stage i+1 has landed (the NST-2 younger ones stay in flight); my reads of stage i are done
        if constexpr (!(OPTIMUS_LAB_DBG & 16)) OPTIMUS_WAIT_VMCNT_LGKM0((NST - 2) * LP);
        if constexpr (!(OPTIMUS_LAB_DBG & 2)) OPTIMUS_BARRIER();
#if OPTIMUS_LAB_DBG & 64
        lab_sum_a += lab_ta;
        lab_sum_b += lab_tb;
        lab_tb = clock64();
#endif
        half(second, yes, yes, st_nxt, st_cur);
        next_stage();
      }
#if OPTIMUS_LAB_DBG & 64
      lab_sum_b += lab_tb;
      if (lane == 0 && blockIdx.x < 2048) g_lab_stall[blockIdx.x * 8 + wave] = lab_sum_b - lab_sum_a;
#endif
      // the last stages: nothing left to load
      for (; i + 1 < n64; ++i) {
        range_end(i);
        half(first, yes, no, st_cur, 0);
        if constexpr (NST > 3) wait_younger(n64 - 2 - i);
        else if (NST > 2 && i + 2 < n64) OPTIMUS_WAIT_VMCNT_LGKM0(LP);
        else OPTIMUS_WAIT_VMCNT_LGKM0(0);
        OPTIMUS_BARRIER();
        half(second, yes, no, st_nxt, st_cur);
        next_stage();
      }
      range_end(i);
      half(first, yes, no, st_cur, 0);
      half(second, no, no, st_nxt, st_cur);
      // the results leave through LDS (see the epilogue): nobody may still be reading the last stage
      OPTIMUS_WAIT_VMCNT_LGKM0(0);
      OPTIMUS_BARRIER();
      OPTIMUS_LAB_STAMP(2);
    } else {
      // Loads per wavefront: a k-strided operand moves one slab per step; a k-contiguous operand moves a pair of
      // slabs (whole 128-byte lines per row) every second step.  The slab count of a workgroup is even (host).
      constexpr int PA1 = DirectPlan<BM, NW>::PER, PB1 = DirectPlan<BN, NW>::PER;
      constexpr int PA = AKC ? 2 * PA1 : PA1, PB = BKC ? 2 * PB1 : PB1;
      constexpr int PKS = (AKC ? 0 : PA1) + (BKC ? 0 : PB1);          // loads of one k-strided slab issue
      constexpr int PKC2 = (AKC ? 2 * PA1 : 0) + (BKC ? 2 * PB1 : 0);  // loads of one k-contiguous pair issue
      unsigned offA[PA], offB[PB];
      direct_offsets<BM, AKC, NW, PA>(offA, a.lda, wave, lane);
      direct_offsets<BN, BKC, NW, PB>(offB, a.ldb, wave, lane);
      int kinA[RAG ? PA : 1], kinB[RAG ? PB : 1];   // RAG: the chunk's k inside its unit
      if constexpr (RAG) {
        direct_cut<BM, AKC, NW, PA>(offA, kinA, a.Mb - m0, wave, lane);
        direct_cut<BN, BKC, NW, PB>(offB, kinB, a.Nb - n0, wave, lane);
      }
      // one load cursor per operand: panel, k offset, buffer resource of the panel, byte offset inside the panel.  LONG: the
      // panels of a k-strided operand are walked in segments of k rows, each with a resource of its own.
      constexpr int KA = AKC ? 2 * BK : BK, KB = BKC ? 2 * BK : BK;  // k advance per issue
      const unsigned stepA = (unsigned)(AKC ? KA : KA * a.lda) * 2u;
      const unsigned stepB = (unsigned)(BKC ? KB : KB * a.ldb) * 2u;
      int lqa = l, kqa = k0, lqb = l, kqb = k0;
      i32x4 ra = make_rsrc(Atile + lqa * a.sAl), rb = make_rsrc(Btile + lqb * a.sBl);
      unsigned sa = (unsigned)(AKC ? kqa : kqa * a.lda) * 2u, sb = (unsigned)(BKC ? kqb : kqb * a.ldb) * 2u;
      constexpr bool SEGA = LONG && !AKC, SEGB = LONG && !BKC;
      [[maybe_unused]] int endA = Kw, endB = Kw;
      [[maybe_unused]] auto segment = [&](i32x4& r, unsigned& off, int& end, const bf16_t* panel, int k, int ld, int seg) {
        r = make_rsrc(panel + (long long)k * ld);
        off = 0;
        end = Kw - k > seg ? k + seg : Kw;
      };
      int segA = 0, segB = 0;
      if constexpr (SEGA) { segA = segment_rows(a.lda); segment(ra, sa, endA, Atile + lqa * a.sAl, kqa, a.lda, segA); }
      if constexpr (SEGB) { segB = segment_rows(a.ldb); segment(rb, sb, endB, Btile + lqb * a.sBl, kqb, a.ldb, segB); }
      const int nslab = t_hi - t_lo;
#define OPTIMUS_NEXT_A()                                                               \
  do {                                                                                 \
    kqa += KA;                                                                         \
    if constexpr (SEGA) {                                                              \
      if (kqa >= endA) {                                                               \
        if (kqa >= Kw) { kqa = 0; ++lqa; }                                             \
        segment(ra, sa, endA, Atile + lqa * a.sAl, kqa, a.lda, segA);                  \
      } else sa += stepA;                                                              \
    } else {                                                                           \
      if (kqa >= Kw) { kqa = 0; ++lqa; sa = 0; ra = make_rsrc(Atile + lqa * a.sAl); }  \
      else sa += stepA;                                                                \
    }                                                                                  \
  } while (0)
#define OPTIMUS_NEXT_B()                                                               \
  do {                                                                                 \
    kqb += KB;                                                                         \
    if constexpr (SEGB) {                                                              \
      if (kqb >= endB) {                                                               \
        if (kqb >= Kw) { kqb = 0; ++lqb; }                                             \
        segment(rb, sb, endB, Btile + lqb * a.sBl, kqb, a.ldb, segB);                  \
      } else sb += stepB;                                                              \
    } else {                                                                           \
      if (kqb >= Kw) { kqb = 0; ++lqb; sb = 0; rb = make_rsrc(Btile + lqb * a.sBl); }  \
      else sb += stepB;                                                                \
    }                                                                                  \
  } while (0)
#define OPTIMUS_ISSUE_A(DST)                                                         \
  do {                                                                               \
    direct_issue<RAG, PA>(ra, sa, offA, kinA, a.Kp - kqa, DST, wave);                \
    OPTIMUS_NEXT_A();                                                                \
  } while (0)
#define OPTIMUS_ISSUE_B(DST)                                                         \
  do {                                                                               \
    direct_issue<RAG, PB>(rb, sb, offB, kinB, a.Kp - kqb, DST, wave);                \
    OPTIMUS_NEXT_B();                                                                \
  } while (0)
      // pair P (0/1) of the k-contiguous operands; slab S (0..3) of the k-strided ones
#define OPTIMUS_ISSUE_KC(P)                                                          \
  do {                                                                               \
    if constexpr (AKC) OPTIMUS_ISSUE_A(ldsA + (P) * 2 * T::A_ELEMS);                 \
    if constexpr (BKC) OPTIMUS_ISSUE_B(ldsB + (P) * 2 * T::B_ELEMS);                 \
  } while (0)
#define OPTIMUS_ISSUE_KS(S)                                                          \
  do {                                                                               \
    if constexpr (!AKC) OPTIMUS_ISSUE_A(ldsA + (S) * T::A_ELEMS);                    \
    if constexpr (!BKC) OPTIMUS_ISSUE_B(ldsB + (S) * T::B_ELEMS);                    \
  } while (0)
      // Continuous pipeline over 16-wide sub-steps; F0 = (fa0, fb0) holds sub-step 0 of the current slab i.
      //   A  sub-step 0: MFMAs on F0; between them the fragment reads of sub-step 1 (F1) and the second half of the
      //      loads of the group opened in the previous step;
      //   B  wait for F1 (after it this wavefront reads slab i no more) and for the loads slab i+1 needs, leaving the
      //      younger ones in flight; barrier: nobody reads slab i any more, slab i+1 is complete in LDS;
      //   C  open the group that refills what slab i freed: its stage for the k-strided operands (slab i+4); after an
      //      odd slab also its pair for the k-contiguous operands (slabs i+3, i+4);
      //   D  sub-step 1: MFMAs on F1; between them the reads of sub-step 0 of slab i+1 (F0) and the first half of
      //      the group's loads.
      // The loads are spread between the MFMAs one by one: issued in one burst after the barrier they fill the
      // CU's memory-instruction queue, and a wavefront stalled on a full queue issues no MFMA either.
      // Loads retire in issue order.  Issue order is [pair 0, slab 0, slab 1, pair 1, slab 2, slab 3], then per even
      // step [slab i+4], per odd step [pair, slab i+4]; the wait counts below are the loads younger than what slab
      // i+1 needs in that order (at B of step i everything up to the group of step i-1 has been issued).
      constexpr int MF = MI * NI;
      constexpr int NF = MI + NI;                                   // fragments per sub-step
      constexpr int FSLOTS = MF / 2 > 0 ? MF / 2 : 1;               // the fragment reads go in front of the first MFMAs
      constexpr int FPS = (NF + FSLOTS - 1) / FSLOTS;               // fragments requested per such slot
      static_assert(BK == 32 && NSTAGE == 4, "the pipeline below is written for two sub-steps per slab, four slabs");
      static_assert(MF <= 16 && FPS <= 3 && PA + PB <= 16, "slot and load lists below");
      constexpr int G_ODD = PA + PB, G_EVEN = PKS;  // loads per group
      bf16x8 fa0[MI], fb0[NI], fa1[MI], fb1[NI];
      bool pend = false;  // the group opened in the previous step still has its second half to issue
      // load N of the group of parity ODD refilling slab S's space: A's chunks first, then B's
#define OPTIMUS_DMA_N(ODD, S, N)                                                                                  \
  do {                                                                                                            \
    constexpr int nA_ = (ODD) ? PA : (AKC ? 0 : PA);                                                              \
    constexpr int nB_ = (ODD) ? PB : (BKC ? 0 : PB);                                                              \
    if constexpr ((N) < nA_)                                                                                      \
      direct_issue_one(ra, sa, cut_off<RAG>(offA[(N) < nA_ ? (N) : 0], kinA[RAG && (N) < nA_ ? (N) : 0], a.Kp - kqa), \
                       ldsA + (AKC ? ((S) >> 1) * 2 : (S)) * T::A_ELEMS, wave * PA + (N));                        \
    else if constexpr ((N) < nA_ + nB_)                                                                           \
      direct_issue_one(rb, sb, cut_off<RAG>(offB[(N) >= nA_ && (N) < nA_ + nB_ ? (N) - nA_ : 0],                  \
                                            kinB[RAG && (N) >= nA_ && (N) < nA_ + nB_ ? (N) - nA_ : 0], a.Kp - kqb), \
                       ldsB + (BKC ? ((S) >> 1) * 2 : (S)) * T::B_ELEMS, wave * PB + (N) - nA_);                  \
  } while (0)
      // in slot M: the loads G0 .. G0+GN-1 of the group whose turn it is
#define OPTIMUS_DMA_SLOT(M, ODD, S, G0, GN, DO)                                                                   \
  do {                                                                                                            \
    if constexpr ((GN) > 0) {                                                                                     \
      if constexpr (dma_slot(0, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 0); }     \
      if constexpr ((GN) > 1 && dma_slot(1, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 1); }\
      if constexpr ((GN) > 2 && dma_slot(2, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 2); }\
      if constexpr ((GN) > 3 && dma_slot(3, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 3); }\
      if constexpr ((GN) > 4 && dma_slot(4, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 4); }\
      if constexpr ((GN) > 5 && dma_slot(5, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 5); }\
      if constexpr ((GN) > 6 && dma_slot(6, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 6); }\
      if constexpr ((GN) > 7 && dma_slot(7, (GN) > 0 ? (GN) : 1, MF) == (M)) { if (DO) OPTIMUS_DMA_N(ODD, S, (G0) + 7); }\
    }                                                                                                             \
  } while (0)
#define OPTIMUS_SLOT(M, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO)                              \
  do {                                                                                                            \
    if constexpr ((M) < MF) {                                                                                     \
      load_frag_r<(M) * FPS, BM, BN, WM, WN, AKC, BKC>(FA_LD, FB_LD, ldsA, ldsB, S_LD, KS_LD, wm, wn, lane); \
      load_frag_r<((FPS > 1) ? (M) * FPS + 1 : NF), BM, BN, WM, WN, AKC, BKC>(FA_LD, FB_LD, ldsA, ldsB, S_LD, KS_LD, wm, wn, lane); \
      load_frag_r<((FPS > 2) ? (M) * FPS + 2 : NF), BM, BN, WM, WN, AKC, BKC>(FA_LD, FB_LD, ldsA, ldsB, S_LD, KS_LD, wm, wn, lane); \
      OPTIMUS_DMA_SLOT(M, ODD, S, G0, GN, DO);                                                                    \
      mfma_m<(((M) < MF) ? (M) : 0), MI, NI>(acc, FA_MM, FB_MM);                                                      \
      __builtin_amdgcn_sched_barrier(0);                                                                          \
    }                                                                                                             \
  } while (0)
#define OPTIMUS_HALF(FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO)                                 \
  do {                                                                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                                            \
    OPTIMUS_SLOT(0, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(1, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(2, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(3, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(4, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(5, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(6, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(7, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(8, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(9, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                 \
    OPTIMUS_SLOT(10, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                \
    OPTIMUS_SLOT(11, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                \
    OPTIMUS_SLOT(12, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                \
    OPTIMUS_SLOT(13, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                \
    OPTIMUS_SLOT(14, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                \
    OPTIMUS_SLOT(15, FA_LD, FB_LD, S_LD, KS_LD, FA_MM, FB_MM, ODD, S, G0, GN, DO);                                \
  } while (0)
      // cursor advance once a group is out: every operand that had loads in it
#define OPTIMUS_ADVANCE(ODD)                                                                  \
  do {                                                                                        \
    if constexpr ((ODD) || !AKC) OPTIMUS_NEXT_A();                                            \
    if constexpr ((ODD) || !BKC) OPTIMUS_NEXT_B();                                            \
  } while (0)
      // S = slab position (0..3) of slab i; the previous step's group refills position (S + 3) & 3.
      // ST = 1: steady state, i >= 4 and i + 8 <= nslab at the top of the four steps: every group exists, so every
      // load is unconditional and every wait count a constant (the conditional form costs about ten scalar branches
      // per step, a third of the time of a step on the small tiles).
#define OPTIMUS_STEP_EVEN(S, ST)                                                                                  \
  do {                                                                                                            \
    OPTIMUS_HALF(fa1, fb1, S, 1, fa0, fb0, true, ((S) + 3) & 3, (G_ODD + 1) / 2, G_ODD / 2, ((ST) || pend));      \
    if ((ST) || pend) OPTIMUS_ADVANCE(true);                                                                      \
    if (!(ST)) pend = false;                                                                                      \
    if constexpr (PKS > 0) { /* all k-contiguous: slab i+1 came with slab i, nothing to hand over */              \
      if ((ST) || i + 2 < nslab) OPTIMUS_WAIT_VMCNT_LGKM0(2 * PKS + PKC2);                                        \
      else OPTIMUS_WAIT_VMCNT_LGKM0(0);                                                                           \
      OPTIMUS_BARRIER();                                                                                          \
      if (!(ST)) pend = i + 4 < nslab;                                                                            \
    }                                                                                                             \
    OPTIMUS_HALF(fa0, fb0, (S) + 1, 0, fa1, fb1, false, S, 0, (G_EVEN + 1) / 2, ((ST) || pend));                  \
    ++i;                                                                                                          \
  } while (0)
#define OPTIMUS_STEP_ODD(S, ST)                                                                                   \
  do {                                                                                                            \
    OPTIMUS_HALF(fa1, fb1, S, 1, fa0, fb0, false, (S) - 1, (G_EVEN + 1) / 2, G_EVEN / 2, ((ST) || pend));         \
    if (PKS > 0 && ((ST) || pend)) OPTIMUS_ADVANCE(false);                                                        \
    if ((ST) || i + 3 < nslab) OPTIMUS_WAIT_VMCNT_LGKM0(2 * PKS);                                                 \
    else if (i + 2 < nslab) OPTIMUS_WAIT_VMCNT_LGKM0(PKS);                                                        \
    else OPTIMUS_WAIT_VMCNT_LGKM0(0);                                                                             \
    OPTIMUS_BARRIER();                                                                                            \
    if (!(ST)) pend = i + 3 < nslab;                                                                              \
    /* after the last slab this reads a slab nobody writes any more; the values are never used */                \
    OPTIMUS_HALF(fa0, fb0, ((S) + 1) & 3, 0, fa1, fb1, true, S, 0, (G_ODD + 1) / 2, ((ST) || pend));              \
    ++i;                                                                                                          \
  } while (0)
      // SEQ: a range ends in front of slab i (ranges are even, so only in front of even steps)
#define OPTIMUS_RANGE_END()                                                        \
  do {                                                                             \
    if constexpr (SEQ) {                                                           \
      if (i == seq_next) {                                                         \
        _Pragma("unroll") for (int mi_ = 0; mi_ < MI; ++mi_)                       \
          _Pragma("unroll") for (int ni_ = 0; ni_ < NI; ++ni_)                     \
            _Pragma("unroll") for (int e_ = 0; e_ < 16; ++e_) {                    \
              tot[mi_][ni_][e_] += acc[mi_][ni_][e_];                              \
              acc[mi_][ni_][e_] = 0.f;                                             \
            }                                                                      \
        seq_next += seq_per;                                                       \
      }                                                                            \
    }                                                                              \
  } while (0)
      // prologue: whole groups at once
      OPTIMUS_ISSUE_KC(0);
      OPTIMUS_ISSUE_KS(0);
      OPTIMUS_ISSUE_KS(1);
      if (nslab > 2) {
        OPTIMUS_ISSUE_KC(1);
        OPTIMUS_ISSUE_KS(2);
        OPTIMUS_ISSUE_KS(3);
        OPTIMUS_WAIT_VMCNT(PKC2 + 2 * PKS);
      } else {
        OPTIMUS_WAIT_VMCNT(0);
      }
      OPTIMUS_BARRIER();
      load_frags<BM, BN, WM, WN, AKC, BKC>(fa0, fb0, ldsA, ldsB, 0, 0, wm, wn, lane);
      int i = 0;
      while (i + 4 <= nslab) {
        OPTIMUS_RANGE_END();
        OPTIMUS_STEP_EVEN(0, 0);
        OPTIMUS_STEP_ODD(1, 0);
        OPTIMUS_RANGE_END();
        OPTIMUS_STEP_EVEN(2, 0);
        OPTIMUS_STEP_ODD(3, 0);
        while (i + 8 <= nslab) {  // i >= 4 here
          OPTIMUS_RANGE_END();
          OPTIMUS_STEP_EVEN(0, 1);
          OPTIMUS_STEP_ODD(1, 1);
          OPTIMUS_RANGE_END();
          OPTIMUS_STEP_EVEN(2, 1);
          OPTIMUS_STEP_ODD(3, 1);
          pend = true;  // the last steady step opened a group
        }
      }
      if (i < nslab) {  // one pair left
        OPTIMUS_RANGE_END();
        OPTIMUS_STEP_EVEN(0, 0);
        OPTIMUS_STEP_ODD(1, 0);
      }
#undef OPTIMUS_RANGE_END
#undef OPTIMUS_STEP_EVEN
#undef OPTIMUS_STEP_ODD
#undef OPTIMUS_HALF
#undef OPTIMUS_SLOT
#undef OPTIMUS_DMA_SLOT
#undef OPTIMUS_DMA_N
#undef OPTIMUS_ADVANCE
#undef OPTIMUS_NEXT_A
#undef OPTIMUS_NEXT_B
#undef OPTIMUS_ISSUE_KS
#undef OPTIMUS_ISSUE_KC
#undef OPTIMUS_ISSUE_A
#undef OPTIMUS_ISSUE_B
    }
  }

  if constexpr (SEQ) {  // the last range joins the sum; the epilogue below works on `acc`
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[mi][ni][e] = tot[mi][ni][e] + acc[mi][ni][e];
  }
  // ---- epilogue: lane holds row (lane%32), columns 8*g + 4*(lane/32) + 0..3 of each 32x32 tile ----
  if (a.splits > 1) {
    // raw fp32 partial tile; the combine kernel adds the splits in order and applies the epilogue
    float* P = a.partials + ((long long)split * a.nz + z) * (long long)a.Mb * a.Nb;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int m = m0 + wm * TM + mi * 32 + (lane & 31);
          const int n = n0 + wn * TN + ni * 32 + g * 8 + ((lane >> 5) << 2);
          if (RAG && (m >= a.Mb || n >= a.Nb)) continue;
          float* p = P + (long long)m * a.Nb + n;
          if (!RAG || (n + 3 < a.Nb && (a.Nb & 3) == 0)) {
            *(float4*)p = make_float4(acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1], acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]);
          } else {
            for (int c = 0; c < 4 && n + c < a.Nb; ++c) p[c] = acc[mi][ni][g * 4 + c];
          }
        }
    return;
  }
  EpiArgs e = a.epi;
  const long long coff = z1 * a.sC1 + z0 * a.sC0;
  if constexpr (RAG) {
    // wavefronts whose tile the block's edge cuts, and blocks whose rows allow no vector accesses
    if (!e.vec_ok || m0 + wm * TM + TM > a.Mb || n0 + wn * TN + TN > a.Nb) {
      if (e.bias) e.bias += z0 * a.sBias0;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int m = m0 + wm * TM + mi * 32 + (lane & 31);
            const int n = n0 + wn * TN + ni * 32 + g * 8 + ((lane >> 5) << 2);
            if (m >= a.Mb || n >= a.Nb) continue;
            const float v[4] = {acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1], acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]};
            epilogue_store4<false>(e, coff, m, n, v, min(4, a.Nb - n));
          }
      return;
    }
  }
  if constexpr (PLAIN) {
    // Stores go through LDS chunk by chunk (see store_chunk_bf16) when rows of C are 16-byte aligned; after the
    // last barrier of the k-loop no wavefront reads operand data from LDS any more.
    const long long tile0 = coff + (long long)(m0 + wm * TM) * e.ldc + n0 + wn * TN;   // first element of the wave tile
    const bool lines16 = ((e.ldc | coff) & 7) == 0;
    // this lane's first element when storing directly: row lane%32, column 4*(lane/32)
    const long long first = tile0 + (long long)(lane & 31) * e.ldc + ((lane >> 5) << 2);
    if (!e.out_fp32) {
      if (lines16) {
        static_assert(ChunkBf16<TN>::BYTES * NW <= LDS_BYTES, "chunk staging must fit in the operand rings");
        char* stage = (char*)lds_all + wave * ChunkBf16<TN>::BYTES;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
          uint2 v[NI][4];
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              v[ni][g] = make_uint2(pack2_bf16(acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1]),
                                    pack2_bf16(acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]));
          store_chunk_bf16<TN>(stage, (bf16_t*)e.C + tile0 + (long long)mi * 32 * e.ldc, e.ldc, v, lane);
        }
      } else {
        bf16_t* crow = (bf16_t*)e.C + first;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              *(uint2*)(crow + ni * 32 + g * 8) = make_uint2(pack2_bf16(acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1]),
                                                             pack2_bf16(acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]));
          crow += 32LL * e.ldc;
        }
      }
    } else {
      static_assert(ChunkF32<TN>::BYTES * NW <= LDS_BYTES, "chunk staging must fit in the operand rings");
      if (((e.ldc | coff) & 3) == 0) {
        char* stage = (char*)lds_all + wave * ChunkF32<TN>::BYTES;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
          float4 v[NI][4];
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              v[ni][g] = make_float4(acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1], acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]);
          store_chunk_f32<TN>(stage, (float*)e.C + tile0 + (long long)mi * 32 * e.ldc, e.ldc, v, lane);
        }
      } else {
        float* crow = (float*)e.C + first;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              *(float4*)(crow + ni * 32 + g * 8) =
                  make_float4(acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1], acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]);
          crow += 32LL * e.ldc;
        }
      }
    }
  } else {
    // General epilogue, vector form (bf16 in, 8- or 16-byte accesses; the host has checked the alignments).
    // Everything it reads is requested in batches ahead of the stores: the compiler cannot prove that C aliases
    // none of the inputs, so a load written after a store waits for it, and 16 * MI * NI dependent round trips
    // to memory would cost more than the product itself.
    const float* bias = e.bias ? e.bias + z0 * a.sBias0 + n0 + wn * TN + ((lane >> 5) << 2) : nullptr;
    const long long tile0 = coff + (long long)(m0 + wm * TM) * e.ldc + n0 + wn * TN;   // first element of the wave tile
    const long long first = tile0 + (long long)(lane & 31) * e.ldc + ((lane >> 5) << 2);
    // results leave through LDS as whole rows of the tile when the rows are 16-byte aligned (see ChunkBf16); the
    // staging piece of a wavefront holds one chunk of C (bf16 or fp32) and one of the pre-activation
    const bool lines16 = ((e.ldc | coff) & 7) == 0;
    constexpr int STAGE_C = ChunkBf16<TN>::BYTES;   // the pre-activation chunk sits behind a bf16 C chunk; an fp32 C chunk uses both
    constexpr int STAGE = ChunkF32<TN>::BYTES > 2 * STAGE_C ? ChunkF32<TN>::BYTES : 2 * STAGE_C;
    const bool pre_lines = lines16 && !e.out_fp32;
    static_assert(STAGE * NW <= LDS_BYTES, "chunk staging must fit in the operand rings");
    char* stage = (char*)lds_all + wave * STAGE;
    const bf16_t* zrow = e.gelu_grad_of ? (const bf16_t*)e.gelu_grad_of + first : nullptr;
    const bf16_t* rrow = e.residual ? (const bf16_t*)e.residual + first : nullptr;
    bf16_t* prow = e.pre_act ? (bf16_t*)e.pre_act + first : nullptr;
    const bool act = e.act == 1, out32 = e.out_fp32 != 0;
    const float alpha = e.alpha;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const long long ro = (long long)mi * 32 * e.ldc;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        float4 b4[4];
        uint2 zz[4], rr[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) b4[g] = bias ? *(const float4*)(bias + ni * 32 + g * 8) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (zrow) {
#pragma unroll
          for (int g = 0; g < 4; ++g) zz[g] = *(const uint2*)(zrow + ro + ni * 32 + g * 8);
        }
        if (rrow) {
#pragma unroll
          for (int g = 0; g < 4; ++g) rr[g] = *(const uint2*)(rrow + ro + ni * 32 + g * 8);
        }
        uint2 pv[4];
        float4 cf[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float t[4] = {acc[mi][ni][g * 4] * alpha + b4[g].x, acc[mi][ni][g * 4 + 1] * alpha + b4[g].y,
                        acc[mi][ni][g * 4 + 2] * alpha + b4[g].z, acc[mi][ni][g * 4 + 3] * alpha + b4[g].w};
          if (prow) pv[g] = make_uint2(pack2_bf16(t[0], t[1]), pack2_bf16(t[2], t[3]));
          if (act) gelu4<false>(t);
          if (zrow) {
            const uint2 w = zz[g];
            const float z[4] = {__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                                __uint_as_float(w.y & 0xffff0000u)};
            gelu_grad_mul4<false>(t, z);
          }
          if (rrow) {
            const uint2 w = rr[g];
            t[0] += __uint_as_float(w.x << 16); t[1] += __uint_as_float(w.x & 0xffff0000u);
            t[2] += __uint_as_float(w.y << 16); t[3] += __uint_as_float(w.y & 0xffff0000u);
          }
          cf[g] = make_float4(t[0], t[1], t[2], t[3]);
        }
        if (prow) {
          if (pre_lines) chunk_write_bf16<TN>(stage + STAGE_C, ni, pv, lane);
          else {
#pragma unroll
            for (int g = 0; g < 4; ++g) *(uint2*)(prow + ro + ni * 32 + g * 8) = pv[g];
          }
        }
        if (out32) {
          if (lines16) chunk_write_f32<TN>(stage, ni, cf, lane);
          else {
#pragma unroll
            for (int g = 0; g < 4; ++g) *(float4*)((float*)e.C + first + ro + ni * 32 + g * 8) = cf[g];
          }
        } else {
          uint2 cv[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) cv[g] = make_uint2(pack2_bf16(cf[g].x, cf[g].y), pack2_bf16(cf[g].z, cf[g].w));
          if (lines16) chunk_write_bf16<TN>(stage, ni, cv, lane);
          else {
#pragma unroll
            for (int g = 0; g < 4; ++g) *(uint2*)((bf16_t*)e.C + first + ro + ni * 32 + g * 8) = cv[g];
          }
        }
      }
      if (lines16) {
        if (prow && pre_lines) chunk_flush_bf16<TN>(stage + STAGE_C, (bf16_t*)e.pre_act + tile0 + ro, e.ldc, lane);
        if (out32) chunk_flush_f32<TN>(stage, (float*)e.C + tile0 + ro, e.ldc, lane);
        else chunk_flush_bf16<TN>(stage, (bf16_t*)e.C + tile0 + ro, e.ldc, lane);
      }
    }
  }
  OPTIMUS_LAB_STAMP(3);
#endif  // __HIP_DEVICE_COMPILE__
}

template <int BM, int BN, int WM, int WN, bool AKC, bool BKC, bool PLAIN, bool SEQ = false, int LOOP = 1, int FORM = 0>
__global__ __launch_bounds__(WM* WN * 64, (Occ<BM, BN, WM, WN>::value)) void gemm_mfma_kernel(const KArgs a) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds_all[lds_elems<BM, BN, LOOP>()];
  gemm_mfma_tile<BM, BN, WM, WN, AKC, BKC, PLAIN, SEQ, LOOP, FORM>(a, blockIdx.x, gridDim.x, lds_all);
}

}  // namespace optimus
