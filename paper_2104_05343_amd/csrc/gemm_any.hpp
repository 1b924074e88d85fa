// Shared by the two product kernels for any shape, stride and alignment (gemm_generic.hip, gemm_short.hip): arguments, the
// staging of an operand's slab in LDS, and the matrix instructions of one eighth of a slab.
#pragma once
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

// One operand's slab of ROWS rows (or columns) by KB = 256 bytes of k (a quarter of it in gemm_short_kernel), in LDS:
//   KC (k contiguous in memory): [ROWS][KB + 16]; a fragment read is 16 bytes of one row, and 16 rows at a pitch of
//     68 (20) banks cover the 64 banks once.
//   !KC, fp32: [64 k][ROWS + 8 floats]; a fragment read is one float per lane, the two half-waves four k-rows apart.
//   !KC, bf16: [128 k][ROWS], 16-column granules XOR 2 * (k & 3), read with the transposing ds_read_b64_tr_b16.
template <typename T, int ROWS, bool KC, bool TINY, int KB = 256, int NT = GT_THREADS>
struct Slab {
  static constexpr int E = 16 / (int)sizeof(T);       // elements per 16-byte chunk
  static constexpr int KS = KB / (int)sizeof(T);      // k per slab
  static constexpr int CHUNKS = ROWS * (KB / 16) / NT;  // chunks per thread
  static constexpr int BYTES = KC ? ROWS * (KB + 16) : (sizeof(T) == 4 ? KS * (ROWS + 8) * 4 : KS * ROWS * 2);

  // element offset of the chunk from the slab's origin, and its place in the tile
  static __device__ __forceinline__ void place(int tid, int it, int& row, int& k) {
    const int c = tid + it * NT;
    constexpr int LOG = KB == 256 ? 4 : 2;   // chunks per row
    if (KC) { row = c >> LOG; k = (c & ((1 << LOG) - 1)) * E; }
    else { k = c / (ROWS / E); row = (c % (ROWS / E)) * E; }
  }
  static __device__ __forceinline__ int lds_off(int row, int k) {   // bytes
    if (KC) return row * (KB + 16) + k * (int)sizeof(T);
    if (sizeof(T) == 4) return (k * (ROWS + 8) + row) * 4;
    return (k * ROWS + ((((row >> 4) ^ (((k & 3) << 1) & (ROWS / 16 - 1)))) << 4) + (row & 15)) * 2;
  }
  static_assert(KB == 256 || KB == 64, "see place");
  static_assert(CHUNKS * NT * E == ROWS * KS, "the threads' chunks cover the slab once");

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

// the launch, arguments prepared (tiles of 64x64); d: for its layout and type
int launch_gemm_short(const GArgs& a, const GemmDesc& d, bool tiny, unsigned nwg, hipStream_t stream);

}  // namespace optimus
