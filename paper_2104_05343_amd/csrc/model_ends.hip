// The two ends of the model around the layer stack in the 2D partition (Sections 3.2.1 / 3.2.2 of the paper):
//   * embedding: the paper's "one-hot matrix times embedding table" product is a row gather.  Device (i, j) holds the
//     token indices of grid row i (every device of a row has them) and the table block (l, j) of every l is resident:
//     out_ij[t] = table block (tok / (v/q), j), row tok % (v/q).  Pure copy: bit exact, HBM bound.
//   * embedding gradient: d_table_lj = sum_i one_hot_il^T dX_ij, the A^T B form reduced within column j onto its owner
//     (l, j).  Computed as the owner sees it: a workgroup owns 128 table rows x 64 columns of the block as fp32
//     accumulators in LDS, scans ALL token indices, adds the rows of dX whose token falls into its rows and writes
//     its piece once.  No atomics, an order of additions fixed by the token order: deterministic, and rows that no
//     token refers to are written as zeros.
//   * cross entropy H = log(sum_i exp(x_i)) - x_label over a logits row that spans the q devices of a grid row: each
//     device reduces its v/q columns to (max, sum exp(x - max)) -- the maximum is subtracted for range, which does
//     not change the value --, the q partials are combined in the order l = 0..q-1 (the row all-reduce), and the
//     device computes the loss and keeps L = log sum exp per row.  Backward: q_j - [j = label] with
//     q_j = exp(x_j - L) recomputed from the saved L (the paper saves the soft-max itself: v/2 times the bytes).
// The lm-head logits are the C = A B^T product of the hidden states with the table: optimus_summa_abt.
#include <type_traits>

#include "common.hpp"

namespace optimus {
namespace {

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}
template <typename T> __device__ __forceinline__ float ldf(const T* p);
template <> __device__ __forceinline__ float ldf<bf16_t>(const bf16_t* p) { return bf16_to_f32(*p); }
template <> __device__ __forceinline__ float ldf<float>(const float* p) { return *p; }
template <typename T> __device__ __forceinline__ void stf(T* p, float v);
template <> __device__ __forceinline__ void stf<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }
template <> __device__ __forceinline__ void stf<float>(float* p, float v) { *p = v; }

__device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }
__device__ __forceinline__ float to_f32(float v) { return v; }

__device__ __forceinline__ int clamp_token(int t, int v) { return min(max(t, 0), v - 1); }

// 16 bytes of a row as floats (8 bf16 or 4 fp32) and back
template <typename T> struct V16;
template <> struct V16<bf16_t> {
  static constexpr int N = 8;
  __device__ static void load(const bf16_t* p, float* f) {
    const uint4 w = *(const uint4*)p;
    const unsigned u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { f[2 * k] = __uint_as_float(u[k] << 16); f[2 * k + 1] = __uint_as_float(u[k] & 0xffff0000u); }
  }
  __device__ static void store(bf16_t* p, const float* f) {
    *(uint4*)p = make_uint4(pack2_bf16(f[0], f[1]), pack2_bf16(f[2], f[3]), pack2_bf16(f[4], f[5]), pack2_bf16(f[6], f[7]));
  }
};
template <> struct V16<float> {
  static constexpr int N = 4;
  __device__ static void load(const float* p, float* f) { const float4 w = *(const float4*)p; f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w; }
  __device__ static void store(float* p, const float* f) { *(float4*)p = make_float4(f[0], f[1], f[2], f[3]); }
};

struct EndArgs {
  int rows;        // M/q: rows of a block
  int vb, hb;      // v/q, h/q
  int q, v;
  int i0, ni, j0, nj;  // devices handled: grid rows i0.., grid columns j0..
};

// ---- embedding forward: one wavefront per output row; 16-byte copies when the block width allows ----
template <typename T>
__global__ __launch_bounds__(256) void embedding_fwd_kernel(const int* __restrict__ tokens, const T* __restrict__ table,
                                                            T* __restrict__ out, EndArgs a) {
  const int lane = threadIdx.x & 63;
  const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= a.rows) return;
  const int dev = blockIdx.y;
  const int i = a.i0 + dev / a.nj, j = a.j0 + dev % a.nj;
  const int tok = clamp_token(tokens[(long long)i * a.rows + r], a.v);
  const int l = tok / a.vb, tr = tok % a.vb;
  const T* src = table + (((long long)l * a.q + j) * a.vb + tr) * a.hb;
  T* dst = out + (((long long)i * a.q + j) * a.rows + r) * a.hb;
  constexpr int VN = 16 / sizeof(T);
  if (a.hb % VN == 0) {
    for (int c = lane * VN; c < a.hb; c += 64 * VN) *(uint4*)(dst + c) = *(const uint4*)(src + c);
  } else {
    for (int c = lane; c < a.hb; c += 64) dst[c] = src[c];
  }
}

// inclusive prefix sums over the lanes, in the vector unit: within rows of 16 lanes, then a row's last lane to the rows behind it
__device__ __forceinline__ unsigned wave_scan(unsigned v) {
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 to rows 1 and 3
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 to rows 2 and 3
  return v;
}

// ---- embedding backward (owner view): workgroup = EB_ROWS table rows x EB_COLS columns of block (l, j) ----
// Token indices are scanned in chunks of 4096; the positions of a chunk that fall into the workgroup's rows are sorted by
// row, in token order within a row (counting sort: ranks from ballots, prefix sums over wavefronts and rounds).  The
// sorted list is cut into 64 consecutive parts of at least four entries, one for each group of 16 lanes; a group adds up a row's run in
// registers, a batch of rows of dX in flight at a time (a lane covers four columns), and touches the accumulators in LDS only
// where the row changes.  Runs that lie inside one part have the row to themselves in this chunk; a part's first and last
// run may continue in the neighbours' and are added in part order afterwards.  The order of all additions is a
// function of the token order alone, so the result is reproducible bit for bit.
// Bound: the workgroup that owns the most frequent rows (text: half of all tokens fall into 128 rows), one CU fetching their columns, a
// 128-byte line of bf16 each; in large tables the fixed chain of a workgroup (scan, sort, one gather), several rounds of them.
// 128 rows x 64 columns against 32 x 256 in as many workgroups: a third of the bytes and of the list on the busiest CU, four parts a
// wavefront.  Zipf tokens, bf16, us, before / now: 4096 tokens, 256 columns, v = 32768 over 4 blocks 37.1 / 18.0 (fp32 36.3 / 17.0), all tokens one
// row 81 / 26, its 16 blocks in one launch 127 / 100; 131072 tokens 1105 / 459; 1024 tokens, 16384 rows of 1024 58 / 45; 64 tokens 11.3 / 6.5.  Widths that are no multiple of four, uniform tokens over
// 500 rows, 16384 of them, fp32, 32 x 256 / 128 x 64 with adjacent columns / with every 16th: width 63 67 / 96 / 49, 127 88 / 97 / 50.
constexpr int EB_ROWS = 128, EB_COLS = 64, EB_WAVES = 16, EB_CHUNK = 4096;
constexpr int EB_LANES = EB_COLS / 4, EB_PARTS = EB_WAVES * 64 / EB_LANES;   // lanes that add up one part of the list, and parts
template <typename T>
__global__ __launch_bounds__(64 * EB_WAVES) void embedding_bwd_kernel(const int* __restrict__ tokens, const T* __restrict__ dX,
                                                                      float* __restrict__ d_table, EndArgs a) {
  constexpr int ROUNDS = EB_CHUNK / (64 * EB_WAVES), SLOTS = EB_WAVES * ROUNDS;   // slot = 64 consecutive tokens
  constexpr int RPW = EB_ROWS / EB_WAVES;
  static_assert(SLOTS == 64 && EB_ROWS == 128 && EB_PARTS == 64, "the prefix sums, the row's bits and the edges below");
  typedef unsigned long long u64;
  __shared__ __attribute__((aligned(16))) float acc[EB_ROWS * EB_COLS];
  __shared__ u64 list[EB_CHUNK];                        // row of dX (in the whole tensor) << 7 | row inside the workgroup's range
  __shared__ __attribute__((aligned(4))) unsigned short hist[SLOTS][EB_ROWS + 2];   // entries of a slot in a row; then how many lie ahead of
                                                        // them in the row; read two rows to a word
  __shared__ int row_first[EB_ROWS + 1];                // entries of a row; then where it starts in the list
  __shared__ float4 edge[2 * EB_PARTS][EB_LANES];       // sums of a part's first and last run
  __shared__ int edge_row[2 * EB_PARTS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = tid / EB_LANES, pl = tid % EB_LANES;
  const int dev = blockIdx.z;
  const int l = a.i0 + dev / a.nj, j = a.j0 + dev % a.nj;
  const int r0 = blockIdx.y * EB_ROWS;                  // first table row (inside block l) of this workgroup
  const int nr = min(EB_ROWS, a.vb - r0);
  typedef T T4 __attribute__((ext_vector_type(4)));
  const bool vec4 = a.hb % 4 == 0;                      // four columns exist or none does, and they are 8/16-byte aligned
  // a lane's four columns inside the block: adjacent ones; or, where they are loaded one by one, every 16th, so that a load of 16 lanes is one
  // piece of memory
  const int c0 = blockIdx.x * EB_COLS + (vec4 ? 4 * pl : pl), dc = vec4 ? 1 : EB_LANES;
  int col[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) col[k] = c0 + k * dc < a.hb ? c0 + k * dc : (vec4 ? k : 0);
  bool used = false;                                    // some token falls into these rows: acc is in use
  const int lo = l * a.vb + r0, hi = lo + nr;           // token indices that land in this workgroup's rows
  const long long total = (long long)a.q * a.rows;      // all tokens, grid row after grid row (below 2^31: host check)
  for (long long base = 0; base < total; base += EB_CHUNK) {
    int row[ROUNDS], rank[ROUNDS];
    int any = 0;
    for (int k = tid; k < SLOTS * (EB_ROWS + 2) / 2; k += 64 * EB_WAVES) ((unsigned*)&hist[0][0])[k] = 0;
    __syncthreads();                                    // (also: the previous chunk's list has been consumed)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const long long t = base + (wave * ROUNDS + r) * 64 + lane;
      const int tok = t < total ? clamp_token(tokens[t], a.v) : -1;
      const bool hit = tok >= lo && tok < hi;
      row[r] = hit ? tok - lo : -1;
      u64 same = __builtin_amdgcn_ballot_w64(hit);      // lanes with this lane's row
      if (same) {
        any = 1;
#pragma unroll
        for (int b = 0; b < 7; ++b) {
          const u64 one = __builtin_amdgcn_ballot_w64(hit && ((row[r] >> b) & 1));
          same &= ((row[r] >> b) & 1) ? one : ~one;
        }
        rank[r] = __builtin_popcountll(same & ((1ull << lane) - 1ull));
        if (hit && rank[r] == 0) hist[wave * ROUNDS + r][row[r]] = (unsigned short)__builtin_popcountll(same);
      }
    }
    if (!__syncthreads_or(any)) continue;               // most workgroups of a large table
    if (!used) {
      for (int k = tid; k < EB_ROWS * EB_COLS / 4; k += 64 * EB_WAVES) ((float4*)acc)[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      used = true;
    }
    {
      // two rows to a word: a chunk's entries fit 16 bits
      unsigned mine[RPW / 2];
      unsigned* const h = (unsigned*)&hist[lane][RPW * wave];
#pragma unroll
      for (int k = 0; k < RPW / 2; ++k) mine[k] = h[k];
#pragma unroll
      for (int k = 0; k < RPW / 2; ++k) {
        const unsigned incl = wave_scan(mine[k]);
        h[k] = incl - mine[k];
        if (lane == 63) { row_first[RPW * wave + 2 * k] = (int)(incl & 0xffffu); row_first[RPW * wave + 2 * k + 1] = (int)(incl >> 16); }
      }
    }
    __syncthreads();
    int n;
    {                                                   // every wavefront: lane k has rows 2k and 2k + 1
      const int even = row_first[2 * lane], odd = row_first[2 * lane + 1];
      const int incl = (int)wave_scan((unsigned)(even + odd));
      n = __builtin_amdgcn_readlane(incl, 63);
      __syncthreads();
      if (wave == 0) { row_first[2 * lane] = incl - odd - even; row_first[2 * lane + 1] = incl - odd; }
      __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
      if (row[r] >= 0) {
        const unsigned t = (unsigned)base + (wave * ROUNDS + r) * 64 + lane, i = t / (unsigned)a.rows;
        const u64 src = ((u64)i * a.q + j) * a.rows + (t - i * (unsigned)a.rows);
        list[row_first[row[r]] + hist[wave * ROUNDS + r][row[r]] + rank[r]] = src << 7 | (unsigned)row[r];
      }
    if (tid < 2 * EB_PARTS) edge_row[tid] = -1;
    __syncthreads();
    const int len = max(4, (n + EB_PARTS - 1) / EB_PARTS), q0 = min(n, part * len), q1 = min(n, q0 + len);
    // No branch between the loads of a batch, and no arithmetic on them before all are requested: columns past the block
    // are read from its first ones and never stored.
    auto add_runs = [&](auto vec_, auto batch_) {
      constexpr int BATCH = decltype(batch_)::value;
      float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
      int cur = (int)list[q0] & (EB_ROWS - 1);
      bool head = true;                                 // still in the part's first run
      for (int m0 = q0; m0 < q1; m0 += BATCH) {
        T4 x[BATCH];
        int rw[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {               // past the end: the last entry again, not added
          const u64 e = list[min(m0 + u, q1 - 1)];
          rw[u] = (int)e & (EB_ROWS - 1);
          const T* src = dX + (e >> 7) * a.hb;
          if constexpr (decltype(vec_)::value) x[u] = *(const T4*)(src + col[0]);
          else x[u] = T4{src[col[0]], src[col[1]], src[col[2]], src[col[3]]};
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const bool there = m0 + u < q1;
          if (there && rw[u] != cur) {
            if (head) {
              edge[2 * part][pl] = sum;
              if (pl == 0) edge_row[2 * part] = cur;
              head = false;
            } else {
              float4* p = (float4*)(acc + cur * EB_COLS) + pl;
              const float4 w = *p;
              *p = make_float4(w.x + sum.x, w.y + sum.y, w.z + sum.z, w.w + sum.w);
            }
            cur = rw[u];
            sum = make_float4(0.f, 0.f, 0.f, 0.f);
          }
          if (there) { sum.x += to_f32(x[u][0]); sum.y += to_f32(x[u][1]); sum.z += to_f32(x[u][2]); sum.w += to_f32(x[u][3]); }
        }
      }
      edge[2 * part + 1][pl] = sum;
      if (pl == 0) edge_row[2 * part + 1] = cur;
    };
    constexpr std::integral_constant<int, sizeof(T) == 2 ? 16 : 8> long_parts{};   // (fp32: 16 spill)
    constexpr std::integral_constant<int, 4> short_parts{};
    if (q0 < q1) {
      if (!vec4) add_runs(std::false_type{}, short_parts);
      else if (n <= 4 * EB_PARTS) add_runs(std::true_type{}, short_parts);
      else add_runs(std::true_type{}, long_parts);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {                       // in part order; wavefront k takes the rows r with r % 16 == k
      const int er = edge_row[h * 64 + lane];
      u64 todo = __builtin_amdgcn_ballot_w64(er >= 0 && (er & (EB_WAVES - 1)) == wave);
      while (todo) {
        const int at = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int r = __builtin_amdgcn_readlane(er, at);
        if (lane < EB_LANES) {
          float4* p = (float4*)(acc + r * EB_COLS) + lane;
          const float4 x = *p, y = edge[h * 64 + at][lane];
          *p = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
        }
      }
    }
  }
  __syncthreads();
  float* const out = d_table + (((long long)l * a.q + j) * a.vb + r0) * a.hb;
  if (vec4 && ((uintptr_t)out & 15) == 0) {
    for (int k = tid; k < nr * EB_LANES; k += 64 * EB_WAVES) {
      const int r = k / EB_LANES, c = blockIdx.x * EB_COLS + 4 * (k % EB_LANES);
      if (c < a.hb) *(float4*)(out + (long long)r * a.hb + c) = used ? ((const float4*)acc)[k] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return;
  }
  for (int k = tid; k < nr * EB_COLS; k += 64 * EB_WAVES) {
    const int r = k / EB_COLS, cc = k % EB_COLS, c = blockIdx.x * EB_COLS + cc;
    const int at = r * EB_COLS + (vec4 ? cc : cc % EB_LANES * 4 + cc / EB_LANES);
    if (c < a.hb) out[(long long)r * a.hb + c] = used ? acc[at] : 0.f;
  }
}

// ---- cross entropy ----
// Loss and log-sum-exp of row r of device (i, j) from the q partials of grid row i, combined in the order l = 0..q-1.
// own_l >= 0: that partial is taken from (own_m, own_s) instead of memory (same values: it has just been computed).
template <typename T>
__device__ __forceinline__ void ce_combine(const T* __restrict__ logits, const int* __restrict__ labels, const float* __restrict__ stats,
                                           float* __restrict__ loss, float* __restrict__ lse, const EndArgs& a, int i, int j,
                                           long long r, int own_l, float own_m, float own_s) {
  float m = -INFINITY;
  for (int l = 0; l < a.q; ++l) m = fmaxf(m, l == own_l ? own_m : stats[(((long long)i * a.q + l) * a.rows + r) * 2]);
  float s = 0.f;
  for (int l = 0; l < a.q; ++l) {
    const float* p = stats + (((long long)i * a.q + l) * a.rows + r) * 2;
    const float ml = l == own_l ? own_m : p[0], sl = l == own_l ? own_s : p[1];
    s += sl * __expf(ml - m);
  }
  const float L = m + __logf(s);
  const int lab = clamp_token(labels[(long long)i * a.rows + r], a.v);
  const float xl = ldf<T>(logits + ((((long long)i * a.q + lab / a.vb) * a.rows + r) * a.vb + lab % a.vb));
  const long long o = ((long long)i * a.q + j) * a.rows + r;
  lse[o] = L;
  loss[o] = L - xl;
}

// partial statistics of one block: (max, sum exp(x - max)) per row; one wavefront per row.  FINAL: the peers'
// partials are already in memory (one device recomputed from resident peers), so the row is finished here.
// WIDE: a whole workgroup per row (its four wavefronts take interleaved 16-byte chunks and their partials are
// combined in wavefront order through LDS): long rows need more loads in flight than one wavefront per SIMD gives.
template <typename T, bool FINAL, bool WIDE>
__global__ __launch_bounds__(256) void ce_stats_kernel(const T* __restrict__ logits, float* __restrict__ stats,
                                                       const int* __restrict__ labels, float* __restrict__ loss,
                                                       float* __restrict__ lse, EndArgs a) {
  __shared__ float part[8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long r = WIDE ? (long long)blockIdx.x : (long long)blockIdx.x * 4 + wave;
  if (r >= a.rows) return;   // (WIDE: the same for the whole workgroup)
  const int first = WIDE ? wave * 64 + lane : lane, step = WIDE ? 256 : 64;
  const int dev = blockIdx.y;
  const int i = a.i0 + dev / a.nj, j = a.j0 + dev % a.nj;
  const long long blk = (long long)i * a.q + j;
  const T* src = logits + (blk * a.rows + r) * a.vb;
  float m = -INFINITY, s = 0.f;
  constexpr int VN = V16<T>::N;
  if (a.vb % VN == 0) {   // 16-byte loads: a chunk's maximum first, then one rescale per chunk
    for (int c = first * VN; c < a.vb; c += step * VN) {
      float f[VN];
      V16<T>::load(src + c, f);
      float cm = f[0];
#pragma unroll
      for (int k = 1; k < VN; ++k) cm = fmaxf(cm, f[k]);
      if (cm > m) { s *= __expf(m - cm); m = cm; }            // exp(-inf - x) = 0 on the first chunk (s is 0 then)
      if (m > -INFINITY) {
#pragma unroll
        for (int k = 0; k < VN; ++k) s += __expf(f[k] - m);
      }
    }
  } else {
    for (int c = first; c < a.vb; c += step) {
      const float x = ldf<T>(src + c);
      if (x > m) { s = s * __expf(m - x) + 1.0f; m = x; }
      else if (m > -INFINITY) s += __expf(x - m);             // (a row of -inf entries contributes nothing)
    }
  }
  float mw = wave_max_f(m);
  s = wave_sum_f(m == -INFINITY ? 0.f : s * __expf(m - mw));
  if (WIDE) {
    if (lane == 0) { part[wave] = mw; part[4 + wave] = s; }
    __syncthreads();
    if (wave != 0) return;
    mw = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    s = 0.f;
    for (int w = 0; w < 4; ++w) s += part[w] == -INFINITY ? 0.f : part[4 + w] * __expf(part[w] - mw);
  }
  if (lane == 0) {
    stats[(blk * a.rows + r) * 2] = mw;
    stats[(blk * a.rows + r) * 2 + 1] = s;
    if (FINAL) ce_combine<T>(logits, labels, stats, loss, lse, a, i, j, r, j, mw, s);
  }
}

// combine the q partials of a grid row in the order l = 0..q-1; loss and log-sum-exp per row of device (i, j)
template <typename T>
__global__ __launch_bounds__(256) void ce_finalize_kernel(const T* __restrict__ logits, const int* __restrict__ labels,
                                                          const float* __restrict__ stats, float* __restrict__ loss,
                                                          float* __restrict__ lse, EndArgs a) {
  const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
  if (r >= a.rows) return;
  const int dev = blockIdx.y;
  const int i = a.i0 + dev / a.nj, j = a.j0 + dev % a.nj;
  ce_combine<T>(logits, labels, stats, loss, lse, a, i, j, r, -1, 0.f, 0.f);
}

// d_logits = scale * (exp(x - L) - [column == label]); one wavefront per row of a block
template <typename T>
__global__ __launch_bounds__(256) void ce_bwd_kernel(const T* __restrict__ logits, const int* __restrict__ labels,
                                                     const float* __restrict__ lse, T* __restrict__ d_logits, float scale, EndArgs a) {
  const int lane = threadIdx.x & 63;
  const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= a.rows) return;
  const int dev = blockIdx.y;
  const int i = a.i0 + dev / a.nj, j = a.j0 + dev % a.nj;
  const long long blk = (long long)i * a.q + j;
  const T* src = logits + (blk * a.rows + r) * a.vb;
  T* dst = d_logits + (blk * a.rows + r) * a.vb;
  const float L = lse[blk * a.rows + r];
  const int lab = clamp_token(labels[(long long)i * a.rows + r], a.v) - j * a.vb;   // label column inside this block, if any
  constexpr int VN = V16<T>::N;
  if (a.vb % VN == 0) {
    for (int c = lane * VN; c < a.vb; c += 64 * VN) {
      float f[VN];
      V16<T>::load(src + c, f);
#pragma unroll
      for (int k = 0; k < VN; ++k) f[k] = scale * (__expf(f[k] - L) - (c + k == lab ? 1.0f : 0.0f));
      V16<T>::store(dst + c, f);
    }
  } else {
    for (int c = lane; c < a.vb; c += 64) {
      const float qv = __expf(ldf<T>(src + c) - L);
      stf<T>(dst + c, scale * (qv - (c == lab ? 1.0f : 0.0f)));
    }
  }
}

}  // namespace

namespace {
template <bool FINAL>
int ce_stats_dispatch(const void* logits, float* stats, const int* labels, float* loss, float* lse, const EndDesc& d,
                      const EndArgs& a, hipStream_t st) {
  const bool wide = d.vb >= 2048;   // a workgroup per row from 2048 columns per block on
  const dim3 grid(wide ? d.rows : (d.rows + 3) / 4, d.ni * d.nj);
  if (d.dtype == OPTIMUS_BF16) {
    if (wide) ce_stats_kernel<bf16_t, FINAL, true><<<grid, 256, 0, st>>>((const bf16_t*)logits, stats, labels, loss, lse, a);
    else ce_stats_kernel<bf16_t, FINAL, false><<<grid, 256, 0, st>>>((const bf16_t*)logits, stats, labels, loss, lse, a);
  } else {
    if (wide) ce_stats_kernel<float, FINAL, true><<<grid, 256, 0, st>>>((const float*)logits, stats, labels, loss, lse, a);
    else ce_stats_kernel<float, FINAL, false><<<grid, 256, 0, st>>>((const float*)logits, stats, labels, loss, lse, a);
  }
  return hip_launch_status();
}
}  // namespace

int launch_embedding_fwd(const int* tokens, const void* table, void* out, const EndDesc& d, hipStream_t st) {
  EndArgs a = {d.rows, d.vb, d.hb, d.q, d.v, d.i0, d.ni, d.j0, d.nj};
  const dim3 grid((d.rows + 3) / 4, d.ni * d.nj);
  if (d.dtype == OPTIMUS_BF16) embedding_fwd_kernel<bf16_t><<<grid, 256, 0, st>>>(tokens, (const bf16_t*)table, (bf16_t*)out, a);
  else embedding_fwd_kernel<float><<<grid, 256, 0, st>>>(tokens, (const float*)table, (float*)out, a);
  return hip_launch_status();
}
int launch_embedding_bwd(const int* tokens, const void* dX, float* d_table, const EndDesc& d, hipStream_t st) {
  EndArgs a = {d.rows, d.vb, d.hb, d.q, d.v, d.i0, d.ni, d.j0, d.nj};
  const dim3 grid((d.hb + EB_COLS - 1) / EB_COLS, (d.vb + EB_ROWS - 1) / EB_ROWS, d.ni * d.nj);
  if ((d.vb + 31) / 32 > 65535 || grid.z > 65535) return OPTIMUS_ESHAPE;   // blocks of at most 2 Mi rows
  if (d.dtype == OPTIMUS_BF16) embedding_bwd_kernel<bf16_t><<<grid, 64 * EB_WAVES, 0, st>>>(tokens, (const bf16_t*)dX, d_table, a);
  else embedding_bwd_kernel<float><<<grid, 64 * EB_WAVES, 0, st>>>(tokens, (const float*)dX, d_table, a);
  return hip_launch_status();
}
int launch_ce_stats(const void* logits, float* stats, const EndDesc& d, hipStream_t st) {
  EndArgs a = {d.rows, d.vb, d.hb, d.q, d.v, d.i0, d.ni, d.j0, d.nj};
  return ce_stats_dispatch<false>(logits, stats, nullptr, nullptr, nullptr, d, a, st);
}
// one device whose peers' partials are resident: statistics and finish in one launch
int launch_ce_stats_final(const void* logits, const int* labels, float* stats, float* loss, float* lse, const EndDesc& d,
                          hipStream_t st) {
  EndArgs a = {d.rows, d.vb, d.hb, d.q, d.v, d.i0, d.ni, d.j0, d.nj};
  return ce_stats_dispatch<true>(logits, stats, labels, loss, lse, d, a, st);
}
int launch_ce_finalize(const void* logits, const int* labels, const float* stats, float* loss, float* lse, const EndDesc& d,
                       hipStream_t st) {
  EndArgs a = {d.rows, d.vb, d.hb, d.q, d.v, d.i0, d.ni, d.j0, d.nj};
  const dim3 grid((d.rows + 255) / 256, d.ni * d.nj);
  if (d.dtype == OPTIMUS_BF16) ce_finalize_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t*)logits, labels, stats, loss, lse, a);
  else ce_finalize_kernel<float><<<grid, 256, 0, st>>>((const float*)logits, labels, stats, loss, lse, a);
  return hip_launch_status();
}
int launch_ce_bwd(const void* logits, const int* labels, const float* lse, void* d_logits, float scale, const EndDesc& d,
                  hipStream_t st) {
  EndArgs a = {d.rows, d.vb, d.hb, d.q, d.v, d.i0, d.ni, d.j0, d.nj};
  const dim3 grid((d.rows + 3) / 4, d.ni * d.nj);
  if (d.dtype == OPTIMUS_BF16)
    ce_bwd_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t*)logits, labels, lse, (bf16_t*)d_logits, scale, a);
  else ce_bwd_kernel<float><<<grid, 256, 0, st>>>((const float*)logits, labels, lse, (float*)d_logits, scale, a);
  return hip_launch_status();
}

}  // namespace optimus
