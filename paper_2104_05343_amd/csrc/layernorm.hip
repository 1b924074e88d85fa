// 2D LayerNorm (Section 3.2.2 of the paper): a row of the hidden dimension is spread over the q devices of a
// grid row; each device sums x and x^2 over its own h/q columns, the q partials are added (the row
// all-reduce), and the device normalises its own block.  Backward treats (sum xhat*g, sum g) the same way.
//
// One wavefront owns one row of a block: the row (<= 2048 columns on the fast path) is read once with
// 16-byte loads, kept in registers, reduced with DPP-free shuffles, and written once.  Wider or unaligned
// rows take a scalar path that re-reads the row.  Statistics are fp32; partials are always added in the
// order l = 0..q-1 so that every device of a row, and grid and device mode, get identical bits.
#include "combine.hpp"

namespace optimus {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

constexpr int LN_MAXCH = 4;  // 16-byte chunks per lane on the fast path (bf16: 8 elems, fp32: 4 elems)

template <typename T> struct Vec;
template <> struct Vec<bf16_t> {
  static constexpr int N = 8;
  __device__ static void load(const bf16_t* p, float* f) {
    uint4 w = *(const uint4*)p;
    unsigned u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { f[2 * k] = __uint_as_float(u[k] << 16); f[2 * k + 1] = __uint_as_float(u[k] & 0xffff0000u); }
  }
  __device__ static void store(bf16_t* p, const float* f) {
    *(uint4*)p = make_uint4(pack2_bf16(f[0], f[1]), pack2_bf16(f[2], f[3]), pack2_bf16(f[4], f[5]), pack2_bf16(f[6], f[7]));
  }
  __device__ static float ld1(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ static void st1(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};
template <> struct Vec<float> {
  static constexpr int N = 4;
  __device__ static void load(const float* p, float* f) { float4 w = *(const float4*)p; f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w; }
  __device__ static void store(float* p, const float* f) { *(float4*)p = make_float4(f[0], f[1], f[2], f[3]); }
  __device__ static float ld1(const float* p) { return *p; }
  __device__ static void st1(float* p, float v) { *p = v; }
};

// The partial tiles of the product that makes X (MODE 3): [splits][blocks of the launch][rows][cols], stride elements from one split to
// the next; the sum, rounded, is X, and is stored there.
struct LnPartials {
  const float* p;
  int splits;
  long long stride;
};

struct LnArgs {
  int rows, cols, H, q;
  int i0, ni, j0, nj;
  float eps;
  int vec;  // fast path allowed
};

// eight columns of X: the splits' sum in their order (as combine_vec adds them), rounded; four splits' loads in flight
__device__ __forceinline__ void ln_sum_partials(const float* p, const LnPartials& part, bf16_t* x, float* v) {
  float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < part.splits; s0 += 4) {
    float4 w[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float* ps = p + (s0 + s < part.splits ? s0 + s : part.splits - 1) * part.stride;
      w[s][0] = *(const float4*)ps; w[s][1] = *(const float4*)(ps + 4);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (s0 + s < part.splits)
#pragma unroll
        for (int h = 0; h < 2; ++h) { t[4 * h] += w[s][h].x; t[4 * h + 1] += w[s][h].y; t[4 * h + 2] += w[s][h].z; t[4 * h + 3] += w[s][h].w; }
  }
  const uint4 u = make_uint4(pack2_bf16(t[0], t[1]), pack2_bf16(t[2], t[3]), pack2_bf16(t[4], t[5]), pack2_bf16(t[6], t[7]));
  *(uint4*)x = u;
  const unsigned k[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[2 * i] = __uint_as_float(k[i] << 16); v[2 * i + 1] = __uint_as_float(k[i] & 0xffff0000u); }
}

// MODE 0: forward stats only.  MODE 1: forward apply (own partial computed here unless own_ready).
// MODE 2: backward stats only. MODE 3: backward apply.
// RG ("row group", MODE 1 and 3, whole grid rows only): a workgroup holds the q wavefronts that own the q segments of
// the same logical row (times a few rows), each computes its partial, the partials meet in LDS, and every
// wavefront adds them in the order l = 0..q-1: the same numbers in the same order as the two-kernel form
// (statistics kernel, then apply with own_ready), in one pass over the input.  The partials are still written
// to `stats`, which device-mode calls of the peers read.
// PART (MODE 3, bf16, vector path): X does not exist yet, its product's partial tiles do (LnPartials).  A launch less, and X is read from
// registers instead of memory: blocks of [1024 x 256], four ranges, 3.7 (combine) and 4.6 us before, now 5.4.
template <typename T, int MODE, bool RG = false, bool PART = false>
__global__ __launch_bounds__(RG ? 1024 : 256) void ln_kernel(const T* __restrict__ X, const T* __restrict__ X2, const float* __restrict__ gamma,
                                                 const float* __restrict__ beta, const float* __restrict__ rstd_in,
                                                 const T* __restrict__ dres, T* __restrict__ Y, T* __restrict__ xhat_out,
                                                 float* __restrict__ rstd_out, float* __restrict__ stats, LnArgs a, int own_ready, LnPartials part) {
  static_assert(!PART || (MODE == 3 && sizeof(T) == 2), "partial tiles: the backward pass, bf16");
  constexpr int VN = Vec<T>::N;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int dev = blockIdx.y;
  // RG: wavefront = (row of the workgroup, segment dj); the host launches whole workgroups only (no partial last one)
  const int di = RG ? a.i0 + dev : a.i0 + dev / a.nj;
  const int dj = RG ? wave % a.q : a.j0 + dev % a.nj;
  const int row = RG ? blockIdx.x * ((int)(blockDim.x >> 6) / a.q) + wave / a.q : blockIdx.x * 4 + wave;
  if (row >= a.rows) return;
  const long long blk = (long long)a.rows * a.cols;
  const long long base = ((long long)di * a.q + dj) * blk + (long long)row * a.cols;
  const T* x = X + base;                    // forward: x ; backward: dy
  const T* x2 = X2 ? X2 + base : nullptr;   // backward: xhat
  const float* gm = gamma ? gamma + (long long)dj * a.cols : nullptr;
  const float* bt = beta ? beta + (long long)dj * a.cols : nullptr;
  float* st_row = stats + ((long long)di * a.q * a.rows + row) * 2;  // + l*rows*2 selects device (di, l)
  const long long st_dev = (long long)a.rows * 2;

  float v[LN_MAXCH * VN];   // forward: x ; backward: g = dy*gamma
  float w[LN_MAXCH * VN];   // backward: xhat
  float s0 = 0.f, s1 = 0.f;
  const bool need_own = !(own_ready && (MODE == 1 || MODE == 3));
  if (a.vec) {
#pragma unroll
    for (int c = 0; c < LN_MAXCH; ++c) {
      int col = (c * 64 + lane) * VN;
      if (col < a.cols) {
        if constexpr (PART) ln_sum_partials(part.p + (RG ? base : (long long)row * a.cols) + col, part, const_cast<T*>(x) + col, v + c * VN);
        else Vec<T>::load(x + col, v + c * VN);
        if (MODE >= 2) {
          Vec<T>::load(x2 + col, w + c * VN);
#pragma unroll
          for (int k = 0; k < VN; ++k) { v[c * VN + k] *= gm[col + k]; s0 += w[c * VN + k] * v[c * VN + k]; s1 += v[c * VN + k]; }
        } else {
#pragma unroll
          for (int k = 0; k < VN; ++k) { s0 += v[c * VN + k]; s1 += v[c * VN + k] * v[c * VN + k]; }
        }
      }
    }
  } else if (need_own) {
    for (int col = lane; col < a.cols; col += 64) {
      float t = Vec<T>::ld1(x + col);
      if (MODE >= 2) { float g = t * gm[col]; s0 += Vec<T>::ld1(x2 + col) * g; s1 += g; }
      else { s0 += t; s1 += t * t; }
    }
  }
  float own0 = 0.f, own1 = 0.f;
  if (need_own) {
    own0 = wave_sum(s0);
    own1 = wave_sum(s1);
    if (lane == 0) { st_row[dj * st_dev] = own0; st_row[dj * st_dev + 1] = own1; }
  }
  if (MODE == 0 || MODE == 2) return;

  // add the q partials of this grid row in fixed order (own partial from registers when computed here)
  float t0 = 0.f, t1 = 0.f;
  if constexpr (RG) {
    __shared__ float part[16][2];
    if (lane == 0) { part[wave][0] = own0; part[wave][1] = own1; }
    __syncthreads();
    const int w0 = wave - dj;  // first wavefront of this row
    for (int l = 0; l < a.q; ++l) { t0 += part[w0 + l][0]; t1 += part[w0 + l][1]; }
  } else {
    for (int l = 0; l < a.q; ++l) {
      float p0, p1;
      if (l == dj && need_own) { p0 = own0; p1 = own1; }
      else { p0 = st_row[l * st_dev]; p1 = st_row[l * st_dev + 1]; }
      t0 += p0; t1 += p1;
    }
  }
  const float invH = 1.0f / (float)a.H;
  if (MODE == 1) {
    float mean = t0 * invH;
    float var = fmaxf(t1 * invH - mean * mean, 0.f);
    float rstd = 1.0f / sqrtf(var + a.eps);
    if (lane == 0) rstd_out[((long long)di * a.q + dj) * a.rows + row] = rstd;
    T* y = Y + base;
    T* xh = xhat_out + base;
    if (a.vec) {
#pragma unroll
      for (int c = 0; c < LN_MAXCH; ++c) {
        int col = (c * 64 + lane) * VN;
        if (col < a.cols) {
          float o[VN], h[VN];
#pragma unroll
          for (int k = 0; k < VN; ++k) { h[k] = (v[c * VN + k] - mean) * rstd; o[k] = h[k] * gm[col + k] + bt[col + k]; }
          Vec<T>::store(xh + col, h);
          Vec<T>::store(y + col, o);
        }
      }
    } else {
      for (int col = lane; col < a.cols; col += 64) {
        float h = (Vec<T>::ld1(x + col) - mean) * rstd;
        Vec<T>::st1(xh + col, h);
        Vec<T>::st1(y + col, h * gm[col] + bt[col]);
      }
    }
  } else {  // MODE 3
    float rstd = rstd_in[((long long)di * a.q + dj) * a.rows + row];
    float mxg = t0 * invH, mg = t1 * invH;
    T* dx = Y + base;
    const T* dr = dres ? dres + base : nullptr;
    if (a.vec) {
#pragma unroll
      for (int c = 0; c < LN_MAXCH; ++c) {
        int col = (c * 64 + lane) * VN;
        if (col < a.cols) {
          float o[VN], r[VN];
          if (dr) Vec<T>::load(dr + col, r);
#pragma unroll
          for (int k = 0; k < VN; ++k) {
            o[k] = rstd * (v[c * VN + k] - w[c * VN + k] * mxg - mg);
            if (dr) o[k] += r[k];
          }
          Vec<T>::store(dx + col, o);
        }
      }
    } else {
      for (int col = lane; col < a.cols; col += 64) {
        float g = Vec<T>::ld1(x + col) * gm[col];
        float o = rstd * (g - Vec<T>::ld1(x2 + col) * mxg - mg);
        if (dr) o += Vec<T>::ld1(dr + col);
        Vec<T>::st1(dx + col, o);
      }
    }
  }
}

static LnArgs make_args(const LnDesc& d, bool ptr_ok, int elem_bytes) {
  LnArgs a;
  a.rows = d.rows; a.cols = d.cols; a.H = d.H; a.q = d.q;
  a.i0 = d.i0; a.ni = d.ni; a.j0 = d.j0; a.nj = d.nj;
  a.eps = d.eps;
  int vn = 16 / elem_bytes;
  a.vec = ptr_ok && (d.cols % vn == 0) && (d.cols <= LN_MAXCH * 64 * vn);
  return a;
}
static bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// rows of one workgroup of the row-group form: q wavefronts per row, four wavefronts or more per workgroup
static int ln_rowgroup_rows(const LnDesc& d) {
  int r = d.q >= 4 ? 1 : 4 / d.q;
  while (r > 1 && d.rows % r) r >>= 1;
  return r;
}
// the call covers whole grid rows (every segment of a logical row), and q wavefronts fit a workgroup
bool ln_rowgroup_ok(const LnDesc& d) { return d.j0 == 0 && d.nj == d.q && d.q >= 1 && d.q <= 16; }

template <typename T, int MODE>
static int run(const void* X, const void* X2, const float* gamma, const float* beta, const float* rstd_in, const void* dres,
               void* Y, void* xhat, float* rstd_out, float* stats, const LnDesc& d, bool own_ready, hipStream_t stream) {
  const LnPartials none = {};
  bool ok = al16(X) && (!X2 || al16(X2)) && (!dres || al16(dres)) && (!Y || al16(Y)) && (!xhat || al16(xhat)) &&
            (!gamma || al16(gamma)) && (!beta || al16(beta));
  LnArgs a = make_args(d, ok, (int)sizeof(T));
  if constexpr (MODE == 1 || MODE == 3) {
    if (!own_ready && ln_rowgroup_ok(d)) {
      const int rpw = ln_rowgroup_rows(d);
      dim3 grid((unsigned)(d.rows / rpw), (unsigned)d.ni);
      hipLaunchKernelGGL((ln_kernel<T, MODE, true>), grid, dim3(64 * d.q * rpw), 0, stream, (const T*)X, (const T*)X2, gamma, beta,
                         rstd_in, (const T*)dres, (T*)Y, (T*)xhat, rstd_out, stats, a, 0, none);
      return hip_launch_status();
    }
  }
  dim3 grid((unsigned)((d.rows + 3) / 4), (unsigned)(d.ni * d.nj));
  hipLaunchKernelGGL((ln_kernel<T, MODE>), grid, dim3(256), 0, stream, (const T*)X, (const T*)X2, gamma, beta, rstd_in,
                     (const T*)dres, (T*)Y, (T*)xhat, rstd_out, stats, a, own_ready ? 1 : 0, none);
  return hip_launch_status();
}

#define LN_DISPATCH(MODE, ...)                                              \
  (d.dtype == OPTIMUS_BF16 ? run<bf16_t, MODE>(__VA_ARGS__) : run<float, MODE>(__VA_ARGS__))

int launch_ln_stats(const void* X, float* stats, const LnDesc& d, hipStream_t stream) {
  return LN_DISPATCH(0, X, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, stats, d, false, stream);
}
int launch_ln_apply(const void* X, const float* gamma, const float* beta, void* Y, void* xhat, float* rstd, float* stats,
                    const LnDesc& d, bool own_ready, hipStream_t stream) {
  return LN_DISPATCH(1, X, nullptr, gamma, beta, nullptr, nullptr, Y, xhat, rstd, stats, d, own_ready, stream);
}
int launch_ln_bwd_stats(const void* dY, const void* xhat, const float* gamma, float* stats, const LnDesc& d, hipStream_t stream) {
  return LN_DISPATCH(2, dY, xhat, gamma, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, stats, d, false, stream);
}
int launch_ln_bwd_apply(const void* dY, const void* xhat, const float* rstd, const float* gamma, const void* dres, void* dX,
                        float* stats, const LnDesc& d, bool own_ready, hipStream_t stream) {
  return LN_DISPATCH(3, dY, xhat, gamma, nullptr, rstd, dres, dX, nullptr, nullptr, stats, d, own_ready, stream);
}

bool ln_bwd_partials_ok(const CombineJob& j, const void* dY, const void* xhat, const float* gamma, const void* dres, const void* dX,
                        const LnDesc& d) {
  const EpiArgs& e = j.epi;
  const long long first = ((long long)d.i0 * d.q + d.j0) * d.rows * d.cols;
  if (!j.vec || d.dtype != OPTIMUS_BF16 || e.C != (const bf16_t*)dY + first || e.alpha != 1.0f || e.bias || e.pre_act || e.act || e.gelu_grad_of || e.residual || e.out_fp32)
    return false;
  const bool grid = ln_rowgroup_ok(d);
  if (j.Mb != d.rows || j.Nb != d.cols || e.ldc != d.cols || j.nz != (grid ? (long long)d.ni * d.nj : 1) || (!grid && d.ni * d.nj != 1)) return false;
  if (grid && (d.i0 != 0 || d.ni != d.q)) return false;
  if (grid && j.nz > 1 && (j.sC0 != (long long)d.rows * d.cols || j.sC1 != j.sC0 * d.q || j.nz0 != d.q)) return false;
  return make_args(d, al16(e.C) && al16(xhat) && al16(gamma) && (!dres || al16(dres)) && al16(dX), 2).vec;
}
int launch_ln_bwd_partials(const CombineJob& j, const void* xhat, const float* rstd, const float* gamma, const void* dres, void* dX, float* stats,
                           const LnDesc& d, hipStream_t stream) {
  const LnArgs a = make_args(d, true, 2);
  const LnPartials part = {j.partials, j.splits, j.nz * j.Mb * (long long)j.Nb};
  // the epilogue's C is the first block of the launch, the kernel's X the grid's first
  const long long first = ((long long)d.i0 * d.q + d.j0) * d.rows * d.cols;
  const bf16_t* X = (const bf16_t*)j.epi.C - first;
  if (ln_rowgroup_ok(d)) {
    const int rpw = ln_rowgroup_rows(d);
    hipLaunchKernelGGL((ln_kernel<bf16_t, 3, true, true>), dim3((unsigned)(d.rows / rpw), (unsigned)d.ni), dim3(64 * d.q * rpw), 0, stream, X,
                       (const bf16_t*)xhat, gamma, (const float*)nullptr, rstd, (const bf16_t*)dres, (bf16_t*)dX, (bf16_t*)nullptr, (float*)nullptr, stats, a, 0, part);
  } else {
    hipLaunchKernelGGL((ln_kernel<bf16_t, 3, false, true>), dim3((unsigned)((d.rows + 3) / 4)), dim3(256), 0, stream, X, (const bf16_t*)xhat, gamma,
                       (const float*)nullptr, rstd, (const bf16_t*)dres, (bf16_t*)dX, (bf16_t*)nullptr, (float*)nullptr, stats, a, 0, part);
  }
  return hip_launch_status();
}

// ---- column sums over the rows of a block: dgamma/dbeta partials, bias gradients ----
// ROWS = 128 or 256 row lanes; a row lane accumulates 8 adjacent columns (16-byte loads) over rows y, y + ROWS, ...  Groups of
// eight row lanes are added by butterfly exchanges, the groups through LDS in order (256 row lanes: group r and group r + 16
// first).  A workgroup covers CL column lanes; a thread is PER row lanes: one, or y and y + ROWS / 2.
// Bound: memory round trips, CUs and loads in flight, not bytes.  The blocks have thousands of rows and a few hundred to a few
// thousand columns, so strips of whole 128-byte lines (CL = 8) give 4 to 64 workgroups, each with a long chain of loads, and
// strips of 8 columns (CL = 1) fetch every line eight times (the strips that share a line run on the same XCD, one after the
// other in its range, and find it in its L2).  The order of the additions depends on ROWS but not on CL: ROWS follows the
// block's shape and CL the launch, and a launch over many blocks gets the same bits as one over a single block.
// Measured, us, bf16, ROWS and CL of 128 and 8, 128 and 1 / as chosen below: [1024 x 256] 4.7, 4.2 / 4.1, 16 blocks of it 4.9,
// 5.2 / 4.4, 16 of [1024 x 1024] 5.6, 11.5 / 5.6, [4096 x 512] 8.7, 8.5 / 5.8, [4096 x 2048] 8.7, 10.8 / 6.6, 16 of [8192 x 64]
// 14.2, 30.0 / 10.8, [32768 x 4096] 101, 109 / 69, [1000 x 250] 12.7, 13.6 / 6.7.  fp32 [1024 x 256] 4.5, 3.7 / 3.7, with products
// 5.1, 3.3 / 3.3.
template <typename T>
__device__ __forceinline__ void cs_load(const T* p, float (&f)[8]) {
  Vec<T>::load(p, f);
  if constexpr (sizeof(T) == 4) Vec<T>::load(p + 4, f + 4);
}
// v: eight columns summed over this lane's rows.  Returns column k = cs_column(lane) summed over the eight row lanes of the
// group: three exchanges that halve the columns a lane is in charge of.
template <int CL>
__device__ __forceinline__ float cs_group(float (&v)[8], int lane) {
#pragma unroll
  for (int half = 4, d = CL; half > 0; half >>= 1, d <<= 1) {
    const bool up = lane & d;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const float give = up ? v[k] : v[k + half], keep = up ? v[k + half] : v[k];
      v[k] = keep + __shfl_xor(give, d, 64);
    }
  }
  return v[0];
}
template <int CL>
__device__ __forceinline__ int cs_column(int lane) {   // the group's row-lane bits, lowest first, are the column's, highest first
  const int g = lane / CL;
  return ((g & 1) << 2) | (g & 2) | ((g >> 2) & 1);
}
// one row's 8 columns from c0 on
template <typename T, bool PROD>
__device__ __forceinline__ void cs_add(float (&acc)[8], float (&acc2)[8], const T* __restrict__ X, const T* __restrict__ W, long long off,
                                       bool vec, int c0, int cols) {
  float x[8], w[8];
  if (vec) {
    cs_load(X + off, x);
    if (PROD) cs_load(W + off, w);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      bool in = c0 + k < cols;
      x[k] = in ? Vec<T>::ld1(X + off + k) : 0.f;
      if (PROD) w[k] = in ? Vec<T>::ld1(W + off + k) : 0.f;
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    acc[k] += x[k];                      // sum x           (dbeta / bias gradient)
    if (PROD) acc2[k] += x[k] * w[k];    // sum x*w         (dgamma)
  }
}
// one strip of one block
template <typename T, bool PROD, int ROWS, int CL, int PER>
__device__ __forceinline__ void colsum_strip(const T* __restrict__ X, const T* __restrict__ W, float* __restrict__ out, float* __restrict__ out2,
                                             int rows, int cols, int ld, int strip, bool vec_rows, float (&red)[ROWS / 8][8 * CL],
                                             float (&red2)[ROWS / 8][8 * CL]) {
  constexpr int CS_COLS = 8 * CL, GROUPS = ROWS / 8;
  const int tx = threadIdx.x & (CL - 1), ty = threadIdx.x / CL;
  const int lane = threadIdx.x & 63;
  const int c0 = strip * CS_COLS + tx * 8;
  float acc[8], acc2[8], bcc[8], bcc2[8];   // bcc: the thread's second row lane
#pragma unroll
  for (int k = 0; k < 8; ++k) { acc[k] = 0.f; acc2[k] = 0.f; bcc[k] = 0.f; bcc2[k] = 0.f; }
  const bool vec = vec_rows && c0 + 8 <= cols;
  constexpr int LANES = ROWS / PER;
  constexpr int IN_FLIGHT = (PROD || (ROWS == 256 && CL == 4) ? 4 : 8) / PER;   // (256 x 4 with eight: 22 us instead of 14)
  int r = ty;
#pragma unroll IN_FLIGHT
  for (; r + (PER - 1) * LANES < rows; r += ROWS) {
    const long long off = (long long)r * ld + c0;
    cs_add<T, PROD>(acc, acc2, X, W, off, vec, c0, cols);
    if constexpr (PER == 2) {
      cs_add<T, PROD>(bcc, bcc2, X, W, off + (long long)LANES * ld, vec, c0, cols);
    }
  }
  if (PER == 2 && r < rows) {
    const long long off = (long long)r * ld + c0;
    cs_add<T, PROD>(acc, acc2, X, W, off, vec, c0, cols);
  }
  const int k = cs_column<CL>(lane);
  red[ty >> 3][tx * 8 + k] = cs_group<CL>(acc, lane);
  if (PROD) red2[ty >> 3][tx * 8 + k] = cs_group<CL>(acc2, lane);
  if constexpr (PER == 2) {
    red[(ty + LANES) >> 3][tx * 8 + k] = cs_group<CL>(bcc, lane);
    if (PROD) red2[(ty + LANES) >> 3][tx * 8 + k] = cs_group<CL>(bcc2, lane);
  }
  __syncthreads();
  if (threadIdx.x < CS_COLS) {
    int c = strip * CS_COLS + threadIdx.x;
    if (c < cols) {
      float s = 0.f, s2 = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s += GROUPS == 16 ? red[r][threadIdx.x] : red[r][threadIdx.x] + red[r + GROUPS - 16][threadIdx.x];
        if (PROD) s2 += GROUPS == 16 ? red2[r][threadIdx.x] : red2[r][threadIdx.x] + red2[r + GROUPS - 16][threadIdx.x];
      }
      out[c] = s;
      if (PROD) out2[c] = s2;
    }
  }
}
// workgroups are dealt round-robin to the 8 XCDs: a contiguous range of strips each (whatever XCD the entry starts on), unless
// a strip is whole lines, which no other shares
template <int CL>
__device__ __forceinline__ int cs_place(int wg, int nwg) {
  if (CL == 8) return wg;
  const int slot = wg >> 3, xcd = wg & 7, rem = nwg & 7;
  return xcd * (nwg >> 3) + (xcd < rem ? xcd : rem) + slot;
}
template <typename T, bool PROD, int ROWS, int CL, int PER>
__global__ __launch_bounds__(ROWS / PER * CL) void colsum_kernel(const T* __restrict__ X, const T* __restrict__ W, float* __restrict__ out,
                                                              float* __restrict__ out2, int rows, int cols, int ld, long long sX,
                                                              long long sOut) {
  __shared__ float red[ROWS / 8][8 * CL];
  __shared__ float red2[ROWS / 8][8 * CL];
  const bool vec_rows = (ld % 8 == 0) && (sX % 8 == 0) && (((uintptr_t)X & 15) == 0) && (!PROD || ((uintptr_t)W & 15) == 0);
  const long long zx = (long long)blockIdx.y * sX, zo = (long long)blockIdx.y * sOut;
  colsum_strip<T, PROD, ROWS, CL, PER>(X + zx, PROD ? W + zx : nullptr, out + zo, PROD ? out2 + zo : nullptr, rows, cols, ld, cs_place<CL>(blockIdx.x, gridDim.x), vec_rows, red, red2);
}
// Several sums in one launch: a layer's vector gradients, whose sources all live until the end of the backward pass.  As six
// launches of 4 to 7 us each, the step of a 1024-wide layer (one device of 4 x 4) takes 250 us, as one 219; of two small
// checkpointed layers on a 2 x 2 grid 362 and 328; of a 1280-wide layer with cut tiles 328 and 292 (four sums, on the branch).
// The combines of panel splits that nothing of the pass waits for (a layer's weight gradients) ride behind them in the same grid:
// 7.9 us for the sums and 15 for four combines of a 1024-wide layer (one device of 4 x 4) before, now 9.6 together.
template <int ROWS, int CL, int PER>
__global__ __launch_bounds__(ROWS / PER * CL) void colsum_jobs_kernel(const ColsumJobs jobs, int rows, unsigned strips, unsigned sums,
                                                                      const CombineJobs combines) {
  __shared__ float red[ROWS / 8][8 * CL];
  __shared__ float red2[ROWS / 8][8 * CL];
  if (blockIdx.x >= sums) {
    unsigned wg = blockIdx.x - sums;
    int k = 0;
    while (k + 1 < combines.n && wg >= combines.blocks[k]) wg -= combines.blocks[k++];
    combine_quad_vec(combines.j[k], wg * (ROWS / PER * CL) + threadIdx.x);
    return;
  }
  const unsigned z = blockIdx.x / strips;
  int strip = cs_place<CL>(blockIdx.x - z * strips, strips), k = 0;
  while (k + 1 < jobs.n && strip >= (jobs.j[k].cols + 8 * CL - 1) / (8 * CL)) strip -= (jobs.j[k++].cols + 8 * CL - 1) / (8 * CL);
  const ColsumJob& j = jobs.j[k];
  const long long zx = (long long)z * rows * j.cols, zo = (long long)z * j.cols;
  const bf16_t* X = (const bf16_t*)j.X + zx;
  const bf16_t* W = j.W ? (const bf16_t*)j.W + zx : nullptr;
  const bool vec_rows = j.cols % 8 == 0 && (((uintptr_t)j.X | (uintptr_t)j.W) & 15) == 0;
  if (W) colsum_strip<bf16_t, true, ROWS, CL, PER>(X, W, j.sum + zo, j.sum_w + zo, rows, j.cols, j.cols, strip, vec_rows, red, red2);
  else colsum_strip<bf16_t, false, ROWS, CL, PER>(X, nullptr, j.sum + zo, nullptr, rows, j.cols, j.cols, strip, vec_rows, red, red2);
}

bool colsum_narrow(int rows, int cols) { return (long long)rows * cols <= (1LL << 20); }

// 256 row lanes for tall bf16 blocks, where the chain of loads is what a launch waits for, and for bf16 rows without 16-byte
// alignment (eight loads a row).  fp32 rows keep twice the loads in flight, and gain nothing.
template <typename T>
static bool cs_tall(int rows, int cols) { return sizeof(T) == 2 && (rows > 2048 || cols % 8 != 0); }
// Column lanes.  Narrow strips where one block is all there is, wider ones as the launch fills the chip.  bf16: 16 columns
// are as fast as 8 there and less to fetch twice; blocks of one 128-byte line or less want half a line as soon as there are
// several (16 blocks of [8192 x 64]: strips of 32, 16, 8 columns 10.8, 16.7, 20.7 us).
template <typename T>
static int cs_lanes(long long width, int cols, unsigned blocks) {
  if (sizeof(T) == 4) return width >= 64 * 256 ? 8 : width >= 32 * 256 ? 4 : width >= 12 * 256 ? 2 : 1;
  if (cols <= 8) return 1;
  if (width >= 64 * 256) return 8;
  return width >= 32 * 256 || (cols <= 64 && blocks > 1) ? 4 : 2;
}
template <typename T, bool PROD>
static void colsum_launch(dim3 batch, const T* X, const T* W, float* out, float* out2, int rows, int cols, int ld, long long sX,
                          long long sOut, hipStream_t stream) {
#define OPTIMUS_COLSUM(ROWS, CL, PER)                                                                                                    \
  hipLaunchKernelGGL((colsum_kernel<T, PROD, ROWS, CL, PER>), dim3((unsigned)((cols + 8 * CL - 1) / (8 * CL)), batch.y),                 \
                     dim3(ROWS / PER * CL), 0, stream, X, W, out, out2, rows, cols, ld, sX, sOut)
  const bool tall = cs_tall<T>(rows, cols);
  const long long width = (long long)cols * batch.y;
  const int cl = cs_lanes<T>(width, cols, batch.y);
  if constexpr (sizeof(T) == 2) {
    if (tall) {
      // two row lanes a thread also where the launch has loads enough without: with products, 4 of [4096 x 2048] 26.0 and 23.3 us
      if (cl == 8) OPTIMUS_COLSUM(256, 8, 2);
      else if (PROD && width >= 32 * 256) OPTIMUS_COLSUM(256, 4, 2);
      else if (cl == 4) OPTIMUS_COLSUM(256, 4, 1);
      else if (cl == 2) OPTIMUS_COLSUM(256, 2, 1);
      else OPTIMUS_COLSUM(256, 1, 1);
      return;
    }
  }
  if (cl == 8) OPTIMUS_COLSUM(128, 8, 1);
  else if (cl == 4) OPTIMUS_COLSUM(128, 4, 1);
  else if (cl == 2) OPTIMUS_COLSUM(128, 2, 1);
  else OPTIMUS_COLSUM(128, 1, 1);
#undef OPTIMUS_COLSUM
}

int launch_colsum_jobs(const ColsumJobs& jobs, int rows, int nz, const CombineJobs* combines, hipStream_t stream) {
  long long width = 0;
  int least = jobs.j[0].cols;
  for (int k = 0; k < jobs.n; ++k) { width += jobs.j[k].cols; least = jobs.j[k].cols < least ? jobs.j[k].cols : least; }
  const bool tall = cs_tall<bf16_t>(rows, least);   // one block's width is a multiple of 8 with all of them (the caller's heads are)
  const int cl = cs_lanes<bf16_t>(width * nz, least, (unsigned)nz);
  unsigned strips = 0;
  for (int k = 0; k < jobs.n; ++k) strips += (unsigned)((jobs.j[k].cols + 8 * cl - 1) / (8 * cl));
  const int threads = (tall ? (cl == 8 ? 128 : 256) : 128) * cl;
  CombineJobs with = {}, alone = {};
  long long blocks = 0;
  for (int k = 0; combines && k < combines->n; ++k) {
    const CombineJob& j = combines->j[k];
    if (!j.vec) { alone.j[alone.n++] = j; continue; }
    blocks += with.blocks[with.n] = (unsigned)((j.nz * j.Mb * (j.Nb / 4) + threads - 1) / threads);
    with.j[with.n++] = j;
  }
  const int rc = launch_gemm_combines(alone, stream);
  if (rc) return rc;
  const unsigned sums = strips * (unsigned)nz;
  const dim3 grid((unsigned)(sums + blocks));
#define OPTIMUS_COLSUM_JOBS(ROWS, CL, PER) \
  hipLaunchKernelGGL((colsum_jobs_kernel<ROWS, CL, PER>), grid, dim3(ROWS / PER * CL), 0, stream, jobs, rows, strips, sums, with)
  if (tall && cl == 8) OPTIMUS_COLSUM_JOBS(256, 8, 2);
  else if (tall && cl == 4) OPTIMUS_COLSUM_JOBS(256, 4, 1);
  else if (tall && cl == 2) OPTIMUS_COLSUM_JOBS(256, 2, 1);
  else if (tall) OPTIMUS_COLSUM_JOBS(256, 1, 1);
  else if (cl == 8) OPTIMUS_COLSUM_JOBS(128, 8, 1);
  else if (cl == 4) OPTIMUS_COLSUM_JOBS(128, 4, 1);
  else if (cl == 2) OPTIMUS_COLSUM_JOBS(128, 2, 1);
  else OPTIMUS_COLSUM_JOBS(128, 1, 1);
#undef OPTIMUS_COLSUM_JOBS
  return hip_launch_status();
}

int launch_colsum(const void* X, float* out, int rows, int cols, int ld, int nz, long long sX, long long sOut, int dtype,
                  hipStream_t stream) {
  dim3 batch(1, (unsigned)nz);
  if (dtype == OPTIMUS_BF16)
    colsum_launch<bf16_t, false>(batch, (const bf16_t*)X, (const bf16_t*)nullptr, out, (float*)nullptr, rows, cols, ld, sX, sOut, stream);
  else
    colsum_launch<float, false>(batch, (const float*)X, (const float*)nullptr, out, (float*)nullptr, rows, cols, ld, sX, sOut, stream);
  return hip_launch_status();
}

// dbeta_part = column sums of dy, dgamma_part = column sums of dy*xhat, for the blocks (i0.., j0..) of d
int launch_ln_param_grads(const void* dY, const void* xhat, float* dgamma_part, float* dbeta_part, const LnDesc& d,
                          hipStream_t stream) {
  const long long blk = (long long)d.rows * d.cols;
  int rc = OPTIMUS_OK;
  // block-major storage: the nj blocks of one grid row are contiguous, and so are whole grid rows that follow each other
  const bool whole_rows = d.nj == d.q;
  const int launches = whole_rows ? 1 : d.ni, per_launch = whole_rows ? d.ni * d.nj : d.nj;
  for (int ii = 0; ii < launches && rc == OPTIMUS_OK; ++ii) {
    const long long first = ((long long)(d.i0 + ii) * d.q + d.j0);
    dim3 batch(1, (unsigned)per_launch);
    if (d.dtype == OPTIMUS_BF16)
      colsum_launch<bf16_t, true>(batch, (const bf16_t*)dY + first * blk, (const bf16_t*)xhat + first * blk, dbeta_part + first * d.cols,
                                  dgamma_part + first * d.cols, d.rows, d.cols, d.cols, blk, (long long)d.cols, stream);
    else
      colsum_launch<float, true>(batch, (const float*)dY + first * blk, (const float*)xhat + first * blk, dbeta_part + first * d.cols,
                                 dgamma_part + first * d.cols, d.rows, d.cols, d.cols, blk, (long long)d.cols, stream);
    rc = hip_launch_status();
  }
  return rc;
}

}  // namespace optimus
