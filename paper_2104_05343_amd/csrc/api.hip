// C ABI of the library: argument validation, block addressing on the q x q grid, and the composition of the
// kernels into the paper's operations (Algorithms 1-3, Section 3.2).  Every entry point validates first and
// enqueues nothing on error.
#include <math.h>

#include <mutex>

#include "common.hpp"
#include "epilogue.hpp"

using namespace optimus;

// Scratch of the entry point that allocates nothing (optimus_attention_fused_bwd_static): one array per GPU the library
// runs on, held until the process ends.  In host code the array's NAME is only a handle for hipGetSymbolAddress, never
// a device address: every use goes through static_scratch(), which looks the address up once per device.
constexpr size_t kStaticScratchBytes = OPTIMUS_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

inline hipStream_t as_stream(void* s) { return (hipStream_t)s; }

int check_coords(int q, int i, int j) {
  if (q <= 0) return OPTIMUS_ESHAPE;
  if (i == OPTIMUS_ALL && j == OPTIMUS_ALL) return OPTIMUS_OK;
  if (i < 0 || j < 0 || i >= q || j >= q) return OPTIMUS_ECOORD;
  return OPTIMUS_OK;
}
inline bool is_grid(int i, int j) { return i == OPTIMUS_ALL && j == OPTIMUS_ALL; }
inline size_t esize(int dtype) { return dtype == OPTIMUS_BF16 ? 2 : 4; }
inline const void* off(const void* p, long long elems, size_t es) { return p ? (const char*)p + elems * (long long)es : nullptr; }
inline void* off(void* p, long long elems, size_t es) { return p ? (char*)p + elems * (long long)es : nullptr; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int check_mkn(int64_t M, int64_t K, int64_t N, int q) {
  if (q <= 0 || M <= 0 || K <= 0 || N <= 0) return OPTIMUS_ESHAPE;
  if (M % q || K % q || N % q) return OPTIMUS_ESHAPE;
  if (M / q > 0x7fffffff || K / q > 0x7fffffff || N / q > 0x7fffffff) return OPTIMUS_ESHAPE;
  return OPTIMUS_OK;
}

// Owner-view descriptor of one SUMMA product for device (i, j), or for the whole grid.
//   AB : C_ij = sum_l A_il B_lj ;  ABT: C_ij = sum_l A_il (B_jl)^T ;  ATB: C_ij = sum_l (A_li)^T B_lj
GemmDesc summa_desc(int form, const void* A, const void* B, void* C, int64_t M, int64_t K, int64_t N, int q, int i, int j,
                    int dtype, const optimus_epilogue* epi) {
  GemmDesc d = {};
  const int Mb = (int)(M / q), Nb = (int)(N / q), Kp = (int)(K / q);
  d.Mb = Mb; d.Nb = Nb; d.Kp = Kp; d.nl = q; d.dtype = dtype;
  const long long blkA = (long long)Mb * Kp, blkB = (long long)Kp * Nb, blkC = (long long)Mb * Nb;
  if (form == OPTIMUS_FORM_ATB) { d.a_kcontig = 0; d.lda = Mb; d.sAl = q * blkA; d.sA1 = blkA; d.sA0 = 0; }
  else { d.a_kcontig = 1; d.lda = Kp; d.sAl = blkA; d.sA1 = q * blkA; d.sA0 = 0; }
  if (form == OPTIMUS_FORM_ABT) { d.b_kcontig = 1; d.ldb = Kp; d.sBl = blkB; d.sB0 = q * blkB; d.sB1 = 0; }
  else { d.b_kcontig = 0; d.ldb = Nb; d.sBl = q * blkB; d.sB0 = blkB; d.sB1 = 0; }
  d.ldc = Nb; d.sC1 = q * blkC; d.sC0 = blkC;
  d.alpha = 1.0f;
  d.splits = 1;
  const size_t es = esize(dtype);
  const bool out32 = epi && epi->out_fp32 && dtype == OPTIMUS_BF16;
  d.out_fp32 = out32 ? 1 : 0;
  const size_t ces = out32 ? 4 : es;
  const float* bias = epi ? epi->bias : nullptr;
  void* pre = epi ? epi->pre_act : nullptr;
  const void* gg = epi ? epi->gelu_grad_of : nullptr;
  const void* res = epi ? epi->residual : nullptr;
  d.act = epi ? epi->act : 0;
  d.sBias0 = Nb;
  if (is_grid(i, j)) {
    d.nz1 = q; d.nz0 = q; d.plan_for_batch = 1;
    d.A = A; d.B = B; d.C = C;
    d.bias = bias; d.pre_act = pre; d.gelu_grad_of = gg; d.residual = res;
  } else {
    d.nz1 = 1; d.nz0 = 1;
    d.A = off(A, i * d.sA1 + j * d.sA0, es);
    d.B = off(B, i * d.sB1 + j * d.sB0, es);
    const long long co = i * d.sC1 + j * d.sC0;
    d.C = off(C, co, ces);
    d.bias = bias ? bias + (long long)j * Nb : nullptr;
    d.pre_act = off(pre, co, es);
    d.gelu_grad_of = off(gg, co, es);
    d.residual = off(res, co, es);
  }
  return d;
}

int run_summa(int form, const void* A, const void* B, void* C, int64_t M, int64_t K, int64_t N, int q, int i, int j, int dtype,
              const optimus_epilogue* epi, void* ws, size_t ws_bytes, void* stream, int corun = 0) {
  if (!A || !B || !C) return OPTIMUS_EINVAL;
  if (form < 0 || form > 2) return OPTIMUS_EINVAL;
  if (dtype != OPTIMUS_FP32 && dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  int rc = check_mkn(M, K, N, q);
  if (rc) return rc;
  rc = check_coords(q, i, j);
  if (rc) return rc;
  if (epi && (epi->act < 0 || epi->act > 1)) return OPTIMUS_EINVAL;
  GemmDesc d = summa_desc(form, A, B, C, M, K, N, q, i, j, dtype, epi);
  d.corun = corun;
  if (gemm_mfma_supported(d)) {
    // a planned panel split writes its partial tiles to the workspace if it is there and large enough; otherwise the
    // same split is emulated inside the workgroups: the bits of a result do not depend on the workspace
    const size_t need = gemm_plan_bytes(d);
    if (need > 0 && ws && ws_bytes >= need) { d.partials = (float*)ws; d.partials_bytes = ws_bytes; }
  }
  return launch_gemm(d, as_stream(stream));
}

// The two products of a linear layer's backward pass, d_in = d_out W^T (with its epilogue) and d_W = in^T d_out in fp32, in one
// launch where they go together; otherwise one after the other.
struct LinearGrads {
  const void *d_out, *w, *in;
  void *d_in, *d_w;
  int64_t M, K, N;              // d_in is [M x K], d_out [M x N], W [K x N]
  const void* gelu_grad_of;     // or nullptr
};
// ws_y: the weight gradient's partial tiles, ws_y_bytes of them.  What is left to be combined is handed out in *in_job (d_in; its C is null
// if there is nothing) and added to *w_jobs.
int run_linear_grads(const LinearGrads& g, int q, int i, int j, void* ws_x, size_t ws_x_bytes, void* ws_y, size_t ws_y_bytes, CombineJob* in_job,
                     CombineJobs* w_jobs, hipStream_t st) {
  optimus_epilogue ex = {}, ey = {};
  ex.gelu_grad_of = g.gelu_grad_of;
  ey.out_fp32 = 1;
  GemmDesc x = summa_desc(OPTIMUS_FORM_ABT, g.d_out, g.w, g.d_in, g.M, g.N, g.K, q, i, j, OPTIMUS_BF16, &ex);
  GemmDesc y = summa_desc(OPTIMUS_FORM_ATB, g.in, g.d_out, g.d_w, g.K, g.M, g.N, q, i, j, OPTIMUS_BF16, &ey);
  const size_t nx = gemm_plan_bytes(x), ny = gemm_plan_bytes(y);
  if (nx > 0 && nx <= ws_x_bytes) { x.partials = (float*)ws_x; x.partials_bytes = ws_x_bytes; }
  if (ny > 0 && ny <= ws_y_bytes) { y.partials = (float*)ws_y; y.partials_bytes = ws_y_bytes; }
  *in_job = CombineJob{};
  CombineJobs jobs = {};
  int rc;
  if (!launch_gemm_pair(x, y, &jobs, st, &rc)) {
    if ((rc = launch_gemm(x, st))) return rc;
    return launch_gemm(y, st);
  }
  for (int k = 0; k < jobs.n; ++k) {
    if (jobs.j[k].epi.C == x.C) *in_job = jobs.j[k];
    else w_jobs->j[w_jobs->n++] = jobs.j[k];
  }
  return rc;
}

struct AttnDims {
  int nb, nh, d, s, ld, ldo;
  long long blk_qkv, blk_attn, blk_probs, nmat;
  long long nmat_dev;   // of one device, whatever a launch covers
};
int attn_dims(int b, int s, int h, int n, int q, AttnDims* a) {
  if (q <= 0 || b <= 0 || s <= 0 || h <= 0 || n <= 0) return OPTIMUS_ESHAPE;
  if (b % q || n % q || h % n) return OPTIMUS_ESHAPE;
  a->nb = b / q; a->nh = n / q; a->d = h / n; a->s = s;
  if (a->d % 8 || s % 8 || s > 4096) return OPTIMUS_ESHAPE;
  a->ld = 3 * h / q; a->ldo = h / q;
  a->blk_qkv = (long long)a->nb * s * a->ld;
  a->blk_attn = (long long)a->nb * s * a->ldo;
  a->nmat = a->nmat_dev = (long long)a->nb * a->nh;
  a->blk_probs = a->nmat * s * s;
  return OPTIMUS_OK;
}
size_t attn_ws_bytes(const AttnDims& a) {
  return align256((size_t)a.blk_probs * 4) + align256((size_t)a.blk_probs * 2);
}

GemmDesc attn_base_desc(const AttnDims& a) {
  GemmDesc d = {};
  d.dtype = OPTIMUS_BF16; d.nl = 1; d.nz1 = a.nb; d.nz0 = a.nh; d.alpha = 1.0f; d.splits = 1;
  return d;
}

// One launch for scores, soft-max and their product, or one each.  The joint kernels walk a row's columns twice in one workgroup,
// so a few long matrices take as long as the separate launches and more; by one device's matrices, as the sums are added in
// another order.  Measured, us, separate / joint.  Forward, causal, width 64: two of s = 512 13 / 12, of 768 15 / 17, of 1024 18 / 21, of
// 4096 68 / 71, three of 1024 20 / 21, of 3072 60 / 54, four of 1024 22 / 22; width 128: six of 384 13 / 15, of 1024 27 / 30, eight of
// 512 16 / 18, of 1024 31 / 30, twelve of 512 19 / 18, four of 4096 138 / 100.  Forward, no mask, width 64: one of 768 14 / 16, two 17 / 16,
// of 2048 34 / 37; width 128: four of 384 13 / 13, six 14 / 14.  Backward (dV and dK included), causal and without a mask, width 64:
// one of 256 19 / 18 and 19 / 17, of 512 22 / 24 and 23 / 24, six of 1024 38 / 40 and 41 / 41, of 1536 53 / 58 and 63 / 59, two of 4096 110 / 131
// and 144 / 132, four 192 / 133 and 269 / 161; width 128: one of 256 19 / 21 and 20 / 21, 16 22 / 23 and 23 / 22, 16 of 512 32 / 32 and 33 / 33,
// eight of 1024 42 / 49 and 47 / 50, 16 60 / 57 and 75 / 62, four of 2048 67 / 90 and 77 / 93, eight 94 / 92 and 169 / 108: one line for
// both, which costs the joint short ones up to a tenth and the separate long ones without a mask up to a third.
bool attn_joint(const AttnDims& a, int causal, bool bwd) {
  const long long n = a.nmat_dev;
  const bool many = n * a.s >= 16384;
  if (bwd) return a.d == 64 ? a.s <= 512 || n >= 6 || many : a.s <= 256 || n >= 16 || many;
  if (!causal) return a.d == 64 ? a.s <= 768 || n >= 2 : a.s <= 256 || n >= 6 || many;
  return a.d == 64 ? a.s <= 512 || n >= 4 || n * a.s > 8192 : a.s <= 256 || n >= 12 || (n >= 8 && a.s > 768) || many;
}

AttnProbsDesc probs_desc(const bf16_t* qkv_blk, const bf16_t* probs_blk, const AttnDims& a, int causal) {
  AttnProbsDesc p = {};
  p.qkv = qkv_blk; p.probs = const_cast<bf16_t*>(probs_blk);
  p.s = a.s; p.d = a.d; p.nh = a.nh; p.ld = a.ld; p.ldo = a.ldo; p.causal = causal;
  p.nmat = a.nmat;
  return p;
}

int attention_fwd_device(const bf16_t* qkv_blk, bf16_t* probs_blk, bf16_t* attn_blk, const AttnDims& a, int causal, void* ws,
                         hipStream_t st) {
  AttnProbsDesc p = probs_desc(qkv_blk, probs_blk, a, causal);
  p.attn = attn_blk;
  if (attn_joint(a, causal, false) && attn_probs_supported(p)) return launch_attn_probs_fwd(p, st);
  float* scores = (float*)ws;
  const long long ss = (long long)a.s * a.s;
  const float scale = 1.0f / sqrtf((float)a.d);
  // S = Q K^T / sqrt(d)
  GemmDesc g = attn_base_desc(a);
  g.A = qkv_blk; g.B = qkv_blk + a.d; g.C = scores;
  g.Mb = a.s; g.Nb = a.s; g.Kp = a.d;
  g.a_kcontig = 1; g.b_kcontig = 1; g.lda = a.ld; g.ldb = a.ld; g.ldc = a.s;
  g.sA1 = (long long)a.s * a.ld; g.sA0 = 3 * a.d; g.sB1 = g.sA1; g.sB0 = g.sA0;
  g.sC1 = a.nh * ss; g.sC0 = ss;
  g.alpha = scale; g.out_fp32 = 1; g.skip_upper = causal;
  int rc = launch_gemm(g, st);
  if (rc) return rc;
  rc = launch_softmax_fwd(scores, probs_blk, (int)a.nmat, a.s, causal, st);
  if (rc) return rc;
  // O = P V
  GemmDesc o = attn_base_desc(a);
  o.A = probs_blk; o.B = qkv_blk + 2 * a.d; o.C = attn_blk;
  o.Mb = a.s; o.Nb = a.d; o.Kp = a.s;
  o.a_kcontig = 1; o.b_kcontig = 0; o.lda = a.s; o.ldb = a.ld; o.ldc = a.ldo;
  o.sA1 = a.nh * ss; o.sA0 = ss; o.sB1 = (long long)a.s * a.ld; o.sB0 = 3 * a.d;
  o.sC1 = (long long)a.s * a.ldo; o.sC0 = a.d;
  o.k_hi_diag = causal;
  return launch_gemm(o, st);
}

int attention_bwd_device(const bf16_t* qkv_blk, const bf16_t* probs_blk, const bf16_t* dattn_blk, bf16_t* dqkv_blk,
                         const AttnDims& a, int causal, void* ws, hipStream_t st) {
  float* dP = (float*)ws;
  bf16_t* dS = (bf16_t*)((char*)ws + align256((size_t)a.blk_probs * 4));
  const long long ss = (long long)a.s * a.s;
  const float scale = 1.0f / sqrtf((float)a.d);
  const long long q1 = (long long)a.s * a.ld, q0 = 3 * a.d;      // (sequence, head) strides inside a qkv block
  const long long o1 = (long long)a.s * a.ldo, o0 = a.d;         // inside an attn block
  const long long p1 = a.nh * ss, p0 = ss;                       // inside probs / scratch
  int rc;
  {  // dV = P^T dO   (contraction over query position t >= key position u)
    GemmDesc g = attn_base_desc(a);
    g.A = probs_blk; g.B = dattn_blk; g.C = dqkv_blk + 2 * a.d;
    g.Mb = a.s; g.Nb = a.d; g.Kp = a.s;
    g.a_kcontig = 0; g.b_kcontig = 0; g.lda = a.s; g.ldb = a.ldo; g.ldc = a.ld;
    g.sA1 = p1; g.sA0 = p0; g.sB1 = o1; g.sB0 = o0; g.sC1 = q1; g.sC0 = q0;
    g.k_lo_diag = causal;
    if ((rc = launch_gemm(g, st))) return rc;
  }
  AttnProbsDesc p = probs_desc(qkv_blk, probs_blk, a, causal);
  p.d_attn = dattn_blk; p.d_scores = dS; p.d_qkv = dqkv_blk;
  const bool joined = attn_joint(a, causal, true) && attn_probs_supported(p);   // dS and dQ in one launch, dP never in memory
  if (joined && (rc = launch_attn_probs_bwd(p, st))) return rc;
  if (!joined) {  // dP = dO V^T
    GemmDesc g = attn_base_desc(a);
    g.A = dattn_blk; g.B = qkv_blk + 2 * a.d; g.C = dP;
    g.Mb = a.s; g.Nb = a.s; g.Kp = a.d;
    g.a_kcontig = 1; g.b_kcontig = 1; g.lda = a.ldo; g.ldb = a.ld; g.ldc = a.s;
    g.sA1 = o1; g.sA0 = o0; g.sB1 = q1; g.sB0 = q0; g.sC1 = p1; g.sC0 = p0;
    g.out_fp32 = 1; g.skip_upper = causal;
    if ((rc = launch_gemm(g, st))) return rc;
  }
  if (!joined && (rc = launch_softmax_bwd(dP, probs_blk, dS, (int)a.nmat, a.s, causal, st))) return rc;
  if (!joined) {  // dQ = dS K / sqrt(d)
    GemmDesc g = attn_base_desc(a);
    g.A = dS; g.B = qkv_blk + a.d; g.C = dqkv_blk;
    g.Mb = a.s; g.Nb = a.d; g.Kp = a.s;
    g.a_kcontig = 1; g.b_kcontig = 0; g.lda = a.s; g.ldb = a.ld; g.ldc = a.ld;
    g.sA1 = p1; g.sA0 = p0; g.sB1 = q1; g.sB0 = q0; g.sC1 = q1; g.sC0 = q0;
    g.alpha = scale; g.k_hi_diag = causal;
    if ((rc = launch_gemm(g, st))) return rc;
  }
  {  // dK = dS^T Q / sqrt(d)
    GemmDesc g = attn_base_desc(a);
    g.A = dS; g.B = qkv_blk; g.C = dqkv_blk + a.d;
    g.Mb = a.s; g.Nb = a.d; g.Kp = a.s;
    g.a_kcontig = 0; g.b_kcontig = 0; g.lda = a.s; g.ldb = a.ld; g.ldc = a.ld;
    g.sA1 = p1; g.sA0 = p0; g.sB1 = q1; g.sB0 = q0; g.sC1 = q1; g.sC0 = q0;
    g.alpha = scale; g.k_lo_diag = causal;
    if ((rc = launch_gemm(g, st))) return rc;
  }
  return OPTIMUS_OK;
}

int run_attention(bool bwd, const void* qkv, const void* probs_in, void* probs_out, const void* d_attn, void* out, int b, int s,
                  int h, int n, int q, int i, int j, int causal, int dtype, void* ws, size_t ws_bytes, void* stream) {
  if (dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  AttnDims a;
  int rc = attn_dims(b, s, h, n, q, &a);
  if (rc) return rc;
  if ((rc = check_coords(q, i, j))) return rc;
  if (!ws || ws_bytes < attn_ws_bytes(a)) return OPTIMUS_EWORKSPACE;
  // Whole grid: the blocks of consecutive devices follow each other in every tensor, and inside a block the
  // sequences do too, so g devices are one batch of g * (b/q) sequences with the same strides.  As many devices per
  // launch as the workspace holds scratch for (one device's worth is the minimum: then device after device).
  const long long first = is_grid(i, j) ? 0 : (long long)i * q + j;
  const long long ndev = is_grid(i, j) ? (long long)q * q : 1;
  long long group = (long long)(ws_bytes / attn_ws_bytes(a));
  if (group > ndev) group = ndev;
  if (group > 0x7fffffffLL / (a.nmat > 0 ? a.nmat : 1)) group = 0x7fffffffLL / a.nmat;   // batch counts are ints
  for (long long dev = first; dev < first + ndev; dev += group) {
    const long long g = dev + group <= first + ndev ? group : first + ndev - dev;
    AttnDims ag = a;
    ag.nb = (int)(a.nb * g); ag.nmat = a.nmat * g; ag.blk_probs = a.blk_probs * g;
    const bf16_t* qb = (const bf16_t*)qkv + dev * a.blk_qkv;
    if (!bwd)
      rc = attention_fwd_device(qb, (bf16_t*)probs_out + dev * a.blk_probs, (bf16_t*)out + dev * a.blk_attn, ag, causal, ws,
                                as_stream(stream));
    else
      rc = attention_bwd_device(qb, (const bf16_t*)probs_in + dev * a.blk_probs, (const bf16_t*)d_attn + dev * a.blk_attn,
                                (bf16_t*)out + dev * a.blk_qkv, ag, causal, ws, as_stream(stream));
    if (rc) return rc;
  }
  return OPTIMUS_OK;
}

// Fused attention: same block geometry, no [s x s] tensors, head width limited to what the kernels are built for.
int attn_fused_dims(int b, int s, int h, int n, int q, AttnDims* a) {
  if (q <= 0 || b <= 0 || s <= 0 || h <= 0 || n <= 0) return OPTIMUS_ESHAPE;
  if (b % q || n % q || h % n) return OPTIMUS_ESHAPE;
  a->nb = b / q; a->nh = n / q; a->d = h / n; a->s = s;
  if (!attn_fused_supported(a->d) || s > (1 << 20)) return OPTIMUS_ESHAPE;
  a->ld = 3 * h / q; a->ldo = h / q;
  a->blk_qkv = (long long)a->nb * s * a->ld;
  a->blk_attn = (long long)a->nb * s * a->ldo;
  a->nmat = a->nmat_dev = (long long)a->nb * a->nh;
  a->blk_probs = 0;
  if (a->nmat > 65535) return OPTIMUS_ESHAPE;
  return OPTIMUS_OK;
}
size_t attn_fused_ws_bytes(const AttnDims& a, int q) { return align256((size_t)q * q * a.nmat * a.s * sizeof(float)); }

int run_attention_fused(bool bwd, const void* qkv, void* attn, float* lse, const void* d_attn, void* d_qkv, int b, int s, int h,
                        int n, int q, int i, int j, int causal, int dtype, void* ws, size_t ws_bytes, void* stream) {
  if (dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  AttnDims a;
  int rc = attn_fused_dims(b, s, h, n, q, &a);
  if (rc) return rc;
  if ((rc = check_coords(q, i, j))) return rc;
  if (bwd && (!ws || ws_bytes < attn_fused_ws_bytes(a, q))) return OPTIMUS_EWORKSPACE;
  const bool grid = is_grid(i, j);
  const long long dev = grid ? 0 : (long long)i * q + j;
  AttnFusedDesc d = {};
  d.qkv = (const bf16_t*)qkv + dev * a.blk_qkv;
  d.attn = (bf16_t*)attn + dev * a.blk_attn;
  d.lse = lse + dev * a.nmat * s;
  d.d_attn = d_attn ? (const bf16_t*)d_attn + dev * a.blk_attn : nullptr;
  d.d_qkv = d_qkv ? (bf16_t*)d_qkv + dev * a.blk_qkv : nullptr;
  d.delta = (float*)ws;
  d.s = s; d.d = a.d; d.nb = a.nb; d.nh = a.nh; d.ld = a.ld; d.ldo = a.ldo;
  d.ndev = grid ? q * q : 1;
  d.dev_qkv = a.blk_qkv; d.dev_attn = a.blk_attn;
  d.causal = causal;
  return bwd ? launch_attn_fused_bwd(d, as_stream(stream)) : launch_attn_fused_fwd(d, as_stream(stream));
}

int end_desc(int64_t M, int64_t v, int64_t h, int q, int i, int j, int dtype, EndDesc* d) {
  if (dtype != OPTIMUS_FP32 && dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  if (q <= 0 || M <= 0 || v <= 0 || h <= 0 || M % q || v % q || h % q) return OPTIMUS_ESHAPE;
  if (M > 0x7fffffff || v > 0x7fffffff || h > 0x7fffffff) return OPTIMUS_ESHAPE;
  int rc = check_coords(q, i, j);
  if (rc) return rc;
  d->rows = (int)(M / q); d->vb = (int)(v / q); d->hb = (int)(h / q); d->q = q; d->v = (int)v; d->dtype = dtype;
  if (is_grid(i, j)) { d->i0 = 0; d->ni = q; d->j0 = 0; d->nj = q; }
  else { d->i0 = i; d->ni = 1; d->j0 = j; d->nj = 1; }
  return OPTIMUS_OK;
}

int ln_desc(int64_t M, int64_t H, int q, int i, int j, int dtype, float eps, LnDesc* d) {
  if (dtype != OPTIMUS_FP32 && dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  if (q <= 0 || M <= 0 || H <= 0 || M % q || H % q) return OPTIMUS_ESHAPE;
  if (M / q > 0x7fffffff / 4 || H > 0x7fffffff) return OPTIMUS_ESHAPE;
  int rc = check_coords(q, i, j);
  if (rc) return rc;
  d->rows = (int)(M / q); d->cols = (int)(H / q); d->H = (int)H; d->q = q; d->dtype = dtype; d->eps = eps;
  if (is_grid(i, j)) { d->i0 = 0; d->ni = q; d->j0 = 0; d->nj = q; }
  else { d->i0 = i; d->ni = 1; d->j0 = j; d->nj = 1; }
  return OPTIMUS_OK;
}

int ln_forward(const void* X, const float* gamma, const float* beta, void* Y, void* xhat, float* rstd, float* stats,
               const LnDesc& d, bool grid, hipStream_t st) {
  if (grid && !ln_rowgroup_ok(d)) {
    int rc = launch_ln_stats(X, stats, d, st);
    if (rc) return rc;
    return launch_ln_apply(X, gamma, beta, Y, xhat, rstd, stats, d, true, st);
  }
  // one device: its own partial, the peers' from `stats`; whole grid: every row's partials meet inside the launch
  return launch_ln_apply(X, gamma, beta, Y, xhat, rstd, stats, d, false, st);
}
int ln_backward(const void* dY, const void* xhat, const float* rstd, const float* gamma, const void* dres, void* dX,
                float* dgamma_part, float* dbeta_part, float* stats, const LnDesc& d, bool grid, hipStream_t st) {
  int rc;
  if (grid && !ln_rowgroup_ok(d)) {
    if ((rc = launch_ln_bwd_stats(dY, xhat, gamma, stats, d, st))) return rc;
    rc = launch_ln_bwd_apply(dY, xhat, rstd, gamma, dres, dX, stats, d, true, st);
  } else {
    rc = launch_ln_bwd_apply(dY, xhat, rstd, gamma, dres, dX, stats, d, false, st);
  }
  if (rc) return rc;
  if (dgamma_part && dbeta_part) rc = launch_ln_param_grads(dY, xhat, dgamma_part, dbeta_part, d, st);
  return rc;
}

int layer_check(const optimus_layer_cfg* c, int i, int j, AttnDims* a) {
  if (!c) return OPTIMUS_EINVAL;
  if (c->dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  int rc = c->fused_attention ? attn_fused_dims(c->b, c->s, c->h, c->n, c->q, a) : attn_dims(c->b, c->s, c->h, c->n, c->q, a);
  if (rc) return rc;
  if (c->h % c->q) return OPTIMUS_ESHAPE;
  if ((long long)c->b * c->s > 0x7fffffffLL) return OPTIMUS_ESHAPE;
  return check_coords(c->q, i, j);
}

struct LayerGemm { int form; int64_t M, K, N; };
// the twelve SUMMA products of a layer (forward 4, backward 8), logical output shapes
void layer_gemms(const optimus_layer_cfg* c, LayerGemm out[12]) {
  const int64_t M = (int64_t)c->b * c->s, h = c->h;
  out[0] = {OPTIMUS_FORM_AB, M, h, 3 * h};      // qkv
  out[1] = {OPTIMUS_FORM_AB, M, h, h};          // dense
  out[2] = {OPTIMUS_FORM_AB, M, h, 4 * h};      // h -> 4h
  out[3] = {OPTIMUS_FORM_AB, M, 4 * h, h};      // 4h -> h
  out[4] = {OPTIMUS_FORM_ABT, M, h, 4 * h};     // d_gelu = d_out W2^T
  out[5] = {OPTIMUS_FORM_ATB, 4 * h, M, h};     // dW2 = gelu^T d_out
  out[6] = {OPTIMUS_FORM_ABT, M, 4 * h, h};     // d_ln2_out = d_pre W1^T
  out[7] = {OPTIMUS_FORM_ATB, h, M, 4 * h};     // dW1 = ln2_out^T d_pre
  out[8] = {OPTIMUS_FORM_ABT, M, h, h};         // d_attn = d_h_mid Wo^T
  out[9] = {OPTIMUS_FORM_ATB, h, M, h};         // dWo = attn^T d_h_mid
  out[10] = {OPTIMUS_FORM_ABT, M, 3 * h, h};    // d_ln1_out = d_qkv Wqkv^T
  out[11] = {OPTIMUS_FORM_ATB, h, M, 3 * h};    // dWqkv = ln1_out^T d_qkv
}

// The parameter gradients of the backward pass (A^T B products, bias column sums) hang off the chain of activation
// gradients but nothing in the chain waits for them: they run on a second stream of the library, forked from and
// joined back into the caller's stream with events (also valid under stream capture: the branch becomes a parallel
// arm of the graph).  One stream and one set of events per device, created on the first call that is not made
// under stream capture; until then, or if they cannot be created, the branch simply runs on the caller's stream.
// The stream and events are shared by all calls on a device: concurrent calls from several host threads on one
// device are not supported.
struct SideStream {
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr, ready[3] = {nullptr, nullptr, nullptr};
  int state = 0;  // 0 = not tried, 1 = usable, -1 = unavailable
};
constexpr int kMaxDevices = 64;
SideStream g_side[kMaxDevices];

SideStream* side_stream(hipStream_t caller) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return nullptr; }
  SideStream& x = g_side[dev];
  if (x.state == 0) {
    // creating a stream while the caller captures a graph is not allowed (and would invalidate the capture):
    // stay on the caller's stream for this call and try again on a later one
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(caller, &cs) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
    if (cs != hipStreamCaptureStatusNone) return nullptr;
    bool ok = hipStreamCreateWithFlags(&x.s, hipStreamNonBlocking) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&x.fork, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&x.join, hipEventDisableTiming) == hipSuccess;
    for (int k = 0; k < 3; ++k) ok = ok && hipEventCreateWithFlags(&x.ready[k], hipEventDisableTiming) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    x.state = ok ? 1 : -1;
  }
  return x.state == 1 ? &x : nullptr;
}
// `to` continues only after everything queued on `from` so far
int stream_after(hipStream_t to, hipStream_t from, hipEvent_t ev) {
  if (hipEventRecord(ev, from) != hipSuccess) return OPTIMUS_EHIP;
  if (hipStreamWaitEvent(to, ev, 0) != hipSuccess) return OPTIMUS_EHIP;
  return OPTIMUS_OK;
}

// Whether both gradients of y = x W, x [M x K], W [K x N], on tensors as they are allocated go in one launch
bool pair_planned(int64_t M, int64_t K, int64_t N, int q, int i, int j) {
  void* const fake = (void*)(uintptr_t)4096;   // a plan depends on shapes, strides and 16-byte alignment only
  optimus_epilogue ey = {};
  ey.out_fp32 = 1;
  GemmDesc x = summa_desc(OPTIMUS_FORM_ABT, fake, fake, fake, M, N, K, q, i, j, OPTIMUS_BF16, nullptr);
  GemmDesc y = summa_desc(OPTIMUS_FORM_ATB, fake, fake, fake, K, M, N, q, i, j, OPTIMUS_BF16, &ey);
  x.partials = y.partials = (float*)fake;
  x.partials_bytes = y.partials_bytes = SIZE_MAX;
  return gemm_pair_planned(x, y);
}

// Whether the second stream pays in a pass that is not captured.  On one stream both products of a linear layer go in one launch
// (launch_gemm_pair) and the combines ride in other launches; on two, a fork or the join costs the host 25 us (the wait on another
// stream's event, for the most part), five of them in a backward pass: the host needs about 200 us for such a pass (a little less with
// q = 1, where no product is split).  Two streams win where the kernels on one take longer than that and the products run beside a long chain: the
// attention of a device with few matrices is one along the sequence (30 us per 1024 rows fused, 36 with the scores in memory); and from 80
// GF of products, where tiles of 256x128 on both are the better use of the chip: not in blocks that the tiles of 64x64 cut, which have no
// such, and from 600 GF not where 128 does not divide the width (64x64 tiles on both streams crowd the L2s); and from 35 GF where the
// products of h -> 4h do not go together.  With q = 1 the weight gradients are few long workgroups that the pair's other product fills up:
// from 200 GF there, below 24 as the kernels' time has it; the grid of one device is that device.
// Measured, step of one layer, two streams / one (us): 3 GF, s = 4096 225 / 209; 6 GF, s = 8200 365 / 390; 13 GF, s = 4096 256 / 230, s = 16384 650 / 730;
// 26 GF, s = 512 217 / 194, 210 / 185; 52 GF, s = 512 256 / 238, 298 / 273, s = 4096 352 / 365; 79 GF 366 / 357; 103 GF, s = 512 384 / 365, 392 / 389, 484 / 436;
// 116 GF 414 / 425, 494 / 447, 430 / 416; 161 GF 542 / 529, 558 / 634; 412 GF 814 / 868, 838 / 895; 825 GF 1369 / 1421; 1649 GF 2269 / 2286.  h -> 4h apart: 40 GF
// 250 / 250, 58 GF 283 / 297, 250 / 261, 79 GF 349 / 371.  Widths that 128 does not divide: 130 GF 526 / 554, 322 GF 1292 / 1264, 522 GF 1665 / 1755, 644 GF 2582 / 2367, 710 GF
// 1927 / 1840, 2447 / 2131, 1450 GF 4631 / 4011, 2013 GF 7732 / 6258.  Cut blocks: 38 GF 282 / 255, 101 GF 379 / 368, 157 GF 602 / 599, 403 GF 1151 / 1082, 806 GF
// 1738 / 1695, 1612 GF 3605 / 3334, 6449 GF 13981 / 11900; s = 4100: 6 GF 284 / 303, 13 GF 277 / 255, 52 GF 412 / 398, 206 GF 815 / 791, 825 GF 2097 / 1906; s = 16400:
// 13 GF 722 / 804, 52 GF 1319 / 1404, 206 GF 1663 / 1614.  q = 1: 1 GF, s = 1536 184 / 133, 6 GF, s = 2048 179 / 165, 13 GF, s = 4096 269 / 277; 52 GF, s = 1024
// 281 / 271, 103 GF 412 / 399, 155 GF 525 / 521, 412 GF 1010 / 1036, 825 GF 1416 / 1443.
// Whole grids: 26 GF 213 / 221, 334 / 326, 52 GF 330 / 333, 273 / 254, 103 GF 374 / 401; cut 34 GF 255 / 280, 259 / 286, 13 GF 205 / 177, 134 GF 457 / 532.
bool two_streams_pay(const optimus_layer_cfg* c, bool grid) {
  if (c->q == 1) grid = false;
  const double devices = grid ? (double)c->q * c->q : 1.0;
  const double gf = 48e-9 * (double)c->b * c->s * (double)c->h * c->h / ((double)c->q * c->q) * devices;
  const double one_us = 120.0 + 0.6 * gf + (c->fused_attention ? 0.030 : 0.036) * c->s;
  const int64_t M = (int64_t)c->b * c->s, h = c->h;
  const bool cut = M / c->q % 64 != 0 || h / c->q % 64 != 0;
  if (grid) return gf >= (cut ? 24.0 : 35.0) || one_us >= 200.0;
  if (cut) return c->s >= 4096 && c->s >= 200.0 * gf;
  if (gf >= 600.0 && h / c->q % 128 != 0) return false;
  if (c->q == 1) return gf >= 200.0 || c->s > 8192 || (gf < 24.0 && one_us >= 185.0);
  return gf >= 80.0 || one_us >= 200.0 || (gf >= 35.0 && !pair_planned(M, h, 4 * h, c->q, 0, 0));
}
// A captured pass pays the host once and keeps both streams (which an earlier pass, short or not, has created): from before the joint launches,
// when two were the shorter ones replayed from 1 GF on.  They are so for the wide layers only by now.  Replayed, one stream / two, us: 4096-wide
// layer, one device of 4 x 4, 914 / 837, fused 893 / 829, of 8 x 8 917 / 855; 39 GF, cut, 273 / 263; 52 GF 236 / 244, 248 / 256; 103 GF 392 / 400; 26 GF 183 / 199;
// 1024-wide layer, one device of 4 x 4, 156 / 173, fused 139 / 154; 3 GF 116 / 132; 0.4 GF 95 / 122; whole grids of small blocks 149 / 192, 165 / 237.
bool captured(hipStream_t caller) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(caller, &cs) != hipSuccess) { (void)hipGetLastError(); return false; }
  return cs != hipStreamCaptureStatusNone;
}

// Whether two matrices of a backward pass share memory in a way that its schedule does not bear.  Steps of the pass, as both schedules keep
// them: 0 d_pre_gelu, d_w2; 1 d_ln2_out, d_w1; 2 LayerNorm 2; 3 d_attn, d_w_o; 4 attention; 5 d_ln1_out, d_w_qkv; 6 LayerNorm 1.  A matrix
// is written in step `first` (-1: before the pass) and read for the last time in `one` (one stream: products in pairs, column sums at the end)
// or in `two` (what the branch reads, it may read until the join, 7).  One stream bears d_x anywhere: optimus_layer_bwd looks for that itself.
bool sharing_breaks(const optimus_layer_cfg* c, const optimus_layer_tensors* t, bool two, bool ln2_sums_on_branch) {
  struct Use { const void* p; int64_t bytes; int first, one, two; };
  const int64_t act = (int64_t)c->b * c->s * c->h * 2, w = (int64_t)c->h * c->h * 2;
  const int64_t heads = (int64_t)c->b * c->n;
  const int ln2 = ln2_sums_on_branch ? 7 : 2;
  const int pre = t->pre_gelu == t->d_pre_gelu ? -1 : 0;   // in place: each element is read by the thread that overwrites it
  const Use use[] = {
      {t->d_out, act, -1, 6, 7}, {t->w2, 4 * w, -1, 0, 0}, {t->pre_gelu, 4 * act, -1, pre, pre}, {t->gelu, 4 * act, -1, 0, 7},
      {t->w1, 4 * w, -1, 1, 1}, {t->ln2_out, act, -1, 1, 7}, {t->xhat2, act, -1, 6, ln2}, {t->w_o, w, -1, 3, 3}, {t->attn, act, -1, 4, 7},
      {t->qkv, 3 * act, -1, 4, 4}, {t->w_qkv, 3 * w, -1, 5, 5}, {t->ln1_out, act, -1, 5, 7}, {t->xhat1, act, -1, 6, 6},
      c->fused_attention ? Use{t->lse, heads * c->s * 4, -1, 4, 4} : Use{t->probs, heads * c->s * c->s * 2, -1, 4, 4},
      {t->d_pre_gelu, 4 * act, 0, 6, 7}, {t->d_w2, 8 * w, 0, 0, 0}, {t->d_ln2_out, act, 1, 6, ln2}, {t->d_w1, 8 * w, 1, 1, 1},
      {t->d_h_mid, act, 2, 6, 7}, {t->d_attn, act, 3, 4, 4}, {t->d_w_o, 2 * w, 3, 3, 3}, {t->d_qkv, 3 * act, 4, 6, 7},
      {t->d_ln1_out, act, 5, 6, 6}, {t->d_w_qkv, 6 * w, 5, 5, 5}, {t->d_x, act, 6, 6, 6}};
  for (const Use& a : use) {
    if (a.first < 0 || (a.first == 6 && !two)) continue;
    for (const Use& b : use)
      if (b.first < a.first && (two ? b.two : b.one) >= a.first && (const char*)a.p < (const char*)b.p + b.bytes &&
          (const char*)b.p < (const char*)a.p + a.bytes)
        return true;
  }
  return false;
}

// Device address of `scratch` on the current device (each GPU holds its own copy at its own address): looked up on
// the first call made with that device current, kept afterwards.
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
int static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return OPTIMUS_EHIP; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return OPTIMUS_EHIP; }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return OPTIMUS_OK;
}

// split workspace of one product as the layer plans it (corun: see GemmDesc)
size_t summa_ws_bytes(int form, int64_t M, int64_t K, int64_t N, int q, int i, int j, int dtype, int corun) {
  if (form < 0 || form > 2 || check_mkn(M, K, N, q) || check_coords(q, i, j)) return 0;
  if (dtype != OPTIMUS_BF16) return 0;
  // pointers only matter for alignment checks; use an aligned dummy
  GemmDesc d = summa_desc(form, (const void*)256, (const void*)256, (void*)256, M, K, N, q, i, j, dtype, nullptr);
  d.corun = corun;
  if (!gemm_mfma_supported(d)) return 0;
  return gemm_plan_bytes(d);
}

size_t layer_gemm_ws(const optimus_layer_cfg* c) {
  LayerGemm g[12];
  layer_gemms(c, g);
  size_t mx = 0;
  for (int k = 0; k < 12; ++k)
    for (int grid = 0; grid < 2; ++grid) {
      // the backward products run in pairs on two streams: chain (A B^T) and branch (A^T B), as optimus_layer_bwd flags them
      const int corun = k < 4 ? 0 : (g[k].form == OPTIMUS_FORM_ABT ? 1 : 2);
      size_t b = summa_ws_bytes(g[k].form, g[k].M, g[k].K, g[k].N, c->q, grid ? -1 : 0, grid ? -1 : 0, c->dtype, corun);
      if (b > mx) mx = b;
    }
  return align256(mx);
}

// Partial tiles of a layer's four weight gradients on one stream, which stay until the end of the pass: each its place behind the last.
// Nothing where two streams run.
bool two_streams_pay(const optimus_layer_cfg* c, bool grid);
void layer_weight_ws(const optimus_layer_cfg* c, int i, int j, size_t at[4], size_t* total) {
  LayerGemm g[12];
  layer_gemms(c, g);
  *total = 0;
  for (int k = 0; k < 4; ++k) {
    at[k] = *total;
    const LayerGemm& w = g[5 + 2 * k];
    *total += align256(summa_ws_bytes(w.form, w.M, w.K, w.N, c->q, i, j, c->dtype, 0));
  }
}
size_t layer_branch_ws(const optimus_layer_cfg* c, size_t gemm_bytes) {
  size_t mx = gemm_bytes, at[4], total;
  for (int grid = 0; grid < 2; ++grid) {
    if (two_streams_pay(c, grid)) continue;
    layer_weight_ws(c, grid ? -1 : 0, grid ? -1 : 0, at, &total);
    if (total > mx) mx = total;
  }
  return mx;
}

}  // namespace

extern "C" {

const char* optimus_error_string(int code) {
  switch (code) {
    case OPTIMUS_OK: return "ok";
    case OPTIMUS_EINVAL: return "invalid argument (null pointer or bad enum)";
    case OPTIMUS_ESHAPE: return "bad shape (non-positive, not divisible by the grid, or beyond a documented limit)";
    case OPTIMUS_ECOORD: return "device coordinates outside the q x q grid";
    case OPTIMUS_EDTYPE: return "dtype not supported by this entry point";
    case OPTIMUS_EWORKSPACE: return "workspace missing or too small";
    case OPTIMUS_EHIP: return "HIP runtime error at launch";
    default: return "unknown error code";
  }
}

int optimus_abi_version(void) { return 2; }

int optimus_pack_blocks(const void* src, void* dst, int64_t R, int64_t C, int q, int elem_bytes, void* stream) {
  if (!src || !dst || src == dst) return OPTIMUS_EINVAL;
  if (elem_bytes != 2 && elem_bytes != 4) return OPTIMUS_EDTYPE;
  if (q <= 0 || R <= 0 || C <= 0 || R % q || C % q) return OPTIMUS_ESHAPE;
  return launch_pack(src, dst, R, C, q, elem_bytes, false, as_stream(stream));
}
int optimus_unpack_blocks(const void* src, void* dst, int64_t R, int64_t C, int q, int elem_bytes, void* stream) {
  if (!src || !dst || src == dst) return OPTIMUS_EINVAL;
  if (elem_bytes != 2 && elem_bytes != 4) return OPTIMUS_EDTYPE;
  if (q <= 0 || R <= 0 || C <= 0 || R % q || C % q) return OPTIMUS_ESHAPE;
  return launch_pack(src, dst, R, C, q, elem_bytes, true, as_stream(stream));
}

int optimus_summa_ab(const void* A, const void* B, void* C, int64_t M, int64_t K, int64_t N, int q, int i, int j, int dtype,
                     void* ws, size_t ws_bytes, void* stream) {
  return run_summa(OPTIMUS_FORM_AB, A, B, C, M, K, N, q, i, j, dtype, nullptr, ws, ws_bytes, stream);
}
int optimus_summa_abt(const void* A, const void* B, void* C, int64_t M, int64_t K, int64_t N, int q, int i, int j, int dtype,
                      void* ws, size_t ws_bytes, void* stream) {
  return run_summa(OPTIMUS_FORM_ABT, A, B, C, M, K, N, q, i, j, dtype, nullptr, ws, ws_bytes, stream);
}
int optimus_summa_atb(const void* A, const void* B, void* C, int64_t M, int64_t K, int64_t N, int q, int i, int j, int dtype,
                      void* ws, size_t ws_bytes, void* stream) {
  return run_summa(OPTIMUS_FORM_ATB, A, B, C, M, K, N, q, i, j, dtype, nullptr, ws, ws_bytes, stream);
}
int optimus_summa_ex(int form, const void* A, const void* B, void* C, int64_t M, int64_t K, int64_t N, int q, int i, int j,
                     int dtype, const optimus_epilogue* epi, void* ws, size_t ws_bytes, void* stream) {
  return run_summa(form, A, B, C, M, K, N, q, i, j, dtype, epi, ws, ws_bytes, stream);
}

size_t optimus_summa_workspace_bytes(int form, int64_t M, int64_t K, int64_t N, int q, int i, int j, int dtype) {
  return summa_ws_bytes(form, M, K, N, q, i, j, dtype, 0);
}

// One step of Algorithms 1-3 as the COMPUTING device (i, j) sees it (the owner view above fuses the q steps).
int optimus_summa_step(int form, const void* A, const void* B, float* c_temp, int64_t M, int64_t K, int64_t N, int q, int i,
                       int j, int l, int dtype, void* stream) {
  if (!A || !B || !c_temp) return OPTIMUS_EINVAL;
  if (form < 0 || form > 2) return OPTIMUS_EINVAL;
  if (dtype != OPTIMUS_FP32 && dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  int rc = check_mkn(M, K, N, q);
  if (rc) return rc;
  if (i < 0 || j < 0 || l < 0 || i >= q || j >= q || l >= q) return OPTIMUS_ECOORD;
  const int Mb = (int)(M / q), Nb = (int)(N / q), Kp = (int)(K / q);
  const long long blkA = (long long)Mb * Kp, blkB = (long long)Kp * Nb;
  const size_t es = esize(dtype);
  GemmDesc d = {};
  d.Mb = Mb; d.Nb = Nb; d.Kp = Kp; d.nl = 1; d.dtype = dtype; d.nz0 = 1; d.nz1 = 1; d.alpha = 1.0f; d.splits = 1;
  d.ldc = Nb; d.out_fp32 = dtype == OPTIMUS_BF16 ? 1 : 0; d.C = c_temp;
  if (form == OPTIMUS_FORM_AB) {          // A_il [Mb x Kp] (received along row i) times B_lj [Kp x Nb] (along column j)
    d.A = off(A, ((long long)i * q + l) * blkA, es); d.a_kcontig = 1; d.lda = Kp;
    d.B = off(B, ((long long)l * q + j) * blkB, es); d.b_kcontig = 0; d.ldb = Nb;
  } else if (form == OPTIMUS_FORM_ABT) {  // own A_ij [Mb x Kp] times (B_lj)^T, B_lj [Nb x Kp] received along column j
    d.A = off(A, ((long long)i * q + j) * blkA, es); d.a_kcontig = 1; d.lda = Kp;
    d.B = off(B, ((long long)l * q + j) * blkB, es); d.b_kcontig = 1; d.ldb = Kp;
  } else {                                // (A_il)^T, A_il [Kp x Mb] received along row i, times own B_ij [Kp x Nb]
    d.A = off(A, ((long long)i * q + l) * blkA, es); d.a_kcontig = 0; d.lda = Mb;
    d.B = off(B, ((long long)i * q + j) * blkB, es); d.b_kcontig = 0; d.ldb = Nb;
  }
  return launch_gemm(d, as_stream(stream));
}

int optimus_summa_reduce(const float* c_temps, int count, void* C, int64_t M, int64_t N, int q, int root_i, int root_j,
                         int dtype, void* stream) {
  if (!c_temps || !C) return OPTIMUS_EINVAL;
  if (dtype != OPTIMUS_FP32 && dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  if (q <= 0 || M <= 0 || N <= 0 || M % q || N % q || count < 1 || count > 65536) return OPTIMUS_ESHAPE;
  if (root_i < 0 || root_j < 0 || root_i >= q || root_j >= q) return OPTIMUS_ECOORD;
  const long long blk = (M / q) * (N / q);
  return launch_reduce_partials(c_temps, off(C, ((long long)root_i * q + root_j) * blk, esize(dtype)), blk, count, dtype,
                                as_stream(stream));
}

int optimus_bias_grad(const void* dY, float* dbias_part, int64_t M, int64_t N, int q, int i, int j, int dtype, void* stream) {
  if (!dY || !dbias_part) return OPTIMUS_EINVAL;
  if (dtype != OPTIMUS_FP32 && dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  if (q <= 0 || M <= 0 || N <= 0 || M % q || N % q || M / q > 0x7fffffff || N / q > 0x7fffffff) return OPTIMUS_ESHAPE;
  int rc = check_coords(q, i, j);
  if (rc) return rc;
  const int rows = (int)(M / q), cols = (int)(N / q);
  const long long blk = (long long)rows * cols;
  if (is_grid(i, j)) return launch_colsum(dY, dbias_part, rows, cols, cols, q * q, blk, cols, dtype, as_stream(stream));
  const long long dev = (long long)i * q + j;
  return launch_colsum(off(dY, dev * blk, esize(dtype)), dbias_part + dev * cols, rows, cols, cols, 1, blk, cols, dtype,
                       as_stream(stream));
}

int optimus_layernorm2d_stats(const void* X, float* stats, int64_t M, int64_t H, int q, int i, int l, int dtype, void* stream) {
  if (!X || !stats) return OPTIMUS_EINVAL;
  LnDesc d;
  int rc = ln_desc(M, H, q, i, l, dtype, 0.f, &d);
  if (rc) return rc;
  return launch_ln_stats(X, stats, d, as_stream(stream));
}
int optimus_layernorm2d(const void* X, const float* gamma, const float* beta, void* Y, void* xhat, float* rstd, float* stats,
                        int64_t M, int64_t H, int q, int i, int j, float eps, int dtype, void* stream) {
  if (!X || !gamma || !beta || !Y || !xhat || !rstd || !stats) return OPTIMUS_EINVAL;
  if (!(eps >= 0.f)) return OPTIMUS_EINVAL;
  LnDesc d;
  int rc = ln_desc(M, H, q, i, j, dtype, eps, &d);
  if (rc) return rc;
  return ln_forward(X, gamma, beta, Y, xhat, rstd, stats, d, is_grid(i, j), as_stream(stream));
}
int optimus_layernorm2d_bwd_stats(const void* dY, const void* xhat, const float* gamma, float* stats, int64_t M, int64_t H, int q,
                                  int i, int l, int dtype, void* stream) {
  if (!dY || !xhat || !gamma || !stats) return OPTIMUS_EINVAL;
  LnDesc d;
  int rc = ln_desc(M, H, q, i, l, dtype, 0.f, &d);
  if (rc) return rc;
  return launch_ln_bwd_stats(dY, xhat, gamma, stats, d, as_stream(stream));
}
int optimus_layernorm2d_bwd(const void* dY, const void* xhat, const float* rstd, const float* gamma, const void* dres, void* dX,
                            float* dgamma_part, float* dbeta_part, float* stats, int64_t M, int64_t H, int q, int i, int j,
                            int dtype, void* stream) {
  if (!dY || !xhat || !rstd || !gamma || !dX || !stats) return OPTIMUS_EINVAL;
  if ((dgamma_part == nullptr) != (dbeta_part == nullptr)) return OPTIMUS_EINVAL;
  LnDesc d;
  int rc = ln_desc(M, H, q, i, j, dtype, 0.f, &d);
  if (rc) return rc;
  return ln_backward(dY, xhat, rstd, gamma, dres, dX, dgamma_part, dbeta_part, stats, d, is_grid(i, j), as_stream(stream));
}

size_t optimus_attention_workspace_bytes(int b, int s, int h, int n, int q) {
  AttnDims a;
  if (attn_dims(b, s, h, n, q, &a)) return 0;
  return attn_ws_bytes(a);
}
int optimus_attention_fwd(const void* qkv, void* probs, void* attn, int b, int s, int h, int n, int q, int i, int j, int causal,
                          int dtype, void* ws, size_t ws_bytes, void* stream) {
  if (!qkv || !probs || !attn) return OPTIMUS_EINVAL;
  return run_attention(false, qkv, nullptr, probs, nullptr, attn, b, s, h, n, q, i, j, causal ? 1 : 0, dtype, ws, ws_bytes, stream);
}
int optimus_attention_bwd(const void* qkv, const void* probs, const void* d_attn, void* d_qkv, int b, int s, int h, int n, int q,
                          int i, int j, int causal, int dtype, void* ws, size_t ws_bytes, void* stream) {
  if (!qkv || !probs || !d_attn || !d_qkv) return OPTIMUS_EINVAL;
  return run_attention(true, qkv, probs, nullptr, d_attn, d_qkv, b, s, h, n, q, i, j, causal ? 1 : 0, dtype, ws, ws_bytes, stream);
}

int optimus_softmax_rows(const float* scores, void* probs, int64_t nmat, int s, int causal, void* stream) {
  if (!scores || !probs) return OPTIMUS_EINVAL;
  if (nmat < 1 || s < 4 || s % 4 || s > 4096 || nmat * s > 0x7fffffffLL) return OPTIMUS_ESHAPE;
  return launch_softmax_fwd(scores, probs, (int)nmat, s, causal ? 1 : 0, as_stream(stream));
}
int optimus_softmax_rows_bwd(const float* d_probs, const void* probs, void* d_scores, int64_t nmat, int s, int causal,
                             void* stream) {
  if (!d_probs || !probs || !d_scores) return OPTIMUS_EINVAL;
  if (nmat < 1 || s < 4 || s % 4 || s > 4096 || nmat * s > 0x7fffffffLL) return OPTIMUS_ESHAPE;
  return launch_softmax_bwd(d_probs, probs, d_scores, (int)nmat, s, causal ? 1 : 0, as_stream(stream));
}

size_t optimus_attention_fused_workspace_bytes(int b, int s, int h, int n, int q) {
  AttnDims a;
  if (attn_fused_dims(b, s, h, n, q, &a)) return 0;
  return attn_fused_ws_bytes(a, q);
}
int optimus_attention_fused_fwd(const void* qkv, void* attn, float* lse, int b, int s, int h, int n, int q, int i, int j, int causal,
                                int dtype, void* stream) {
  if (!qkv || !attn || !lse) return OPTIMUS_EINVAL;
  return run_attention_fused(false, qkv, attn, lse, nullptr, nullptr, b, s, h, n, q, i, j, causal ? 1 : 0, dtype, nullptr, 0, stream);
}
int optimus_attention_fused_bwd(const void* qkv, const void* attn, const float* lse, const void* d_attn, void* d_qkv, int b, int s,
                                int h, int n, int q, int i, int j, int causal, int dtype, void* ws, size_t ws_bytes, void* stream) {
  if (!qkv || !attn || !lse || !d_attn || !d_qkv) return OPTIMUS_EINVAL;
  return run_attention_fused(true, qkv, const_cast<void*>(attn), const_cast<float*>(lse), d_attn, d_qkv, b, s, h, n, q, i, j,
                             causal ? 1 : 0, dtype, ws, ws_bytes, stream);
}

int optimus_attention_fused_bwd_static(const void* qkv, const void* attn, const float* lse, const void* d_attn, void* d_qkv, int b,
                                       int s, int h, int n, int q, int i, int j, int causal, int dtype, void* stream) {
  if (!qkv || !attn || !lse || !d_attn || !d_qkv) return OPTIMUS_EINVAL;
  if (dtype != OPTIMUS_BF16) return OPTIMUS_EDTYPE;
  AttnDims a;
  int rc = attn_fused_dims(b, s, h, n, q, &a);
  if (rc) return rc;
  if ((rc = check_coords(q, i, j))) return rc;
  // one fp32 per query row of every matrix of the launch (one device's, or the whole grid's)
  const size_t need = (size_t)(is_grid(i, j) ? q * q : 1) * (size_t)a.nmat * (size_t)s * sizeof(float);
  if (need > kStaticScratchBytes) return OPTIMUS_EWORKSPACE;
  void* ws = nullptr;
  if ((rc = static_scratch(&ws))) return rc;
  // the kernels index the scratch by the launch's own device count, so `need` bytes are all they touch; the size
  // check of the shared code path is against the whole-grid size, which the array is not required to hold
  return run_attention_fused(true, qkv, const_cast<void*>(attn), const_cast<float*>(lse), d_attn, d_qkv, b, s, h, n, q, i, j,
                             causal ? 1 : 0, dtype, ws, attn_fused_ws_bytes(a, q), stream);
}

size_t layer_attn_ws(const optimus_layer_cfg* c, const AttnDims& a) {
  return c->fused_attention ? attn_fused_ws_bytes(a, c->q) : attn_ws_bytes(a);
}
int layer_attention(bool bwd, const optimus_layer_cfg* c, const optimus_layer_tensors* t, int i, int j, void* ws, size_t ws_bytes,
                    void* stream) {
  const int causal = c->causal ? 1 : 0;
  if (c->fused_attention)
    return run_attention_fused(bwd, t->qkv, t->attn, t->lse, bwd ? t->d_attn : nullptr, bwd ? t->d_qkv : nullptr, c->b, c->s, c->h,
                               c->n, c->q, i, j, causal, c->dtype, ws, ws_bytes, stream);
  if (bwd)
    return run_attention(true, t->qkv, t->probs, nullptr, t->d_attn, t->d_qkv, c->b, c->s, c->h, c->n, c->q, i, j, causal, c->dtype,
                         ws, ws_bytes, stream);
  return run_attention(false, t->qkv, nullptr, t->probs, nullptr, t->attn, c->b, c->s, c->h, c->n, c->q, i, j, causal, c->dtype, ws,
                       ws_bytes, stream);
}

int optimus_embedding_fwd(const int32_t* tokens, const void* table, void* x, int64_t M, int64_t v, int64_t h, int q, int i, int j,
                          int dtype, void* stream) {
  if (!tokens || !table || !x) return OPTIMUS_EINVAL;
  EndDesc d;
  int rc = end_desc(M, v, h, q, i, j, dtype, &d);
  if (rc) return rc;
  return launch_embedding_fwd(tokens, table, x, d, as_stream(stream));
}
int optimus_embedding_bwd(const int32_t* tokens, const void* d_x, float* d_table, int64_t M, int64_t v, int64_t h, int q, int l,
                          int j, int dtype, void* stream) {
  if (!tokens || !d_x || !d_table) return OPTIMUS_EINVAL;
  EndDesc d;
  int rc = end_desc(M, v, h, q, l, j, dtype, &d);
  if (rc) return rc;
  return launch_embedding_bwd(tokens, d_x, d_table, d, as_stream(stream));
}
int optimus_cross_entropy2d_stats(const void* logits, float* stats, int64_t M, int64_t v, int q, int i, int l, int dtype,
                                  void* stream) {
  if (!logits || !stats) return OPTIMUS_EINVAL;
  EndDesc d;
  int rc = end_desc(M, v, q, q, i, l, dtype, &d);
  if (rc) return rc;
  return launch_ce_stats(logits, stats, d, as_stream(stream));
}
int optimus_cross_entropy2d(const void* logits, const int32_t* labels, float* loss, float* lse, float* stats, int64_t M, int64_t v,
                            int q, int i, int j, int dtype, void* stream) {
  if (!logits || !labels || !loss || !lse || !stats) return OPTIMUS_EINVAL;
  EndDesc d;
  int rc = end_desc(M, v, q, q, i, j, dtype, &d);
  if (rc) return rc;
  if (!is_grid(i, j)) return launch_ce_stats_final(logits, labels, stats, loss, lse, d, as_stream(stream));  // peers resident
  if ((rc = launch_ce_stats(logits, stats, d, as_stream(stream)))) return rc;   // every device's partial first
  return launch_ce_finalize(logits, labels, stats, loss, lse, d, as_stream(stream));
}
int optimus_cross_entropy2d_bwd(const void* logits, const int32_t* labels, const float* lse, void* d_logits, float scale, int64_t M,
                                int64_t v, int q, int i, int j, int dtype, void* stream) {
  if (!logits || !labels || !lse || !d_logits) return OPTIMUS_EINVAL;
  EndDesc d;
  int rc = end_desc(M, v, q, q, i, j, dtype, &d);
  if (rc) return rc;
  return launch_ce_bwd(logits, labels, lse, d_logits, scale, d, as_stream(stream));
}

size_t optimus_layer_workspace_bytes(const optimus_layer_cfg* cfg) {
  AttnDims a;
  if (layer_check(cfg, 0, 0, &a)) return 0;
  // scores scratch of attention + split partials of the activation chain + split partials of the gradient branch
  const size_t gemm_bytes = layer_gemm_ws(cfg);
  return layer_attn_ws(cfg, a) + gemm_bytes + layer_branch_ws(cfg, gemm_bytes);
}

size_t optimus_layer_workspace_bytes_grid(const optimus_layer_cfg* cfg) {
  const size_t base = optimus_layer_workspace_bytes(cfg);
  AttnDims a;
  if (base == 0 || cfg->fused_attention || layer_check(cfg, 0, 0, &a)) return base;
  // scratch for as many devices' attention per launch as stay inside the 256 MB Infinity Cache (at least one)
  const size_t one = attn_ws_bytes(a);
  size_t g = ((size_t)256 << 20) / one;
  const size_t all = (size_t)cfg->q * cfg->q;
  if (g > all) g = all;
  if (g < 1) g = 1;
  return base + (g - 1) * one;
}

}  // extern "C"

// The forward pass; with skip_out the last product (out = h_mid + gelu W2 + b2) is left out: no gradient needs it, so a
// forward pass that is recomputed inside a backward pass with activation checkpointing stops before it (the third
// of the memory-management remarks at the end of Section 3.2.3).
int optimus::layer_forward(const optimus_layer_cfg* c, const optimus_layer_tensors* t, int i, int j, void* ws, size_t ws_bytes,
                           void* stream, bool skip_out) {
  AttnDims a;
  int rc = layer_check(c, i, j, &a);
  if (rc) return rc;
  if (!t) return OPTIMUS_EINVAL;
  if (!t->x || !t->ln1_g || !t->ln1_b || !t->w_qkv || !t->b_qkv || !t->w_o || !t->b_o || !t->ln2_g || !t->ln2_b || !t->w1 ||
      !t->b1 || !t->w2 || !t->b2 || !t->ln1_out || !t->xhat1 || !t->rstd1 || !t->stats1 || !t->qkv ||
      !(c->fused_attention ? (const void*)t->lse : (const void*)t->probs) || !t->attn ||
      !t->h_mid || !t->ln2_out || !t->xhat2 || !t->rstd2 || !t->stats2 || !t->pre_gelu || !t->gelu || (!skip_out && !t->out))
    return OPTIMUS_EINVAL;
  const size_t gemm_bytes = layer_gemm_ws(c);
  if (!ws || ws_bytes < layer_attn_ws(c, a) + 2 * gemm_bytes) return OPTIMUS_EWORKSPACE;
  const int q = c->q, dt = c->dtype;
  const int64_t M = (int64_t)c->b * c->s, h = c->h;
  const bool grid = is_grid(i, j);
  hipStream_t st = as_stream(stream);
  // workspace: [products, chain][products, branch][attention: everything that is left]
  void* gemm_ws = ws;
  void* attn_ws = (char*)ws + 2 * gemm_bytes;
  const size_t attn_bytes = ws_bytes - 2 * gemm_bytes;
  LnDesc ln;
  if ((rc = ln_desc(M, h, q, i, j, dt, c->eps, &ln))) return rc;
  // a1 = LN1(x)
  if ((rc = ln_forward(t->x, t->ln1_g, t->ln1_b, t->ln1_out, t->xhat1, t->rstd1, t->stats1, ln, grid, st))) return rc;
  // qkv = a1 Wqkv + b
  optimus_epilogue e = {};
  e.bias = t->b_qkv;
  if ((rc = run_summa(OPTIMUS_FORM_AB, t->ln1_out, t->w_qkv, t->qkv, M, h, 3 * h, q, i, j, dt, &e, gemm_ws, gemm_bytes, stream))) return rc;
  // local attention
  if ((rc = layer_attention(false, c, t, i, j, attn_ws, attn_bytes, stream))) return rc;
  // h_mid = x + attn Wo + b
  e = {};
  e.bias = t->b_o; e.residual = t->x;
  if ((rc = run_summa(OPTIMUS_FORM_AB, t->attn, t->w_o, t->h_mid, M, h, h, q, i, j, dt, &e, gemm_ws, gemm_bytes, stream))) return rc;
  // a2 = LN2(h_mid)
  if ((rc = ln_forward(t->h_mid, t->ln2_g, t->ln2_b, t->ln2_out, t->xhat2, t->rstd2, t->stats2, ln, grid, st))) return rc;
  // pre = a2 W1 + b ; g = GeLU(pre)
  e = {};
  e.bias = t->b1; e.pre_act = t->pre_gelu; e.act = 1;
  if ((rc = run_summa(OPTIMUS_FORM_AB, t->ln2_out, t->w1, t->gelu, M, h, 4 * h, q, i, j, dt, &e, gemm_ws, gemm_bytes, stream))) return rc;
  if (skip_out) return OPTIMUS_OK;
  // out = h_mid + g W2 + b
  e = {};
  e.bias = t->b2; e.residual = t->h_mid;
  return run_summa(OPTIMUS_FORM_AB, t->gelu, t->w2, t->out, M, 4 * h, h, q, i, j, dt, &e, gemm_ws, gemm_bytes, stream);
}

extern "C" {

int optimus_layer_fwd(const optimus_layer_cfg* c, const optimus_layer_tensors* t, int i, int j, void* ws, size_t ws_bytes,
                      void* stream) {
  return layer_forward(c, t, i, j, ws, ws_bytes, stream, false);
}

int optimus_layer_bwd(const optimus_layer_cfg* c, const optimus_layer_tensors* t, int i, int j, void* ws, size_t ws_bytes,
                      void* stream) {
  AttnDims a;
  int rc = layer_check(c, i, j, &a);
  if (rc) return rc;
  if (!t) return OPTIMUS_EINVAL;
  if (!t->x || !t->ln1_g || !t->w_qkv || !t->w_o || !t->ln2_g || !t->w1 || !t->w2 || !t->ln1_out || !t->xhat1 || !t->rstd1 ||
      !t->qkv || !(c->fused_attention ? (const void*)t->lse : (const void*)t->probs) || !t->attn || !t->ln2_out || !t->xhat2 ||
      !t->rstd2 || !t->pre_gelu || !t->gelu || !t->d_out ||
      !t->d_pre_gelu || !t->d_ln2_out || !t->d_h_mid || !t->d_attn || !t->d_qkv || !t->d_ln1_out || !t->d_x || !t->bstats1 ||
      !t->bstats2 || !t->d_w_qkv || !t->d_w_o || !t->d_w1 || !t->d_w2 || !t->d_b_qkv || !t->d_b_o || !t->d_b1 || !t->d_b2 ||
      !t->d_ln1_g || !t->d_ln1_b || !t->d_ln2_g || !t->d_ln2_b)
    return OPTIMUS_EINVAL;
  const size_t gemm_bytes = layer_gemm_ws(c);
  if (!ws || ws_bytes < layer_attn_ws(c, a) + 2 * gemm_bytes) return OPTIMUS_EWORKSPACE;
  const int q = c->q, dt = c->dtype;
  const int64_t M = (int64_t)c->b * c->s, h = c->h;
  const bool grid = is_grid(i, j);
  hipStream_t st = as_stream(stream);
  // workspace: [products, chain][products, branch][attention: everything that is left]
  void* gemm_ws = ws;
  void* attn_ws = (char*)ws + 2 * gemm_bytes;
  size_t attn_bytes = ws_bytes - 2 * gemm_bytes;
  LnDesc ln;
  if ((rc = ln_desc(M, h, q, i, j, dt, c->eps, &ln))) return rc;
  // gradient branch: its own stream and its own split workspace (see SideStream)
  SideStream* ss = side_stream(st);   // asked for in any case: a later call may be captured, and then it has to be there
  if (ss && !two_streams_pay(c, grid) && !captured(st)) ss = nullptr;
  // LayerNorm 2's parameter gradients need d_ln2_out only.  Small blocks: the chain is a string of short kernels and
  // the column sums are one more serial step of it, so they go to the branch (measured: the step 5 % shorter at
  // [1024 x 256] blocks).  Large blocks: the branch, with its transposing products, is the longer stream already.
  const bool narrow = colsum_narrow((int)(M / q), (int)(h / q));
  // Matrices that share memory: one stream where the branch could still read what the chain overwrites; and step after step in the order
  // of the header where a pair of products or a column sum at the end could.
  if (ss && sharing_breaks(c, t, true, narrow)) ss = nullptr;
  const bool in_order = !ss && sharing_breaks(c, t, false, false);
  const int co_chain = ss ? 1 : 0, co_branch = ss ? 2 : 0;   // products planned for company only where they have it
  hipStream_t gst = ss ? ss->s : st;
  void* gstream = (void*)gst;
  void* grad_ws = ss ? (char*)gemm_ws + gemm_bytes : gemm_ws;
  const bool ln2_grads_on_branch = ss && narrow;
  const bool sums_at_end = ss ? narrow : !in_order;   // small blocks: the column sums are launches, not bytes
  optimus_epilogue e = {};
  optimus_epilogue e32 = {};
  e32.out_fp32 = 1;
  // After the fork the branch stream depends on the caller's stream; whatever happens afterwards, the caller's stream
  // must be joined with it again before this call returns (a stream capture that is left forked cannot be ended).
  // So the first failing step only switches the remaining steps off, and the join below still runs.
  rc = OPTIMUS_OK;
  bool forked = false;
#define RUN(...) do { if (rc == OPTIMUS_OK) rc = (__VA_ARGS__); } while (0)
#define BRANCH_AFTER_MAIN(EV) do { if (ss && rc == OPTIMUS_OK) { rc = stream_after(gst, st, EV); forked = forked || rc == OPTIMUS_OK; } } while (0)
  BRANCH_AFTER_MAIN(ss->fork);
  // ---- out = h_mid + gelu W2 + b2 ----
  // One stream: both products of a linear layer in one launch, the partial tiles of a panel split combined where they are needed: those
  // of d_ln1_out and d_ln2_out by the LayerNorm, the weight gradients' at the end of the pass (if the workspace holds them that long;
  // otherwise at once).  Two: the gradient of the weight on the branch.
  CombineJob in_job = {};
  CombineJobs w_jobs = {};
  size_t w_at[4], w_total = 0;
  if (!ss && !in_order) layer_weight_ws(c, i, j, w_at, &w_total);
  const size_t branch_bytes = w_total > gemm_bytes ? w_total : gemm_bytes;
  const bool keep = w_total > 0 && ws_bytes >= layer_attn_ws(c, a) + gemm_bytes + branch_bytes;
  if (keep) {
    attn_ws = (char*)ws + gemm_bytes + branch_bytes;
    attn_bytes = ws_bytes - gemm_bytes - branch_bytes;
  }
  const auto linear = [&](int nth, const void* d_y, const void* w, const void* in, void* d_in, float* d_w, int64_t k, int64_t n,
                          const void* gelu_grad_of) {
    const LinearGrads g = {d_y, w, in, d_in, d_w, M, k * h, n * h, gelu_grad_of};
    if (!ss && !in_order) {
      char* const branch = (char*)gemm_ws + gemm_bytes;
      const size_t bytes = !keep ? gemm_bytes : nth < 3 ? w_at[nth + 1] - w_at[nth] : w_total - w_at[nth];
      int r = run_linear_grads(g, q, i, j, gemm_ws, gemm_bytes, branch + (keep ? w_at[nth] : 0), bytes, &in_job, &w_jobs, st);
      if (r) return r;
      CombineJobs now = {};
      if (in_job.partials && nth % 2 == 0) { now.j[now.n++] = in_job; in_job = CombineJob{}; }   // no LayerNorm follows
      if (!keep) {
        for (int m = 0; m < w_jobs.n; ++m) now.j[now.n++] = w_jobs.j[m];
        w_jobs.n = 0;
      }
      return launch_gemm_combines(now, st);
    }
    e = {}; e.gelu_grad_of = gelu_grad_of;
    const int r = run_summa(OPTIMUS_FORM_ABT, d_y, w, d_in, M, n * h, k * h, q, i, j, dt, &e, gemm_ws, gemm_bytes, stream, co_chain);
    if (r) return r;
    return run_summa(OPTIMUS_FORM_ATB, in, d_y, d_w, k * h, M, n * h, q, i, j, dt, &e32, grad_ws, gemm_bytes, gstream, co_branch);
  };
  // LayerNorm backward behind linear(): its input, d_y, is complete or the partial tiles of in_job
  const auto norm_bwd = [&](const void* d_y, const void* xhat, const float* rstd, const float* gamma, const void* d_res, void* d_in, float* d_g,
                            float* d_b, float* stats) {
    if (in_job.partials) {
      if (!d_g && ln_bwd_partials_ok(in_job, d_y, xhat, gamma, d_res, d_in, ln))
        return launch_ln_bwd_partials(in_job, xhat, rstd, gamma, d_res, d_in, stats, ln, st);
      CombineJobs now = {};
      now.j[now.n++] = in_job;
      const int r = launch_gemm_combines(now, st);
      if (r) return r;
    }
    if (in_order) {   // the sums first: d_in may take d_y's place
      const int r = launch_ln_param_grads(d_y, xhat, d_g, d_b, ln, st);
      return r ? r : ln_backward(d_y, xhat, rstd, gamma, d_res, d_in, nullptr, nullptr, stats, ln, grid, st);
    }
    return ln_backward(d_y, xhat, rstd, gamma, d_res, d_in, d_g, d_b, stats, ln, grid, st);
  };
  RUN(linear(0, t->d_out, t->w2, t->gelu, t->d_pre_gelu, t->d_w2, 4, 1, t->pre_gelu));   // d_pre = (d_out W2^T) * GeLU'(pre)
  if (ss || in_order) RUN(optimus_bias_grad(t->d_out, t->d_b2, M, h, q, i, j, dt, gstream));
  // ---- pre = ln2_out W1 + b1 ----
  BRANCH_AFTER_MAIN(ss->ready[0]);  // d_pre_gelu is complete
  RUN(linear(1, t->d_pre_gelu, t->w1, t->ln2_out, t->d_ln2_out, t->d_w1, 1, 4, nullptr));
  if (!sums_at_end) RUN(optimus_bias_grad(t->d_pre_gelu, t->d_b1, M, 4 * h, q, i, j, dt, gstream));
  // ---- LN2 backward, plus the residual branch: d_h_mid = d_out + LN2'(d_ln2_out) ----
  RUN(norm_bwd(t->d_ln2_out, t->xhat2, t->rstd2, t->ln2_g, t->d_out, t->d_h_mid, sums_at_end ? nullptr : t->d_ln2_g,
               sums_at_end ? nullptr : t->d_ln2_b, t->bstats2));
  // ---- h_mid = x + attn Wo + bo ----
  BRANCH_AFTER_MAIN(ss->ready[1]);  // d_h_mid is complete
  RUN(linear(2, t->d_h_mid, t->w_o, t->attn, t->d_attn, t->d_w_o, 1, 1, nullptr));
  if (!sums_at_end) RUN(optimus_bias_grad(t->d_h_mid, t->d_b_o, M, h, q, i, j, dt, gstream));
  // ---- local attention backward ----
  RUN(layer_attention(true, c, t, i, j, attn_ws, attn_bytes, stream));
  // ---- qkv = ln1_out Wqkv + b ----
  BRANCH_AFTER_MAIN(ss->ready[2]);  // d_qkv is complete
  RUN(linear(3, t->d_qkv, t->w_qkv, t->ln1_out, t->d_ln1_out, t->d_w_qkv, 1, 3, nullptr));
  if (!sums_at_end) RUN(optimus_bias_grad(t->d_qkv, t->d_b_qkv, M, 3 * h, q, i, j, dt, gstream));
  // ---- LN1 backward, plus the residual branch: d_x = d_h_mid + LN1'(d_ln1_out) ----
  // On one stream ahead of the sums, which then find d_ln1_out complete; behind them if d_x takes the place of what they read.
  const auto takes = [&](const void* p, int64_t k) {
    const char *x0 = (const char*)t->d_x, *p0 = (const char*)p;
    return x0 < p0 + M * k * h * 2 && p0 < x0 + M * h * 2;
  };
  const bool norm_last = ss || in_order || takes(t->d_pre_gelu, 4) || takes(t->d_qkv, 3) || takes(t->d_ln2_out, 1) || takes(t->xhat2, 1) ||
                         takes(t->d_h_mid, 1) || takes(t->d_ln1_out, 1) || takes(t->xhat1, 1) || takes(t->d_out, 1);
  if (norm_last && in_job.partials) {
    CombineJobs now = {};
    now.j[now.n++] = in_job;
    in_job = CombineJob{};
    RUN(launch_gemm_combines(now, st));
  }
  const auto norm1 = [&]() {
    return norm_bwd(t->d_ln1_out, t->xhat1, t->rstd1, t->ln1_g, t->d_h_mid, t->d_x, ss || in_order ? t->d_ln1_g : nullptr,
                    ss || in_order ? t->d_ln1_b : nullptr, t->bstats1);
  };
  if (!norm_last) RUN(norm1());
  if (sums_at_end) {   // column sums, and the combines kept so far, in one launch; the sources are still there; on a branch without the two that
                       // would wait
    const int rows = (int)(M / q), hb = (int)(h / q);
    const long long dev = grid ? 0 : (long long)i * q + j;
    const auto job = [&](const void* X, const void* W, float* sum, float* sum_w, int k) {
      const long long at = dev * rows * k * hb, to = dev * k * hb;
      return ColsumJob{off(X, at, 2), off(W, at, 2), sum + to, W ? sum_w + to : nullptr, k * hb};
    };
    const ColsumJobs jobs = {{job(t->d_pre_gelu, nullptr, t->d_b1, nullptr, 4), job(t->d_qkv, nullptr, t->d_b_qkv, nullptr, 3),
                              job(t->d_ln2_out, t->xhat2, t->d_ln2_b, t->d_ln2_g, 1), job(t->d_h_mid, nullptr, t->d_b_o, nullptr, 1),
                              job(t->d_ln1_out, t->xhat1, t->d_ln1_b, t->d_ln1_g, 1), job(t->d_out, nullptr, t->d_b2, nullptr, 1)}, ss ? 4 : 6};
    RUN(launch_colsum_jobs(jobs, rows, grid ? q * q : 1, &w_jobs, gst));
  }
  if (norm_last) RUN(norm1());
  // the caller's stream owns every result again
  if (ss && forked) {
    const int jr = stream_after(st, gst, ss->join);
    if (rc == OPTIMUS_OK) rc = jr;
  }
#undef BRANCH_AFTER_MAIN
#undef RUN
  return rc;
}

int64_t optimus_gemm_flops(int64_t M, int64_t K, int64_t N, int q) {
  if (check_mkn(M, K, N, q)) return -1;
  return 2 * (M / q) * K * (N / q);
}

int64_t optimus_layer_flops(const optimus_layer_cfg* c, int what) {
  AttnDims a;
  if (layer_check(c, 0, 0, &a) || what < 0 || what > 1) return -1;
  const int64_t b = c->b, s = c->s, h = c->h, p = (int64_t)c->q * c->q;
  const int64_t fwd = 2 * (12 * b * s * h * h + 2 * b * s * s * h) / p;
  return what == 0 ? fwd : 2 * fwd;
}

int optimus_debug_mfma_rate(float* out, int workgroups, int iters, int random_data, void* stream) {
  if (!out) return OPTIMUS_EINVAL;
  if (workgroups < 1 || workgroups > 65536 || iters < 1 || iters > (1 << 24)) return OPTIMUS_ESHAPE;
  return launch_mfma_rate(out, workgroups, iters, random_data ? 1 : 0, as_stream(stream));
}

// ---- tuning hook used by the benchmark (not part of the method): force a matrix-core tile variant, -1 = automatic ----
void optimus_debug_set_gemm_variant(int v) { gemm_set_variant(v); }
void optimus_debug_set_corun_variants(int chain_v, int branch_v) { gemm_set_corun_variants(chain_v, branch_v); }
int optimus_debug_plan_summa(int form, int64_t M, int64_t K, int64_t N, int q, int i, int j, int corun, int have_ws, int* out3) {
  if (!out3 || form < 0 || form > 2 || corun < 0 || corun > 2) return OPTIMUS_EINVAL;
  int rc = check_mkn(M, K, N, q);
  if (rc) return rc;
  rc = check_coords(q, i, j);
  if (rc) return rc;
  // the plan depends on shapes, strides and 16-byte alignment only: a fixed aligned address stands in for the tensors
  void* const fake = (void*)(uintptr_t)4096;
  GemmDesc d = summa_desc(form, fake, fake, fake, M, K, N, q, i, j, OPTIMUS_BF16, nullptr);
  d.corun = corun;
  return gemm_plan_of(d, have_ws != 0, out3) ? OPTIMUS_OK : OPTIMUS_EDTYPE;
}
int optimus_debug_plan_pair(int64_t M, int64_t K, int64_t N, int q, int i, int j) {
  if (check_mkn(M, K, N, q) || check_coords(q, i, j)) return -1;
  return pair_planned(M, K, N, q, i, j) ? 1 : 0;
}
int optimus_debug_last_gemm_plan(void) { return gemm_last_plan(); }
int optimus_debug_layer_bwd_streams(const optimus_layer_cfg* c, int i, int j) {
  AttnDims a;
  if (layer_check(c, i, j, &a)) return -1;
  return two_streams_pay(c, is_grid(i, j)) ? 2 : 1;
}

}  // extern "C"
