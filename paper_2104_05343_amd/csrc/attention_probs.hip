// Local attention that keeps the probabilities (the paper's Sections 2.1 / 3.2.1: whole sequences and n/q heads are local to a
// device), without the score matrices in memory.
//
//   forward   P = softmax(Q K^T / sqrt(d)) and O = P V:                     one launch for scores, soft-max and P V
//   backward  dS = P o (dO V^T - rowsum(P o dO V^T)) and dQ = dS K / sqrt(d): one launch for dP, the soft-max's gradient and dQ
//             (dV = P^T dO and dK = dS^T Q contract over the rows and stay products of their own)
//
// Both are the same kernel: the rows a workgroup owns ("own": Q or dO) against all rows of one [s x d] matrix ("x": K or V) give a
// tile of numbers that needs one statistic per row (maximum and sum, or the rowsum) before it is final; the final tile goes to
// memory in bf16 and multiplies the rows of the other matrix ("y": V or K).  So the tiles are walked twice, first for the
// statistic, then, computed again, for the results: the matrix instructions spent twice (0.25 of the pass's at d = 64) cost
// less than fp32 scores written and read (four times the bytes of P).  The products, layouts and the two wavefront parities
// are those of attention_fused_kernel.hpp.  P is rounded to bf16 before it meets V, as what is saved.
//
// What bounds it: P itself (s * s * 2 bytes a matrix; with the mask half of it is zeros that are written all the same).  A
// lane's accumulators are 16 numbers of one row, 8 bytes side by side; stored so, every 128-byte line would be completed by
// sixteen writes.  A wavefront's 32 rows pass through LDS of its own and leave as 64 or 128 bytes a row, and a wait for the
// next tiles leaves those stores in flight.
//
// Measured, us, whole calls (the backward with dV and dK), separate launches / these, causal and without a mask.  128 matrices, s = 512,
// d = 64 (all devices of a 1024-wide layer on a 4 x 4 grid): forward 61 / 27 (64 MiB of P: 2.5 TB/s) and 78 / 32, backward 94 / 58 and
// 134 / 78.  16 matrices, s = 1024, d = 128 (one device of a 4096-wide layer): forward 39 / 31 and 51 / 31, backward 60 / 57 and 75 / 61.
// Passes with the separate launches and with these: checkpointed stack of four such 1024-wide layers 3721 / 3112, 4096-wide layer
// 871 / 846, two 256-wide layers 321 / 301.
#include "attention_fused_kernel.hpp"

namespace optimus {
namespace {

struct ProbArgs {
  const bf16_t* own;       // Q (inside qkv) or dO
  const bf16_t* x;         // K or V, inside qkv
  const bf16_t* y;         // V or K, inside qkv
  const bf16_t* p_in;      // backward: P
  bf16_t* tile_out;        // [matrix][s][s]: P or dS
  bf16_t* out;             // O or dQ
  int s, nh;
  int ld, ld_own, ld_out;  // row lengths of qkv, own and out
  int h_own, h_out;        // distance of two heads in own and out (3d inside qkv)
  float scale, scale_log2;
};

// s_waitcnt vmcnt(n) lgkmcnt(0), gfx9 encoding; the builtin, so that the compiler's own wait counts know what has landed
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Zeros of dS beyond the diagonal are read by dK's tiles only, which start at their first row: up to the end of a tile's rows.
constexpr int kTileRows = 256;

template <int D, bool CAUSAL, int NRG, bool BWD>
__global__ __launch_bounds__(NRG * 128) void attn_probs_kernel(ProbArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int KS = D / 16, DT = D / 32, BQ = NRG * 32, NW = 2 * NRG;
  constexpr int TPC = D == 128 && NRG == 4 ? 1 : 2;   // 32-column tiles that leave together (LDS: 160 KiB)
  constexpr int PITCH = TPC * 64 + 16, LPR = TPC * 4, RPI = 64 / LPR, NIT = 32 / RPI;
  constexpr int STORES = 2 / TPC * NIT;               // per block and wavefront
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][PAIR * D];   // [stage][x, y][pair tile]
  __shared__ __attribute__((aligned(16))) char lds_out[NW][32 * PITCH];
  __shared__ float lds_stat[NW][2][64];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave % NRG, par = wave / NRG;
  const int tile = gridDim.y - 1 - blockIdx.y;        // all matrices' longest causal loops first
  const int mat = blockIdx.x, s = a.s;
  const int seq = mat / a.nh, head = mat % a.nh;
  const bf16_t* Xp = a.x + (long long)seq * s * a.ld + head * 3 * D;
  const bf16_t* Yp = a.y + (long long)seq * s * a.ld + head * 3 * D;
  const int q0 = tile * BQ + rg * 32;
  const int row = q0 + (lane & 31);
  const int rowc = min(row, s - 1);
  const bf16_t* Op = a.own + ((long long)seq * s + rowc) * a.ld_own + head * a.h_own;
  bf16x8 of[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) of[ks] = *(const bf16x8*)(Op + ks * 16 + g * 8);
  const int wg_hi = min(tile * BQ + BQ, s) - 1;
  const int nkb_all = (s + BLK - 1) / BLK;
  const int nkb = CAUSAL ? wg_hi / BLK + 1 : nkb_all;
  const int n_it = (nkb + 1) / 2;
  const int wave_nkb = q0 >= s ? 0 : (CAUSAL ? min(q0 + 31, s - 1) / BLK + 1 : nkb);
  const int limit = CAUSAL ? rowc : s - 1;            // last column this lane's row has
  bf16_t* const Tp = a.tile_out + (long long)mat * s * s;

  TileLoader<D, NW, PAIR, true> ldr;
  ldr.init(a.ld, wave, lane);
  u32x4 p_next[4];   // backward: P of the next block, 16 bytes a lane: columns 16 * n + 8 * g + 0..7 of the lane's row
  auto load_p = [&](int kb) {
    const bf16_t* src = a.p_in + ((long long)mat * s + rowc) * s;
#pragma unroll
    for (int n = 0; n < 4; ++n) p_next[n] = *(const u32x4*)(src + min(kb * BLK + n * 16 + g * 8, s - 8));
  };
  // 32 of the block's 64 columns of this wavefront's rows, transposed: own rows x rows of tile tX
  auto scores = [&](f32x16& acc, const bf16_t* tX, int t2) {
    acc = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<D>(tX, t2 * 32, ks, lane), of[ks], acc, 0, 0, 0);
  };
  const auto column = [&](int kbase, int t2, int r) { return kbase + t2 * 32 + 8 * (r >> 2) + 4 * g + (r & 3); };   // of slot r
  // P as loaded -> P of tile t2 in accumulator order, fp32, zero past the row's last column
  auto spread_p = [&](f32x16& p, const u32x4 (&w)[4], int kbase, int t2, bool need_mask) {
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(w[2 * t2 + n][k], w[2 * t2 + n][2 + k], false, false);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          p[(2 * n + c) * 4 + 2 * k] = __uint_as_float(r[c] << 16);
          p[(2 * n + c) * 4 + 2 * k + 1] = __uint_as_float(r[c] & 0xffff0000u);
        }
      }
    if (need_mask) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (column(kbase, t2, r) > limit) p[r] = 0.f;
    }
  };
  // exp of a score against the row's largest.  The difference first: it is 0 for the largest itself, where one fused multiply-add
  // keeps the rounding error of the largest's product, which is beyond any exponent for scores of 1e9.  The second operation is 2 to
  // 5 % of the forward: 16 matrices, s = 2048, d = 64, causal 44.6 -> 46.7 us, 20 without a mask 84 -> 89.
  auto weight = [&](float score, float largest) { return __builtin_amdgcn_exp2f((score - largest) * a.scale_log2); };
  auto masked = [&](int kbase) { return CAUSAL ? kbase + BLK - 1 > q0 : kbase + BLK > s; };   // uniform

  // ---- first walk: maximum and sum of a row (forward), or its rowsum (backward)
  // The maximum starts at a finite number: blocks whose scores are all -inf add exp(-inf) = 0.  A row of nothing else is 0 / 0.
  float m_run = -__FLT_MAX__, l_run = 0.f;            // backward: l_run only
  ldr.issue(Xp, 0, s, lds[0][0]);
  if constexpr (BWD) load_p(par);
  wait_and_barrier<0>();
  for (int it = 0; it < n_it; ++it) {
    const int st = it & 1, kb = 2 * it + par, kbase = kb * BLK;
    u32x4 p_cur[4];
    if constexpr (BWD) {
#pragma unroll
      for (int n = 0; n < 4; ++n) p_cur[n] = p_next[n];
      load_p(it + 1 < n_it ? kb + 2 : par);
    }
    if (it + 1 < n_it) {
      ldr.issue(Xp, (it + 1) * PAIR, s, lds[st ^ 1][0]);
    } else {                                          // the second walk's first pair
      ldr.issue(Xp, 0, s, lds[st ^ 1][0]);
      ldr.issue(Yp, 0, s, lds[st ^ 1][1]);
    }
    if (kb < wave_nkb) {
      const bf16_t* tX = lds[st][0] + par * BLK * D;
      const bool need_mask = masked(kbase);
      if constexpr (BWD) {
        float dot = 0.f;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          f32x16 acc, p;
          scores(acc, tX, t2);
          spread_p(p, p_cur, kbase, t2, need_mask);
#pragma unroll
          for (int r = 0; r < 16; ++r) dot = fmaf(p[r], need_mask && column(kbase, t2, r) > limit ? 0.f : acc[r], dot);
        }
        l_run += dot;
      } else {
        f32x16 acc[2];
        float mx = -INFINITY;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          scores(acc[t2], tX, t2);
          if (need_mask) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (column(kbase, t2, r) > limit) acc[t2][r] = -INFINITY;
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[t2][r]);
        }
        const float m_new = fmaxf(m_run, halfwave_max(mx));
        float sum = 0.f;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int r = 0; r < 16; ++r) sum += weight(acc[t2][r], m_new);
        l_run = fmaf(l_run, weight(m_run, m_new), sum);
        m_run = m_new;
      }
    }
    if (it + 1 == n_it) {
      lds_stat[wave][0][lane] = halfwave_sum(l_run);
      if constexpr (!BWD) lds_stat[wave][1][lane] = m_run;
    }
    wait_and_barrier<0>();
  }
  // of both parities, the even one first: the two wavefronts of a row agree on every bit
  float stat_m = 0.f, stat_l;
  {
    const float l0 = lds_stat[rg][0][lane], l1 = lds_stat[rg + NRG][0][lane];
    if constexpr (BWD) {
      stat_l = l0 + l1;
    } else {
      const float m0 = lds_stat[rg][1][lane], m1 = lds_stat[rg + NRG][1][lane];
      stat_m = fmaxf(m0, m1);                         // where the odd parity had no block l1 is 0
      stat_l = 1.0f / (l0 * weight(m0, stat_m) + l1 * weight(m1, stat_m));
    }
  }

  // ---- second walk: the final tiles, and their product with y
  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) oacc[dt] = zero16();
  for (int it = 0; it < n_it; ++it) {
    const int st = (n_it + it) & 1, kb = 2 * it + par, kbase = kb * BLK;
    u32x4 p_cur[4];
    if constexpr (BWD) {
#pragma unroll
      for (int n = 0; n < 4; ++n) p_cur[n] = p_next[n];
      load_p(kb + 2);
    }
    if (it + 1 < n_it) {
      ldr.issue(Xp, (it + 1) * PAIR, s, lds[st ^ 1][0]);
      ldr.issue(Yp, (it + 1) * PAIR, s, lds[st ^ 1][1]);
    }
    const bool inside = kb < wave_nkb && q0 + 32 <= s && kbase + BLK <= s;   // uniform: all rows and columns exist
    if (kb < wave_nkb) {
      const bf16_t* tX = lds[st][0] + par * BLK * D;
      const bf16_t* tY = lds[st][1] + par * BLK * D;
      const bool need_mask = masked(kbase);
      char* const chunk = lds_out[wave];
      f32x16 acc[2];
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) scores(acc[t2], tX, t2);
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        if constexpr (BWD) {
          f32x16 p;
          spread_p(p, p_cur, kbase, t2, need_mask);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[t2][r] = p[r] * (acc[t2][r] - stat_l);
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[t2][r] = weight(acc[t2][r], stat_m) * stat_l;
        }
        if (need_mask) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (column(kbase, t2, r) > limit) acc[t2][r] = 0.f;
        }
        const bf16x8 pf[2] = {pack_acc<0>(acc[t2]), pack_acc<1>(acc[t2])};
        char* wr = chunk + (lane & 31) * PITCH + (t2 % TPC) * 64 + g * 8;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const u32x4 w = __builtin_bit_cast(u32x4, pf[u]);
          *(u32x2*)(wr + u * 32) = u32x2{w[0], w[1]};
          *(u32x2*)(wr + u * 32 + 16) = u32x2{w[2], w[3]};
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_acc_order<D>(tY, t2 * 32 + u * 16, dt * 32, lane), pf[u],
                                                               oacc[dt], 0, 0, 0);
        if ((t2 + 1) % TPC == 0) {   // LDS operations of one wavefront execute in order
          asm volatile("" ::: "memory");
          const int col = kbase + (t2 + 1 - TPC) * 32 + (lane % LPR) * 8;
#pragma unroll
          for (int k = 0; k < NIT; ++k) {
            const int r = k * RPI + lane / LPR;
            const u32x4 v = *(const u32x4*)(chunk + r * PITCH + (lane % LPR) * 16);
            if (inside) *(u32x4*)(Tp + (long long)(q0 + r) * s + col) = v;
            else if (q0 + r < s && col < s) *(u32x4*)(Tp + (long long)(q0 + r) * s + col) = v;
          }
          asm volatile("" ::: "memory");
        }
        if constexpr (BWD && D == 128) __builtin_amdgcn_sched_barrier(0);   // (registers)
      }
    }
    // the next pair's loads are older than this block's stores, which may stay in flight
    if (inside) wait_and_barrier<STORES>();
    else wait_and_barrier<0>();
  }
  // merge the two parities; all tiles are free
  float* xch = (float*)&lds[0][0][0] + rg * (DT * 16) * 64;
  if (par == 1) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[(dt * 16 + r) * 64 + lane] = oacc[dt][r];
  }
  __syncthreads();
  if (par == 0 && row < s) {
    const float w = BWD ? a.scale : 1.0f;
    bf16_t* dst = a.out + ((long long)seq * s + row) * a.ld_out + head * a.h_out;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (oacc[dt][4 * c + e] + xch[(dt * 16 + 4 * c + e) * 64 + lane]) * w;
        *(u32x2*)(dst + dt * 32 + 8 * c + 4 * g) = u32x2{pack2_bf16(o[0], o[1]), pack2_bf16(o[2], o[3])};
      }
  }
  if constexpr (CAUSAL) {   // exact zeros in the blocks that were not walked
    const int end = BWD ? min(s, (q0 / kTileRows + 1) * kTileRows) : s;
    const int col = (lane & 7) * 8;
    if (q0 < s)
      for (int kb = wave_nkb + ((wave_nkb ^ par) & 1); kb * BLK < end; kb += 2)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = q0 + k * 8 + (lane >> 3);
          if (r < s && kb * BLK + col < s) *(u32x4*)(Tp + (long long)r * s + kb * BLK + col) = u32x4{0, 0, 0, 0};
        }
  }
#endif
}

template <int D, bool CAUSAL, bool BWD>
void launch_rows(const ProbArgs& a, long long nmat, hipStream_t st) {
  // Workgroups of 64 or of 128 rows (half the tiles' bytes per row); the sums are the same, and either kind has a compute unit to
  // itself (LDS).  A workgroup of 64 is 0.85 of the time, so without a mask 64 rows where those workgroups are one round, 128 from
  // the first that would be the second on.  With the mask the second round is short tiles behind long ones: 128 rows from one
  // workgroup of theirs per compute unit on.  64 / 128 rows, us, forward: 256 of 64 rows, mask 22 / 25 (16 matrices, s = 1024, d = 64),
  // none 22 / 26; 288 (12, 1536, 64) 30 / 34 and 55 / 35; 384 (24, 1024, 64) 25 / 26 and 40 / 27; 512 (32, 1024, 64) 30 / 26 and 41 / 28;
  // the backward the same way, 0.86 of the time to 1.02 with the mask, 0.86 to 1.2 without.  Short rows have little to
  // fill in behind: 384 of (96, 256, 64) with the mask 15 / 11.
  const long long cus = num_cus();
  const bool big = CAUSAL ? (a.s + 127) / 128 * nmat >= cus : (a.s + BLK - 1) / BLK * nmat > cus;
  const int rows = big ? 128 : BLK;
  const dim3 grid((unsigned)nmat, (a.s + rows - 1) / rows);
  if (big) attn_probs_kernel<D, CAUSAL, 4, BWD><<<grid, 512, 0, st>>>(a);
  else attn_probs_kernel<D, CAUSAL, 2, BWD><<<grid, 256, 0, st>>>(a);
}
template <bool BWD>
int launch_form(const ProbArgs& a, int d, int causal, long long nmat, hipStream_t st) {
  if (d == 64 && causal) launch_rows<64, true, BWD>(a, nmat, st);
  else if (d == 64) launch_rows<64, false, BWD>(a, nmat, st);
  else if (causal) launch_rows<128, true, BWD>(a, nmat, st);
  else launch_rows<128, false, BWD>(a, nmat, st);
  return hip_launch_status();
}
ProbArgs make_args(const AttnProbsDesc& d) {
  ProbArgs a = {};
  a.s = d.s; a.nh = d.nh; a.ld = d.ld;
  a.scale = 1.0f / sqrtf((float)d.d);
  a.scale_log2 = a.scale * LOG2E;
  return a;
}

}  // namespace

bool attn_probs_supported(const AttnProbsDesc& d) {
  const auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if (!attn_fused_supported(d.d) || d.s % 8 || d.s < 8 || d.ld % 8 || d.ldo % 8) return false;
  if ((long long)PAIR * d.ld * 2 >= (1ll << 31) || d.nmat > 0x7fffffffll) return false;   // offsets inside a pair tile; grid x
  return al16(d.qkv) && al16(d.probs) && al16(d.attn) && al16(d.d_attn) && al16(d.d_scores) && al16(d.d_qkv);
}

int launch_attn_probs_fwd(const AttnProbsDesc& d, hipStream_t st) {
  ProbArgs a = make_args(d);
  const bf16_t* qkv = (const bf16_t*)d.qkv;
  a.own = qkv; a.ld_own = d.ld; a.h_own = 3 * d.d;
  a.x = qkv + d.d; a.y = qkv + 2 * d.d;
  a.tile_out = (bf16_t*)d.probs;
  a.out = (bf16_t*)d.attn; a.ld_out = d.ldo; a.h_out = d.d;
  return launch_form<false>(a, d.d, d.causal, d.nmat, st);
}

int launch_attn_probs_bwd(const AttnProbsDesc& d, hipStream_t st) {
  ProbArgs a = make_args(d);
  const bf16_t* qkv = (const bf16_t*)d.qkv;
  a.own = (const bf16_t*)d.d_attn; a.ld_own = d.ldo; a.h_own = d.d;
  a.x = qkv + 2 * d.d; a.y = qkv + d.d;
  a.p_in = (const bf16_t*)d.probs;
  a.tile_out = (bf16_t*)d.d_scores;
  a.out = (bf16_t*)d.d_qkv; a.ld_out = d.ld; a.h_out = 3 * d.d;
  return launch_form<true>(a, d.d, d.causal, d.nmat, st);
}

}  // namespace optimus
