// The backward of the fused attention in workgroups of eight wavefronts (see attention_fused_kernel.hpp).  A translation unit of
// its own: compiled together with these kernels, the forward at head width 128 came out with other address arithmetic (30
// instructions more) and 2 to 5 % slower.
#include "attention_fused_kernel.hpp"

namespace optimus {
namespace {

// Head width 128: 128 keys per workgroup, eight wavefronts, two per SIMD, so that one's matrix instructions run beside the
// other's soft-max arithmetic and LDS reads.  A lane has 256 registers then, and 128 of them are the dK and dV
// accumulators: the wavefront's own V fragments and half of its K fragments stay in LDS (with all of K in registers a
// dozen were spilled, and with the mask in a branch of its own), the blocks come one at a time, and a wavefront takes one
// 32-query half (par) of every 64-query block instead of every second block.
// The queries' lse and rowsum(dO * O) go through a register and reach LDS at the end of an iteration: stored at its top,
// the store would wait for its load and for all the tile loads issued before it.
// Bound: LDS reads (44 KiB per wavefront and 32 x 32 scores, beside 1024 clk of matrix instructions).  Measured, 16
// matrices, s = 4096, causal: four wavefronts with every fragment in registers, 64 keys per workgroup, 456 us; with that 313, and with fragments read ahead of their use 282 for the whole backward.
template <int D>
struct WideLds {
  bf16_t block[2][2][BLK * D];   // [stage][Q, dO]
  bf16_t v[128 * D], k[128 * D]; // the workgroup's own rows
  float l[2][BLK], d[2][BLK];
};
// 32 x 32 scores S (rows: queries q0 .., columns: keys) and dP = dO V^T in accumulators -> P and dS in their place.
// l, d: lse * log2(e) and rowsum(dO * O) of the 32 queries.
template <bool CAUSAL>
__device__ __forceinline__ void dkv_scores(f32x16& sacc, f32x16& pacc, const float* l, const float* d, int q0, int key, int s, bool need_mask,
                                           float scale_log2, int g) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int qi = 8 * c + 4 * g;
    const float4 l4 = *(const float4*)(l + qi);
    const float4 d4 = *(const float4*)(d + qi);
    const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 4 * c + e, qy = q0 + qi + e;
      float p = __builtin_amdgcn_exp2f(fmaf(sacc[r], scale_log2, -lv[e]));
      float ds = p * (pacc[r] - dv[e]);
      if (need_mask && (qy >= s || (CAUSAL && qy < key))) { p = 0.f; ds = 0.f; }
      sacc[r] = p;
      pacc[r] = ds;
    }
  }
}
template <int D, bool CAUSAL>
__device__ __forceinline__ void bwd_dkv_wide_body(const FusedArgs& a, WideLds<D>& lds, int tile, int mat, int dev) {
  constexpr int KS = D / 16, DT = D / 32, BKW = 128, KREG = KS / 2;   // KREG: K fragments kept in registers
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave & 3, par = wave >> 2;
  const int s = a.s;
  const int seq = mat / a.nh, head = mat % a.nh;
  const bf16_t* Qp = a.qkv + dev * a.dev_qkv + (long long)seq * s * a.ld + head * 3 * D;
  const bf16_t* Kp = Qp + D;
  const bf16_t* Gp = a.d_attn + dev * a.dev_attn + (long long)seq * s * a.ldo + head * D;
  const float* Lp = a.lse + dev * a.dev_vec + (long long)mat * s;
  const float* Dp = a.delta + dev * a.dev_vec + (long long)mat * s;
  const int k0 = tile * BKW + rg * 32;
  const int key = k0 + (lane & 31);
  const int krow = min(key, s - 1);
  bf16x8 kf[KREG];
#pragma unroll
  for (int ks = 0; ks < KREG; ++ks) kf[ks] = *(const bf16x8*)(Kp + (long long)krow * a.ld + ks * 16 + g * 8);
  const int nqb = (s + BLK - 1) / BLK;
  const int qb_lo = CAUSAL ? (tile * BKW) / BLK : 0;
  const int n_it = nqb - qb_lo;

  f32x16 dkacc[DT], dvacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    dkacc[dt] = zero16();
    dvacc[dt] = zero16();
  }
  {
    TileLoader<D, 8, BKW> ldv;
    ldv.init(a.ld, wave, lane);
    ldv.issue(Qp + 2 * D, tile * BKW, s, lds.v);
    ldv.issue(Kp, tile * BKW, s, lds.k);
  }
  TileLoader<D, 8, BLK> ldq, ldg;
  ldq.init(a.ld, wave, lane);
  ldg.init(a.ldo, wave, lane);
  float next_l = 0.f, next_d = 0.f;
  auto load_block = [&](int it, int st) {
    const int row0 = (qb_lo + it) * BLK;
    if (tid < BLK) {
      const int row = min(row0 + tid, s - 1);
      next_l = Lp[row];
      next_d = Dp[row];
    }
    ldq.issue(Qp, row0, s, lds.block[st][0]);
    ldg.issue(Gp, row0, s, lds.block[st][1]);
  };
  auto store_rows = [&](int st) {
    if (tid < BLK) {
      lds.l[st][tid] = next_l * LOG2E;
      lds.d[st][tid] = next_d;
    }
  };
  load_block(0, 0);
  store_rows(0);
  wait_loads_and_barrier();
  for (int it = 0; it < n_it; ++it) {
    const int st = it & 1;
    if (it + 1 < n_it) load_block(it + 1, st ^ 1);
    const int q0 = (qb_lo + it) * BLK + par * 32;   // this wavefront's queries
    if (k0 < s && q0 < s && (!CAUSAL || q0 + 31 >= k0)) {
      const bf16_t* tQ = lds.block[st][0];
      const bf16_t* tG = lds.block[st][1];
      f32x16 sacc = zero16(), pacc = zero16();
      struct Two { bf16x8 q, own; };
      pipelined<2 * KS, 2>([&](int n) {
                            const int ks = n / 2;
                            Two f;
                            f.q = frag_rows<D>(n & 1 ? tG : tQ, par * 32, ks, lane);
                            if (n & 1) f.own = frag_rows<D>(lds.v, rg * 32, ks, lane);
                            else f.own = ks < KREG ? kf[ks < KREG ? ks : 0] : frag_rows<D>(lds.k, rg * 32, ks, lane);
                            return f;
                          },
                          [&](int n, const Two& f) {
                            f32x16& acc = n & 1 ? pacc : sacc;
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.q, f.own, acc, 0, 0, 0);
                          });
      const bool need_mask = (CAUSAL && q0 < k0 + 31) || (q0 + 32 > s);
      dkv_scores<CAUSAL>(sacc, pacc, lds.l[st] + par * 32, lds.d[st] + par * 32, q0, key, s, need_mask, a.scale_log2, g);
      const bf16x8 pf[2] = {pack_acc<0>(sacc), pack_acc<1>(sacc)}, dsf[2] = {pack_acc<0>(pacc), pack_acc<1>(pacc)};
      pipelined<4 * DT, 2>([&](int n) { return frag_cols_acc_order<D>(n & 1 ? tQ : tG, par * 32 + n / (2 * DT) * 16, n / 2 % DT * 32, lane); },
                          [&](int n, const bf16x8& f) {
                            const int dt = n / 2 % DT, u = n / (2 * DT);
                            f32x16& acc = n & 1 ? dkacc[dt] : dvacc[dt];
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, n & 1 ? dsf[u] : pf[u], acc, 0, 0, 0);
                          });
    }
    if (it + 1 < n_it) store_rows(st ^ 1);
    wait_loads_and_barrier();
  }
  // merge the two halves' sums, dV first: the odd one hands over through LDS (64 KiB, all block tiles are free)
  float* xch = (float*)&lds.block[0][0][0] + rg * (DT * 16) * 64;
  bf16_t* dKp = a.d_qkv + dev * a.dev_qkv + ((long long)seq * s + key) * a.ld + head * 3 * D + D;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    f32x16 (&acc)[DT] = which == 0 ? dvacc : dkacc;
    if (which == 1) __syncthreads();
    if (par == 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) xch[(dt * 16 + r) * 64 + lane] = acc[dt][r];
    }
    __syncthreads();
    if (par == 0 && key < s) {
      const float w = which == 0 ? 1.0f : a.scale;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (acc[dt][4 * c + e] + xch[(dt * 16 + 4 * c + e) * 64 + lane]) * w;
          u32x2 x = {pack2_bf16(o[0], o[1]), pack2_bf16(o[2], o[3])};
          *(u32x2*)(dKp + (which == 0 ? D : 0) + dt * 32 + 8 * c + 4 * g) = x;
        }
    }
  }
}

// The same for launches with a 128-row workgroup for every compute unit: eight wavefronts share the tiles of K/V or Q/dO.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(512) void attn_fused_bwd_wide_kernel(FusedArgs a) {
  const int rank = blockIdx.y, mat = blockIdx.x >> 1, kind = blockIdx.x & 1, ntiles = gridDim.y, dev = blockIdx.z;
  if constexpr (D == 128) {
    __shared__ __attribute__((aligned(1024))) char lds[sizeof(WideLds<D>)];
    static_assert(sizeof(WideLds<D>) >= 2 * 2 * PAIR * D * sizeof(bf16_t), "room for the dQ body's tiles");
    if (kind) bwd_dq_body<D, CAUSAL, 4, false>(a, (bf16_t (*)[2][PAIR * D])lds, ntiles - 1 - rank, mat, dev);
    else bwd_dkv_wide_body<D, CAUSAL>(a, *(WideLds<D>*)lds, rank, mat, dev);
  } else {
    __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][PAIR * D];
    __shared__ __attribute__((aligned(16))) float ldsL[2][PAIR];
    __shared__ __attribute__((aligned(16))) float ldsD[2][PAIR];
    if (kind) bwd_dq_body<D, CAUSAL, 4, false>(a, lds, ntiles - 1 - rank, mat, dev);
    else bwd_dkv_body<D, CAUSAL, 4>(a, lds, ldsL, ldsD, rank, mat, dev);
  }
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(512) void attn_fused_bwd_dkv_wide_kernel(FusedArgs a) {
  __shared__ __attribute__((aligned(1024))) WideLds<D> lds;
  bwd_dkv_wide_body<D, CAUSAL>(a, lds, blockIdx.x, blockIdx.y, blockIdx.z);
}

}  // namespace

void launch_attn_fused_bwd_wide(const FusedArgs& a, int d, bool causal, dim3 grid, hipStream_t st) {
  const dim3 both(2 * grid.y, grid.x, grid.z);
  if (d == 64) attn_fused_bwd_wide_kernel<64, true><<<both, 512, 0, st>>>(a);   // (without a mask: one kind after the other)
  else if (causal) attn_fused_bwd_wide_kernel<128, true><<<both, 512, 0, st>>>(a);
  else attn_fused_bwd_wide_kernel<128, false><<<both, 512, 0, st>>>(a);
}
void launch_attn_fused_bwd_dkv_wide(const FusedArgs& a, dim3 grid, hipStream_t st) {
  attn_fused_bwd_dkv_wide_kernel<128, false><<<grid, 512, 0, st>>>(a);
}

}  // namespace optimus
