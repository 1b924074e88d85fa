// Forward and backward kernels of the fused attention (attention_fused_kernel.hpp) and the choice between the forms.
#include "attention_fused_kernel.hpp"

namespace optimus {
namespace {

// ---------------------------------------------------------------- forward
// NRG: row groups of 32 queries per workgroup (2: 64 rows, four wavefronts; 4: 128 rows, eight wavefronts -- half the
// K/V bytes per flop and two wavefronts per SIMD, for launches with more workgroups than compute units).
// TILES_FIRST: a matrix's tiles first instead of all matrices' tiles of a rank first (see fwd_launch).
template <int D, bool CAUSAL, int NRG, bool TILES_FIRST = false>
__global__ __launch_bounds__(NRG * 128, D == 64 ? NRG : NRG / 2) void attn_fused_fwd_kernel(FusedArgs a) {   // two workgroups a CU of width 64
  constexpr int KS = D / 16, DT = D / 32, BQ = NRG * 32;
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][PAIR * D];  // [stage][K, V][pair tile]
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave % NRG, par = wave / NRG;
  // the tiles with the longest causal loops start first
  const int tile = TILES_FIRST ? gridDim.x - 1 - blockIdx.x : gridDim.y - 1 - blockIdx.y;
  const int mat = TILES_FIRST ? blockIdx.y : blockIdx.x, dev = blockIdx.z, s = a.s;
  const int seq = mat / a.nh, head = mat % a.nh;
  const bf16_t* Qp = a.qkv + dev * a.dev_qkv + (long long)seq * s * a.ld + head * 3 * D;
  const bf16_t* Kp = Qp + D;
  const bf16_t* Vp = Qp + 2 * D;
  const int q0 = tile * BQ + rg * 32;
  const int query = q0 + (lane & 31);
  const int qrow = min(query, s - 1);
  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(Qp + (long long)qrow * a.ld + ks * 16 + g * 8);
  const int wg_hi = min(tile * BQ + BQ, s) - 1;  // last query row of the workgroup
  const int nkb = CAUSAL ? wg_hi / BLK + 1 : (s + BLK - 1) / BLK;
  const int n_it = (nkb + 1) / 2;
  const int wave_nkb = q0 >= s ? 0 : (CAUSAL ? min(q0 + 31, s - 1) / BLK + 1 : nkb);
  const int limit = CAUSAL ? qrow : s - 1;  // last key this lane's row may see

  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) oacc[dt] = zero16();
  float m_run = -INFINITY, l_run = 0.f;

  TileLoader<D, 2 * NRG> ldr;
  ldr.init(a.ld, wave, lane);
  ldr.issue(Kp, 0, s, lds[0][0]);
  ldr.issue(Vp, 0, s, lds[0][1]);
  wait_loads_and_barrier();
  for (int it = 0; it < n_it; ++it) {
    const int st = it & 1;
    if (it + 1 < n_it) {
      ldr.issue(Kp, (it + 1) * PAIR, s, lds[st ^ 1][0]);
      ldr.issue(Vp, (it + 1) * PAIR, s, lds[st ^ 1][1]);
    }
    const int kb = 2 * it + par;
    if (kb < wave_nkb) {
      const bf16_t* tK = lds[st][0] + par * BLK * D;
      const bf16_t* tV = lds[st][1] + par * BLK * D;
      const int kbase = kb * BLK;
      f32x16 sacc[2];
      sacc[0] = zero16();
      sacc[1] = zero16();
      pipelined<2 * KS, D == 64 ? 1 : 2>([&](int n) { return frag_rows<D>(tK, n / KS * 32, n % KS, lane); },
                          [&](int n, const bf16x8& f) {
                            sacc[n / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[n % KS], sacc[n / KS], 0, 0, 0);
                          });
      // keys of this block past the row's limit exist only in the last blocks of the loop (wave-uniform test)
      const bool need_mask = CAUSAL ? (kbase + BLK - 1 > q0) : (kbase + BLK > s);
      if (need_mask) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = kbase + t2 * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
            if (key > limit) sacc[t2][r] = -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[t2][r]);
      mx = halfwave_max(mx) * a.scale_log2;  // the scale is positive: it commutes with the maximum
      // Every block a wavefront works on holds a visible key for each of its rows (the first key of a block is
      // never past the wavefront's first row), so mx is finite.
      // The running maximum only has to keep exp2 in range, not to be the true maximum: it follows the block
      // maximum only when that is more than 2^8 above it (wave-uniform decision), which spares the rescaling of
      // the accumulators in nearly every block.  p <= 2^8 then; the normalisation by l and the log-sum-exp
      // m + log2(l) are unchanged by the choice of m.
      const bool move = __builtin_amdgcn_ballot_w64(mx > m_run + 8.0f) != 0;
      const float m_new = move ? fmaxf(m_run, mx) : m_run;
      float sum = 0.f;
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(fmaf(sacc[t2][r], a.scale_log2, -m_new));  // masked: exp2(-inf) = 0
          sacc[t2][r] = p;
          sum += p;
        }
      sum = halfwave_sum(sum);
      if (move) {  // rescale what was accumulated
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
        m_run = m_new;
      }
      l_run += sum;
      bf16x8 pf[2][2];
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        pf[t2][0] = pack_acc<0>(sacc[t2]);
        pf[t2][1] = pack_acc<1>(sacc[t2]);
      }
      pipelined<4 * DT, D == 64 ? 1 : 2>([&](int n) { return frag_cols_acc_order<D>(tV, n / DT * 16, n % DT * 32, lane); },
                          [&](int n, const bf16x8& f) {
                            oacc[n % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pf[n / (2 * DT)][n / DT & 1], oacc[n % DT], 0, 0, 0);
                          });
    }
    wait_loads_and_barrier();
  }
  // merge the two parities: the odd one hands (m, l, O) over through LDS (all tiles are free after the last barrier)
  float* xch = (float*)&lds[0][0][0] + rg * (DT * 16 + 2) * 64;
  if (par == 1) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[(dt * 16 + r) * 64 + lane] = oacc[dt][r];
    xch[(DT * 16) * 64 + lane] = m_run;
    xch[(DT * 16 + 1) * 64 + lane] = l_run;
  }
  __syncthreads();
  if (par == 0 && wave_nkb > 0 && query < s) {
    const float m1 = xch[(DT * 16) * 64 + lane], l1 = xch[(DT * 16 + 1) * 64 + lane];
    const float m = fmaxf(m_run, m1);  // m_run is finite: block 0 belongs to this parity
    const float a0 = __builtin_amdgcn_exp2f(m_run - m), a1 = __builtin_amdgcn_exp2f(m1 - m);  // a1 = 0 if the other had no block
    const float l = l_run * a0 + l1 * a1;
    const float inv = 1.0f / l;
    const float w0 = a0 * inv, w1 = a1 * inv;
    bf16_t* Op = a.attn + dev * a.dev_attn + ((long long)seq * s + query) * a.ldo + head * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = oacc[dt][4 * c + e] * w0 + xch[(dt * 16 + 4 * c + e) * 64 + lane] * w1;
        u32x2 w = {pack2_bf16(o[0], o[1]), pack2_bf16(o[2], o[3])};
        *(u32x2*)(Op + dt * 32 + 8 * c + 4 * g) = w;
      }
    if (g == 0) a.lse[dev * a.dev_vec + (long long)mat * s + query] = (m + __log2f(l)) * LN2;
  }
}

template <int D, bool CAUSAL, int NRG>
__global__ __launch_bounds__(NRG * 128) void attn_fused_bwd_dq_kernel(FusedArgs a) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][PAIR * D];
  bwd_dq_body<D, CAUSAL, NRG, true>(a, lds, gridDim.x - 1 - blockIdx.x, blockIdx.y, blockIdx.z);  // longest causal rows first
}

// rowsum(dO * O) for every query row of the launch: a wavefront takes 32 rows, lane pair (l, l ^ 32) one row.
template <int D>
__global__ __launch_bounds__(256) void attn_fused_delta_kernel(FusedArgs a) {
  const int lane = threadIdx.x & 63, g = lane >> 5, wave = threadIdx.x >> 6;
  const int mat = blockIdx.y, dev = blockIdx.z, s = a.s;
  const int seq = mat / a.nh, head = mat % a.nh;
  const int query = blockIdx.x * 128 + wave * 32 + (lane & 31);
  const int qrow = min(query, s - 1);
  const long long orow = dev * a.dev_attn + ((long long)seq * s + qrow) * a.ldo + head * D;
  float delta = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
    delta += delta_piece(*(const bf16x8*)(a.d_attn + orow + ks * 16 + g * 8), *(const bf16x8*)(a.attn + orow + ks * 16 + g * 8));
  delta = halfwave_sum(delta);
  if (g == 0 && query < s) a.delta[dev * a.dev_vec + (long long)mat * s + qrow] = delta;
}

template <int D, bool CAUSAL, int NRG>
__global__ __launch_bounds__(NRG * 128) void attn_fused_bwd_dkv_kernel(FusedArgs a) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][PAIR * D];
  __shared__ __attribute__((aligned(16))) float ldsL[2][PAIR];
  __shared__ __attribute__((aligned(16))) float ldsD[2][PAIR];
  bwd_dkv_body<D, CAUSAL, NRG>(a, lds, ldsL, ldsD, blockIdx.x, blockIdx.y, blockIdx.z);  // early key tiles: longest causal loops
}

// dQ and dK/dV of one launch side by side.  A causal launch of either kernel alone is as long as its longest row or
// column tile while the average tile is half as long, and one workgroup fills a compute unit (registers), so with
// about one workgroup per compute unit half the chip idles.  Here the workgroups of both are one grid, ordered by loop
// length (longest first, the two kinds alternating): a compute unit that finishes a short tile picks up the next one
// of either kind.  rowsum(dO * O) comes from attn_fused_delta_kernel (launched before), so no workgroup waits for
// another.  Same arithmetic per workgroup as the two separate kernels: same bits.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_fused_bwd_kernel(FusedArgs a, int ntiles, int nmat) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][PAIR * D];
  __shared__ __attribute__((aligned(16))) float ldsL[2][PAIR];
  __shared__ __attribute__((aligned(16))) float ldsD[2][PAIR];
  const unsigned per_rank = 2u * (unsigned)nmat;   // grid: x = (rank of the loop length, matrix, kind), y = device
  const unsigned rank = blockIdx.x / per_rank, rem = blockIdx.x % per_rank;
  const int mat = (int)(rem >> 1), dev = (int)blockIdx.y;
  if (rem & 1) bwd_dq_body<D, CAUSAL, 2, false>(a, lds, ntiles - 1 - (int)rank, mat, dev);
  else bwd_dkv_body<D, CAUSAL, 2>(a, lds, ldsL, ldsD, (int)rank, mat, dev);
}
FusedArgs make_args(const AttnFusedDesc& d) {
  FusedArgs a = {};
  a.qkv = (const bf16_t*)d.qkv; a.attn = (bf16_t*)d.attn; a.lse = d.lse;
  a.d_attn = (const bf16_t*)d.d_attn; a.d_qkv = (bf16_t*)d.d_qkv; a.delta = d.delta;
  a.s = d.s; a.nh = d.nh; a.ld = d.ld; a.ldo = d.ldo;
  a.dev_qkv = d.dev_qkv; a.dev_attn = d.dev_attn; a.dev_vec = (long long)d.nb * d.nh * d.s;
  a.scale = 1.0f / sqrtf((float)d.d);
  a.scale_log2 = a.scale * LOG2E;
  return a;
}

bool desc_ok(const AttnFusedDesc& d) {
  if (!attn_fused_supported(d.d)) return false;
  if (d.s < 1 || d.nb < 1 || d.nh < 1 || d.ndev < 1 || d.ndev > 65535) return false;
  if ((long long)d.nb * d.nh > 65535) return false;
  if (d.ld % 8 || d.ldo % 8 || d.ld < 3 * d.d * d.nh || d.ldo < d.d * d.nh) return false;
  if ((long long)PAIR * d.ld * 2 >= (1ll << 31)) return false;  // per-lane byte offsets inside a pair tile are 32-bit
  return true;
}

template <int D>
void fwd_launch(const FusedArgs& a, const AttnFusedDesc& d, hipStream_t st) {
  // 128-row workgroups from one per two compute units on (measured: equal or faster than 64-row ones from there)
  const bool big = (long long)((d.s + 127) / 128) * d.nb * d.nh * d.ndev >= 128;
  // Without a mask all loops are alike and the order is a matter of caches: once a matrix's K and V fill an XCD's L2 (4 MiB)
  // its tiles run together (8 matrices, s = 8192, width 128: 275 us, by rank 286; 2 matrices, 16384: 265, 277), below that
  // the matrices side by side (16, 4096: 149, 149; 64, 1024: 58, 49).
  const int rows = big ? 128 : BLK;
  const dim3 grid(d.nb * d.nh, (d.s + rows - 1) / rows, d.ndev);
  if (big) {
    if (d.causal) attn_fused_fwd_kernel<D, true, 4><<<grid, 512, 0, st>>>(a);
    else if (4ll * D * d.s >= 4ll << 20) attn_fused_fwd_kernel<D, false, 4, true><<<dim3(grid.y, grid.x, grid.z), 512, 0, st>>>(a);
    else attn_fused_fwd_kernel<D, false, 4><<<grid, 512, 0, st>>>(a);
  } else {
    if (d.causal) attn_fused_fwd_kernel<D, true, 2><<<grid, 256, 0, st>>>(a);
    else attn_fused_fwd_kernel<D, false, 2><<<grid, 256, 0, st>>>(a);
  }
}
// Which form of the backward.  The forms of head width 128 add up dK and dV in different orders, so there the choice follows
// one device's matrices, whatever the launch covers; at 64 they do not, and it follows the launch.
// Measured, us, 128-row form against the others, head width 128.  Not causal: 512 workgroups (8 matrices, s = 4096) 298
// against 510, 256 (8, 2048) 87 against 138, 128 (4, 2048) 81 against 75: below a workgroup per compute unit the longest
// tile's loop is what counts, and two blocks per iteration walk it faster.  Causal: 512 157 against 267, 256 (16, 1024) 48
// against 54 alone, but beside the products of the layer's gradient branch, which take compute units away, the longest
// tiles then start second: the 4096-wide layer step 874 against 850.  Both kinds in one grid against one after the other, 16
// matrices, s = 4096: causal 308 against 477 (width 64: 189 against 279), not causal 596 against 507 (327 against 295).
// Width 64, causal, one tile per matrix: 512 matrices of s = 128 43 against 38, 1024 of 64 53 against 48; two or three tiles
// between 0.87 and 1.07 of one after the other, from 512 on 0.92 and less.
template <int D, bool CAUSAL>
void bwd_launch_c(const FusedArgs& a, const AttnFusedDesc& d, hipStream_t st) {
  const long long tiles64 = (d.s + BLK - 1) / BLK, tiles128 = (d.s + 127) / 128, nmat = (long long)d.nb * d.nh;
  const bool big = tiles128 * nmat * d.ndev >= 512;
  const dim3 grid128((unsigned)tiles128, (unsigned)nmat, d.ndev);
  const bool wide = D == 128 ? 2 * tiles128 * nmat >= (CAUSAL ? 512 : 256) : big;
  if (wide && (CAUSAL || !big) && !(D == 64 && tiles128 == 1)) {
    attn_fused_delta_kernel<D><<<grid128, 256, 0, st>>>(a);
    launch_attn_fused_bwd_wide(a, D, CAUSAL, grid128, st);
    return;
  }
  if (!big) {
    // small launches (about a workgroup per compute unit or less): both kinds of workgroup in one grid
    attn_fused_delta_kernel<D><<<grid128, 256, 0, st>>>(a);
    attn_fused_bwd_kernel<D, CAUSAL><<<dim3((unsigned)(2 * tiles64 * nmat), d.ndev), 256, 0, st>>>(a, (int)tiles64, (int)nmat);
    return;
  }
  // Without a mask, or with one tile per matrix, all loops are alike: one kind after the other, which saves the delta kernel and
  // mixes no tile sizes.
  attn_fused_bwd_dq_kernel<D, CAUSAL, 4><<<grid128, 512, 0, st>>>(a);
  if constexpr (D == 64) attn_fused_bwd_dkv_kernel<D, CAUSAL, 4><<<grid128, 512, 0, st>>>(a);
  else if (wide) launch_attn_fused_bwd_dkv_wide(a, grid128, st);
  else attn_fused_bwd_dkv_kernel<D, CAUSAL, 2><<<dim3((unsigned)tiles64, (unsigned)nmat, d.ndev), 256, 0, st>>>(a);   // many devices' blocks of few matrices
}
template <int D>
void bwd_launch(const FusedArgs& a, const AttnFusedDesc& d, hipStream_t st) {
  if (d.causal) bwd_launch_c<D, true>(a, d, st);
  else bwd_launch_c<D, false>(a, d, st);
}

}  // namespace

bool attn_fused_supported(int d) { return d == 64 || d == 128; }

int launch_attn_fused_fwd(const AttnFusedDesc& d, hipStream_t st) {
  if (!desc_ok(d) || !d.qkv || !d.attn || !d.lse) return OPTIMUS_ESHAPE;
  const FusedArgs a = make_args(d);
  if (d.d == 64) fwd_launch<64>(a, d, st);
  else fwd_launch<128>(a, d, st);
  return hip_launch_status();
}

int launch_attn_fused_bwd(const AttnFusedDesc& d, hipStream_t st) {
  if (!desc_ok(d) || !d.qkv || !d.attn || !d.lse || !d.d_attn || !d.d_qkv || !d.delta) return OPTIMUS_ESHAPE;
  const FusedArgs a = make_args(d);
  if (d.d == 64) bwd_launch<64>(a, d, st);
  else bwd_launch<128>(a, d, st);
  return hip_launch_status();
}

}  // namespace optimus
