// Fixed-order combine of the partial tiles of a panel split, and the epilogue: the short path.
#pragma once
#include "epilogue.hpp"

namespace optimus {

// Four columns of a row a thread.  What bounds it is the launch and one round trip to memory: all partial tiles' loads and what the
// epilogue reads are on their way before the first is waited for.  (In a loop over the splits the compiler waited for each load in turn.)
template <int S>   // splits <= S: the loads past the last one repeat it
__device__ __forceinline__ void combine_vec(const CombineJob& j, unsigned z, unsigned m, unsigned n) {
  const long long block = (long long)j.Mb * j.Nb, stride = j.nz * block;
  const float* p = j.partials + z * block + (long long)m * j.Nb + n;
  const EpiArgs& e = j.epi;
  const unsigned z1 = z / (unsigned)j.nz0, z0 = z - z1 * (unsigned)j.nz0;
  const long long off = z1 * j.sC1 + z0 * j.sC0 + (long long)m * e.ldc + n;
  float4 w[S];
#pragma unroll
  for (int s = 0; s < S; ++s) w[s] = *(const float4*)(p + (s < j.splits ? s : j.splits - 1) * stride);
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  uint2 zz = make_uint2(0, 0), rr = zz;
  if (e.bias) bias = *(const float4*)(e.bias + z0 * j.sBias0 + n);
  if (e.gelu_grad_of) zz = *(const uint2*)((const bf16_t*)e.gelu_grad_of + off);
  if (e.residual) rr = *(const uint2*)((const bf16_t*)e.residual + off);
  float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s < j.splits) { t[0] += w[s].x; t[1] += w[s].y; t[2] += w[s].z; t[3] += w[s].w; }
#pragma unroll
  for (int c = 0; c < 4; ++c) t[c] *= e.alpha;
  if (e.bias) { t[0] += bias.x; t[1] += bias.y; t[2] += bias.z; t[3] += bias.w; }
  if (e.pre_act) *(uint2*)((bf16_t*)e.pre_act + off) = make_uint2(pack2_bf16(t[0], t[1]), pack2_bf16(t[2], t[3]));
  if (e.act == 1) gelu4<false>(t);
  if (e.gelu_grad_of) {
    const float g[4] = {__uint_as_float(zz.x << 16), __uint_as_float(zz.x & 0xffff0000u), __uint_as_float(zz.y << 16),
                        __uint_as_float(zz.y & 0xffff0000u)};
    gelu_grad_mul4<false>(t, g);
  }
  if (e.residual) {
    t[0] += __uint_as_float(rr.x << 16); t[1] += __uint_as_float(rr.x & 0xffff0000u);
    t[2] += __uint_as_float(rr.y << 16); t[3] += __uint_as_float(rr.y & 0xffff0000u);
  }
  if (e.out_fp32) *(float4*)((float*)e.C + off) = make_float4(t[0], t[1], t[2], t[3]);
  else *(uint2*)((bf16_t*)e.C + off) = make_uint2(pack2_bf16(t[0], t[1]), pack2_bf16(t[2], t[3]));
}
// quad idx of a job that takes combine_vec (CombineJob::vec).  The first workgroups wait for every line of code they run: the short path
// is a kernel of its own, without 64-bit divisions, and divides by the block's rows only where there are several blocks.
__device__ __forceinline__ void combine_quad_vec(const CombineJob& j, unsigned idx) {
  const unsigned quads_per_row = (unsigned)j.Nb >> 2, r = idx / quads_per_row, n = (idx - r * quads_per_row) * 4;
  unsigned z = 0, m = r;
  if (j.nz > 1) { z = r / (unsigned)j.Mb; m = r - z * (unsigned)j.Mb; }
  if (r >= (unsigned)j.nz * (unsigned)j.Mb) return;
  if (j.splits <= 4) combine_vec<4>(j, z, m, n);
  else combine_vec<8>(j, z, m, n);
}

}  // namespace optimus
