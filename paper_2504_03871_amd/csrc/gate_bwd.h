// Pieces of the gate backward that two kernels share: the gradient of a token's selected logits, and the dense form of the
// gate weight gradient.
#pragma once
#include "common.h"

namespace moe {

#ifdef __HIPCC__
// Softmax-over-selected backward of token t: ds_j = w_j (dw_j - sum_i w_i dw_i).  An expert id outside [0, E) contributes
// nothing (id -1, ds 0).
__device__ __forceinline__ void gate_dsel(const int32_t* __restrict__ topk_idx, const float* __restrict__ topk_w,
                                          const float* __restrict__ d_topk_w, int t, int E, int k, float (&ds)[MOE_MAX_K], int (&ej)[MOE_MAX_K]) {
  float gsum = 0.f;
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j)
    if (j < k) gsum = fmaf(topk_w[(size_t)t * k + j], d_topk_w[(size_t)t * k + j], gsum);
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    ds[j] = 0.f;
    ej[j] = 0;
    if (j < k) {
      ds[j] = topk_w[(size_t)t * k + j] * (d_topk_w[(size_t)t * k + j] - gsum);
      ej[j] = topk_idx[(size_t)t * k + j];
      if (ej[j] < 0 || ej[j] >= E) { ej[j] = -1; ds[j] = 0.f; }
    }
  }
}
// d_logits[t][:] of a wave's token
__device__ __forceinline__ void gate_dlogits_row(float* __restrict__ d_logits, int t, int E, int k, int lane, const float (&ds)[MOE_MAX_K],
                                                 const int (&ej)[MOE_MAX_K]) {
  for (int e = lane; e < E; e += WAVE) {
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j) v = (j < k && ej[j] == e) ? ds[j] : v;
    d_logits[(size_t)t * E + e] = v;
  }
}

// Gate weight gradient dWr = x^T d_logits.  Experts in groups of EB <= 16 (bz): every thread keeps an [EB] x
// (16-byte column group) block of the weight gradient in registers and adds d_logits[t][:] (x) x[t][cols] token after token,
// zeros of the unselected experts included; no LDS read-modify-write, no branches, one 16-byte load of
// x per token.  The slice's d_logits rows are staged in LDS once, padded with zeros to EB per row, and
// read back as 16-byte broadcasts.  Geometry: RouteBwdGeom; s_dl4: [slices_per_block][tps][EB] floats.
// SELECTED: the rows are not read but computed from the selection (topk_*, one expert group).
template <typename T, int EB, bool SELECTED>
__device__ __forceinline__ void gate_dwr_dense(
    const T* __restrict__ x, const float* __restrict__ d_logits, const int32_t* __restrict__ topk_idx, const float* __restrict__ topk_w,
    const float* __restrict__ d_topk_w, float* __restrict__ partials, int Tn, int d, int E, int k, const RouteBwdGeom& gm, int bx, int by, int bz,
    float4* s_dl4) {
  float* s_dl = reinterpret_cast<float*>(s_dl4);
  constexpr int VN = Vec16<T>::N, U = 8;   // tokens whose x pieces a thread keeps in flight
  const int c = threadIdx.x & (gm.cg_pow2 - 1), slice = threadIdx.x / gm.cg_pow2;
  const int col = (bx * gm.cg_pow2 + c) * VN;
  const int row = by * gm.slices_per_block + slice;   // row of partial sums = token slice
  const int e0 = bz * EB;                             // this block's group of experts (more than EB experts: x is read once per group)
  const int t0 = row * gm.tps;
  const int nt = max(0, min(gm.tps, Tn - t0));
  // The first U pieces of x are requested before the rows are staged where the accumulators leave registers for it (fp32, up
  // to 8 experts): with few tokens a block is a chain of latencies.  input_grad_kernel, fp32, us: T 512, d 128, k 2
  // 9.7 -> 6.5, T 2000, d 516 15.0 -> 9.3; in 16-bit types, whose 64 or 128 accumulators it pushes to fewer waves, T 8192,
  // d 1024 26.7 -> 28.6, T 3001, d 1088 13.9 -> 17.6.
  constexpr bool FIRST = EB * VN <= 32;
  Vec16<T> xv[U];
  auto load_x = [&](int tb) {   // a piece past the slice's last token is that token's again
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u].load_nt(x + (size_t)(t0 + min(tb + u, nt - 1)) * d + col);
  };
  if (FIRST && col < d && nt > 0) load_x(0);
  {   // the block's slices are adjacent tokens: one pass over them, zero past the last token and past E
    const int tb = by * gm.slices_per_block * gm.tps, n = gm.slices_per_block * gm.tps * EB;
    if constexpr (SELECTED) {
      for (int i = threadIdx.x; i < n / 4; i += 256) s_dl4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      __syncthreads();
      for (int i = threadIdx.x; i < n / EB && tb + i < Tn; i += 256) {
        float ds[MOE_MAX_K];
        int ej[MOE_MAX_K];
        gate_dsel(topk_idx, topk_w, d_topk_w, tb + i, E, k, ds, ej);
#pragma unroll
        for (int j = 0; j < MOE_MAX_K; ++j)
          if (j < k && ej[j] >= 0) s_dl[i * EB + ej[j]] = ds[j];
      }
    } else {
      for (int i = threadIdx.x; i < n; i += 256) {
        const int t = tb + i / EB, e = i % EB;
        s_dl[i] = (t < Tn && e0 + e < E) ? d_logits[(size_t)t * E + e0 + e] : 0.f;
      }
    }
  }
  __syncthreads();
  if (col >= d) return;
  const float4* dl = s_dl4 + (size_t)slice * gm.tps * (EB / 4);
  float acc[EB][VN];
#pragma unroll
  for (int e = 0; e < EB; ++e)
#pragma unroll
    for (int v = 0; v < VN; ++v) acc[e][v] = 0.f;
  for (int tb = 0; tb < nt; tb += U) {
    if (!FIRST || tb > 0) load_x(tb);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xf[VN];
      xv[u].unpack(xf);
      const float live = (tb + u < nt) ? 1.f : 0.f;   // the clamped reload of the last token counts once
#pragma unroll
      for (int q = 0; q < EB / 4; ++q) {
        const float4 g4 = dl[min(tb + u, nt - 1) * (EB / 4) + q];
        const float g[4] = {g4.x * live, g4.y * live, g4.z * live, g4.w * live};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int v = 0; v < VN; ++v) acc[q * 4 + j][v] = fmaf(g[j], xf[v], acc[q * 4 + j][v]);
      }
    }
  }
  float* out = partials + (size_t)row * E * d + col;   // [row][e][col]: 16-byte stores, adjacent lanes adjacent
#pragma unroll
  for (int e = 0; e < EB; ++e)
    if (e0 + e < E) {
#pragma unroll
      for (int v = 0; v < VN; v += 4)
        *reinterpret_cast<float4*>(out + (size_t)(e0 + e) * d + v) = make_float4(acc[e][v], acc[e][v + 1], acc[e][v + 2], acc[e][v + 3]);
    }
}
#endif

}  // namespace moe
