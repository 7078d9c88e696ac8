// Gradient of the layer's input in one pass: the rows that come back through the experts, summed over a token's slots
// (what moe_combine does with unit weights), and the gate's share d_logits Wr^T (moe_route_bwd), with the gate weight
// gradient's partial sums in blocks of the same launch where they are cheap to stage.
//
// HBM-bound: k rows in and one out per token; the two calls in a row write dx, read it back and write it again (128 experts,
// d 2048, 8192 tokens, k 8: 56 + 30 us -> 61).  The sum over the experts is rounded to the storage type before the gate's share
// is added, as the two calls do it: same bits.
#include "common.h"
#include "gate_bwd.h"

namespace moe {

struct InputGradArgs {
  const void* dx_perm;
  const void* x;
  const float* WrT;   // [E][d]
  const int32_t *topk_idx, *row_of, *offsets, *kept, *lo, *hi;
  const float *topk_w, *d_topk_w;
  float *d_logits, *partials;
  void* dx;
  int Tn, d, E, k, dwr_blocks;
  RouteBwdGeom gm;
};

// EB > 0: the first dwr_blocks blocks compute the gate weight gradient's partial sums, EB experts per row
template <typename T, int KMAX, int CU, int EB>
__global__ __launch_bounds__(256) void input_grad_kernel(InputGradArgs g) {
  constexpr int VN = Vec16<T>::N;
  if constexpr (EB > 0) {
    extern __shared__ float4 s_dl4[];
    if ((int)blockIdx.x < g.dwr_blocks)
      return gate_dwr_dense<T, EB, true>((const T*)g.x, nullptr, g.topk_idx, g.topk_w, g.d_topk_w, g.partials, g.Tn, g.d, g.E, g.k, g.gm,
                                         blockIdx.x % g.gm.col_blocks, blockIdx.x / g.gm.col_blocks, 0, s_dl4);
  }
  const int lane = threadIdx.x & (WAVE - 1);
  const int t = ((blockIdx.x - (EB > 0 ? g.dwr_blocks : 0)) * 256 + threadIdx.x) / WAVE;
  if (t >= g.Tn) return;
  int rows[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) rows[j] = j < g.k ? live_row(t * g.k + j, g.topk_idx, g.row_of, g.offsets, g.kept, g.lo, g.hi) : -1;
  float ds[MOE_MAX_K];
  int ej[MOE_MAX_K];
  gate_dsel(g.topk_idx, g.topk_w, g.d_topk_w, t, g.E, g.k, ds, ej);
  gate_dlogits_row(g.d_logits, t, g.E, g.k, lane, ds, ej);
  const T* src = (const T*)g.dx_perm;
  T* dst = (T*)g.dx + (size_t)t * g.d;
  for (int c0 = lane * VN; c0 < g.d; c0 += WAVE * VN * CU) {
    Vec16<T> v[KMAX][CU];
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (rows[j] >= 0) {
#pragma unroll
        for (int u = 0; u < CU; ++u)
          if (c0 + u * WAVE * VN < g.d) v[j][u].load_nt(src + (size_t)rows[j] * g.d + c0 + u * WAVE * VN);
      }
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int c = c0 + u * WAVE * VN;
      if (c >= g.d) break;
      float acc[VN];
#pragma unroll
      for (int i = 0; i < VN; ++i) acc[i] = 0.f;
#pragma unroll
      for (int j = 0; j < KMAX; ++j)     // fixed slot order: the sum is deterministic
        if (rows[j] >= 0) {
          float f[VN];
          v[j][u].unpack(f);
#pragma unroll
          for (int i = 0; i < VN; ++i) acc[i] += f[i];
        }
      Vec16<T> o;
      o.pack(acc);
      o.unpack(acc);
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (j < g.k) {
          const float* w = g.WrT + (size_t)max(ej[j], 0) * g.d + c;
#pragma unroll
          for (int i = 0; i < VN; i += 4) {
            const float4 w4 = *reinterpret_cast<const float4*>(w + i);
            acc[i] = fmaf(ds[j], w4.x, acc[i]);
            acc[i + 1] = fmaf(ds[j], w4.y, acc[i + 1]);
            acc[i + 2] = fmaf(ds[j], w4.z, acc[i + 2]);
            acc[i + 3] = fmaf(ds[j], w4.w, acc[i + 3]);
          }
        }
      o.pack(acc);
      o.store_nt(dst + c);
    }
  }
}

// The weight gradient shares the launch up to 16 experts (one group) while its staged rows leave the other blocks' LDS alone.
constexpr size_t DWR_SHARED_LDS = 16 * 1024;
static size_t dwr_lds(const RouteBwdGeom& gm, int eb) { return (size_t)gm.slices_per_block * gm.tps * eb * 4; }
bool input_grad_has_dwr(const moe_cfg* c) {
  return c->E <= 16 && dwr_lds(route_bwd_geom(c->T, c->d_model, (int)elt_size(c), c->E), c->E <= 8 ? 8 : 16) <= DWR_SHARED_LDS;
}

template <typename T, int KMAX, int CU>
static void launch_cu(const moe_cfg* c, InputGradArgs& g, bool dwr, hipStream_t s) {
  const int blocks = (c->T + 3) / 4;
  if (!dwr) { input_grad_kernel<T, KMAX, CU, 0><<<blocks, 256, 0, s>>>(g); return; }
  g.gm = route_bwd_geom(c->T, c->d_model, (int)sizeof(T), c->E);
  g.dwr_blocks = g.gm.col_blocks * g.gm.row_blocks;
  if (c->E <= 8) input_grad_kernel<T, KMAX, CU, 8><<<blocks + g.dwr_blocks, 256, dwr_lds(g.gm, 8), s>>>(g);
  else input_grad_kernel<T, KMAX, CU, 16><<<blocks + g.dwr_blocks, 256, dwr_lds(g.gm, 16), s>>>(g);
}
// column units in flight per lane: as in moe_combine
template <typename T>
static void launch_typed(const moe_cfg* c, InputGradArgs& g, bool dwr, hipStream_t s) {
  auto long_row = [&](int units) { return c->d_model > units * WAVE * Vec16<T>::N; };
  if (c->k <= 2) { if (long_row(4)) launch_cu<T, 2, 8>(c, g, dwr, s); else launch_cu<T, 2, 4>(c, g, dwr, s); }
  else if (c->k <= 4) { if (long_row(2)) launch_cu<T, 4, 4>(c, g, dwr, s); else launch_cu<T, 4, 2>(c, g, dwr, s); }
  else { if (long_row(2)) launch_cu<T, 8, 4>(c, g, dwr, s); else launch_cu<T, 8, 2>(c, g, dwr, s); }
}

// dx and d_logits; with `dwr` also the rows of partial sums of dWr (route_bwd_geom) that the gate's reduction adds up
int launch_input_grad(const moe_cfg* c, const moe_layer_bufs* b, const float* WrT, float* partials, bool dwr, hipStream_t s) {
  InputGradArgs g = {};
  g.dx_perm = b->dx_perm; g.x = b->x; g.WrT = WrT;
  g.topk_idx = b->topk_idx; g.row_of = b->row_of; g.offsets = b->offsets; g.kept = b->kept; g.lo = b->slice_lo; g.hi = b->slice_hi;
  g.topk_w = b->topk_w; g.d_topk_w = b->d_topk_w; g.d_logits = b->d_logits; g.partials = partials; g.dx = b->dx;
  g.Tn = c->T; g.d = c->d_model; g.E = c->E; g.k = c->k;
  if (c->dtype == MOE_DTYPE_BF16) launch_typed<bf16>(c, g, dwr, s);
  else if (c->dtype == MOE_DTYPE_F16) launch_typed<f16>(c, g, dwr, s);
  else launch_typed<float>(c, g, dwr, s);
  return launch_status();
}

}  // namespace moe
