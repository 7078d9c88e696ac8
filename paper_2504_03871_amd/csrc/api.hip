// C ABI of the MoE library: argument validation, workspace layout, kernel sequencing.
#include "common.h"
#include "gemm.h"
#include "prof.h"
#include "tile_map.h"
#include <algorithm>

namespace moe {

static thread_local int g_last_hip_error = 0;
int set_hip_error(hipError_t e) {
  g_last_hip_error = (int)e;
  return MOE_ERR_HIP;
}

int check_cfg(const moe_cfg* c) {
  if (c == nullptr) return MOE_ERR_NULL;
  if (c->dtype != MOE_DTYPE_F32 && c->dtype != MOE_DTYPE_BF16 && c->dtype != MOE_DTYPE_F16) return MOE_ERR_BAD_DTYPE;
  if (c->act != MOE_ACT_GELU && c->act != MOE_ACT_SWIGLU) return MOE_ERR_BAD_DTYPE;
  if (c->T < 0 || c->d_model <= 0 || c->d_ff <= 0) return MOE_ERR_BAD_SHAPE;
  if (c->E < 1 || c->E > MOE_MAX_E) return MOE_ERR_BAD_SHAPE;
  if (c->k < 1 || c->k > MOE_MAX_K || c->k > c->E) return MOE_ERR_BAD_SHAPE;
  const int mult = is_half(c) ? 64 : 4;
  if (c->d_model % mult != 0 || c->d_ff % mult != 0) return MOE_ERR_BAD_SHAPE;
  if ((long long)c->T * c->k > (1ll << 30)) return MOE_ERR_BAD_SHAPE;
  if (!offsets_fit_32_bits(c->T, c->k, c->d_model, c->d_ff, (int)elt_size(c))) return MOE_ERR_BAD_SHAPE;
  return MOE_OK;
}

static int tile_rows_for(const moe_cfg* c) {   // both row-tile GEMMs of a pass share one map: the wider decides
  if (is_half(c)) return mid_applies((long long)c->T * c->k, c->E) ? MID_ROWS : gemm_bf16_tile_rows();
  return f32_tile_rows((long long)c->T * c->k, c->E / 2, std::max(c->d_model, c->d_ff));
}
// The smallest row tiles of a 16-bit GEMM with K = d_ff are split along K (gemm.h): 256-row tiles only
static bool splits_small_tiles(const moe_cfg* c) { return is_half(c) && tile_rows_for(c) != MID_ROWS && split_k_applies(c->E, c->d_ff); }
// Forward GEMMs of few rows per expert
static bool fwd_skinny(const moe_cfg* c) {
  return is_half(c) && skinny_applies((long long)c->T * c->k, c->E, c->d_model, c->d_ff, c->act == MOE_ACT_SWIGLU, (int)elt_size(c));
}
static int weights_streamed_from(const moe_cfg* c, int tile_rows) {
  return is_half(c) ? streamed_from((long long)c->T * c->k, tile_rows, c->E, c->d_model, c->d_ff, c->act == MOE_ACT_SWIGLU ? 3 : 2, (int)elt_size(c)) : 0;
}
// backward: a row-tile GEMM of N columns with at most about eight rounds of tiles shares its launch (moe_expert_ffn_bwd)
static bool shares_launch(const moe_cfg* c, int N, int max_tiles) {
  const int cols = is_half(c) ? gemm_bf16_tile_rows() : F32_TILE_COLS;
  return (long long)((N + cols - 1) / cols) * max_tiles <= 8 * (is_half(c) ? 256 : F32_LOW_TILES);
}

WsLayout ws_layout(const moe_cfg* c) {
  WsLayout w{};
  const size_t A = (size_t)c->T * c->k;
  size_t off = 0;
  w.dispatch_blk_cnt = off;
  off += align_up(((A + DISPATCH_CHUNK - 1) / DISPATCH_CHUNK + 1) * (size_t)c->E * 4, 256);   // + a row of totals
  w.tile_map = off;
  off += align_up(tile_map_bytes(max_row_tiles((int)A, c->E, TILE_ROWS_MIN), c->E), 256);
  w.route_partials = off;
  const size_t partial_rows = route_bwd_uses_mfma(c->dtype != MOE_DTYPE_F32, c->E)
                                  ? (size_t)route_bwd_mfma_geom(c->T, c->d_model, c->E).rows
                                  : (size_t)route_bwd_geom(c->T, c->d_model, (int)elt_size(c), c->E).partial_rows;
  off += align_up(partial_rows * c->d_model * c->E * 4, 256);
  w.route_wrt = off;   // shared with the forward's gate weight in MFMA operand layout (never live together)
  off += align_up(std::max((size_t)c->d_model * c->E * 4, route_wfrag_bytes(c->d_model, c->E)), 256);
  // Partial sums of split-K tiles: the forward's (y) may reach into the region of dA, which only a backward call fills and
  // reads; the GELU dx reads dA while it writes its own, so those lie in front of it.
  w.ffn_split = off;
  const size_t dact = align_up((c->act == MOE_ACT_SWIGLU ? 2 : 1) * A * c->d_ff * elt_size(c), 256);
  size_t fwd = 0, bwd = 0;
  if (is_half(c) && c->d_ff >= SPLIT_MIN_K) {
    const int max_tiles = max_row_tiles((int)A, c->E, tile_rows_for(c));
    const bool skinny = fwd_skinny(c), small = splits_small_tiles(c);
    const size_t rows = split_ws_bytes(c->E, c->d_model), tail = tail_ws_bytes(max_tiles, c->d_model);
    fwd = skinny ? (skinny_split(c->E, c->d_ff) ? rows : 0) : std::max(small ? rows : 0, tail);
    if (c->act == MOE_ACT_GELU) bwd = std::max(small ? rows : 0, shares_launch(c, c->d_model, max_tiles) ? 0 : tail);
  }
  off += align_up(std::max(bwd, fwd > dact ? fwd - dact : 0), 256);
  w.ffn_bwd_dact = off;
  off += dact;
  w.total = off;
  return w;
}

// defined in the kernel files
int launch_route(const moe_cfg*, const void*, const float*, const float*, const float*, float*, int32_t*, float*, void*,
                 hipStream_t);
int launch_route_bwd(const moe_cfg*, const void*, const float*, const int32_t*, const float*, const float*, float*,
                     float*, void*, int, float*, float*, hipStream_t);
int launch_dispatch(const moe_cfg*, const void*, const int32_t*, const int32_t*, const int32_t*, int32_t*, int32_t*,
                    int32_t*, int32_t*, int32_t*, void*, int32_t*, const SideWork*, hipStream_t);
int dispatch_static_scratch(int32_t** out);
int launch_combine(const moe_cfg*, const void*, const float*, const int32_t*, const int32_t*, const int32_t*,
                   const int32_t*, const int32_t*, const int32_t*, void*, int, hipStream_t);
int launch_combine_bwd(const moe_cfg*, const void*, const void*, const float*, const int32_t*, const int32_t*,
                       const int32_t*, const int32_t*, const int32_t*, const int32_t*, void*, float*, const SideWork*, hipStream_t);
bool input_grad_has_dwr(const moe_cfg*);
int launch_input_grad(const moe_cfg*, const moe_layer_bufs*, const float*, float*, bool, hipStream_t);
int launch_gate_dwr(const moe_cfg*, const void*, const float*, float*, int, float*, bool, hipStream_t);

__global__ void fill_zero_kernel(float* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// Streaming copy / fill for the benchmark: 16-byte vectors, four per thread in flight, grid-stride.
typedef unsigned bs_u32x4 __attribute__((ext_vector_type(4)));
template <bool FILL>
__global__ __launch_bounds__(256) void bench_stream_kernel(bs_u32x4* __restrict__ dst, const bs_u32x4* __restrict__ src, size_t n16) {
  const size_t stride = (size_t)gridDim.x * 256 * 4;
  for (size_t i = (size_t)blockIdx.x * 256 * 4 + threadIdx.x; i < n16; i += stride) {
    bs_u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[u] = bs_u32x4{0u, 0u, 0u, 0u};
      if (!FILL && i + u * 256 < n16) v[u] = __builtin_nontemporal_load(src + i + u * 256);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * 256 < n16) __builtin_nontemporal_store(v[u], dst + i + u * 256);
  }
}

// One lane samples the shader-clock counter and the 100 MHz real-time counter n times, sleeping in between
// (a bounded loop: the kernel always ends).  Two consecutive samples give the shader clock over that interval.
__global__ void clock_probe_kernel(unsigned long long* __restrict__ out, int n, int sleeps) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  for (int i = 0; i < n; ++i) {
    out[2 * i] = __builtin_amdgcn_s_memtime();
    out[2 * i + 1] = __builtin_amdgcn_s_memrealtime();
    for (int s = 0; s < sleeps; ++s) __builtin_amdgcn_s_sleep(127);
  }
}

// Nothing but MFMAs on register operands: 32 accumulations per round, each on an accumulator of its own
// (16 x 16 x 32: 32 accumulators of 4 registers; 32 x 32 x 16: 8 accumulators of 16 registers, four rounds of them).
typedef __bf16 ml_bf16x8 __attribute__((ext_vector_type(8)));
typedef float ml_f32x4 __attribute__((ext_vector_type(4)));
typedef float ml_f32x16 __attribute__((ext_vector_type(16)));
template <int KIND>
__global__ __launch_bounds__(512, 1) void mfma_loop_kernel(const ml_bf16x8* __restrict__ in, float* __restrict__ out, int iters) {
  ml_bf16x8 a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = in[(threadIdx.x * 8 + i) % 4096];
    b[i] = in[(threadIdx.x * 8 + 4 + i) % 4096];
  }
  float s = 0.f;
  if constexpr (KIND == 0) {
    ml_f32x4 acc[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i] = ml_f32x4{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int i = 0; i < 32; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i % 4], b[(i / 4) % 4], acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) s += acc[i][0] + acc[i][1] + acc[i][2] + acc[i][3];
  } else {
    ml_f32x16 acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    for (int it = 0; it < 2 * iters; ++it) {   // 16 instructions of twice the FLOP = the FLOP of a round above
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i % 4], b[(i / 4) % 4], acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) s += acc[i][v];
  }
  out[blockIdx.x * blockDim.x + threadIdx.x] = s;
}

static int check_ws(const moe_cfg* c, const void* ws, size_t ws_bytes) {
  return (ws != nullptr && ws_bytes < ws_layout(c).total) ? MOE_ERR_WORKSPACE : MOE_OK;
}

static int check_slices(const int32_t* lo, const int32_t* hi) {
  return ((lo == nullptr) != (hi == nullptr)) ? MOE_ERR_BAD_SLICE : MOE_OK;
}

static int launch_gemm(const moe_cfg* c, int mode, int epi, bool dual, bool chain, const GemmArgs& g, int max_tiles,
                       hipStream_t s) {
  return is_half(c) ? launch_gemm_half(c->dtype, mode, epi, dual, chain, g, max_tiles, s)
                    : launch_gemm_f32(mode, epi, dual, chain, g, tile_rows_for(c), max_tiles, s);
}
static int launch_pair(const moe_cfg* c, int epi1, bool chain1, const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  return is_half(c) ? launch_gemm_half_pair(c->dtype, epi1, chain1, g1, max_tiles, g2, s)
                    : launch_gemm_f32_pair(epi1, chain1, g1, tile_rows_for(c), max_tiles, g2, s);
}

}  // namespace moe

using namespace moe;

#define REQUIRE(p) do { if ((p) == nullptr) return MOE_ERR_NULL; } while (0)
#define ALIGNED(p) do { if (misaligned(p)) return MOE_ERR_ALIGN; } while (0)
#define CHECK(expr) do { int rc_ = (expr); if (rc_ != MOE_OK) return rc_; } while (0)

extern "C" {

const char* moe_error_string(int code) {
  switch (code) {
    case MOE_OK: return "ok";
    case MOE_ERR_NULL: return "a required pointer is NULL";
    case MOE_ERR_BAD_SHAPE: return "unsupported shape (T, d_model, d_ff, E or k)";
    case MOE_ERR_BAD_DTYPE: return "unknown dtype or activation";
    case MOE_ERR_BAD_SLICE: return "slice_lo and slice_hi must both be given or both be NULL";
    case MOE_ERR_ALIGN: return "device pointer not 16-byte aligned";
    case MOE_ERR_HIP: return "HIP launch failed (see moe_last_hip_error)";
    case MOE_ERR_WORKSPACE: return "workspace smaller than moe_workspace_bytes(cfg), or problem too large for the static scratch";
    default: return "unknown error code";
  }
}

int moe_last_hip_error(void) { return g_last_hip_error; }

int moe_bench_stream(void* dst, const void* src, size_t bytes, int32_t mode, void* stream) {
  REQUIRE(dst);
  if (mode != 0 && mode != 1) return MOE_ERR_BAD_DTYPE;
  if (mode == 0) REQUIRE(src);
  ALIGNED(dst); ALIGNED(src);
  if (bytes % 16 != 0) return MOE_ERR_BAD_SHAPE;
  if (bytes == 0) return MOE_OK;
  const size_t n16 = bytes / 16;
  const size_t want = (n16 + 1023) / 1024;
  const unsigned grid = (unsigned)(want < 256 * 16 ? want : 256 * 16);
  if (mode == 0) bench_stream_kernel<false><<<grid, 256, 0, (hipStream_t)stream>>>((bs_u32x4*)dst, (const bs_u32x4*)src, n16);
  else bench_stream_kernel<true><<<grid, 256, 0, (hipStream_t)stream>>>((bs_u32x4*)dst, nullptr, n16);
  return launch_status();
}

int moe_bench_clock_probe(uint64_t* samples, int32_t n, int32_t sleeps, void* stream) {
  REQUIRE(samples);
  ALIGNED(samples);
  if (n < 1 || n > (1 << 20) || sleeps < 0 || sleeps > 1000) return MOE_ERR_BAD_SHAPE;
  clock_probe_kernel<<<1, 64, 0, (hipStream_t)stream>>>(reinterpret_cast<unsigned long long*>(samples), n, sleeps);
  return launch_status();
}

int moe_bench_mfma_loop(int32_t kind, int32_t iters, const void* operand, float* sink, void* stream) {
  REQUIRE(operand);
  REQUIRE(sink);
  ALIGNED(operand);
  ALIGNED(sink);
  if (kind < 0 || kind > 1 || iters < 1 || iters > 1000000) return MOE_ERR_BAD_SHAPE;
  if (kind == 0)
    mfma_loop_kernel<0><<<1024, 512, 0, (hipStream_t)stream>>>(reinterpret_cast<const ml_bf16x8*>(operand), sink, iters);
  else
    mfma_loop_kernel<1><<<1024, 512, 0, (hipStream_t)stream>>>(reinterpret_cast<const ml_bf16x8*>(operand), sink, iters);
  return launch_status();
}

int moe_gemm_block_tile(int32_t kind, int64_t block, int32_t n_rt, int32_t n_full_rt, int32_t n_split, int32_t ntm,
                        int32_t ntn, int32_t* out) {
  REQUIRE(out);
  if (block < 0 || block > 0x7fffffffll || ntn < 1 || n_rt < 0 || n_full_rt < 0 || n_full_rt > n_rt || n_split < 0 ||
      n_split > n_rt - n_full_rt)
    return MOE_ERR_BAD_SHAPE;
  // the kernels count tiles, K parts and K values in 32 bits
  const long long parts = kind == 5 ? (long long)(n_split ? SPLIT_K : 1) * n_rt : n_rt + (long long)(SPLIT_K - 1) * n_split;
  const long long tiles = kind == 1 ? (long long)ntm * ntn : kind == 6 ? (block / MID_ROWS + n_rt) * ntn : kind == 7 ? 0 : parts * ntn;
  if (tiles > 0x7fffffffll - NUM_XCD || ((kind == 4 || kind == 6) && ntm > 0x7fffffff / 64)) return MOE_ERR_BAD_SHAPE;
  for (int i = 0; i < 6; ++i) out[i] = -1;
  if (kind == 0 || kind == 3) {
    RowBlock r;
    out[0] = row_tile_block((int)block, n_rt, n_full_rt, n_split, ntn, kind == 3, r) ? 1 : 0;
    if (out[0]) { out[1] = r.rt; out[3] = r.nt; out[4] = r.split_tile; out[5] = r.ksplit; }
    return MOE_OK;
  }
  if (kind == 4) {
    if (ntm < 1) return MOE_ERR_BAD_SHAPE;
    const TailSplit t = tail_split(n_rt * ntn, ntm * 64);
    RowBlock r;
    out[0] = tail_split_block((int)block, n_rt, n_full_rt, ntn, false, t, r) ? 1 : 0;
    if (out[0]) { out[1] = r.rt; out[2] = t.parts; out[3] = r.nt; out[4] = r.split_tile; out[5] = r.ksplit; }
    return MOE_OK;
  }
  if (kind == 6) {
    if (ntm < 1) return MOE_ERR_BAD_SHAPE;
    out[0] = tail_may_split((int)block, n_rt, n_split == 0, ntn, ntm * 64, n_full_rt == 1 ? MID_ROWS : gemm_bf16_tile_rows()) ? 1 : 0;
    return MOE_OK;
  }
  if (kind == 7) {
    if (n_full_rt > 1) return MOE_ERR_BAD_SHAPE;
    const moe_cfg c = {(int)block, ntm, ntn, n_rt, 1, MOE_DTYPE_BF16, n_full_rt == 1 ? MOE_ACT_SWIGLU : MOE_ACT_GELU, 0, nullptr};
    CHECK(check_cfg(&c));
    out[0] = fwd_skinny(&c) ? SKINNY_ROWS : tile_rows_for(&c);
    out[1] = fwd_skinny(&c) ? 0 : weights_streamed_from(&c, out[0]);
    out[2] = tile_rows_for(&c);
    out[3] = weights_streamed_from(&c, out[2]);
    return MOE_OK;
  }
  if (kind == 5) {
    if (ntm < 1 || n_full_rt > 1 || n_split > 1) return MOE_ERR_BAD_SHAPE;
    const SkinnyOrder o = skinny_order(n_rt, n_full_rt == 1, ntm, n_split == 1);
    RowBlock r;
    out[0] = skinny_block((int)block, o, ntn, r) ? 1 : 0;
    if (out[0]) { out[1] = r.rt; out[2] = 1 << o.shift; out[3] = r.nt; out[4] = r.split_tile; out[5] = r.ksplit; }
    return MOE_OK;
  }
  if (kind == 1) {
    if (ntm < 1) return MOE_ERR_BAD_SHAPE;
    int slot, mt, nt;
    out[0] = dw_block((int)block, ntm, ntn, slot, mt, nt) ? 1 : 0;
    if (out[0]) { out[1] = slot; out[2] = mt; out[3] = nt; }
    return MOE_OK;
  }
  return MOE_ERR_BAD_DTYPE;
}

int moe_workspace_bytes(const moe_cfg* cfg, size_t* bytes) {
  CHECK(check_cfg(cfg));
  REQUIRE(bytes);
  *bytes = ws_layout(cfg).total;
  return MOE_OK;
}

int moe_saved_bytes(const moe_cfg* cfg, size_t* bytes) {
  CHECK(check_cfg(cfg));
  REQUIRE(bytes);
  *bytes = (size_t)(cfg->act == MOE_ACT_SWIGLU ? 3 : 2) * cfg->T * cfg->k * cfg->d_ff * elt_size(cfg);
  return MOE_OK;
}

int moe_route(const moe_cfg* cfg, const void* x, const float* Wr, const float* bias, const float* logits_in,
              float* logits_out, int32_t* topk_idx, float* topk_w, void* ws, size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  if (logits_in == nullptr) { REQUIRE(x); REQUIRE(Wr); REQUIRE(logits_out); }
  if (logits_in == nullptr && cfg->dtype != MOE_DTYPE_F32) REQUIRE(ws);   // the matrix-core gate (16-bit storage)
  REQUIRE(topk_idx);
  REQUIRE(topk_w);
  ALIGNED(x); ALIGNED(Wr); ALIGNED(bias); ALIGNED(logits_in); ALIGNED(logits_out); ALIGNED(topk_idx); ALIGNED(topk_w);
  ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  if (cfg->T == 0) return MOE_OK;
  void* wfrag = ws != nullptr ? static_cast<char*>(ws) + ws_layout(cfg).route_wrt : nullptr;
  ProfScope ps(cfg, MOE_PROF_ROUTE, (hipStream_t)stream);
  return launch_route(cfg, x, Wr, bias, logits_in, logits_out, topk_idx, topk_w, wfrag, (hipStream_t)stream);
}

int moe_dispatch(const moe_cfg* cfg, const void* x, const int32_t* topk_idx, const int32_t* slice_lo,
                 const int32_t* slice_hi, int32_t* counts, int32_t* kept, int32_t* offsets, int32_t* row_of,
                 int32_t* src_of, void* x_perm, void* ws, size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(topk_idx); REQUIRE(counts); REQUIRE(kept); REQUIRE(offsets); REQUIRE(row_of); REQUIRE(src_of); REQUIRE(ws);
  if (x_perm != nullptr) REQUIRE(x);
  ALIGNED(x); ALIGNED(topk_idx); ALIGNED(slice_lo); ALIGNED(slice_hi); ALIGNED(counts); ALIGNED(kept);
  ALIGNED(offsets); ALIGNED(row_of); ALIGNED(src_of); ALIGNED(x_perm); ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  const WsLayout w = ws_layout(cfg);
  int32_t* blk_cnt = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + w.dispatch_blk_cnt);
  // T == 0 still has to produce zero counts and offsets: the kernels handle an empty assignment list
  return launch_dispatch(cfg, x, topk_idx, slice_lo, slice_hi, counts, kept, offsets, row_of, src_of, x_perm, blk_cnt,
                         nullptr, (hipStream_t)stream);
}

int moe_dispatch_static(const moe_cfg* cfg, const void* x, const int32_t* topk_idx, const int32_t* slice_lo,
                        const int32_t* slice_hi, int32_t* counts, int32_t* kept, int32_t* offsets, int32_t* row_of,
                        int32_t* src_of, void* x_perm, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(topk_idx); REQUIRE(counts); REQUIRE(kept); REQUIRE(offsets); REQUIRE(row_of); REQUIRE(src_of);
  if (x_perm != nullptr) REQUIRE(x);
  ALIGNED(x); ALIGNED(topk_idx); ALIGNED(slice_lo); ALIGNED(slice_hi); ALIGNED(counts); ALIGNED(kept);
  ALIGNED(offsets); ALIGNED(row_of); ALIGNED(src_of); ALIGNED(x_perm);
  // the same per-block histogram region as the workspace version, held to the size of the static array
  const size_t A = (size_t)cfg->T * cfg->k;
  const size_t need = ((A + DISPATCH_CHUNK - 1) / DISPATCH_CHUNK + 1) * (size_t)cfg->E * 4;
  if (need > MOE_DISPATCH_STATIC_BYTES) return MOE_ERR_WORKSPACE;
  int32_t* blk_cnt = nullptr;
  CHECK(dispatch_static_scratch(&blk_cnt));
  return launch_dispatch(cfg, x, topk_idx, slice_lo, slice_hi, counts, kept, offsets, row_of, src_of, x_perm, blk_cnt,
                         nullptr, (hipStream_t)stream);
}

namespace {
// the row-tile map of a forward or backward FFN call and its table
TileMapArgs tile_map_args(const moe_cfg* cfg, const int32_t* offsets, const int32_t* kept, const int32_t* lo, const int32_t* hi, bool forward, void* ws) {
  TileMapArgs t = {offsets, kept, lo, hi, cfg->E};
  const bool skinny = forward && fwd_skinny(cfg);
  t.tile_rows = skinny ? SKINNY_ROWS : tile_rows_for(cfg);
  t.by_expert = skinny || (is_half(cfg) && t.tile_rows == MID_ROWS);
  t.table = cfg->act != MOE_ACT_GELU || cfg->dtype != MOE_DTYPE_BF16 ? GELU_TAB_NONE : forward ? GELU_TAB_PHI : GELU_TAB_GRAD;
  t.map = tile_map_at(static_cast<char*>(ws) + ws_layout(cfg).tile_map, max_row_tiles(cfg->T * cfg->k, cfg->E, TILE_ROWS_MIN), cfg->E);
  return t;
}
// GEMM1 with its activation epilogue into `saved` (or, saved == NULL, its hidden activation alone into
// `hidden`), then (y_perm != NULL) GEMM2.
int ffn_fwd_impl(const moe_cfg* cfg, const void* x_perm, const void* W1, const void* W1b, const void* W2,
                 const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo, const int32_t* slice_hi,
                 void* saved, void* hidden, void* y_perm, void* ws, bool map_built, hipStream_t s) {
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  const WsLayout w = ws_layout(cfg);
  const int A = cfg->T * cfg->k, d = cfg->d_model, f = cfg->d_ff;
  const bool skinny = fwd_skinny(cfg);
  const TileMapArgs tm = tile_map_args(cfg, offsets, kept, slice_lo, slice_hi, true, ws);
  const TileMap& map = tm.map;
  const int tr = tm.tile_rows, max_tiles = max_row_tiles(A, cfg->E, tr);
  if (!map_built) CHECK(launch_tile_map(tm, s));
  const size_t plane = (size_t)A * f * elt_size(cfg);
  char* sv = static_cast<char*>(saved);
  GemmArgs g = {};
  g.tiles = map.tiles; g.ntiles = map.header; g.order = map.order; g.gelu_tab = map.gelu_tab; g.tile_rows = tr;
  g.stream = weights_streamed_from(cfg, tr);
  g.offsets = offsets; g.kept = kept; g.lo = slice_lo; g.hi = slice_hi; g.E = cfg->E;
  // hidden = act(x_perm W1)
  g.A = x_perm; g.B = W1; g.B2 = W1b; g.N = f; g.K = d;
  g.chunked = row_tiles_chunked(A, d, f, cfg->E, swiglu ? 2 : 1, (int)elt_size(cfg));
  g.near = hidden_near(A, f);
  g.C = sv; g.C2 = sv + plane; g.C3 = sv + 2 * plane;
  char* hid = swiglu ? sv + 2 * plane : sv + plane;
  if (saved == nullptr) {   // keep nothing but the hidden activation
    hid = static_cast<char*>(hidden);
    g.C = nullptr; g.C2 = swiglu ? nullptr : hid; g.C3 = swiglu ? hid : nullptr;
  }
  {
    ProfScope ps(cfg, MOE_PROF_GEMM1_FWD, s);
    const int epi = swiglu ? EPI_SWIGLU_FWD : EPI_GELU_FWD;
    if (skinny) CHECK(launch_gemm_half_skinny(cfg->dtype, epi, swiglu, g, max_tiles, s));
    else CHECK(launch_gemm(cfg, MODE_NN, epi, swiglu, false, g, max_tiles, s));
  }
  if (y_perm == nullptr) return MOE_OK;
  // y = hidden W2
  g.A = hid; g.B = W2; g.B2 = nullptr; g.N = d; g.K = f;
  g.chunked = row_tiles_chunked(A, f, d, cfg->E, 1, (int)elt_size(cfg));
  g.C = y_perm; g.C2 = g.C3 = nullptr;
  g.split_all = skinny && skinny_split(cfg->E, f);
  g.split_small = !skinny && splits_small_tiles(cfg);   // split-K: smallest row tiles, last round (gemm.h)
  const bool exact = cfg->capacity == 0 && slice_lo == nullptr;
  g.split_tail = is_half(cfg) && !skinny && tail_may_split(A, cfg->E, exact, (d + 255) / 256, f, tr);
  if (g.split_all || g.split_small || g.split_tail) g.split_ws = reinterpret_cast<float*>(static_cast<char*>(ws) + w.ffn_split);
  ProfScope ps(cfg, MOE_PROF_GEMM2_FWD, s);
  if (skinny) return launch_gemm_half_skinny(cfg->dtype, EPI_STORE, false, g, max_tiles, s);
  return launch_gemm(cfg, MODE_NN, EPI_STORE, false, false, g, max_tiles, s);
}
}  // namespace

int moe_expert_ffn_fwd(const moe_cfg* cfg, const void* x_perm, const void* W1, const void* W1b, const void* W2,
                       const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo, const int32_t* slice_hi,
                       void* saved, void* y_perm, void* ws, size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(x_perm); REQUIRE(W1); REQUIRE(W2); REQUIRE(offsets); REQUIRE(kept); REQUIRE(saved); REQUIRE(y_perm); REQUIRE(ws);
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  if (swiglu) REQUIRE(W1b);
  if (!swiglu && W1b != nullptr) return MOE_ERR_BAD_DTYPE;
  ALIGNED(x_perm); ALIGNED(W1); ALIGNED(W1b); ALIGNED(W2); ALIGNED(offsets); ALIGNED(kept); ALIGNED(slice_lo);
  ALIGNED(slice_hi); ALIGNED(saved); ALIGNED(y_perm); ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  if (cfg->T == 0) return MOE_OK;
  return ffn_fwd_impl(cfg, x_perm, W1, W1b, W2, offsets, kept, slice_lo, slice_hi, saved, nullptr, y_perm, ws,
                      false, (hipStream_t)stream);
}

int moe_expert_ffn_fwd_light(const moe_cfg* cfg, const void* x_perm, const void* W1, const void* W1b, const void* W2,
                             const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo,
                             const int32_t* slice_hi, void* hidden, void* y_perm, void* ws, size_t ws_bytes,
                             void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(x_perm); REQUIRE(W1); REQUIRE(W2); REQUIRE(offsets); REQUIRE(kept); REQUIRE(hidden); REQUIRE(y_perm); REQUIRE(ws);
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  if (swiglu) REQUIRE(W1b);
  if (!swiglu && W1b != nullptr) return MOE_ERR_BAD_DTYPE;
  ALIGNED(x_perm); ALIGNED(W1); ALIGNED(W1b); ALIGNED(W2); ALIGNED(offsets); ALIGNED(kept); ALIGNED(slice_lo);
  ALIGNED(slice_hi); ALIGNED(hidden); ALIGNED(y_perm); ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  if (cfg->T == 0) return MOE_OK;
  return ffn_fwd_impl(cfg, x_perm, W1, W1b, W2, offsets, kept, slice_lo, slice_hi, nullptr, hidden, y_perm, ws,
                      false, (hipStream_t)stream);
}

int moe_expert_ffn_recompute(const moe_cfg* cfg, const void* x_perm, const void* W1, const void* W1b,
                             const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo,
                             const int32_t* slice_hi, void* saved, void* ws, size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(x_perm); REQUIRE(W1); REQUIRE(offsets); REQUIRE(kept); REQUIRE(saved); REQUIRE(ws);
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  if (swiglu) REQUIRE(W1b);
  if (!swiglu && W1b != nullptr) return MOE_ERR_BAD_DTYPE;
  ALIGNED(x_perm); ALIGNED(W1); ALIGNED(W1b); ALIGNED(offsets); ALIGNED(kept); ALIGNED(slice_lo); ALIGNED(slice_hi);
  ALIGNED(saved); ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  if (cfg->T == 0) return MOE_OK;
  return ffn_fwd_impl(cfg, x_perm, W1, W1b, nullptr, offsets, kept, slice_lo, slice_hi, saved, nullptr, nullptr, ws,
                      false, (hipStream_t)stream);
}

int moe_combine(const moe_cfg* cfg, const void* y_perm, const float* topk_w, const int32_t* topk_idx,
                const int32_t* row_of, const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo,
                const int32_t* slice_hi, void* out, int32_t accumulate, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(y_perm); REQUIRE(topk_idx); REQUIRE(row_of); REQUIRE(offsets); REQUIRE(kept); REQUIRE(out);
  ALIGNED(y_perm); ALIGNED(topk_w); ALIGNED(topk_idx); ALIGNED(row_of); ALIGNED(offsets); ALIGNED(kept);
  ALIGNED(slice_lo); ALIGNED(slice_hi); ALIGNED(out);
  if (cfg->T == 0) return MOE_OK;
  ProfScope ps(cfg, MOE_PROF_COMBINE, (hipStream_t)stream);
  return launch_combine(cfg, y_perm, topk_w, topk_idx, row_of, offsets, kept, slice_lo, slice_hi, out, accumulate,
                        (hipStream_t)stream);
}

int moe_combine_bwd(const moe_cfg* cfg, const void* d_out, const void* y_perm, const float* topk_w,
                    const int32_t* topk_idx, const int32_t* row_of, const int32_t* offsets, const int32_t* kept,
                    const int32_t* slice_lo, const int32_t* slice_hi, void* dy_perm, float* d_topk_w, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(d_out); REQUIRE(y_perm); REQUIRE(topk_w); REQUIRE(topk_idx); REQUIRE(row_of); REQUIRE(offsets);
  REQUIRE(kept); REQUIRE(dy_perm); REQUIRE(d_topk_w);
  ALIGNED(d_out); ALIGNED(y_perm); ALIGNED(topk_w); ALIGNED(topk_idx); ALIGNED(row_of); ALIGNED(offsets);
  ALIGNED(kept); ALIGNED(slice_lo); ALIGNED(slice_hi); ALIGNED(dy_perm); ALIGNED(d_topk_w);
  if (cfg->T == 0) return MOE_OK;
  ProfScope ps(cfg, MOE_PROF_COMBINE_BWD, (hipStream_t)stream);
  return launch_combine_bwd(cfg, d_out, y_perm, topk_w, topk_idx, row_of, offsets, kept, slice_lo, slice_hi, dy_perm,
                            d_topk_w, nullptr, (hipStream_t)stream);
}

namespace {
// inputs_only: dA and dx_perm, no weight gradients; dx_sums: room for dx's partial sums (inputs_split_bytes), or NULL
int ffn_bwd_impl(const moe_cfg* cfg, const void* dy_perm, const void* x_perm, const void* saved, const void* W1, const void* W1b,
                 const void* W2, const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo, const int32_t* slice_hi,
                 void* dx_perm, float* dW1, float* dW1b, float* dW2, int32_t accumulate, void* ws, bool map_built, hipStream_t s,
                 bool inputs_only = false, float* dx_sums = nullptr) {
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  const WsLayout w = ws_layout(cfg);
  const int A = cfg->T * cfg->k, d = cfg->d_model, f = cfg->d_ff;
  const TileMapArgs tm = tile_map_args(cfg, offsets, kept, slice_lo, slice_hi, false, ws);
  const TileMap& map = tm.map;
  const int tr = tm.tile_rows, max_tiles = max_row_tiles(A, cfg->E, tr);
  if (!map_built) CHECK(launch_tile_map(tm, s));
  const size_t plane = (size_t)A * f * elt_size(cfg);
  const char* sv = static_cast<const char*>(saved);
  char* dact = static_cast<char*>(ws) + w.ffn_bwd_dact;
  const void* hidden = swiglu ? sv + 2 * plane : sv + plane;
  GemmArgs g = {};
  g.tiles = map.tiles; g.ntiles = map.header; g.order = map.order; g.gelu_tab = map.gelu_tab; g.tile_rows = tr;
  g.stream = weights_streamed_from(cfg, tr);
  g.offsets = offsets; g.kept = kept; g.lo = slice_lo; g.hi = slice_hi; g.E = cfg->E;
  g.accumulate = accumulate;
  // Four GEMMs: dH = dy W2^T fused with the activation derivative -> dA (GELU) or dG, dU (SwiGLU);
  // dW2[e] = H^T dy;  dW1[e] = x_perm^T dA (SwiGLU: dW1 from dG, dW1b from dU);
  // dx_perm = dA W1^T (SwiGLU: dG W1^T + dU W1b^T).
  GemmArgs gh = g, gw2 = g, gw1 = g, gx = g;
  gh.A = dy_perm; gh.B = W2; gh.N = f; gh.K = d; gh.C = dact; gh.C2 = dact + plane; gh.S1 = sv; gh.S2 = sv + plane;
  gw2.A = hidden; gw2.B = dy_perm; gw2.M = f; gw2.N = d;  gw2.C = dW2;
  gw1.A = x_perm; gw1.B = dact; gw1.M = d; gw1.N = f; gw1.C = dW1;
  gx.A = dact; gx.A2 = dact + plane; gx.B = W1; gx.B2 = W1b; gx.N = d; gx.K = f; gx.C = dx_perm;
  gh.chunked = row_tiles_chunked(A, d, f, cfg->E, 1, (int)elt_size(cfg));
  gx.chunked = row_tiles_chunked((swiglu ? 2ll : 1ll) * A, f, d, cfg->E, swiglu ? 2 : 1, (int)elt_size(cfg));
  const int epi_h = swiglu ? EPI_SWIGLU_BWD : EPI_GELU_BWD;
  // A row-tile GEMM with few rounds of tiles shares its launch with the weight-gradient GEMM that follows it (dH with
  // dW2, dx with dW1, and dW1b where there is one), whose tiles then start on the compute units that its last, partly
  // filled round leaves idle.  With many rounds that idle share is small and separate launches keep the cache to one
  // GEMM at a time.  dW1 and dW1b are one launch in any case.  (Timing brackets: a shared launch counts under the
  // row-tile GEMM.)  Three to five launches before: fp32, T 2000, d 516, f 1540, SwiGLU step 743 -> 681 us, T 512, d 128,
  // f 256, GELU 101 -> 92; bf16 SwiGLU (dW1b had its own), 3001 rows, d 1088, f 2880 624 -> 609, 128 experts of 512 rows
  // 3735 -> 3695.
  const bool bf = is_half(cfg);
  const bool pair_h = !inputs_only && shares_launch(cfg, f, max_tiles), pair_x = !inputs_only && shares_launch(cfg, d, max_tiles);
  if (swiglu) { gw1.B2 = dact + plane; gw1.C2 = dW1b; }
  {
    ProfScope ps(cfg, MOE_PROF_DH_BWD, s);
    if (pair_h) CHECK(launch_pair(cfg, epi_h, false, gh, max_tiles, gw2, s));
    else CHECK(launch_gemm(cfg, MODE_NT, epi_h, false, false, gh, max_tiles, s));
  }
  if (!pair_h && !inputs_only) {
    ProfScope ps(cfg, MOE_PROF_DW2_BWD, s);
    CHECK(launch_gemm(cfg, MODE_TN, EPI_DW, false, false, gw2, 0, s));
  }
  if (!pair_x && !inputs_only) {
    ProfScope ps(cfg, MOE_PROF_DW1_BWD, s);
    CHECK(launch_gemm(cfg, MODE_TN, EPI_DW, false, false, gw1, 0, s));
  }
  ProfScope ps(cfg, MOE_PROF_DX_BWD, s);
  // split-K of the GELU dx: the smallest row tiles; the last round only in a launch of its own (in a shared one the
  // weight-gradient tiles fill it), for SwiGLU where the caller gives room for the partial sums
  const bool may_split = !pair_x && tail_may_split(A, cfg->E, cfg->capacity == 0 && slice_lo == nullptr, (d + 255) / 256, swiglu ? 2 * f : f, tr);
  gx.split_small = !swiglu && splits_small_tiles(cfg);
  gx.split_tail = bf && may_split && (dx_sums != nullptr || (!swiglu && !shares_launch(cfg, d, max_tiles)));
  if (gx.split_small || gx.split_tail) gx.split_ws = dx_sums != nullptr ? dx_sums : reinterpret_cast<float*>(static_cast<char*>(ws) + w.ffn_split);
  if (pair_x) return launch_pair(cfg, EPI_STORE, swiglu, gx, max_tiles, gw1, s);
  return launch_gemm(cfg, MODE_NT, EPI_STORE, false, swiglu, gx, max_tiles, s);
}
}  // namespace

int moe_expert_ffn_bwd(const moe_cfg* cfg, const void* dy_perm, const void* x_perm, const void* saved, const void* W1,
                       const void* W1b, const void* W2, const int32_t* offsets, const int32_t* kept,
                       const int32_t* slice_lo, const int32_t* slice_hi, void* dx_perm, float* dW1, float* dW1b,
                       float* dW2, int32_t accumulate, void* ws, size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(dy_perm); REQUIRE(x_perm); REQUIRE(saved); REQUIRE(W1); REQUIRE(W2); REQUIRE(offsets); REQUIRE(kept);
  REQUIRE(dx_perm); REQUIRE(dW1); REQUIRE(dW2); REQUIRE(ws);
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  if (swiglu) { REQUIRE(W1b); REQUIRE(dW1b); }
  if (!swiglu && (W1b != nullptr || dW1b != nullptr)) return MOE_ERR_BAD_DTYPE;
  ALIGNED(dy_perm); ALIGNED(x_perm); ALIGNED(saved); ALIGNED(W1); ALIGNED(W1b); ALIGNED(W2); ALIGNED(offsets);
  ALIGNED(kept); ALIGNED(slice_lo); ALIGNED(slice_hi); ALIGNED(dx_perm); ALIGNED(dW1); ALIGNED(dW1b); ALIGNED(dW2);
  ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  if (cfg->T == 0) return MOE_OK;
  return ffn_bwd_impl(cfg, dy_perm, x_perm, saved, W1, W1b, W2, offsets, kept, slice_lo, slice_hi, dx_perm, dW1, dW1b, dW2, accumulate,
                      ws, false, (hipStream_t)stream);
}

namespace {
// Room for dx's partial sums in a backward that leaves the weight gradients to a later call: the chip has nothing else to
// do beside dx's last round then
size_t inputs_split_bytes(const moe_cfg* c) {
  if (!is_half(c) || (c->act == MOE_ACT_SWIGLU ? 2 : 1) * c->d_ff < SPLIT_MIN_K) return 0;
  const bool small = c->act == MOE_ACT_GELU && splits_small_tiles(c);
  return align_up(std::max(small ? split_ws_bytes(c->E, c->d_model) : 0, tail_ws_bytes(max_row_tiles(c->T * c->k, c->E, tile_rows_for(c)), c->d_model)), 256);
}
// A caller's room for them: refused if it is too small, not used where nothing is split
int check_room(const moe_cfg* c, const void* room, size_t room_bytes, float** sums) {
  ALIGNED(room);
  const size_t need = inputs_split_bytes(c);
  if (room != nullptr && room_bytes < need) return MOE_ERR_WORKSPACE;
  *sums = need > 0 ? static_cast<float*>(const_cast<void*>(room)) : nullptr;
  return MOE_OK;
}
}  // namespace

int moe_expert_ffn_bwd_inputs(const moe_cfg* cfg, const void* dy_perm, const void* saved, const void* W1, const void* W1b, const void* W2,
                              const int32_t* offsets, const int32_t* kept, const int32_t* slice_lo, const int32_t* slice_hi,
                              void* dx_perm, void* room, size_t room_bytes, void* ws, size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  CHECK(check_slices(slice_lo, slice_hi));
  REQUIRE(dy_perm); REQUIRE(saved); REQUIRE(W1); REQUIRE(W2); REQUIRE(offsets); REQUIRE(kept); REQUIRE(dx_perm); REQUIRE(ws);
  if (cfg->act == MOE_ACT_SWIGLU) REQUIRE(W1b);
  else if (W1b != nullptr) return MOE_ERR_BAD_DTYPE;
  ALIGNED(dy_perm); ALIGNED(saved); ALIGNED(W1); ALIGNED(W1b); ALIGNED(W2); ALIGNED(offsets); ALIGNED(kept); ALIGNED(slice_lo);
  ALIGNED(slice_hi); ALIGNED(dx_perm); ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  float* sums = nullptr;
  CHECK(check_room(cfg, room, room_bytes, &sums));
  if (cfg->T == 0) return MOE_OK;
  return ffn_bwd_impl(cfg, dy_perm, nullptr, saved, W1, W1b, W2, offsets, kept, slice_lo, slice_hi, dx_perm, nullptr, nullptr, nullptr, 0, ws, false,
                      (hipStream_t)stream, true, sums);
}

int moe_route_bwd(const moe_cfg* cfg, const void* x, const float* Wr, const int32_t* topk_idx, const float* topk_w,
                  const float* d_topk_w, float* d_logits, float* dWr, void* dx, int32_t accumulate, void* ws,
                  size_t ws_bytes, void* stream) {
  CHECK(check_cfg(cfg));
  REQUIRE(x); REQUIRE(Wr); REQUIRE(topk_idx); REQUIRE(topk_w); REQUIRE(d_topk_w); REQUIRE(d_logits);
  REQUIRE(ws);
  ALIGNED(x); ALIGNED(Wr); ALIGNED(topk_idx); ALIGNED(topk_w); ALIGNED(d_topk_w); ALIGNED(d_logits); ALIGNED(dWr);
  ALIGNED(dx); ALIGNED(ws);
  CHECK(check_ws(cfg, ws, ws_bytes));
  hipStream_t s = (hipStream_t)stream;
  if (cfg->T == 0) {
    if (accumulate || dWr == nullptr) return MOE_OK;
    const int n = cfg->d_model * cfg->E;
    fill_zero_kernel<<<(n + 255) / 256, 256, 0, s>>>(dWr, n);   // a kernel, not a memset: safe under graph capture
    return launch_status();
  }
  const WsLayout w = ws_layout(cfg);
  float* partials = reinterpret_cast<float*>(static_cast<char*>(ws) + w.route_partials);
  float* wrt = reinterpret_cast<float*>(static_cast<char*>(ws) + w.route_wrt);
  return launch_route_bwd(cfg, x, Wr, topk_idx, topk_w, d_topk_w, d_logits, dWr, dx, accumulate != 0, partials, wrt, s);
}

namespace {
// Arguments of the calls that a whole-layer call stands for, checked before anything is launched
int check_layer(const moe_cfg* cfg, const moe_layer_bufs* b, bool combine, bool backward, bool dw = true) {
  CHECK(check_cfg(cfg));
  REQUIRE(b);
  CHECK(check_slices(b->slice_lo, b->slice_hi));
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  REQUIRE(b->x); REQUIRE(b->Wr); REQUIRE(b->W1); REQUIRE(b->topk_idx); REQUIRE(b->topk_w); REQUIRE(b->kept); REQUIRE(b->offsets);
  REQUIRE(b->row_of); REQUIRE(b->x_perm); REQUIRE(b->saved); REQUIRE(b->ws);
  if (!backward) { REQUIRE(b->logits); REQUIRE(b->counts); REQUIRE(b->src_of); }
  if (combine || backward) { REQUIRE(b->W2); REQUIRE(b->y_perm); }
  if (combine) REQUIRE(b->out);
  if (backward) {
    REQUIRE(b->d_out); REQUIRE(b->dy_perm); REQUIRE(b->d_topk_w); REQUIRE(b->dx_perm); REQUIRE(b->dWr); REQUIRE(b->d_logits); REQUIRE(b->dx);
    if (dw) { REQUIRE(b->dW1); REQUIRE(b->dW2); }
  }
  if (swiglu) { REQUIRE(b->W1b); if (backward && dw) REQUIRE(b->dW1b); }
  if (!swiglu && (b->W1b != nullptr || (backward && b->dW1b != nullptr))) return MOE_ERR_BAD_DTYPE;
  const void* const fwd[] = {b->x, b->Wr, b->bias, b->W1, b->W1b, b->W2, b->slice_lo, b->slice_hi, b->logits, b->topk_idx, b->topk_w, b->counts, b->kept,
                             b->offsets, b->row_of, b->src_of, b->x_perm, b->saved, b->y_perm, b->out, b->ws};
  for (const void* p : fwd) ALIGNED(p);
  const void* const bwd[] = {b->d_out, b->dy_perm, b->d_topk_w, b->dx_perm, b->dW1, b->dW1b, b->dW2, b->dWr, b->d_logits, b->dx};
  if (backward)
    for (const void* p : bwd) ALIGNED(p);
  return check_ws(cfg, b->ws, b->ws_bytes);
}
}  // namespace

int moe_layer_fwd(const moe_cfg* cfg, const moe_layer_bufs* b, int32_t mode, void* stream) {
  if (mode < MOE_FWD_FULL || mode > MOE_FWD_RECOMPUTE) return MOE_ERR_BAD_DTYPE;
  CHECK(check_layer(cfg, b, mode != MOE_FWD_RECOMPUTE, false));
  hipStream_t s = (hipStream_t)stream;
  char* ws = static_cast<char*>(b->ws);
  const WsLayout w = ws_layout(cfg);
  if (cfg->T > 0) {
    ProfScope ps(cfg, MOE_PROF_ROUTE, s);
    CHECK(launch_route(cfg, b->x, b->Wr, b->bias, nullptr, b->logits, b->topk_idx, b->topk_w, ws + w.route_wrt, s));
  }
  const SideWork side = side_work(tile_map_args(cfg, b->offsets, b->kept, b->slice_lo, b->slice_hi, true, b->ws), nullptr, nullptr, 0);
  CHECK(launch_dispatch(cfg, b->x, b->topk_idx, b->slice_lo, b->slice_hi, b->counts, b->kept, b->offsets, b->row_of, b->src_of, b->x_perm,
                        reinterpret_cast<int32_t*>(ws + w.dispatch_blk_cnt), &side, s));
  if (cfg->T == 0) return MOE_OK;
  void* hidden = nullptr;
  if (mode == MOE_FWD_LIGHT)
    hidden = static_cast<char*>(b->saved) + (size_t)(cfg->act == MOE_ACT_SWIGLU ? 2 : 1) * cfg->T * cfg->k * cfg->d_ff * elt_size(cfg);
  CHECK(ffn_fwd_impl(cfg, b->x_perm, b->W1, b->W1b, b->W2, b->offsets, b->kept, b->slice_lo, b->slice_hi, mode == MOE_FWD_LIGHT ? nullptr : b->saved,
                     hidden, mode == MOE_FWD_RECOMPUTE ? nullptr : b->y_perm, b->ws, true, s));
  if (mode == MOE_FWD_RECOMPUTE) return MOE_OK;
  ProfScope ps(cfg, MOE_PROF_COMBINE, s);
  return launch_combine(cfg, b->y_perm, b->topk_w, b->topk_idx, b->row_of, b->offsets, b->kept, b->slice_lo, b->slice_hi, b->out, 0, s);
}

namespace {
// room: inputs_split_bytes for dx's partial sums, or NULL
int layer_bwd(const moe_cfg* cfg, const moe_layer_bufs* b, int32_t accumulate, bool inputs_only, float* room, void* stream) {
  CHECK(check_layer(cfg, b, false, true, !inputs_only));
  if (cfg->T == 0)
    return moe_route_bwd(cfg, b->x, b->Wr, b->topk_idx, b->topk_w, b->d_topk_w, b->d_logits, b->dWr, b->dx, accumulate, b->ws, b->ws_bytes, stream);
  hipStream_t s = (hipStream_t)stream;
  char* ws = static_cast<char*>(b->ws);
  const WsLayout w = ws_layout(cfg);
  float *wrt = reinterpret_cast<float*>(ws + w.route_wrt), *partials = reinterpret_cast<float*>(ws + w.route_partials);
  const SideWork side = side_work(tile_map_args(cfg, b->offsets, b->kept, b->slice_lo, b->slice_hi, false, b->ws), b->Wr, wrt, cfg->d_model);
  {
    ProfScope ps(cfg, MOE_PROF_COMBINE_BWD, s);
    CHECK(launch_combine_bwd(cfg, b->d_out, b->y_perm, b->topk_w, b->topk_idx, b->row_of, b->offsets, b->kept, b->slice_lo, b->slice_hi, b->dy_perm,
                             b->d_topk_w, &side, s));
  }
  CHECK(ffn_bwd_impl(cfg, b->dy_perm, b->x_perm, b->saved, b->W1, b->W1b, b->W2, b->offsets, b->kept, b->slice_lo, b->slice_hi, b->dx_perm, b->dW1,
                     b->dW1b, b->dW2, accumulate, b->ws, true, s, inputs_only, room));
  const bool dwr = input_grad_has_dwr(cfg);
  CHECK(launch_input_grad(cfg, b, wrt, partials, dwr, s));
  return launch_gate_dwr(cfg, b->x, b->d_logits, b->dWr, accumulate != 0, partials, dwr, s);
}
}  // namespace

int moe_layer_bwd(const moe_cfg* cfg, const moe_layer_bufs* b, int32_t accumulate, void* stream) { return layer_bwd(cfg, b, accumulate, false, nullptr, stream); }

int moe_layer_bwd_inputs(const moe_cfg* cfg, const moe_layer_bufs* b, int32_t accumulate, void* stream) {
  CHECK(check_layer(cfg, b, false, true, false));
  const size_t room = inputs_split_bytes(cfg), behind = align_up(ws_layout(cfg).total, 256);
  const bool there = room > 0 && b->ws_bytes >= behind + room;
  return layer_bwd(cfg, b, accumulate, true, there ? reinterpret_cast<float*>(static_cast<char*>(b->ws) + behind) : nullptr, stream);
}

int moe_layer_bwd_inputs_in(const moe_cfg* cfg, const moe_layer_bufs* b, void* room, size_t room_bytes, int32_t accumulate, void* stream) {
  CHECK(check_cfg(cfg));
  float* sums = nullptr;
  CHECK(check_room(cfg, room, room_bytes, &sums));
  return layer_bwd(cfg, b, accumulate, true, sums, stream);
}

int moe_layer_bwd_inputs_room_bytes(const moe_cfg* cfg, size_t* bytes) {
  CHECK(check_cfg(cfg));
  REQUIRE(bytes);
  *bytes = inputs_split_bytes(cfg);
  return MOE_OK;
}

int moe_layer_bwd_inputs_ws_bytes(const moe_cfg* cfg, size_t* bytes) {
  CHECK(check_cfg(cfg));
  REQUIRE(bytes);
  *bytes = align_up(ws_layout(cfg).total, 256) + inputs_split_bytes(cfg);
  return MOE_OK;
}

int moe_layer_expert_dw(const moe_cfg* cfg, const moe_layer_bufs* const* calls, int32_t n, int32_t accumulate, void* stream) {
  CHECK(check_cfg(cfg));
  REQUIRE(calls);
  if (n < 1) return MOE_ERR_BAD_SHAPE;
  const bool swiglu = cfg->act == MOE_ACT_SWIGLU;
  for (int i = 0; i < n; ++i) {
    const moe_layer_bufs* b = calls[i];
    REQUIRE(b);
    CHECK(check_slices(b->slice_lo, b->slice_hi));
    REQUIRE(b->offsets); REQUIRE(b->kept); REQUIRE(b->x_perm); REQUIRE(b->saved); REQUIRE(b->dy_perm); REQUIRE(b->ws);
    const void* const in[] = {b->offsets, b->kept, b->slice_lo, b->slice_hi, b->x_perm, b->saved, b->dy_perm, b->ws};
    for (const void* p : in) ALIGNED(p);
    CHECK(check_ws(cfg, b->ws, b->ws_bytes));
  }
  const moe_layer_bufs* out = calls[0];
  REQUIRE(out->dW1); REQUIRE(out->dW2);
  if (swiglu) REQUIRE(out->dW1b);
  if (!swiglu && out->dW1b != nullptr) return MOE_ERR_BAD_DTYPE;
  ALIGNED(out->dW1); ALIGNED(out->dW1b); ALIGNED(out->dW2);
  if (cfg->T == 0) return MOE_OK;
  hipStream_t s = (hipStream_t)stream;
  const WsLayout w = ws_layout(cfg);
  const size_t plane = (size_t)cfg->T * cfg->k * cfg->d_ff * elt_size(cfg);
  auto hidden = [&](const moe_layer_bufs* b) { return static_cast<const char*>(b->saved) + (swiglu ? 2 : 1) * plane; };
  auto dact = [&](const moe_layer_bufs* b) { return static_cast<const char*>(b->ws) + w.ffn_bwd_dact; };
  const int per = is_half(cfg) ? DW_MAX_SEGS : 1;
  for (int i = 0; i < n; i += per) {
    const moe_layer_bufs* b = calls[i];
    GemmArgs g = {};
    g.order = tile_map_args(cfg, b->offsets, b->kept, b->slice_lo, b->slice_hi, false, b->ws).map.order;
    g.offsets = b->offsets; g.kept = b->kept; g.lo = b->slice_lo; g.hi = b->slice_hi; g.E = cfg->E;
    g.accumulate = accumulate || i > 0;
    GemmArgs gw2 = g, gw1 = g;   // dW2[e] = H^T dy;  dW1[e] = x_perm^T dA (SwiGLU: dW1 from dG, dW1b from dU)
    gw2.A = hidden(b); gw2.B = b->dy_perm; gw2.M = cfg->d_ff; gw2.N = cfg->d_model; gw2.C = out->dW2;
    gw1.A = b->x_perm; gw1.B = dact(b); gw1.M = cfg->d_model; gw1.N = cfg->d_ff; gw1.C = out->dW1;
    if (swiglu) { gw1.B2 = dact(b) + plane; gw1.C2 = out->dW1b; }
    ProfScope ps(cfg, MOE_PROF_DW2_BWD, s);
    if (!is_half(cfg)) {
      CHECK(launch_gemm(cfg, MODE_TN, EPI_DW, false, false, gw2, 0, s));
      CHECK(launch_gemm(cfg, MODE_TN, EPI_DW, false, false, gw1, 0, s));
      continue;
    }
    DwSegs s2 = {}, s1 = {};
    s1.n = s2.n = std::min(per, n - i);
    for (int q = 0; q < s1.n; ++q) {
      const moe_layer_bufs* c = calls[i + q];
      s2.A[q] = hidden(c); s2.B[q] = s2.B2[q] = c->dy_perm;
      s1.A[q] = c->x_perm; s1.B[q] = dact(c); s1.B2[q] = dact(c) + (swiglu ? plane : 0);
      s1.offsets[q] = s2.offsets[q] = c->offsets; s1.kept[q] = s2.kept[q] = c->kept;
      s1.lo[q] = s2.lo[q] = c->slice_lo; s1.hi[q] = s2.hi[q] = c->slice_hi;
    }
    CHECK(launch_gemm_half_dw_segs(cfg->dtype, gw2, s2, gw1, s1, s));
  }
  return MOE_OK;
}

}  // extern "C"
