// Grouped GEMM kernel for the gfx950 matrix cores with 16-bit storage: bf16 (v_mfma_f32_16x16x32_bf16) or
// fp16 (v_mfma_f32_16x16x32_f16), fp32 accumulate.  The storage type ST is a template parameter of the one
// kernel; it selects the MFMA instruction, the conversions of the epilogues, and whether the GELU epilogues
// look their function up (bf16: a table over all bf16 numbers fits in LDS) or evaluate it (fp16).
//
// Why the 16 x 16 x 32 instruction and not 32 x 32 x 16 (same FLOP per cycle): the chip lowers its clock under
// matrix-core load, and by how much depends on the instruction.  A loop of nothing but MFMAs (the library's
// moe_bench_mfma_loop), matrix cores busy 99 % of the cycles in both cases, runs 1.14 times faster with
// 16 x 16 x 32 (about 2.0-2.1 PFLOP/s against 1.7-1.9): 32 x 32 x 16 moves twice the accumulator registers per
// FLOP.  In this kernel the change was worth 4-6 % on x W and dy W^T and 1-2 % on x^T dy, and the shader clock
// sampled during a whole layer step rose from 1.66 to 1.80 GHz.
//
// Work decomposition: block tile BM x BN, WGM x WGN waves; a wave owns BN/WGN adjacent columns and the
// 32-row bands b = wm, wm + WGM, ... of the tile, each band two 16-row MFMA tiles; K advances BKT elements
// per stage, 32 per MFMA ("K step").  Interleaving the bands spreads a partly filled row tile over every
// wave row.
//
// Pipeline: LDS stages of 64 K values, two of one operand and three of the other, filled by buffer loads that write LDS
// directly (no staging registers, no LDS store instructions).  An iteration multiplies one stage in two K steps; the first
// reads the fragments of the second, then every wave waits for its own loads of the next stage and joins the
// iteration's one block barrier; the second K step reads the first fragments of the next stage.  The loads of the
// stage after that go where stages have been read: the barrier releases the LDS of this one to the operand with two, that of
// the one before has been free since the last barrier, and the operand with three is loaded in the first K step already.
// 64-wide because a 32-wide stage fetches an operand with contiguous K as 64-byte pieces of 128-byte lines, which fills the address FIFO of the
// memory pipe (counters: full thirteen times as often); the operands with strided K gain a little from the
// halved number of barriers (weight gradients +2 % against a ring of four 32-wide stages).
// 160 KB of LDS hold two stages of 256 x 256 and a third of one operand.  Its loads have half an iteration more to land, and
// those of the other can go first in their half; waits for loads were what the loop lost (two stages of both: 0.27 to 0.40 of the
// wave cycles).  us, two stages of both, requested in the second K step -> three of A -> three of B, as the loads are now (LSH below):
//   16384 rows in 16 skewed experts, d 2048, f 8192, fp16 GELU: GEMM1 632 -> 607 -> 609, y 506 -> 474 -> 473, dH 629 -> 598 -> 603,
//     dW2 636 -> 626 -> 639, dx + dW1 1197 -> 1103 -> 1109; bf16: GEMM1 594 -> 562 -> 563, dx + dW1 1167 -> 1090 -> 1086, step 3604 -> 3402 -> 3421
//   65536 rows in 8, d 4096, f 14336, SwiGLU: GEMM1 12.52 -> 12.15 -> 12.23 ms, y 5.74 -> 5.51 -> 5.50, dH 6.53 -> 6.35 -> 6.39,
//     dW1 + dW1b 11.67 -> 11.63 -> 11.57, dx 12.03 -> 11.10 -> 11.13
//   65536 rows in 128, d 2048, f 1024, SwiGLU: GEMM1 604 -> 540 -> 551, y 335 -> 303 -> 312, dx 575 -> 501 -> 499, dW1 + dW1b 856 -> 876 -> 880
//   16384 rows in 8, d 1024, f 4096, GELU: GEMM1 174 -> 172 -> 178, y 142 -> 129 -> 132, dx + dW1 257 -> 241 -> 249
//   16384 rows in 8, d 2048, f 8192, SwiGLU, dx alone: bf16 1129 -> 945 -> 928, fp16 1146 -> 1001 -> 976
// so three of B where two products are chained (dx of SwiGLU), three of A elsewhere.
// A tile of 160 rows and 256 columns (or twice 128) leaves LDS for three stages of both (156 of 160 KB): loads then have two
// stages' worth of MFMAs to land instead of one, which is what a GEMM of few rows per expert waits for, and the chip is
// left with smaller remainders (512 micro-batch rows per expert, d 1024, f 4096: GEMM1 59 -> 53 us, y 63 -> 53, dx + dW1 116 -> 92).
// It moves 13 % more bytes per product from L2, so 256 rows stay ahead where tiles are
// many and full (the line: mid_applies).  Its five bands of 32 rows go three and two to the two wave rows, one wave of
// either on each SIMD.
// The direct loads are raw instructions: if the compiler knew that they write LDS it would wait for
// every outstanding load before each LDS read it cannot prove disjoint.  The pipeline orders loads and
// reads itself (explicit vmcnt waits, block barriers); the LDS reads stay compiler-tracked.
//
// Operands: one whose K index is contiguous in memory is kept as [rows][BKT] in LDS and read with
// 16-byte LDS reads; one whose K index is strided is kept exactly as it lies in memory, [BKT][cols],
// and read with the transposing 8-byte LDS read of gfx950, so nothing is ever transposed in global
// memory and the same kernel serves x W (NN), dy W^T (NT) and x^T dy (TN).
//
// Epilogue: straight from the accumulators.  The weights are the MFMA's first operand, so that a lane ends up with four
// adjacent columns of one row; exchanges between lanes turn that into 16 bytes per lane and whole 128-byte lines, for
// the outputs and for the saved tensors that the backward epilogues read ("accumulator layout -> memory layout" below).
//
// MFMA 16x16x32 register layout: lane l supplies row/column l%16 and the eight K values (l/16)*8..+7 of
// the step; accumulator register v of lane l is row (l/16)*4 + v of the first operand, row l%16 of the second.
#pragma once
#include "gemm.h"

namespace moe {

typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// What depends on the 16-bit storage type: packing two fp32 values, unpacking, and the MFMA instruction.
template <typename ST> struct Half16;
template <> struct Half16<bf16> {
  static constexpr bool GELU_TABLE = true;
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) { return pack_bf16x2(lo, hi); }
  static __device__ __forceinline__ float lo(uint32_t u) { return __uint_as_float(u << 16); }
  static __device__ __forceinline__ float hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
  static __device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Half16<f16> {
  static constexpr bool GELU_TABLE = false;
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) { return pack_f16x2(lo, hi); }
  static __device__ __forceinline__ float lo(uint32_t u) { return f16_bits_to_f32(u & 0xffffu); }
  static __device__ __forceinline__ float hi(uint32_t u) { return f16_bits_to_f32(u >> 16); }
  static __device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};

constexpr int BKT = 64;   // K values per LDS stage: two MFMA K steps; an operand row with contiguous K is one 128-byte line
// bytes of an LDS stage of either operand and how many stages of it there are: three where the LDS holds them (160 x 256: 156 KB),
// else (256 x 256: 160 KB) three of one operand and two of the other
constexpr int LDS_BYTES = 160 * 1024;
template <int BM> constexpr int gemm_bf16_a_bytes() { return BM * BKT * 2; }
template <int BN, bool DUAL> constexpr int gemm_bf16_b_bytes() { return BN * BKT * 2 * (DUAL ? 2 : 1); }
template <int BM, int BN, bool DUAL>
constexpr bool gemm_bf16_three() { return (gemm_bf16_a_bytes<BM>() + gemm_bf16_b_bytes<BN, DUAL>()) * 3 <= LDS_BYTES; }
template <int BM, int BN, bool DUAL>
constexpr int gemm_bf16_lds_bytes() {
  constexpr int A = gemm_bf16_a_bytes<BM>(), B = gemm_bf16_b_bytes<BN, DUAL>();
  return gemm_bf16_three<BM, BN, DUAL>() ? 3 * (A + B) : 2 * (A + B) + (A > B ? A : B);
}
// ---- LDS layouts -------------------------------------------------------------------------------
// K-contiguous tile: [rows][BKT] bf16.  The 16-byte chunks of a row are XOR-swizzled with the index
// of the 256-byte LDS line the row lies in, so 16 lanes reading the same chunk of 16 consecutive
// rows hit 16 distinct 16-byte bank groups (the LDS serves 64 banks x 4 bytes per clock).
__device__ __forceinline__ int kc_off(int row, int chunk) {
  constexpr int CPR = BKT / 8, RP = 256 / (BKT * 2);
  return row * (BKT * 2) + ((chunk ^ ((row / RP) & (CPR - 1))) << 4);
}
// K-strided tile: [BKT][W] bf16; the 64-byte granules of a K row are XOR-swizzled with k%4, so the four
// K rows that one 16-lane block of a transposing read touches fall into different bank groups, and the
// 32-byte halves of a granule with (k/8)%2, which separates two blocks that read the same columns eight K
// rows apart (counters: no bank conflicts).
template <int W>
__device__ __forceinline__ int ks_off(int krow, int col_byte) {
  return krow * (W * 2) + (col_byte ^ (((krow & 3) << 6) | (((krow >> 3) & 1) << 5)));
}

// Fragment reads.  The eight K values of one lane (column l%16, K chunk l/16 of the step) of a K-strided
// tile come from two transposing reads: the instruction works on blocks of 16 lanes, lane s of a block
// reads 8 bytes at (K row s/4, columns 4*(s%4)..+3) and receives the four K rows of column s; the second
// read lies four K rows further on.  `p` is the lane's address of the first read.
template <int W>
__device__ __forceinline__ bf16x8 lds_read_ks2(const char* p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * W * 2));
  union { struct { s16x4 a, b; } q; bf16x8 v; } u;
  u.q.a = lo;
  u.q.b = hi;
  return u.v;
}

// ---- global -> LDS loads of one stage ------------------------------------------------------------
// Global loads are raw buffer loads: the descriptor's byte count is set to the part of the operand
// this tile may read, and the hardware returns zero for anything past it.  That gives the ragged
// edges (rows past an expert's share, K rows past the share in the weight-gradient GEMM, columns past
// the matrix) for free, with no predicates, no branches and one 32-bit offset register per load.

// One operand tile of one stage, cut into 16-byte chunks; thread tid moves chunks tid + NT*i.
// KC: [ROWS][BKT], chunk id -> (row id/CPR, chunk id%CPR).
// KS: [BKT][ROWS] (ROWS = tile width), chunk id -> (K row id/(ROWS/8), chunk id%(ROWS/8)).
template <bool KC, int ROWS, int NT>
struct Stage {
  static constexpr int CPR = KC ? BKT / 8 : ROWS / 8;
  static constexpr int CH = (ROWS * BKT / 8 + NT - 1) / NT;
  static constexpr int LAST = ROWS * BKT / 8 - (CH - 1) * NT;   // threads that move a chunk with the last load: all, or whole waves
  static_assert(CH >= 1 && LAST % 64 == 0, "a load is made by whole waves");
  // A direct load places lane l of a wave at byte 16*l of the instruction's LDS window, so chunk id
  // lands at byte 16*id of the tile; this is the operand byte offset (pitch in bytes) whose data
  // belongs there: the tile's swizzle, inverted.
  static __device__ __forceinline__ unsigned goff(int i, int tid, unsigned pitch) {
    const int id = tid + NT * i, r = id / CPR, pc = id % CPR;
    if constexpr (KC) {
      constexpr int RP = 256 / (BKT * 2);
      return (unsigned)r * pitch + (unsigned)(pc ^ ((r / RP) & (CPR - 1))) * 16u;
    } else {
      return (unsigned)r * pitch + (unsigned)(pc ^ (((r & 3) << 2) | (((r >> 3) & 1) << 1))) * 16u;
    }
  }
};

// ---- fast activation pieces for bf16 outputs ----------------------------------------------------
__device__ __forceinline__ float sigmoid_fast(float g) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.44269504088896340736f));
}

// Entry of the LDS copy of a GELU table (layout: gemm.h) for the bf16 number with bit pattern `bits`.
__device__ __forceinline__ float gelu_tab_lookup(const float* tab, uint32_t bits) {
  const int m = min(max((int)(bits & 0x7fffu) - (GELU_TAB_EXP0 << 7), 0), GELU_TAB_NMAG - 1);
  return tab[m + (int)(bits >> 15) * GELU_TAB_NMAG];
}

// Four adjacent columns of one row: the accumulator(s) and the saved values (packed) -> the packed 16-bit outputs.
template <typename ST, int EPI>
__device__ __forceinline__ void activate4(const f32x4& a, const f32x4& a2, const u32x2& sv1, const u32x2& sv2, const float* tab,
                                          u32x2& c, u32x2& c2, u32x2& c3) {
  typedef Half16<ST> H;
  auto pk = [](float v0, float v1, float v2, float v3) { return u32x2{H::pack2(v0, v1), H::pack2(v2, v3)}; };
  auto up = [](const u32x2& r, float* f) { f[0] = H::lo(r.x); f[1] = H::hi(r.x); f[2] = H::lo(r.y); f[3] = H::hi(r.y); };
  if constexpr (EPI == EPI_STORE) {
    c = pk(a[0], a[1], a[2], a[3]);
  } else if constexpr (EPI == EPI_GELU_FWD) {
    // h = a Phi(v), v = the pre-activation as stored: GELU of the saved tensor; Phi looked up (bf16) or evaluated (fp16)
    c = pk(a[0], a[1], a[2], a[3]);
    if constexpr (H::GELU_TABLE) {
      c2 = pk(a[0] * gelu_tab_lookup(tab, c.x & 0xffffu), a[1] * gelu_tab_lookup(tab, c.x >> 16),
              a[2] * gelu_tab_lookup(tab, c.y & 0xffffu), a[3] * gelu_tab_lookup(tab, c.y >> 16));
    } else {
      c2 = pk(a[0] * phi_fast(H::lo(c.x)), a[1] * phi_fast(H::hi(c.x)), a[2] * phi_fast(H::lo(c.y)), a[3] * phi_fast(H::hi(c.y)));
    }
  } else if constexpr (EPI == EPI_SWIGLU_FWD) {
    c = pk(a[0], a[1], a[2], a[3]);
    c2 = pk(a2[0], a2[1], a2[2], a2[3]);
    float h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = a[i] * sigmoid_fast(a[i]) * a2[i];
    c3 = pk(h[0], h[1], h[2], h[3]);
  } else if constexpr (EPI == EPI_GELU_BWD) {
    // the derivative at the saved pre-activation: looked up (bf16) or evaluated (fp16)
    if constexpr (H::GELU_TABLE) {
      c = pk(a[0] * gelu_tab_lookup(tab, sv1.x & 0xffffu), a[1] * gelu_tab_lookup(tab, sv1.x >> 16),
             a[2] * gelu_tab_lookup(tab, sv1.y & 0xffffu), a[3] * gelu_tab_lookup(tab, sv1.y >> 16));
    } else {
      c = pk(a[0] * gelu_grad_fast(H::lo(sv1.x)), a[1] * gelu_grad_fast(H::hi(sv1.x)),
             a[2] * gelu_grad_fast(H::lo(sv1.y)), a[3] * gelu_grad_fast(H::hi(sv1.y)));
    }
  } else if constexpr (EPI == EPI_SWIGLU_BWD) {
    float gg[4], uu[4], dg[4], du[4];
    up(sv1, gg);
    up(sv2, uu);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float sg = sigmoid_fast(gg[i]);
      dg[i] = a[i] * uu[i] * sg * fmaf(gg[i], 1.f - sg, 1.f);
      du[i] = a[i] * gg[i] * sg;
    }
    c = pk(dg[0], dg[1], dg[2], dg[3]);
    c2 = pk(du[0], du[1], du[2], du[3]);
  }
}

// ---- accumulator layout -> memory layout ----
// The weights are the MFMA's first operand, so a lane holds four adjacent columns (of group g = lane / 16) of one row
// (lane % 16) per 16 x 16 tile.  Memory wants 16 bytes per lane and whole 128-byte lines per instruction: with half lines
// (the four lanes of a row, 64 bytes) the stores of an fp32 tile take 20 us instead of 13 as streaming stores, and saved
// tensors read by halves cost 10 us more per tile.  Two exchanges between registers and lanes do it, both their own inverse:
//  * join: the odd 16-lane groups of one tile against the even ones of its neighbour (one instruction per register pair):
//    a lane then has eight adjacent columns of the two tiles' 32, from lane_col8(g) on;
//  * swap8: lanes 8-15 of every 16 of one register against lanes 0-7 of another: two registers of 16 rows x 64 bytes
//    become two of 8 rows x 128 bytes.
__device__ __forceinline__ int lane_col8(int g) { return (g & 1) * 16 + (g >> 1) * 8; }
__device__ __forceinline__ u32x2 join16(unsigned a, unsigned b) { return __builtin_amdgcn_permlane16_swap(a, b, false, false); }
__device__ __forceinline__ u32x4 join_tiles(const u32x2& p0, const u32x2& p1) {   // 16-bit: four columns of each -> eight
  const u32x2 x = join16(p0.x, p1.x), y = join16(p0.y, p1.y);
  return u32x4{x.x, y.x, x.y, y.y};
}
__device__ __forceinline__ void join_tiles(f32x4& a, f32x4& b) {    // fp32: a = the first four of the eight columns, b = the rest
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const u32x2 x = join16(__float_as_uint(a[v]), __float_as_uint(b[v]));
    a[v] = __uint_as_float(x.x);
    b[v] = __uint_as_float(x.y);
  }
}
template <typename V>   // u32x4 or f32x4
__device__ __forceinline__ void swap8(V& a, V& b) {
  constexpr int ROR8 = 0x128;
  const u32x4 x = __builtin_bit_cast(u32x4, a), y = __builtin_bit_cast(u32x4, b);
  u32x4 p, q;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    p[v] = (unsigned)__builtin_amdgcn_update_dpp((int)x[v], (int)y[v], ROR8, 0xf, 0xc, false);
    q[v] = (unsigned)__builtin_amdgcn_update_dpp((int)y[v], (int)x[v], ROR8, 0xf, 0x3, false);
  }
  a = __builtin_bit_cast(V, p);
  b = __builtin_bit_cast(V, q);
}

// ---- epilogue accesses through buffer descriptors: 32-bit offsets; what lies past the byte count is not touched ----
// Outputs are streamed, which keeps them from displacing operand panels in the L2 (dH -1.3 %, whole GELU steps -0.4 to
// -1.5 % against plain stores).  What a writer costs the blocks beside it: the two-stage main loop of 128 tiles (K 4096, 34 MB
// of operands) on half of the compute units takes 76 us alone; with 134 | 268 | 537 MB written by others meanwhile (at 4.0 |
// 5.4 | 5.7 TB/s) 84 | 116 | 188 us beside plain stores, 85 | 95 | 122 beside streaming ones, 81 | 93 | 116 if those are written
// through (which takes the writer longer: 56 us instead of 34, 67 instead of 50, 100 instead of 94).  A streaming writer thus
// costs the loops beside it a quarter to half of the time it takes, a plain one all of it and more.
constexpr int AUX_NT = 2;    // streaming access
constexpr int AUX_WT = 18;   // streaming and written through: for half lines
__device__ __forceinline__ __amdgpu_buffer_rsrc_t out_rsrc(const void* base, size_t bytes) {
  const unsigned long long p = (unsigned long long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
  const unsigned n = __builtin_amdgcn_readfirstlane(bytes > 0xffffffffull ? 0xffffffffu : (unsigned)bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(lo | (unsigned long long)hi << 32), 0, (int)n, 0x00020000);
}
template <int AUX>
__device__ __forceinline__ void buf_store16(__amdgpu_buffer_rsrc_t r, unsigned off, const u32x4& v) { __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, AUX); }
__device__ __forceinline__ u32x4 buf_load16_nt(__amdgpu_buffer_rsrc_t r, unsigned off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX_NT); }

// The 16-bit output planes of an epilogue from element `first` on.
struct OutPlanes { __amdgpu_buffer_rsrc_t c, c2, c3; bool pre, near; };   // pre: the forward keeps its pre-activation plane(s); near: GemmArgs.near
template <typename ST, int EPI>
__device__ __forceinline__ OutPlanes out_planes(const GemmArgs& g, size_t first, size_t bytes) {
  auto at = [&](void* base) { return out_rsrc(reinterpret_cast<ST*>(base) + first, bytes); };
  OutPlanes o;
  o.pre = g.C != nullptr;
  o.near = g.near != 0;
  o.c = at(g.C);
  o.c2 = (EPI == EPI_GELU_FWD || EPI == EPI_SWIGLU_FWD || EPI == EPI_SWIGLU_BWD) ? at(g.C2) : o.c;
  o.c3 = EPI == EPI_SWIGLU_FWD ? at(g.C3) : o.c;
  return o;
}
// Forward epilogues of 16 rows x 32 NP columns (NP pairs of tiles), eight columns per lane: NP == 2 leaves as two stores
// of 8 rows x 128 bytes at off[0], off[1], NP == 1 as one of 16 rows x 64 bytes.
template <typename ST, int EPI, int NP, int AUX>
__device__ __forceinline__ void epilogue_fwd(const OutPlanes& o, const unsigned (&off)[NP], const f32x4* a, const f32x4* b, const float* tab) {
  u32x4 v[3][NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    u32x2 c[2] = {}, c2[2] = {}, c3[2] = {};
#pragma unroll
    for (int h = 0; h < 2; ++h) activate4<ST, EPI>(a[2 * q + h], b[EPI == EPI_SWIGLU_FWD ? 2 * q + h : 0], u32x2{}, u32x2{}, tab, c[h], c2[h], c3[h]);
    v[0][q] = join_tiles(c[0], c[1]);
    v[1][q] = join_tiles(c2[0], c2[1]);
    v[2][q] = join_tiles(c3[0], c3[1]);
  }
  auto put = [&](__amdgpu_buffer_rsrc_t r, u32x4* w) {
    if constexpr (NP == 2) swap8(w[0], w[1]);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      if (EPI == EPI_GELU_FWD && w == v[1] && o.near) buf_store16<0>(r, off[q], w[q]);
      else buf_store16<AUX>(r, off[q], w[q]);
    }
  };
  if (EPI == EPI_STORE || o.pre) put(o.c, v[0]);
  if constexpr (EPI == EPI_GELU_FWD) put(o.c2, v[1]);
  if constexpr (EPI == EPI_SWIGLU_FWD) {
    if (o.pre) put(o.c2, v[1]);
    put(o.c3, v[2]);
  }
}

// One output tile; vb = the tile's number in dispatch order.  Block-uniform control flow; returns at
// once for numbers past the last tile (the grid is sized for the worst case).
// SEGS (weight gradients): the K range is that of several calls, one after the other through one pipeline, each call's
// products in a sum of their own that is added to the total: the sums, and their rounding, of call after call.
// STREAM (row tiles): the weights of an expert with a single row tile are requested as streaming data (streamed_from).  A
// template parameter because the choice, once per load, costs a main loop that never takes it 1 to 3 %.
template <typename ST, int MODE, int EPI, bool DUAL, bool CHAIN, int BM, int BN, int WGM, int WGN, bool SEGS = false, bool STREAM = false>
__device__ __forceinline__ void gemm_bf16_tile(const GemmArgs& g, const int vb, char* smem, const DwSegs* segs = nullptr) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = (BM / 32 + WGM - 1) / WGM, WTN = BN / WGN / 32;   // (an odd number of bands: the last wave row has one less)
  constexpr int KS = BKT / 32;               // MFMA K steps per stage
  constexpr int TM = 2 * WTM, TNN = 2 * WTN; // 16 x 16 MFMA tiles of a wave
  constexpr bool A_KC = (MODE != MODE_TN);   // A stored with K contiguous
  constexpr bool B_KC = (MODE == MODE_NT);
  constexpr int A_BYTES = gemm_bf16_a_bytes<BM>(), B_BYTES = BN * BKT * 2, B_STAGE = gemm_bf16_b_bytes<BN, DUAL>();   // B_STAGE: of both matrices
  constexpr bool THREE = gemm_bf16_three<BM, BN, DUAL>(), THREE_B = THREE || CHAIN;
  constexpr int NA = THREE || !THREE_B ? 3 : 2, NB = THREE_B ? 3 : 2, B_AT = NA * A_BYTES;   // LDS: the stages of A, then those of B
  constexpr bool TAB = (EPI == EPI_GELU_BWD || EPI == EPI_GELU_FWD) && Half16<ST>::GELU_TABLE;
  static_assert(KS == 2, "the pipeline below: stages of two K steps");
  static_assert(NA * A_BYTES + NB * B_STAGE <= gemm_bf16_lds_bytes<BM, BN, DUAL>(), "the caller's LDS");
  // the GELU table takes a stage that is free before the loop's last two iterations
  constexpr int TAB_AT = NB == 3 ? B_AT : 0, TAB_STAGE = NB == 3 ? B_STAGE : A_BYTES;
  static_assert(!TAB || TAB_STAGE >= GELU_TAB_FLOATS * 4, "room for the table");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps wave-dependent values scalar
  const int wm = wave / WGN, wn = wave % WGN;

  int e, row0, mvalid, klen, m0 = 0, n0;
  int kbase = 0, skip = 0, part_stages = 0;   // CHAIN: first stage and number of stages of this block's K part (0: all)
  int seg_rows = 0, seg_row0 = 0, seg_stages = 0;          // SEGS: lane s holds segment s's rows and first row; stages in all
  unsigned seg_a[2] = {}, seg_b[2] = {};                   // and its operands' addresses
  bool second = false;          // TN with two gradients: this block's tile is one of the second's (B2, C2)
  bool once = false;            // STREAM: no other row tile takes the same weights, and those of all do not fit the caches
  float* part_sums = nullptr;   // this block computes one K part of a split tile: where its fp32 sums go, and their pitch
  int part_pitch = 0;
  {
    const int ntn = (g.N + BN - 1) / BN;
    int rt, nt;
    if constexpr (MODE == MODE_TN) {
      // weight gradients: tile (expert, m tile, n tile), order in gemm.h (dw_block)
      const int ntm = (g.M + BM - 1) / BM;
      int slot, mt;
      if (!dw_block(vb, ntm, ntn, slot, mt, nt)) return;
      if (g.C2 != nullptr) { slot = __builtin_amdgcn_readfirstlane(slot); second = slot & 1; slot >>= 1; }   // the two gradients of an expert follow each other
      e = g.order[slot];
      m0 = mt * BM;
      rt = 0;
      int l, h;
      if constexpr (SEGS) {
        static_assert(MODE == MODE_TN, "weight gradients");
        int all = 0;
#pragma unroll
        for (int q = 0; q < DW_MAX_SEGS; ++q)
          if (q < segs->n) {
            share_of(segs->lo[q], segs->hi[q], segs->kept[q][e], e, l, h);
            const unsigned long long pa = (unsigned long long)segs->A[q], pb = (unsigned long long)(second ? segs->B2[q] : segs->B[q]);
            if (lane == q) {
              seg_rows = h - l;
              seg_row0 = segs->offsets[q][e] + l;
              seg_a[0] = (unsigned)pa; seg_a[1] = (unsigned)(pa >> 32);
              seg_b[0] = (unsigned)pb; seg_b[1] = (unsigned)(pb >> 32);
            }
            all += (h - l + BKT - 1) / BKT;
          }
        seg_stages = __builtin_amdgcn_readfirstlane(all);
        row0 = 0;
        klen = seg_stages;
      } else {
        share_of(g.lo, g.hi, g.kept[e], e, l, h);
        row0 = g.offsets[e] + l;
        klen = h - l;
      }
      mvalid = min(BM, g.M - m0);
      if (klen == 0 && g.accumulate) return;
    } else {
      constexpr bool CAN_SPLIT = EPI == EPI_STORE;
      const int kall = CHAIN ? 2 * g.K : g.K;
      const int n_rt = g.ntiles[0];
      RowBlock rb;
      klen = g.K;
      TailSplit ts = {0, 1};
      if (CAN_SPLIT && g.split_tail) ts = tail_split(n_rt * ntn, kall);
      if (CAN_SPLIT && ts.parts > 1) {          // the tiles of the last round are split along K
        if (!tail_split_block(vb, n_rt, g.ntiles[1], ntn, g.chunked != 0, ts, rb)) return;
        if (rb.split_tile >= 0) {
          const int stages = kall / BKT, k0 = rb.ksplit * stages / ts.parts, k1 = (rb.ksplit + 1) * stages / ts.parts;
          if constexpr (CHAIN) { skip = k0; part_stages = k1 - k0; }
          else { kbase = k0 * BKT; klen = (k1 - k0) * BKT; }
          part_sums = g.split_ws + (size_t)(rb.split_tile * ts.parts + rb.ksplit) * (BM * BN);
          part_pitch = BN;
        }
      } else {
        // or the smallest row tiles: the last n_sp row tiles are not part of the regular numbering; their blocks
        // follow it, SPLIT_K per (row tile, column tile), each with a K range of its own
        const int n_sp = (CAN_SPLIT && !CHAIN && g.split_small) ? g.ntiles[2] : 0;
        if (!row_tile_block(vb, n_rt, g.ntiles[1], n_sp, ntn, g.chunked != 0, rb)) return;
        if (CAN_SPLIT && !CHAIN && rb.split_tile >= 0) {
          klen = g.K / SPLIT_K;
          kbase = rb.ksplit * klen;
          part_sums = g.split_ws + (size_t)(rb.split_tile * SPLIT_K + rb.ksplit) * SPLIT_ROWS * g.N + rb.nt * BN;
          part_pitch = g.N;
        }
      }
      // block-uniform, but divided in vector registers: back to scalar ones
      rt = __builtin_amdgcn_readfirstlane(rb.rt);
      nt = __builtin_amdgcn_readfirstlane(rb.nt);
      kbase = __builtin_amdgcn_readfirstlane(kbase);
      klen = __builtin_amdgcn_readfirstlane(klen);
      skip = __builtin_amdgcn_readfirstlane(skip);
      part_stages = __builtin_amdgcn_readfirstlane(part_stages);
      const RowTile t = g.tiles[rt];
      e = t.e;
      row0 = t.row0;
      mvalid = t.nrows;
      if constexpr (STREAM) once = __builtin_amdgcn_readfirstlane(t.mates) == 0 && n_rt >= g.stream;
    }
    n0 = nt * BN;
  }
  const int nvalid = min(BN, g.N - n0);

  f32x4 acc[TM][TNN], acc2[DUAL ? TM : 1][DUAL ? TNN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TNN; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (DUAL) acc2[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  f32x4 total[SEGS ? TM : 1][SEGS ? TNN : 1] = {};

  const int KT = (klen + BKT - 1) / BKT;
  int tab_stage = 0;   // the stage that ends up with the GELU table
  // MFMA row bands of this wave that contain valid rows
  // (row band b of the tile belongs to wave row b % WGM, as its band b / WGM: a partly filled tile then
  // spreads its valid bands over all wave rows instead of loading the first ones only)
  const int ni = (MODE == MODE_TN) ? WTM : min(max(((mvalid + 31) / 32 - wm + WGM - 1) / WGM, 0), WTM);
  typedef Stage<A_KC, BM, NT> StA;
  typedef Stage<B_KC, BN, NT> StB;

  // fragment read offsets inside a stage.  Lane l of a 16 x 16 x 32 MFMA holds row (column) l % 16 and the
  // eight K values of chunk l / 16.  K-contiguous: one offset per K step (MFMA tiles are a constant 16 rows
  // apart); K-strided: one per MFMA tile (K steps are a constant apart).
  int a_fr[A_KC ? KS : TM], b_fr[B_KC ? KS : TNN];
  if constexpr (A_KC) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a_fr[ks] = kc_off(wm * 32 + (lane & 15), ks * 4 + (lane >> 4));
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
      a_fr[i] = ks_off<BM>((lane >> 4) * 8 + ((lane & 15) >> 2),
                           (((i >> 1) * WGM + wm) * 32 + (i & 1) * 16 + (lane & 3) * 4) * 2);
  }
  if constexpr (B_KC) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      b_fr[ks] = B_AT + kc_off(wn * WTN * 32 + (lane & 15), ks * 4 + (lane >> 4));
  } else {
#pragma unroll
    for (int j = 0; j < TNN; ++j)
      b_fr[j] = B_AT + ks_off<BN>((lane >> 4) * 8 + ((lane & 15) >> 2),
                                  (wn * WTN * 32 + j * 16 + (lane & 3) * 4) * 2);
  }

  {
    // operand bases of this tile (a chained GEMM has two operand pairs and runs their K ranges back to
    // back through one pipeline), byte counts the tile may read, pitches and the advance per K stage
    const bf16* A0 = reinterpret_cast<const bf16*>(g.A);
    const bf16* A1 = reinterpret_cast<const bf16*>(CHAIN ? g.A2 : g.A);
    const bf16* B0 = reinterpret_cast<const bf16*>(MODE == MODE_TN && second ? g.B2 : g.B);
    const bf16* B1 = reinterpret_cast<const bf16*>(g.B2);   // SwiGLU: second weight matrix
    size_t aoff, boff, abytes, bbytes;
    unsigned pa, pb, astep, bstep;
    if constexpr (MODE == MODE_TN) {
      // A = [rows][M] from (row0, m0), B = [rows][N] from (row0, n0); rows past the share read as zero
      aoff = (size_t)row0 * g.M + m0;  abytes = ((size_t)klen * g.M - m0) * 2;
      boff = (size_t)row0 * g.N + n0;  bbytes = ((size_t)klen * g.N - n0) * 2;
      pa = g.M * 2; pb = g.N * 2; astep = BKT * pa; bstep = BKT * pb;
    } else if constexpr (MODE == MODE_NN) {
      // A = [rows][K] rows row0..row0+mvalid; B = W_e [K][N] from column n0; both from K index kbase on
      aoff = (size_t)row0 * g.K + kbase;  abytes = ((size_t)mvalid * g.K - kbase) * 2;
      boff = ((size_t)e * g.K + kbase) * g.N + n0;  bbytes = ((size_t)(g.K - kbase) * g.N - n0) * 2;
      pa = g.K * 2; pb = g.N * 2; astep = BKT * 2; bstep = BKT * pb;
    } else {
      // A as above; B = W_e [N][K] rows n0..N
      aoff = (size_t)row0 * g.K + kbase;  abytes = ((size_t)mvalid * g.K - kbase) * 2;
      boff = ((size_t)e * g.N + n0) * g.K + kbase;  bbytes = ((size_t)(g.N - n0) * g.K - kbase) * 2;
      pa = g.K * 2; pb = g.K * 2; astep = BKT * 2; bstep = BKT * 2;
    }
    rsrc_t ra = make_rsrc(A0 + aoff, abytes), rb = make_rsrc(B0 + boff, bbytes);
    const rsrc_t ra1 = make_rsrc(A1 + aoff, abytes), rb1 = make_rsrc(B1 + boff, bbytes);
    // SEGS: the segment whose stages are being requested, the next stage of it and how many it has; stages are requested
    // strictly in order, and never more than there are, so a segment with rows follows whenever one is asked for
    int seg = -1, seg_k = 0, seg_n = 0;
    auto next_stage = [&]() {
      if (seg_k < seg_n) return;
      int rows;
      do rows = __builtin_amdgcn_readlane(seg_rows, ++seg); while (rows == 0 && seg + 1 < DW_MAX_SEGS);
      const size_t r0 = __builtin_amdgcn_readlane(seg_row0, seg);
      const unsigned long long a = (unsigned)__builtin_amdgcn_readlane(seg_a[0], seg) | (unsigned long long)(unsigned)__builtin_amdgcn_readlane(seg_a[1], seg) << 32;
      const unsigned long long b = (unsigned)__builtin_amdgcn_readlane(seg_b[0], seg) | (unsigned long long)(unsigned)__builtin_amdgcn_readlane(seg_b[1], seg) << 32;
      ra = make_rsrc(reinterpret_cast<const bf16*>(a) + r0 * g.M + m0, ((size_t)rows * g.M - m0) * 2);
      rb = make_rsrc(reinterpret_cast<const bf16*>(b) + r0 * g.N + n0, ((size_t)rows * g.N - n0) * 2);
      seg_k = 0;
      seg_n = (rows + BKT - 1) / BKT;
    };
    int mul_seg = -1, mul_end = 0;   // SEGS: the segment that is being multiplied and the stage behind its last
    auto next_product = [&]() {
      int rows;
      do rows = __builtin_amdgcn_readlane(seg_rows, ++mul_seg); while (rows == 0 && mul_seg + 1 < DW_MAX_SEGS);
      mul_end += (rows + BKT - 1) / BKT;
    };
    auto end_of_stage = [&](int stage) {   // the last one of a segment: its sum joins the total
      if (stage + 1 != mul_end) return;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TNN; ++j) {
          total[SEGS ? i : 0][SEGS ? j : 0] += acc[i][j];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      if (mul_end < seg_stages) next_product();
    };
    const int KT1 = KT;                      // stages of one operand pair
    const int KTT = SEGS ? seg_stages : !CHAIN ? KT1 : part_stages > 0 ? part_stages : 2 * KT1;   // stages in all
    tab_stage = KTT % 3;
    constexpr int LB = StB::CH * (DUAL ? 2 : 1), L = StA::CH + LB;   // loads per thread per stage: of B, in all
    constexpr int LA_MIN = StA::CH - (StA::LAST < NT ? 1 : 0);       // of A by the waves that sit out the last one
    // Which K step makes a stage's loads (numbered q, below): where one operand has two LDS stages, its LSH loads are K step 1's,
    // in the first half of its regions, and those of the other are K step 0's, over all of its regions; else all are K step 1's.
    // (All in K step 1 -> as it is, us: SwiGLU, 65536 rows in 8 experts, d 4096, f 14336, GEMM1 12150 -> 12100, dx 11190 -> 10940, dH
    // 6360 -> 6290, dW 8670 -> 8570, y 5440 -> 5440; in 128, d 2048, f 1024, GEMM1 588 -> 569, y 324 -> 309, dx 539 -> 514; fp16 GELU, 16384
    // in 16, d 2048, f 8192, dx + dW1 1167 -> 1120, dH 628 -> 611.  K step 1's over all its regions: dx of the first 11630; in the
    // first quarter: 10980.)
    constexpr int LSH = THREE ? L : NB == 2 ? LB : StA::CH;
    constexpr int B_Q = NB == 2 ? 0 : StA::CH, A_Q = NB == 2 ? LB : 0;   // where the loads of B and of A start among a stage's
    static_assert(StB::LAST == NT, "whole loads of B");
    static_assert(!SEGS || NA == NB, "a segment's operands are requested together");
    constexpr int DEPTH = THREE ? 3 : 2;                      // stages requested before the loop
    constexpr int PEND = (DEPTH - 1) * (LA_MIN + LB);         // loads that may stay in flight at the prologue's barrier: all but stage 0's
    constexpr int AHEAD_MIN = (NA == 3 ? LA_MIN : 0) + (NB == 3 ? LB : 0);    // of the newest stage that may stay in flight in the loop: A's alone where B has two
    static_assert(PEND < 64 && AHEAD_MIN < 16, "the wait counter has six bits");
    constexpr int WAIT_P = (PEND & 15) | ((PEND >> 4) << 14) | 0x70 | (15 << 8);   // s_waitcnt vmcnt(PEND) only
    constexpr int WAIT_0 = 0x70 | (15 << 8);                                       // s_waitcnt vmcnt(0) only
    constexpr int WAIT_AHEAD = AHEAD_MIN | 0x70;                                   // s_waitcnt vmcnt(AHEAD_MIN) lgkmcnt(0)
    constexpr int WAIT_LGKM0 = 0xC07F;                                             // s_waitcnt lgkmcnt(0) only
    unsigned a_vo[StA::CH], b_vo[StB::CH];
#pragma unroll
    for (int i = 0; i < StA::CH; ++i) a_vo[i] = StA::goff(i, tid, pa);
#pragma unroll
    for (int i = 0; i < StB::CH; ++i) b_vo[i] = StB::goff(i, tid, pb);
    const int wbase = wave * 1024;   // a wave's 64 lanes fill 1 KB of the tile per load
    const unsigned smem_base = lds_addr(smem);
    // A K step is the 32 K values of one MFMA: TM x TNN instructions per wave, cut into TM regions that the
    // scheduler may not move instructions across (sched_barrier).  Region i holds the MFMAs of row tile i;
    // behind them, the read of row tile i's A fragment for the NEXT K step, into the same registers (their
    // last use has just been issued, and the fragment is not needed for another TM - 1 regions), in the
    // first TNN regions one B fragment of the next step (into the other of two B register sets), and this
    // region's share of the global -> LDS loads.  LDS reads and, above all, the global loads then arrive as a
    // steady trickle: loads issued in one burst fill the address FIFO of the memory pipe, and a wave that
    // cannot issue a load cannot issue the MFMAs behind it either.
    constexpr int NR = TM;                           // regions per K step
    auto load_region = [](int q) { return THREE ? q * NR / L : q < LSH ? q * NR / (2 * LSH) : (q - LSH + 1) * NR / (L - LSH) - 1; };
    static_assert(THREE || NR % (L - LSH) == 0, "every load has a region");
    bf16x8 af[TM], bfr[2][TNN], bfr2[2][DUAL ? TNN : 1];
// load q_ of a stage: the chunks of A and those of B (DUAL: both weight matrices in turn).  Where B has two stages, its loads go
// first: they have to land an iteration earlier
#define MOE_LOAD1(akt_, abuf_, bkt_, bbuf_, q_)                                                             \
  do {                                                                                                      \
    const int kq__ = SEGS ? seg_k : ((q_) >= B_Q && (q_) < B_Q + LB ? (bkt_) : (akt_)) + (CHAIN ? skip : 0);                     \
    const bool sec__ = CHAIN && kq__ >= KT1;                                                                \
    const unsigned kl__ = (unsigned)(sec__ ? kq__ - KT1 : kq__);                                            \
    if ((q_) >= B_Q && (q_) < B_Q + LB) {                                                                   \
      const int c__ = ((q_) - B_Q) / (DUAL ? 2 : 1);                                                        \
      const unsigned st__ = smem_base + B_AT + (bbuf_) + wbase + NT * 16 * c__;                             \
      const bool first__ = !DUAL || ((q_) - B_Q) % 2 == 0;                                                  \
      if (STREAM && once)                                                                                   \
        load_to_lds16_nt(!first__ || sec__ ? rb1 : rb, st__ + (first__ ? 0 : B_BYTES), b_vo[c__] + kl__ * bstep); \
      else load_to_lds16(!first__ || sec__ ? rb1 : rb, st__ + (first__ ? 0 : B_BYTES), b_vo[c__] + kl__ * bstep); \
    } else {                                                                                                \
      const int c__ = (q_) - A_Q;                                                                           \
      if (c__ < StA::CH - 1 || StA::LAST == NT || wave < StA::LAST / 64)                                    \
        load_to_lds16(sec__ ? ra1 : ra, smem_base + (abuf_) + wbase + NT * 16 * c__, a_vo[c__] + kl__ * astep); \
    }                                                                                                       \
  } while (0)
// A fragment of row tile i_ / B fragment(s) of column tile j_ for K step ks_ of the stage at buf_
#define MOE_FRAG_A(i_, buf_, ks_)                                                                           \
  do {                                                                                                      \
    const char* st__ = smem + (buf_);                                                                       \
    if constexpr (A_KC)                                                                                     \
      af[i_] = *reinterpret_cast<const bf16x8*>(st__ + a_fr[ks_] + ((i_) >> 1) * WGM * 32 * BKT * 2 + ((i_) & 1) * 16 * BKT * 2); \
    else af[i_] = lds_read_ks2<BM>(st__ + a_fr[i_] + (ks_) * 32 * BM * 2);                                  \
  } while (0)
#define MOE_FRAG_B(set_, j_, buf_, ks_)                                                                     \
  do {                                                                                                      \
    const char* st__ = smem + (buf_);                                                                       \
    if constexpr (B_KC) bfr[set_][j_] = *reinterpret_cast<const bf16x8*>(st__ + b_fr[ks_] + (j_) * 16 * BKT * 2); \
    else bfr[set_][j_] = lds_read_ks2<BN>(st__ + b_fr[j_] + (ks_) * 32 * BN * 2);                           \
    if constexpr (DUAL) bfr2[set_][j_] = lds_read_ks2<BN>(st__ + B_BYTES + b_fr[j_] + (ks_) * 32 * BN * 2); \
  } while (0)
#define MOE_FRAGS(set_, abuf_, bbuf_, ks_)                                                                  \
  do {                                                                                                      \
    _Pragma("unroll") for (int i__ = 0; i__ < TM; ++i__) MOE_FRAG_A(i__, abuf_, ks_);                       \
    _Pragma("unroll") for (int j__ = 0; j__ < TNN; ++j__) MOE_FRAG_B(set_, j__, bbuf_, ks_);                \
  } while (0)
// One K step on B register set set_; DO_NEXT_: read the fragments of K step rks_ of the stages at rabuf_, rbbuf_;
// request the loads Q0_ .. Q1_-1 of stage S_+DEPTH.
#define MOE_STEP(set_, DO_NEXT_, rabuf_, rbbuf_, rks_, S_, Q0_, Q1_, NI_)                                  \
  do {                                                                                                      \
    _Pragma("unroll") for (int r__ = 0; r__ < NR; ++r__) {                                                  \
      if ((r__ >> 1) < (NI_)) {                                                                             \
        _Pragma("unroll") for (int j__ = 0; j__ < TNN; ++j__) {                                             \
          acc[r__][j__] = Half16<ST>::mfma(bfr[set_][j__], af[r__], acc[r__][j__]);                         \
          if constexpr (DUAL) acc2[r__][j__] = Half16<ST>::mfma(bfr2[set_][j__], af[r__], acc2[r__][j__]);  \
        }                                                                                                   \
      }                                                                                                     \
      if (DO_NEXT_) {                                                                                       \
        MOE_FRAG_A(r__, rabuf_, rks_);                                                                      \
        if (r__ < TNN) MOE_FRAG_B((set_) ^ 1, r__ < TNN ? r__ : 0, rbbuf_, rks_);                           \
      }                                                                                                     \
      _Pragma("unroll") for (int q__ = 0; q__ < L; ++q__)                                                   \
        if (q__ >= (Q0_) && q__ < (Q1_) && load_region(q__) == r__)                                         \
          MOE_LOAD1((S_) + DEPTH, THREE || NA == 2 ? a0 : a2, (S_) + DEPTH, THREE || NB == 2 ? bb0 : bb2, q__); \
      __builtin_amdgcn_sched_barrier(0);                                                                    \
    }                                                                                                       \
  } while (0)
#define MOE_BLOCK_BARRIER()                                                                                 \
  do {                                                                                                      \
    asm volatile("" ::: "memory");                                                                          \
    __builtin_amdgcn_s_barrier();                                                                           \
    asm volatile("" ::: "memory");                                                                          \
  } while (0)
    // GELU table into LDS at `at`, 1 KB per wave and instruction
    auto load_table = [&](unsigned at) {
      static_assert(GELU_TAB_FLOATS * 4 % (NT * 16) == 0, "whole block-wide loads");
      const rsrc_t rt = make_rsrc(g.gelu_tab, (size_t)GELU_TAB_FLOATS * 4);
      const unsigned to = __builtin_amdgcn_readfirstlane(smem_base + at + wbase);
#pragma unroll
      for (int i = 0; i < GELU_TAB_FLOATS * 4 / (NT * 16); ++i)
        load_to_lds16(rt, to + i * NT * 16, (unsigned)(i * NT + tid) * 16u);
    };
    {
      // Iteration S multiplies stage S (two K steps).  K step 0 reads the fragments of K step 1; then every wave waits for its
      // own loads of stage S+1 (of stage S+2 those stay in flight that are made by now: all, with three stages of both, else
      // this K step's) and for its fragment reads and joins the one block barrier of the iteration, after which stage S+1 is
      // visible to all and nobody reads stage S's LDS again; K step 1 reads the fragments of step 0 of stage S+1.
      // DO_LOAD_: stage S+DEPTH is requested; MORE_: stage S+2 exists and is on its way.
#define MOE_ITER(S_, DO_NEXT_, DO_LOAD_, MORE_, NI_)                                                        \
  do {                                                                                                      \
    MOE_STEP(0, true, a0, bb0, 1, S_, LSH, !THREE && (DO_LOAD_) ? L : 0, NI_);                              \
    if (DO_NEXT_) {                                                                                         \
      if (MORE_) __builtin_amdgcn_s_waitcnt(WAIT_AHEAD);                                                    \
      else __builtin_amdgcn_s_waitcnt(0);   /* vmcnt(0) lgkmcnt(0) */                                       \
      MOE_BLOCK_BARRIER();                                                                                  \
    }                                                                                                       \
    if constexpr (SEGS) { if (DO_LOAD_) next_stage(); }                                                     \
    MOE_STEP(1, DO_NEXT_, a1, bb1, 0, S_, 0, (DO_LOAD_) ? LSH : 0, NI_);                                    \
    if constexpr (SEGS) { if (DO_LOAD_) ++seg_k; }                                                          \
    if constexpr (NA == 2) { const int t__ = a0; a0 = a1; a1 = t__; }                                       \
    else { const int t__ = a0; a0 = a1; a1 = a2; a2 = t__; }                                                   \
    if constexpr (NB == 2) { const int t__ = bb0; bb0 = bb1; bb1 = t__; }                                   \
    else { const int t__ = bb0; bb0 = bb1; bb1 = bb2; bb2 = t__; }                                          \
  } while (0)
      if (KTT > 0) {
        if constexpr (SEGS) next_product();
        int a0 = 0, a1 = A_BYTES, a2 = NA == 3 ? 2 * A_BYTES : 0, bb0 = 0, bb1 = B_STAGE, bb2 = NB == 3 ? 2 * B_STAGE : 0;
#pragma unroll
        for (int q = 0; q < DEPTH; ++q)
          if (q < KTT) {
            if constexpr (SEGS) next_stage();
#pragma unroll
            for (int l = 0; l < L; ++l)
              MOE_LOAD1(q, q * A_BYTES, q, q * B_STAGE, l);
            if constexpr (SEGS) ++seg_k;
          }
        if (KTT >= 3 || (!TAB && KTT >= DEPTH)) {
          __builtin_amdgcn_s_waitcnt(WAIT_P);   // stage 0 has landed, the others may be in flight
        } else {
          if constexpr (TAB) load_table(TAB_AT + KTT * TAB_STAGE);
          __builtin_amdgcn_s_waitcnt(WAIT_0);
        }
        MOE_BLOCK_BARRIER();
        // the table takes the place of stage KTT - 3, free from that iteration's barrier on; the wait and the barrier of the next
        // iteration make it visible to all.
        // CHAIN: the empty asm, another one in each copy of the loop, keeps the copies' first reads in them.  Hoisted in front, as
        // equal code, they took registers beside the loop's own, and nine to eleven others were spilled; with STREAM two of those
        // were reloaded in every iteration, which waits for all loads in flight.  dx of 200 rows per expert in 256, d 2048, f 1024,
        // bf16 570 -> 457 us, fp16 582 -> 474 (plain loads, nothing reloaded in the loop: 472, 490); in 64, d 2048, f 2048 289 -> 268 (285).
#define MOE_MAINLOOP(NI_)                                                                        \
  do {                                                                                          \
    if constexpr (CHAIN) asm volatile("; " #NI_ ::: "memory");                                  \
    MOE_FRAGS(0, a0, bb0, 0);                                                                   \
    __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);   /* nothing pending at the loop head: the waits inside the loop then count only its own reads */ \
    int S = 0;                                                                                  \
    _Pragma("unroll 1") for (; S + DEPTH < KTT; ++S) {                                              \
      MOE_ITER(S, true, true, true, NI_);                                                          \
      if constexpr (SEGS) end_of_stage(S);                                                      \
    }                                                                                           \
    _Pragma("unroll 1") for (; S < KTT; ++S) {                                                   \
      if constexpr (TAB) { if (S + 2 == KTT && S > 0) load_table(TAB_AT + (NB == 3 ? bb2 : a2)); } \
      MOE_ITER(S, S + 1 < KTT, false, THREE && S + 2 < KTT, NI_);                               \
      if constexpr (SEGS) end_of_stage(S);                                                      \
    }                                                                                           \
  } while (0)
        if (ni == WTM) MOE_MAINLOOP(WTM);
        else if (NB == 3 && ni == WTM - 1) MOE_MAINLOOP(WTM - 1);
        else MOE_MAINLOOP(ni);
#undef MOE_MAINLOOP
      }
#undef MOE_ITER
    }
#undef MOE_LOAD1
#undef MOE_FRAG_A
#undef MOE_FRAG_B
#undef MOE_FRAGS
#undef MOE_STEP
#undef MOE_BLOCK_BARRIER
  }

  // Epilogue, straight from the accumulators (layouts above).  A wave's columns are all valid or all past the matrix
  // (widths are multiples of 64).  A round trip through LDS took 2.4-2.7 us per tile instead.  Launches of four rounds,
  // with it -> without, us: plain store x W K 1024 132 -> 123, GELU forward 157 -> 150, GELU backward 163 -> 155, weight
  // gradient of 1024 rows 153 -> 143; at K 4096 1-2 %; the SwiGLU epilogues (two planes in, two out) stay within 1 %.
  // What is left is the memory's time: 128 KB per plane and tile, 4 us, of which blocks that are out of step hide about half
  // (what a writer costs: AUX_NT above).
  constexpr int C = WTN * 32;
  if (wn * C >= nvalid) return;
  if constexpr (SEGS) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TNN; ++j) acc[i][j] = total[i][j];
  }
  const int grp = lane >> 4, r8 = lane & 7, right = (lane >> 3) & 1;   // after swap8: row of eight, left or right half of a line
  auto band_row = [&](int i) { return ((i >> 1) * WGM + wm) * 32 + (i & 1) * 16; };   // first row of row tile i
  auto empty = [&](int i) { return band_row(i) >= mvalid; };
  if (MODE != MODE_TN && EPI == EPI_STORE && part_sums != nullptr) {   // fp32 partial sums of this block's K part
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if (!empty(i)) {
#pragma unroll
        for (int j = 0; j < TNN; j += 2) {
          swap8(acc[i][j], acc[i][j + 1]);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int m = band_row(i) + h * 8 + r8;
            if (m < mvalid) *reinterpret_cast<f32x4*>(part_sums + (size_t)m * part_pitch + wn * C + j * 16 + right * 16 + grp * 4) = acc[i][j + h];
          }
        }
      }
    return;
  }
  if constexpr (MODE == MODE_TN) {   // fp32 weight gradient of expert e; M is a multiple of 64: whole bands
    static_assert(TNN % 2 == 0, "pairs of column tiles");
    const size_t first = ((size_t)e * g.M + m0) * g.N + n0;
    const __amdgpu_buffer_rsrc_t rc = out_rsrc(reinterpret_cast<float*>(second ? g.C2 : g.C) + first, ((size_t)mvalid * g.N - n0) * 4);
    const unsigned col = (unsigned)(wn * C + right * 16 + grp * 4) * 4u, pitch = (unsigned)g.N * 4u;
    auto at = [&](int i, int j) { return (unsigned)(band_row(i) + (j & 1) * 8 + r8) * pitch + col + (unsigned)(j >> 1) * 128u; };
    auto rows_of_8 = [&](int i) {
#pragma unroll
      for (int j = 0; j < TNN; j += 2) swap8(acc[i][j], acc[i][j + 1]);
    };
    if (g.accumulate) {
      // The old values are requested AHEAD row tiles ahead, so that a row tile's latency runs beside the others' sums.
      // (Loaded piece by piece between the stores, which the compiler must not move a load across, this is a chain of
      // memory round trips: 21-25 us per tile against 4 without accumulation.)
      constexpr int AHEAD = 4;
      u32x4 old[AHEAD][TNN];
      auto load_old = [&](int i) {
#pragma unroll
        for (int j = 0; j < TNN; ++j) old[i % AHEAD][j] = buf_load16_nt(rc, empty(i) ? OUT_OF_RANGE : at(i, j));
      };
#pragma unroll
      for (int i = 0; i < AHEAD - 1; ++i) load_old(i);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (i + AHEAD - 1 < TM) load_old(i + AHEAD - 1);
        if (!empty(i)) {
          rows_of_8(i);
#pragma unroll
          for (int j = 0; j < TNN; ++j)
            buf_store16<AUX_NT>(rc, at(i, j), __builtin_bit_cast(u32x4, __builtin_bit_cast(f32x4, old[i % AHEAD][j]) + acc[i][j]));
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        if (!empty(i)) {
          rows_of_8(i);
#pragma unroll
          for (int j = 0; j < TNN; ++j) buf_store16<AUX_NT>(rc, at(i, j), __builtin_bit_cast(u32x4, acc[i][j]));
        }
    }
  } else {
    const size_t first = (size_t)row0 * g.N + n0, bytes = ((size_t)mvalid * g.N - n0) * 2;
    const OutPlanes o = out_planes<ST, EPI>(g, first, bytes);
    const unsigned pitch = (unsigned)g.N * 2u;
    const float* tab_lds = reinterpret_cast<const float*>(smem + TAB_AT + tab_stage * TAB_STAGE);
    if constexpr (TNN == 2) {   // 32 columns per wave and matrix, half lines (the neighbouring wave has the other half)
      const unsigned col = (unsigned)(wn * C + lane_col8(grp)) * 2u;
#pragma unroll
      for (int i = 0; i < TM; ++i)
        if (!empty(i)) {
          const int m = band_row(i) + (lane & 15);
          const unsigned off[1] = {m < mvalid ? (unsigned)m * pitch + col : OUT_OF_RANGE};
          epilogue_fwd<ST, EPI, 1, AUX_WT>(o, off, acc[i], acc2[DUAL ? i : 0], tab_lds);
        }
    } else {
      static_assert(TNN == 4, "two pairs of column tiles");
      const unsigned col = (unsigned)(wn * C + right * 32 + lane_col8(grp)) * 2u;
      auto at = [&](int i, int h) { const int m = band_row(i) + h * 8 + r8; return m < mvalid ? (unsigned)m * pitch + col : OUT_OF_RANGE; };
      if constexpr (EPI == EPI_STORE || EPI == EPI_GELU_FWD || EPI == EPI_SWIGLU_FWD) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          if (!empty(i)) {
            const unsigned off[2] = {at(i, 0), at(i, 1)};
            epilogue_fwd<ST, EPI, 2, AUX_NT>(o, off, acc[i], DUAL ? acc2[DUAL ? i : 0] : acc[i], tab_lds);
          }
      } else {
        // The saved tensors are requested AHEAD row tiles ahead, the first ones before anything else.
        constexpr bool TWO = EPI == EPI_SWIGLU_BWD;
        constexpr int AHEAD = 4;
        u32x4 s1[AHEAD][2], s2[TWO ? AHEAD : 1][2] = {};
        const __amdgpu_buffer_rsrc_t r1 = out_rsrc(reinterpret_cast<const ST*>(g.S1) + first, bytes);
        const __amdgpu_buffer_rsrc_t r2 = TWO ? out_rsrc(reinterpret_cast<const ST*>(g.S2) + first, bytes) : r1;
        auto load_saved = [&](int i) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            s1[i % AHEAD][h] = buf_load16_nt(r1, at(i, h));
            if constexpr (TWO) s2[TWO ? i % AHEAD : 0][h] = buf_load16_nt(r2, at(i, h));
          }
        };
#pragma unroll
        for (int i = 0; i < AHEAD - 1; ++i) load_saved(i);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if (i + AHEAD - 1 < TM) load_saved(i + AHEAD - 1);
          if (!empty(i)) {
            join_tiles(acc[i][0], acc[i][1]);
            join_tiles(acc[i][2], acc[i][3]);
            swap8(acc[i][0], acc[i][2]);
            swap8(acc[i][1], acc[i][3]);   // rows 0-7: columns 0-3 in [0], 4-7 in [1]; rows 8-15: [2], [3]
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              u32x2 c[2] = {}, c2[2] = {}, unused;
              const u32x4 p = s1[i % AHEAD][h], q = s2[TWO ? i % AHEAD : 0][h];
              activate4<ST, EPI>(acc[i][2 * h], f32x4{}, u32x2{p.x, p.y}, u32x2{q.x, q.y}, tab_lds, c[0], c2[0], unused);
              activate4<ST, EPI>(acc[i][2 * h + 1], f32x4{}, u32x2{p.z, p.w}, u32x2{q.z, q.w}, tab_lds, c[1], c2[1], unused);
              buf_store16<AUX_NT>(o.c, at(i, h), u32x4{c[0].x, c[0].y, c[1].x, c[1].y});
              if constexpr (TWO) buf_store16<AUX_NT>(o.c2, at(i, h), u32x4{c2[0].x, c2[0].y, c2[1].x, c2[1].y});
            }
          }
        }
      }
    }
  }
}

// Second half of split-K: adds the parts of every split tile in part order and writes the 16-bit rows; a thread owns
// four adjacent columns of one row.  Whether the tiles of the last round or the smallest row tiles are split follows
// from the tile counts, as in the GEMM; surplus blocks exit.
constexpr int TAIL_REDUCE_ROWS = 16;   // rows of a tile a block adds up
template <typename ST>
__global__ __launch_bounds__(256) void split_reduce_kernel(GemmArgs g) {
  const int n_rt = g.ntiles[0], ntn = (g.N + 255) / 256;
  TailSplit ts = {0, 1};
  if (g.split_tail) ts = tail_split(n_rt * ntn, g.B2 != nullptr ? 2 * g.K : g.K);   // B2: two products chained
  auto put = [&](size_t row, int n, const f32x4& v) {
    *reinterpret_cast<u32x2*>(reinterpret_cast<ST*>(g.C) + row * g.N + n) = u32x2{Half16<ST>::pack2(v[0], v[1]), Half16<ST>::pack2(v[2], v[3])};
  };
  if (ts.parts > 1) {
    const int PER = g.tile_rows / TAIL_REDUCE_ROWS, slot = g.tile_rows * 256;   // blocks per tile, floats per part
    const int q = blockIdx.x / PER, n = (threadIdx.x & 63) * 4;
    if (q >= n_rt * ntn - ts.first) return;
    int rt, nt;
    block_to_tile(ts.first + q, n_rt, g.ntiles[1], ntn, g.chunked != 0, rt, nt);
    const RowTile t = g.tiles[rt];
    if (nt * 256 + n >= g.N) return;
#pragma unroll
    for (int i = 0; i < TAIL_REDUCE_ROWS / 4; ++i) {
      const int m = (blockIdx.x % PER) * TAIL_REDUCE_ROWS + i * 4 + threadIdx.x / 64;
      if (m >= t.nrows) return;
      const float* src = g.split_ws + (size_t)q * ts.parts * slot + m * 256 + n;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < TAIL_MAX_PARTS; ++p)
        if (p < ts.parts) sum += *reinterpret_cast<const f32x4*>(src + (size_t)p * slot);
      put(t.row0 + m, nt * 256 + n, sum);
    }
    return;
  }
  const bool all = g.split_all;
  if (!g.split_small && !all) return;
  const int n_sp = all ? n_rt : g.ntiles[2], parts = all ? 1 << skinny_order(n_rt, g.ntiles[2] != 0, g.E, true).shift : SPLIT_K;
  const int per_row = g.N / 4, per_tile = (SPLIT_ROWS * per_row + 255) / 256, st = blockIdx.x / per_tile;
  if (st >= n_sp) return;
  const RowTile t = g.tiles[n_rt - n_sp + st];
  const int i = (blockIdx.x % per_tile) * 256 + threadIdx.x, m = i / per_row, n = (i % per_row) * 4;
  if (m >= t.nrows) return;
  const float* src = g.split_ws + ((size_t)st * parts * SPLIT_ROWS + m) * g.N + n;
  const size_t pitch = (size_t)SPLIT_ROWS * g.N;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < SPLIT_K / 2; ++ks) sum += *reinterpret_cast<const f32x4*>(src + ks * pitch);
  if (parts == SPLIT_K) {
#pragma unroll
    for (int ks = SPLIT_K / 2; ks < SPLIT_K; ++ks) sum += *reinterpret_cast<const f32x4*>(src + ks * pitch);
  }
  put(t.row0 + m, n, sum);
}

template <typename ST, int MODE, int EPI, bool DUAL, bool CHAIN, int BM, int BN, int WGM, int WGN, bool STREAM>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void gemm_bf16_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_bf16_tile<ST, MODE, EPI, DUAL, CHAIN, BM, BN, WGM, WGN, false, STREAM>(g, blockIdx.x, smem);
}

// Two independent GEMMs in one launch: blocks below `first_blocks` take a tile of the first, the others a
// tile of the second.  Blocks are dispatched in order, so the second GEMM's tiles start on the compute
// units that the first one's last, partly filled round leaves idle (no stream or event in between,
// and the two never compete for the cache from the start as two concurrent kernels would).
template <typename ST, int MODE1, int EPI1, bool CHAIN1, int BM1, int MODE2, int EPI2, int BM, int BN, int WGM, int WGN, bool STREAM>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void gemm_bf16_pair_kernel(GemmArgs g1, GemmArgs g2, int first_blocks) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if ((int)blockIdx.x < first_blocks)
    gemm_bf16_tile<ST, MODE1, EPI1, false, CHAIN1, BM1, BN, WGM, WGN, false, STREAM>(g1, blockIdx.x, smem);
  else
    gemm_bf16_tile<ST, MODE2, EPI2, false, false, BM, BN, WGM, WGN>(g2, blockIdx.x - first_blocks, smem);
}

// Both weight gradients over the rows of several calls: blocks below `first_blocks` take a tile of the first.
// Per call, a micro-batch of 512 rows per expert has eight K stages of arithmetic per tile and moves 512 KB of old and new
// sums for it; over all calls the sums are written once.  Tiles of 256 x 128, whose registers hold the call's sum and the
// total: one chain over all calls would round more often (four calls of 512 rows, simulated: 0.85e-7 -> 1.4e-7 of the
// gradient).  Four micro-batches of 2048 tokens, d 1024, f 4096, eight experts: backward GEMMs 1040 us with the gradients
// accumulated call by call in launches shared with dH and dx; 4 x 88 + 335 now, 284 of them in 256 x 256 tiles and one chain.
struct DwSegsPair { GemmArgs g[2]; DwSegs s[2]; int first_blocks; };
template <typename ST, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void gemm_bf16_dw_segs_kernel(DwSegsPair p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int w = (int)blockIdx.x >= p.first_blocks;
  gemm_bf16_tile<ST, MODE_TN, EPI_DW, false, false, BM, BN, WGM, WGN, true>(p.g[w], blockIdx.x - w * p.first_blocks, smem, &p.s[w]);
}

inline unsigned gemm_bf16_grid(long long tiles) { return (unsigned)(tiles > 0 ? tiles : 1); }

}  // namespace moe
