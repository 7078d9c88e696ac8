// Grouped (per-expert, ragged) GEMM plumbing shared by the fp32 and the bf16 MFMA kernels.
//
// The expert FFN of the paper is "mainly GEMMs" (Section 2.1) and its cost must follow the number
// of token rows an expert receives, not the number of experts (Section 4.2, the remark on
// T_E^Exp).  So every GEMM here walks a device-resident list of row tiles built from
// offsets / kept / shares: no padding of experts to a common size and no host read-back of counts.
#pragma once
#include "common.h"

namespace moe {

// One tile of consecutive permuted rows belonging to one expert.
struct RowTile {
  int32_t e;      // expert
  int32_t row0;   // first row (absolute index into the permuted buffers)
  int32_t nrows;  // valid rows in this tile (1..tile height)
  int32_t mates;  // whether the expert has other tiles too
};

// Tables over the bf16 numbers for the bf16 GELU epilogues.  The pre-activation is stored as a bf16
// number, so the forward applies GELU to exactly that number (as a separate activation kernel on the
// stored tensor would) and the backward takes the derivative at it; both are looked up instead of
// computed: Phi(v) for the forward (h = a Phi(v)), gelu'(v) for the backward.  Entry [sign][m],
// m = (bits & 0x7fff) - (GELU_TAB_EXP0 << 7) clamped to [0, GELU_TAB_NMAG): magnitudes from 2^-16 up to
// (not including) 8; smaller ones read the first entry (Phi and gelu' are 0.5 there to within 1.3e-5),
// larger ones the last (gelu' is 1 or 0 there to within 1e-13; the last Phi entries are set to exactly 1 and 0).
enum GeluTable { GELU_TAB_NONE = 0, GELU_TAB_PHI = 1, GELU_TAB_GRAD = 2 };
// Split-K for the smallest row tiles.  A partly filled row tile of at most SPLIT_ROWS rows has almost no
// MFMA work, but a block still walks all K stages for it at the pace of memory latency, and such tiles
// run last, on a mostly idle chip.  For the plain-store GEMMs each of them is therefore cut into
// SPLIT_K blocks along K that write fp32 partial sums [tile][k part][SPLIT_ROWS][N] into the workspace;
// split_reduce adds the parts in fixed order and writes the bf16 rows.  Used when K is long enough
// to matter and the experts are few (the partial sums take E * SPLIT_K * SPLIT_ROWS * N * 4 bytes).
constexpr int SPLIT_ROWS = 64;
constexpr int SPLIT_K = 8;
constexpr int SPLIT_MAX_E = 32;
constexpr int SPLIT_MIN_K = 2048;
// (each K part must be whole 64-wide stages of the row-tile GEMMs)
inline bool split_k_applies(int E, int K) { return E <= SPLIT_MAX_E && K >= SPLIT_MIN_K && K % (SPLIT_K * 64) == 0; }
inline size_t split_ws_bytes(int E, int N) { return (size_t)E * SPLIT_K * SPLIT_ROWS * N * 4; }

constexpr int GELU_TAB_EXP0 = 111;                 // biased exponent of 2^-16
constexpr int GELU_TAB_NMAG = (130 - 111) * 128;   // 2432 magnitudes per sign
constexpr int GELU_TAB_FLOATS = 6144;              // 2 * 2432 entries, padded to 24 KB (whole 1 KB wave loads)

// Tile map in the workspace: header[0] = number of tiles, header[1] = number of tiles at the head of the
// list that are walked XCD by XCD (the full tiles; with many experts of few tiles each the list is
// expert-major and this is all of it), header[2] = number of tiles of at most SPLIT_ROWS rows at the
// end of the list that may be split along K (0 for an expert-major list; in the few-row kernel's list, which is always
// expert-major, the number of experts with more than one tile); then the tiles; then order[E] = the experts by
// descending share length (heaviest first); then one table as above.
struct TileMap {
  int32_t* header;
  RowTile* tiles;
  int32_t* order;
  float* gelu_tab;
};
inline size_t tile_map_bytes(int max_tiles, int E) {
  return 16 + (size_t)max_tiles * sizeof(RowTile) + (((size_t)E * 4 + 15) & ~(size_t)15) + (size_t)GELU_TAB_FLOATS * 4;
}
inline TileMap tile_map_at(void* ws_region, int max_tiles, int E) {
  TileMap m;
  char* base = reinterpret_cast<char*>(ws_region);
  m.header = reinterpret_cast<int32_t*>(base);
  m.tiles = reinterpret_cast<RowTile*>(base + 16);
  m.order = reinterpret_cast<int32_t*>(base + 16 + (size_t)max_tiles * sizeof(RowTile));
  m.gelu_tab = reinterpret_cast<float*>(base + 16 + (size_t)max_tiles * sizeof(RowTile) + (((size_t)E * 4 + 15) & ~(size_t)15));
  return m;
}
inline int max_row_tiles(int A, int E, int tile_rows) { return (A + tile_rows - 1) / tile_rows + E; }

// ---- block -> tile numbering of the MFMA grouped GEMMs (host and device: a host-side test enumerates it) ----
#ifdef __HIPCC__
#define MOE_HD __host__ __device__
#else
#define MOE_HD
#endif
constexpr int NUM_XCD = 8;

// Workgroups go to the eight XCDs round-robin (block b runs on XCD b % 8), each XCD has an L2 of its own, and all of
// them share the memory-side cache.  The order of the tiles serves both levels.  A compute unit holds one block, so
// an XCD runs 32 tiles at a time and the chip 256: the tile list is cut into chunks of 256, and XCD x takes the x-th
// run of 32 tiles of every chunk.  The list itself (patch_tile) goes through the tile matrix so that 32 consecutive
// tiles are a patch of 4 x 8 (twelve operand panels in the XCD's L2) and 256 consecutive ones a compact block (8 x 32
// or 16 x 16), whose panels the XCDs read at about the same time and therefore mostly from the memory-side cache.
// Before, every XCD walked a contiguous eighth of the whole list: the same L2 patches, but eight XCDs in eight
// different places (different experts, on the Mixtral-like shape) shared nothing beyond their L2.  Eight experts of
// 8192 rows, d 4096, f 14336, plain store, 256 x 256 tiles: x W 5.89 -> 5.36 ms (1307 -> 1437 TFLOP/s), dy W^T 5.95 ->
// 5.41 ms; 16 experts of 2048 rows, d 2048, f 8192: 0.92 -> 0.89 and 0.88 -> 0.85 ms.
constexpr int PATCH_R = 4, PATCH_C = 8, CHUNK_TILES = PATCH_R * PATCH_C * NUM_XCD;

// Position in the tile list of block b of n, `run` tiles per XCD and chunk; the last chunk is shared out evenly as
// well, its m % 8 last blocks by index.
MOE_HD inline int chunk_position(int b, int n, int run) {
  const int chunk = run * NUM_XCD, c0 = b / chunk * chunk, q = b - c0;
  const int m = (chunk < n - c0) ? chunk : n - c0, per = m / NUM_XCD;
  return (q < per * NUM_XCD) ? c0 + (q % NUM_XCD) * per + q / NUM_XCD : b;
}

// Tile p of an nr x nc tile matrix: bands of `band` rows; in a band, column strips PATCH_C wide; in a strip, patches
// of PATCH_R rows; in a patch, column by column.  Ragged ends shrink the patch, the numbering stays gapless.
MOE_HD inline void patch_tile(int p, int nr, int nc, int band, int& r, int& c) {
  const int b = p / (band * nc), in = p - b * (band * nc), first = b * band;
  const int rows = (band < nr - first) ? band : nr - first;
  const int strip = in / (rows * PATCH_C), in2 = in - strip * (rows * PATCH_C);
  const int cols = (PATCH_C < nc - strip * PATCH_C) ? PATCH_C : nc - strip * PATCH_C;
  const int sub = in2 / (PATCH_R * cols), in3 = in2 - sub * (PATCH_R * cols);
  const int pr = (PATCH_R < rows - sub * PATCH_R) ? PATCH_R : rows - sub * PATCH_R;
  r = first + sub * PATCH_R + in3 % pr;
  c = strip * PATCH_C + in3 / pr;
}

// Row-tile GEMMs.  Tiles are numbered (row tile, column tile) with the full row tiles first, in patch order.  The
// partly filled row tiles follow in dispatch order: they are the last blocks to start and fill the chip's final round.
// Chunked order for operands that do not fit the memory-side cache, in bands of eight row tiles: with 16 the large
// shapes lose 1-4 %, with 32 4-6 % (a weight panel that all eight XCDs want at the same moment costs more than an
// activation panel that four of them want).  Operands that do fit are served from that cache in any order; for them
// one run per XCD in bands of four stays (the tiles an XCD takes one after the other then share their four activation
// panels, which its L2 keeps from one patch to the next: 61 full row tiles, d 1024, f 4096, dH + dW2 292 against 300
// us in chunks, GELU forward 176 against 179; SwiGLU forward of d 1088, f 2880: 100 against 104).
constexpr int ROW_BAND = 8;
MOE_HD inline bool block_to_tile(int b, int n_rt, int n_full_rt, int ntn, bool chunked, int& rt, int& nt) {
  const int n_full = n_full_rt * ntn, n_all = n_rt * ntn;
  if (b >= n_all) return false;
  if (b >= n_full) {                          // partial row tiles, largest first, in dispatch order
    rt = n_full_rt + (b - n_full) / ntn;
    nt = (b - n_full) % ntn;
    return true;
  }
  const int run = chunked ? PATCH_R * PATCH_C : n_full / NUM_XCD + 1;   // + 1: the whole list is one chunk
  patch_tile(chunk_position(b, n_full, run), n_full_rt, ntn, chunked ? ROW_BAND : PATCH_R, rt, nt);
  return true;
}
// (host) whether the operands of a row-tile GEMM exceed the 256 MB memory-side cache; rows = the most it can have
constexpr long long MEMORY_SIDE_CACHE = 256ll << 20;
inline bool row_tiles_chunked(long long rows, long long K, long long N, int E, int matrices, int elt) {
  return (rows * K + (long long)E * K * N * matrices) * elt > MEMORY_SIDE_CACHE;
}

// Block vb of a row-tile GEMM launch over n_rt row tiles (the first n_full_rt of them walked XCD by XCD), of
// which the last n_sp are split along K: those are not part of the regular numbering; their blocks follow it,
// SPLIT_K per (row tile, column tile), each with a K part of its own.  False: no tile (surplus block).
struct RowBlock { int rt, nt, split_tile, ksplit; };
MOE_HD inline bool row_tile_block(int vb, int n_rt, int n_full_rt, int n_sp, int ntn, bool chunked, RowBlock& r) {
  const int n_reg = n_rt - n_sp;
  r.split_tile = -1;
  r.ksplit = 0;
  if (vb < n_reg * ntn) return block_to_tile(vb, n_reg, n_full_rt, ntn, chunked, r.rt, r.nt);
  const int q = vb - n_reg * ntn;
  if (q >= n_sp * ntn * SPLIT_K) return false;
  r.ksplit = q % SPLIT_K;
  r.nt = (q / SPLIT_K) % ntn;
  r.split_tile = q / (SPLIT_K * ntn);
  r.rt = n_reg + r.split_tile;
  return true;
}

// Few-row GEMMs (gemm_skinny_kernel.h) on an expert-major list.  Lists without an expert of several row tiles (`mates`)
// read every weight once: up to 32 experts a block's neighbours are the next columns and K parts of its tile, so that the
// chip streams whole weight rows; more experts go in patches, one contiguous run per XCD.  With such an expert the XCDs
// take runs of 64 tiles, 8 rows x 8 columns, in turn: the row tiles that share weights run together on an XCD and find
// them in its L2, while the chip as a whole reads whole weight rows (runs that walk down a strip of eight columns leave
// the other half of 4 KB rows, and half of the memory channels, untouched: 256 experts of 48 rows, d 2048, f 1024, second
// GEMM 244 us against 199; runs of 32 tiles are within 5 % either way, bands of 16 row tiles up to 10 % slower).
// Split along K (up to 32 experts): eight parts, four where an expert has several tiles, which are at most 1.5 E then
// (SKINNY_AVERAGE rows per expert, SKINNY_ROWS per tile).
constexpr int SKINNY_RUN = 64, SKINNY_BAND = 8;
struct SkinnyOrder { int n_rt, E, shift; bool mates; };   // 1 << shift K parts per tile
MOE_HD inline SkinnyOrder skinny_order(int n_rt, bool mates, int E, bool split) {
  return SkinnyOrder{n_rt, E, !split ? 0 : mates ? 2 : 3, mates};
}
MOE_HD inline bool skinny_block(int vb, const SkinnyOrder& o, int ntn, RowBlock& r) {
  const int nc = ntn << o.shift, n = o.n_rt * nc;
  if (vb >= n) return false;
  int c;
  if (!o.mates && o.E <= SPLIT_MAX_E) {
    r.ksplit = vb & ((1 << o.shift) - 1);
    c = vb >> o.shift;
    r.rt = c / ntn;
    r.nt = c - r.rt * ntn;
  } else {
    if (o.mates) patch_tile(chunk_position(vb, n, SKINNY_RUN), o.n_rt, nc, SKINNY_BAND, r.rt, c);
    else patch_tile(chunk_position(vb, n, n / NUM_XCD + 1), o.n_rt, nc, PATCH_R, r.rt, c);
    r.ksplit = c / ntn;
    r.nt = c - r.ksplit * ntn;
  }
  r.split_tile = o.shift > 0 ? r.rt : -1;
  return true;
}

// Split-K of the last round.  256 blocks run at a time; the tiles behind the last whole round of 256 (all of them, when
// there are fewer) leave most of the chip idle for the length of one tile.  In the plain-store GEMMs with long K these
// r tiles are cut along K into `parts` blocks each, at most 256 in all, whose fp32 partial sums [slot][rows of a tile][256] go to
// the workspace; split_reduce adds them in part order.  A round costs about 26 us per 1024 K values, a slot about
// 0.1 us (256 KB written and read again); the parts minimise the sum of the two, and a gain below 2 us, the model's
// error, is left.  The reduction is a launch of its own, and the GEMM alone knows how many tiles there are: it is paid
// (2 us) wherever tail_may_split cannot rule a split out, split or not, and takes no part in the comparison.  (8 us asked
// for instead, forward pass: d 2048, f 2048, 96 tiles 102.6 -> 95.6 us with 2, 112 tiles 103.0 -> 99.2; d 2560, f 2560,
// 120 tiles 126.7 -> 115.3.)
// y = hidden W2, with the reduction: 16 experts of 125 rows, d 2048, f 8192 (128 tiles) 198 -> 131 us; eight experts of 512
// rows, d 1024, f 4096 (about 80 tiles) 101 -> 60; d 2048, f 8192, 16384 rows in 16 skewed experts, per step 4.56 -> 4.38 ms.
constexpr int TAIL_SLOTS = 256, TAIL_MAX_PARTS = 8;
struct TailSplit { int first, parts; };   // tiles from `first` on are split; parts == 1: none
MOE_HD inline TailSplit tail_split(int n_tiles, int K) {
  TailSplit t = {n_tiles, 1};
  const int r = n_tiles % TAIL_SLOTS, round = K / 4;   // tenths of a microsecond
  if (K < SPLIT_MIN_K || r == 0) return t;
  int best = round - 20;
  for (int p = 2; p <= TAIL_MAX_PARTS && p * r <= TAIL_SLOTS; ++p)
    if (round / p + p * r < best) { best = round / p + p * r; t.parts = p; }
  if (t.parts > 1) t.first = n_tiles - r;
  return t;
}
// (host) whether any number of row tiles that `rows` rows of E experts can have is split; exact: all of them are computed
// (no capacity, no slices), else there may be any number of tiles.
inline bool tail_may_split(int rows, int E, bool exact, int ntn, int K, int tile_rows = 256) {
  if (K < SPLIT_MIN_K) return false;
  if (!exact) return true;
  for (int n = (rows + tile_rows - 1) / tile_rows; n <= rows / tile_rows + E && n <= rows; ++n)
    if (tail_split(n * ntn, K).parts > 1) return true;
  return false;
}
inline size_t tail_ws_bytes(int max_tiles, int N) {   // room for slots of 256 x 256; lower tiles pack theirs
  const long long slots = (long long)max_tiles * ((N + 255) / 256) * TAIL_MAX_PARTS;
  return (size_t)(slots < TAIL_SLOTS ? slots : TAIL_SLOTS) * 256 * 256 * 4;
}
// Block vb of a row-tile GEMM launch whose last round is split: r.split_tile = the tile's index among the split ones.
// Part p of a tile takes the K stages of 64 from p * stages / parts on.
MOE_HD inline bool tail_split_block(int vb, int n_rt, int n_full_rt, int ntn, bool chunked, const TailSplit& t, RowBlock& r) {
  r.split_tile = -1;
  r.ksplit = 0;
  if (vb >= t.first) {
    r.split_tile = (vb - t.first) / t.parts;
    r.ksplit = (vb - t.first) % t.parts;
    vb = t.first + r.split_tile;
  }
  return block_to_tile(vb, n_rt, n_full_rt, ntn, chunked, r.rt, r.nt);
}

// Block vb of a weight-gradient launch: tile (expert slot in descending-size order, m tile, n tile).  A tile costs its
// expert's row count, so every expert's ntm x ntn tiles are split evenly over the XCDs and a skewed load is even
// across them; within the expert the order is the chunked patch order above, in bands of 16 (256 tiles at a time are
// 16 x 16).  With more than one chunk the bands run along the shorter side: dW2 of eight experts of 8192 rows (14336 x
// 4096) 5.89 -> 5.79 ms, 16 of 2048 rows (8192 x 2048) 1.007 -> 0.985 ms, against one contiguous run of the expert's
// tiles per XCD; with one chunk that turn costs 3 % instead (4096 x 1024, 2048 rows: 127 -> 131 us).  Wide matrices
// (4096 x 14336) take the same time in either order.
constexpr int DW_BAND = 16;
MOE_HD inline bool dw_block(int vb, int ntm, int ntn, int& slot, int& mt, int& nt) {
  const int P = ntm * ntn, P8 = (P + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
  slot = vb / P8;
  const int q = vb - slot * P8;
  if (q >= P) return false;
  const int p = chunk_position(q, P, PATCH_R * PATCH_C);
  if (ntm > ntn && P > CHUNK_TILES) patch_tile(p, ntn, ntm, DW_BAND, nt, mt); else patch_tile(p, ntm, ntn, DW_BAND, mt, nt);
  return true;
}

enum GemmMode {
  MODE_NN = 0,  // C[rows, N] = A[rows, K] * B_e[K, N]          (forward GEMMs)
  MODE_NT = 1,  // C[rows, N] = A[rows, K] * B_e[N, K]^T        (dH, dX)
  MODE_TN = 2   // C_e[M, N] (+)= A[rows_e, M]^T * B[rows_e, N]  (weight gradients)
};

enum Epilogue {
  EPI_STORE = 0,       // C = acc
  EPI_GELU_FWD = 1,    // C = acc (pre-activation; skipped when C is NULL), C2 = gelu(acc)
  EPI_SWIGLU_FWD = 2,  // dual accumulators g,u: C = g, C2 = u (both skipped when C is NULL), C3 = silu(g)*u
  EPI_GELU_BWD = 3,    // C = acc * gelu'(S1)
  EPI_SWIGLU_BWD = 4,  // C = dG = acc * S2 * silu'(S1), C2 = dU = acc * silu(S1)   (S1 = G, S2 = U)
  EPI_DW = 5           // fp32 C_e = acc (+ C_e)
};

struct GemmArgs {
  const void* A;
  const void* A2;   // second activation operand (SwiGLU dX: dU)
  const void* B;
  const void* B2;   // second weight operand (SwiGLU: W1b); weight gradients: dU, where C2 is given
  void* C;
  void* C2;         // weight gradients: a second one of the same A (SwiGLU: dW1b), in the same launch
  void* C3;
  const void* S1;
  const void* S2;
  const RowTile* tiles;
  const int32_t* ntiles;
  const int32_t* order;     // experts by descending share length (weight-gradient GEMMs start the heaviest first)
  const float* gelu_tab;    // bf16 GELU epilogues: Phi (forward) or gelu' (backward) over the bf16 numbers
  float* split_ws;          // fp32 partial sums of split tiles, or NULL: no split-K
  int near;                      // GELU forward: the hidden plane is stored for the caches (hidden_near)
  int split_small, split_tail;   // which tiles may be split: the smallest row tiles (SPLIT_K), those of the last round (tail_split)
  int split_all;                 // few-row GEMMs: every tile is split (skinny_order)
  const int32_t* offsets;
  const int32_t* kept;
  const int32_t* lo;
  const int32_t* hi;
  int M, N, K;   // NN/NT: N and K fixed (M unused); TN: M and N fixed (K is the expert's row count)
  int E;
  int accumulate;
  int chunked;   // row-tile GEMMs: order of the full tiles (block_to_tile)
  int stream;    // row-tile GEMMs: row tiles from which on weights that one of them takes are requested as streaming data, 0: never (streamed_from)
  int tile_rows; // row-tile GEMMs: rows per entry of the tile map
};

// blocks of a weight-gradient launch of bm x bn tiles (dw_block), of two gradients where the second is asked for
inline long long dw_blocks(const GemmArgs& g, int bm, int bn) {
  const long long p = (long long)((g.N + bn - 1) / bn) * ((g.M + bm - 1) / bm);
  return (p + NUM_XCD - 1) / NUM_XCD * NUM_XCD * g.E * (g.C2 != nullptr ? 2 : 1);
}

struct TileMapArgs;   // tile_map.h
int launch_tile_map(const TileMapArgs& tm, hipStream_t s);

// fp32 storage, fp32 MFMA (any shape that passes check_cfg)
int launch_gemm_f32(int mode, int epi, bool dual, bool chain, const GemmArgs& g, int tile_rows, int max_tiles, hipStream_t s);
int launch_gemm_f32_pair(int epi1, bool chain1, const GemmArgs& g1, int tile_rows, int max_tiles, const GemmArgs& g2, hipStream_t s);
// Height of its tiles (64 columns wide): 32 rows where 64 would leave the chip short of its three blocks per compute
// unit; `parts`: partly filled tiles to expect.  64 -> 32 rows, us: SwiGLU forward T 100, d 1024, f 4096 (8 experts, 512
// tiles of 64) 203 -> 149, GELU step T 1000, d 512, f 1024 (576 tiles) 261 -> 248,
// SwiGLU step T 300, d 1024, f 1024 285 -> 276; above the line, forced: T 1000, d 700,
// f 2048, E 32 forward 218 -> 225, step T 2000, d 1024, f 1024, E 16 639 -> 653, T 4096, d 1024, f 4096 3592 -> 3787.
constexpr long long F32_LOW_TILES = 768;
constexpr int F32_TILE_COLS = 64;
inline int f32_tile_rows(long long rows, int parts, int N) { return ((rows + 63) / 64 + parts) * ((N + F32_TILE_COLS - 1) / F32_TILE_COLS) < F32_LOW_TILES ? 32 : 64; }
// 16-bit storage (dtype = MOE_DTYPE_BF16 or MOE_DTYPE_F16), MFMA with fp32 accumulation
int launch_gemm_half(int dtype, int mode, int epi, bool dual, bool chain, const GemmArgs& g, int max_tiles, hipStream_t s);
// one launch for an NT GEMM (epilogue epi1, chained or not) followed by a TN weight-gradient GEMM
int launch_gemm_half_pair(int dtype, int epi1, bool chain1, const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s);
int gemm_bf16_tile_rows();
// Height of the 16-bit row tiles.  256 rows move the fewest bytes per product; LDS holds three stages of one operand and two of the
// other.  160 rows leave room for three of both, so all loads have the longer time to land, and fill the chip more evenly where
// an expert has few tiles.  The host sees the average rows per expert, not the load, and the line is drawn on that.
// 256 -> 160 rows, geometric mean over 1800 layers of random sizes (d 512 to 4096, d_ff 512 to 14336, both activations and
// types), forward pass | forward and backward, at an even load and router biases of -0.7 and -1.2 log(e + 1):
//   rows per expert          even           -0.7           -1.2                                even           -0.7           -1.2
//   up to 32 experts                                                   more
//   100 - 128          0.94 | 0.95    0.94 | 0.94    0.93 | 0.92                         0.95 | 0.99    0.96 | 0.98    0.97 | 0.98
//   129 - 160          0.98 | 0.98    0.93 | 0.93    0.99 | 0.95                         1.01 | 1.01    0.97 | 0.99    0.96 | 0.98
//   161 - 256          1.02 | 0.98    0.96 | 0.96    0.97 | 0.95                         1.13 | 1.08    1.00 | 1.01    1.00 | 1.01
//   257 - 320          0.88 | 0.91    1.00 | 0.97    0.97 | 0.97                         0.97 | 0.99    0.99 | 1.01    1.00 | 1.00
//   321 - 512          0.99 | 0.96    1.02 | 1.00    0.97 | 0.97                         1.06 | 1.04    1.03 | 1.02    1.03 | 1.02
//   513 - 650          0.98 | 0.97    1.02 | 0.99    1.01 | 1.00                         1.04 | 1.03    1.03 | 1.03    1.04 | 1.03
//   650 - 1000         1.04 | 1.01    1.03 | 1.01    0.99 | 1.00                         1.05 | 1.04    1.06 | 1.04    1.05 | 1.04
// (a layer's own ratio lies within about a tenth of these.)
constexpr int MID_ROWS = 160;
constexpr int MID_FEW_EXPERTS = 32, MID_AVERAGE_FEW = 512, MID_AVERAGE_MANY = 128;
inline bool mid_applies(long long rows, int E) { return rows <= (long long)(E <= MID_FEW_EXPERTS ? MID_AVERAGE_FEW : MID_AVERAGE_MANY) * E; }
// Whether the weights of an expert with a single row tile are requested as streaming data: they are read once per launch, and
// as plain loads they push each other through the caches.  Asked for where experts have a tile each on average and the layer's
// weights do not fit the memory-side cache with room to spare; smaller ones are found there by the launch that reads them next
// (dx after GEMM1, dH after y, the next step).  90 rows per expert, us, plain -> streaming, forward pass | step, by the
// megabytes of a layer's weights:
//    64  d 1024, f 2048, 8 experts, GELU       57 ->  62 | 139 -> 152      192  d 1024, f 4096, 8, SwiGLU      73 ->  80 | 262 -> 293
//   256  d 1024, f 4096, 16, GELU              87 ->  88 | 301 -> 302      256  d 1024, f 1024, 64, GELU       94 ->  92 | 307 -> 300
//   288  d 2048, f 3072, 8, SwiGLU            102 ->  96 | 332 -> 341      384  d 1536, f 4096, 16, GELU      123 -> 116 | 402 -> 397
//   384  d 1024, f 4096, 16, SwiGLU           130 -> 116 | 430 -> 424      384  d 1024, f 1024, 64, SwiGLU    132 -> 119 | 424 -> 398
//   512  d 1024, f 4096, 32, GELU             158 -> 146 | 541 -> 508      576  d 1536, f 4096, 16, SwiGLU    165 -> 154 | 570 -> 550
// 160-row tiles: 125 rows, d 2048, f 8192, 16 experts, fp16 GELU 280 -> 265 | 1109 -> 1036; 75 rows, d 4096, f 14336, 8, SwiGLU 577
// -> 534 | 2397 -> 2253.  256-row tiles: 160 rows, d 2048, f 2048, 128, GELU 558 -> 536 | 2339 -> 2264; 200 rows, d 2048, f 1024, 256,
// GELU 710 -> 684 | 2804 -> 2729, SwiGLU 941 -> 906 | 3734 -> 3663; where experts have two or three tiles (512 rows, 128 experts,
// SwiGLU) 1003 -> 1001 | 3299 -> 3323.  1250 layers of random sizes beyond 320 MB, the line drawn at all experts: step x0.94 to 0.98 in
// each class of weights, rows and load but one (up to 32 experts, 320 to 400 MB, bias -1.2: 1.00, see the last lines); 225 of 200
// to 320 MB: x1.02 to 1.03 up to 32 experts, 1.00 beyond.
// In launches shared with a weight gradient too: 256-row tiles, whole step, us, 140 rows, d 1024, f 1536, 64, SwiGLU 675 -> 631; 160,
// d 2048, f 1024, 128, fp16 GELU 1307 -> 1250; 200, d 2048, f 4096, 48, SwiGLU 2645 -> 2563; 250, d 1024, f 768, 128 1039 -> 1037; 150,
// d 1024, f 1024, 96, GELU, router bias -1.2 log(e + 1), 553 -> 521.
// The weights that count are those of experts with rows.  The host does not know these; the kernel knows the row tiles, at least
// one per such expert, so the answer is how many of those it takes (0: no number passes the line).  Backward, us, the line drawn
// at all experts -> at those with rows: 26 experts, d 512, f 4352, SwiGLU (332 MB), 32 tokens of four at a router bias of
// -1.2 log(e + 1) 265 -> 207; 14, d 1024, f 7168, GELU (392 MB), 70 tokens of one, the same bias 267 -> 214.
inline int streamed_from(long long rows, int tile_rows, long long E, long long d, long long f, int matrices, int elt) {
  const long long expert = d * f * matrices * elt, least = MEMORY_SIDE_CACHE / 4 * 5 / expert + 1;
  return rows <= tile_rows * E && least <= E ? (int)least : 0;
}
// Whether GELU's hidden plane, which GEMM2 reads next, is stored plainly instead of streamed.  Up to about twice the L2
// caches' 32 MB much of it is still near when GEMM2 starts; beyond, it only displaces operands.  Forward pass, us, streamed
// -> plain: eight experts of 1000 rows, d 832, f 3264 (52 MB) 168 -> 158; six of 1200, d 1088, f 2880 (41 MB) 138 -> 126;
// 12 of the same (83 MB) 225 -> 230; eight of 2048, d 1024, f 4096 (134 MB) 303 -> 313.  SwiGLU: from -4 to +4 %.
constexpr long long NEAR_BYTES = 64ll << 20;
inline bool hidden_near(long long rows, int f) { return rows * f * 2 <= NEAR_BYTES; }
// forward GEMMs of experts with few rows (gemm_skinny_kernel.h), on a map of SKINNY_ROWS-row tiles
constexpr int SKINNY_ROWS = 64;
// GEMM2, long K and few experts: the column tiles alone do not fill the chip
inline bool skinny_split(int E, int K) { return E <= SPLIT_MAX_E && K >= SPLIT_MIN_K; }
int launch_gemm_half_skinny(int dtype, int epi, bool dual, const GemmArgs& g, int max_tiles, hipStream_t s);
// An expert's weights are read again for every 64 rows: the line lies where that evens out over the loads.  Both GEMMs
// with their map, us, 160-row kernel -> this one (above the line: forced), for an even load and router biases of
// -0.7 and -1.2 log(e + 1):
//   rows per expert                                 even          -0.7          -1.2
//   d 4096, f 14336, 8 experts, SwiGLU     16   502 -> 494   500 -> 493   507 -> 496
//                                          32   522 -> 527   525 -> 520   540 -> 515
//                                          48   537 -> 552   549 -> 540   570 -> 582
//   d 4096, f 14336, 8 experts, GELU       16   325 -> 331   328 -> 332   301 -> 303
//                                          32   332 -> 364   344 -> 335   356 -> 336
//                                          48   342 -> 387   360 -> 390   376 -> 392
//   d 2048, f 8192, 16 experts, GELU       16   206 -> 200   195 -> 189   187 -> 175
//                                          32   211 -> 220   219 -> 215   244 -> 225
//                                          48   218 -> 234   252 -> 239   244 -> 234
//   d 4096, f 1024, 40 experts, SwiGLU     16   214 -> 190   207 -> 183   134 -> 136
//                                          32   218 -> 201   217 -> 210   142 -> 168
//                                          48   225 -> 210   219 -> 234   195 -> 197
//   d 2048, f 1024, 128 experts, SwiGLU    16   304 -> 282   286 -> 284   194 -> 192
//                                          32   318 -> 298   319 -> 310   250 -> 250
//                                          48   327 -> 316   336 -> 351   272 -> 285
//   d 2048, f 1024, 256 experts, GELU      16   380 -> 375   320 -> 322   155 -> 167
//                                          32   392 -> 408   396 -> 415   221 -> 240
//                                          48   406 -> 426   432 -> 482   252 -> 312
//   d 1024, f 512, 64 experts, SwiGLU      16    44 ->  46    44 ->  48    37 ->  41
//                                          32    46 ->  47    65 ->  52    40 ->  45
//                                          48    47 ->  55    65 ->  62    43 ->  54
//   d 1024, f 512, 128 experts, SwiGLU     16    90 ->  74    84 ->  74    44 ->  50
//                                          32    98 ->  84   116 ->  99    66 ->  67
//                                          48   103 -> 101   115 -> 108    70 ->  84
// These are with plain loads on the left.  Where 160-row tiles stream the weights too (streamed_from), both stream, and the
// ring of 64 KB per block in whole rounds of 256 blocks is ahead: forward pass, us, this kernel -> 160-row tiles,
//   rows per expert                                 even          -0.7          -1.2
//   d 4096, f 14336, 8 experts, SwiGLU      4   479 -> 458                 441 -> 427
//                                          16   517 -> 481   517 -> 481   517 -> 484
//   d 4096, f 14336, 8 experts, GELU        4   322 -> 307                 227 -> 240
//                                           8   330 -> 313   334 -> 313   334 -> 316
//                                          24   371 -> 334   369 -> 340   346 -> 349
//   d 2048, f 8192, 16 experts, GELU        4   194 -> 197                 132 -> 142
//                                           8   201 -> 201   195 -> 191   175 -> 173
//                                          24   227 -> 209   220 -> 215   223 -> 218
//                                          32   237 -> 212   233 -> 220   240 -> 257
//   d 2048, f 1024, 128 experts, SwiGLU     4   299 -> 294                 156 -> 161
//                                           8   314 -> 305   273 -> 280   174 -> 176
//                                          32   343 -> 324   367 -> 345   273 -> 245
//   d 2048, f 1024, 256 experts, GELU       8   424 -> 406   324 -> 310   201 -> 203
//                                          32   485 -> 439   496 -> 451   329 -> 288
//   d 4096, f 1024, 40 experts, SwiGLU     16   230 -> 235   223 -> 243   175 -> 165   (GEMM1: 320 tiles, 1.25 rounds)
//   d 3200, f 5120, 12 experts, SwiGLU      8   219 -> 223   211 -> 217   203 -> 215   (y: 156 tiles, neither a round nor split)
//   d 4096, f 8192, 16 experts, SwiGLU      1   404 -> 379   231 -> 229   205 -> 214
//                                           2   535 -> 529   290 -> 289   262 -> 265
//                                          16   584 -> 553   598 -> 550   589 -> 523
// so from 8 rows on (16 with more than 32 experts) where the rounds of both GEMMs are at least four fifths full or the last one
// is split, up to 24 with few experts (at a skewed load their y has too many tiles for the split); and from 2 rows on where
// a SwiGLU expert's matrices have 64 MB each.
// GEMM1's loop is d long, and a block that has its compute unit to itself waits for the fill in front of it and the stores behind it
// (here the other block runs on; y, f long, loses less): the wider the layer, the more the 160-row tiles gain.  Forward pass,
// this kernel -> 160-row tiles where the lines above take them, geometric mean over the three loads and layers of random
// width (multiples of 64, d 512 to 4096, d_ff 512 to 14336, 4 to 256 experts, more than 320 MB of weights):
//   d                            512 - 767   768 - 1279   1280 - 1791   1792 - 2303   2304 - 3071   from 3072
//   up to 32 experts, GELU            1.12         1.04          1.04          1.01          1.00        0.97   (d 2048: 1.00)
//   up to 32 experts, SwiGLU          1.16         1.07          1.06          1.00          0.99        0.97   (d 2048: 0.98)
//   more, GELU                        1.01         0.97          0.97          0.96          0.96        0.95
//   more, SwiGLU                      1.05         0.99          0.97          0.95          0.95        0.94   (d 1024: 0.98)
// so from d 2048 on with few experts, and with many from 1024 on for SwiGLU, which has twice as much in front of and behind its
// loop.  The 64 MB: d from 2048, 2 to 8 rows, 40 to 64 MB 1.01, 64 to 100 MB 0.98.
constexpr int SKINNY_AVERAGE = 32;
inline bool few_rows_streamed(long long rows, int E, int d, int f, bool swiglu, int elt) {
  if (!streamed_from(rows, MID_ROWS, E, d, f, swiglu ? 3 : 2, elt) || rows > (long long)(E <= MID_FEW_EXPERTS ? 24 : SKINNY_AVERAGE) * E) return false;
  if (d < (E <= MID_FEW_EXPERTS ? 2048 : swiglu ? 1024 : 0)) return false;
  const int cols = swiglu ? 128 : 256, tiles1 = E * ((f + cols - 1) / cols), tiles2 = E * ((d + 255) / 256);
  auto full = [](int tiles) { return (long long)tiles * 5 >= (tiles + 255) / 256 * 256ll * 4; };
  if (!full(tiles1) || !(full(tiles2) || tail_split(tiles2, f).parts > 1)) return false;
  const bool large = swiglu && E <= MID_FEW_EXPERTS && (long long)d * f * elt >= 64ll << 20;
  return rows >= (long long)(large ? 2 : E <= MID_FEW_EXPERTS ? 8 : 16) * E;
}
inline bool skinny_applies(long long rows, int E, int d, int f, bool swiglu, int elt) {
  return rows <= (long long)SKINNY_AVERAGE * E && !few_rows_streamed(rows, E, d, f, swiglu, elt);
}

// A weight gradient over the rows of several calls (micro-batches) at once: operand s of call s, each with its own share
// bounds.  GemmArgs holds what they have in common.
constexpr int DW_MAX_SEGS = 8;
struct DwSegs {
  const void *A[DW_MAX_SEGS], *B[DW_MAX_SEGS], *B2[DW_MAX_SEGS];
  const int32_t *offsets[DW_MAX_SEGS], *kept[DW_MAX_SEGS], *lo[DW_MAX_SEGS], *hi[DW_MAX_SEGS];
  int n;
};
// both weight gradients (g1 over s1, then g2 over s2) in one launch
int launch_gemm_half_dw_segs(int dtype, const GemmArgs& g1, const DwSegs& s1, const GemmArgs& g2, const DwSegs& s2, hipStream_t s);

#ifdef __HIPCC__
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// ---- global -> LDS loads, shared by both kernels ----
// Buffer loads: the descriptor's byte count is the part of the operand a tile may read; anything past it reads as zero.
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ unsigned lds_addr(const char* p) { return (unsigned)(uintptr_t)(const lds_char*)p; }
typedef u32x4 rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, size_t bytes) {
  // block-uniform; values that went through a vector division come back to scalar registers here
  const unsigned long long p = (unsigned long long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
  const unsigned n = __builtin_amdgcn_readfirstlane(bytes > 0xffffffffull ? 0xffffffffu : (unsigned)bytes);
  // raw buffer: base address, stride 0, byte count, 32-bit untyped data format
  return rsrc_t{lo, hi & 0xffffu, n, 0x00020000u};
}

// 16 bytes per lane from a buffer straight into LDS: lane l of the wave lands at LDS byte address
// lds + 16*l (lds is wave-uniform; the instruction takes it from M0).  Completion is tracked by
// vmcnt like any other buffer load.  Written as a raw instruction on purpose: the compiler must not
// know that this load writes LDS, or it waits for every outstanding load before each LDS read it
// cannot prove disjoint (the transposing reads).  The pipeline orders loads and reads itself with
// explicit vmcnt waits and block barriers; the memory clobber keeps LDS reads from moving across.
__device__ __forceinline__ void load_to_lds16(rsrc_t rs, unsigned lds, unsigned voffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds), "v"(voffset), "s"(rs) : "memory", "m0");
}
// load_to_lds16 for data that one block reads once: the weights do not displace anything in the caches
__device__ __forceinline__ void load_to_lds16_nt(rsrc_t rs, unsigned lds, unsigned voffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
               :: "s"(lds), "v"(voffset), "s"(rs) : "memory", "m0");
}
// a byte offset past any operand: they are multiples of 16 bytes below 4 GiB (offsets_fit_32_bits)
constexpr unsigned OUT_OF_RANGE = 0xfffffff0u;
#endif

}  // namespace moe
