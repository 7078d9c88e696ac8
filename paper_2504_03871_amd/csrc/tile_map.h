// Row-tile map builder (layout: gemm.h) and the small jobs that ride in front of another kernel's blocks.
#pragma once
#include "gemm.h"

namespace moe {

struct TileMapArgs {
  const int32_t* offsets;
  const int32_t* kept;
  const int32_t* lo;
  const int32_t* hi;
  int E, tile_rows;
  int by_expert;     // an expert-major list in any case
  int table;         // which GELU table to fill as well (bf16 GELU layers: GELU_TAB_PHI before the forward GEMMs, GELU_TAB_GRAD before the backward ones)
  TileMap map;
};

// A launch whose work does not need them can carry the tile map (with its table) and the transposed gate weight in blocks
// in front of its own: launches of 3 to 7 us each (two maps and the transpose per step) then cost less than 1 us together.
// With them, with the input gradient in one pass (input_grad.hip) and two calls instead of eight from the host: fp32 step
// of 512 tokens, d 128, f 256 92 -> 67 us, bf16 step of 8192 tokens, d 1024, f 4096 980 -> 964, of 3001 tokens, d 1088,
// f 2880 590 -> 578, four micro-batches of 2048 tokens 2027 -> 1939.
constexpr int SIDE_THREADS = 256;
constexpr int WRT_PER_THREAD = 4;
struct SideWork {
  TileMapArgs tm;
  const float* Wr;   // [d][E] -> WrT [E][d]
  float* WrT;
  int d;
  int map_blocks, wrt_blocks;
  int blocks() const { return map_blocks + wrt_blocks; }
};
inline int tile_map_blocks(int table) { return table == GELU_TAB_NONE ? 1 : 1 + GELU_TAB_FLOATS / SIDE_THREADS; }
inline SideWork side_work(const TileMapArgs& tm, const float* Wr, float* WrT, int d) {
  SideWork s = {};
  s.tm = tm;
  s.map_blocks = tile_map_blocks(tm.table);
  if (WrT != nullptr) {
    s.Wr = Wr; s.WrT = WrT; s.d = d;
    s.wrt_blocks = (int)(((long long)d * tm.E + SIDE_THREADS * WRT_PER_THREAD - 1) / (SIDE_THREADS * WRT_PER_THREAD));
  }
  return s;
}

#ifdef __HIPCC__
// Tile order: every full tile (tile_rows valid rows) first, in expert order, then the experts' last,
// partly filled tiles by descending row count.  Blocks are dispatched in tile order, so the short
// tiles fill the chip's last round instead of each costing a full round.
// header[0] = number of tiles, header[1] = tiles walked XCD by XCD, header[2] = trailing tiles that may be split along K, or,
// by_expert, the number of experts with several tiles (gemm.h).
static_assert(MOE_MAX_E == SIDE_THREADS && MOE_MAX_E == 4 * WAVE, "one thread per expert; one wave scans four per lane");
__device__ inline void build_tile_map(const TileMapArgs& a) {
  // sort keys: (value << 32) | (MOE_MAX_E - 1 - id), so that "ahead of me" (larger value, ties by lower id) is
  // one 64-bit comparison; entries from E on hold value 0 and ids above every real one: never ahead
  __shared__ __align__(16) unsigned long long s_klen[MOE_MAX_E], s_krem[MOE_MAX_E];
  __shared__ int s_full[MOE_MAX_E], s_rem[MOE_MAX_E], s_start[MOE_MAX_E], s_base[MOE_MAX_E], s_rank[MOE_MAX_E];
  __shared__ int s_nfull, s_major;
  const int tid = threadIdx.x, E = a.E, tile_rows = a.tile_rows;
  {
    int l = 0, h = 0, base = 0;
    if (tid < E) {
      share_of(a.lo, a.hi, a.kept[tid], tid, l, h);
      base = a.offsets[tid] + l;
    }
    const int rem = (h - l) % tile_rows;
    s_full[tid] = (h - l) / tile_rows;
    s_rem[tid] = rem;
    s_base[tid] = base;
    s_klen[tid] = ((unsigned long long)(h - l) << 32) | (unsigned)(MOE_MAX_E - 1 - tid);
    s_krem[tid] = ((unsigned long long)rem << 32) | (unsigned)(MOE_MAX_E - 1 - tid);
  }
  __syncthreads();
  if (tid < E) {   // number of entries ahead of this thread's expert, by share length and by remainder
    const unsigned long long my_len = s_klen[tid], my_rem = s_krem[tid];
    int rank_len = 0, rank_rem = 0;
#pragma unroll 4
    for (int o = 0; o < E; o += 2) {   // entries in pairs (16-byte LDS reads)
      const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(s_klen + o), r = *reinterpret_cast<const ulonglong2*>(s_krem + o);
      rank_len += (v.x > my_len) + (v.y > my_len);
      rank_rem += (r.x > my_rem) + (r.y > my_rem);
    }
    a.map.order[rank_len] = tid;   // experts by descending share length, ties by id
    s_rank[tid] = rank_rem;
  }
  if (tid < WAVE) {   // the first wave scans the experts, four per lane
    int full[4], some[4], sum_full = 0, sum_part = 0, sum_small = 0, sum_more = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      full[i] = s_full[tid * 4 + i];
      const int rem = s_rem[tid * 4 + i];
      some[i] = rem > 0;
      sum_full += full[i];
      sum_part += some[i];
      sum_small += (rem > 0 && rem <= SPLIT_ROWS);
      sum_more += full[i] + some[i] > 1;
    }
    const int run = wave_sum_i(sum_full), parts = wave_sum_i(sum_part), small = wave_sum_i(sum_small);
    sum_more = wave_sum_i(sum_more);
    // Many experts of few row tiles each: an expert's weight panels are used by two or three tiles only,
    // so these must run together (same XCD, same time) or the panels are fetched once per tile.  The
    // list is then expert-major (each expert's full tiles, then its partly filled one) and the whole of
    // it is walked as the full region is.
    const bool major = a.by_expert || (E > SPLIT_MAX_E && run < 3 * E);
    const int mine = major ? sum_full + sum_part : sum_full;
    int pos = wave_scan_i(mine) - mine;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s_start[tid * 4 + i] = pos;
      pos += full[i] + (major ? some[i] : 0);
    }
    if (tid == 0) {
      s_nfull = run;
      s_major = major;
      a.map.header[0] = run + parts;
      a.map.header[1] = major ? run + parts : run;
      a.map.header[2] = a.by_expert ? sum_more : major ? 0 : small;   // the last entries: the partly filled tiles are sorted by descending size
    }
  }
  __syncthreads();
  const int per_expert = SIDE_THREADS / E, e = tid / per_expert, part = tid % per_expert;   // the threads share out an expert's tiles
  if (e < E) {
    const int base = s_base[e], nfull = s_full[e], rem = s_rem[e];
    // Expert-major list: an expert's rows are cut into its ceil(len / tile_rows) tiles evenly (in steps of 64
    // rows, two MFMA row bands) instead of full tiles plus a remainder.  A remainder of a few rows costs a
    // block the whole weight panel for next to no arithmetic; two tiles of 140 rows cost less than one of
    // 256 and one of 24, and every output row is computed the same way wherever its tile starts.
    const int len = nfull * tile_rows + rem, ntile = s_major ? nfull + (rem > 0) : nfull;
    int per = tile_rows;
    if (s_major && ntile > 1) {
      per = min(tile_rows, ((len + ntile - 1) / ntile + 63) & ~63);
      if ((ntile - 1) * per >= len) per = tile_rows;   // many tiles: the rounding would leave the last one empty
    }
    for (int i = part; i < ntile; i += per_expert) {
      RowTile t;
      t.e = e;
      t.row0 = base + i * per;
      t.nrows = min(per, len - i * per);
      t.mates = nfull + (rem > 0) > 1;
      a.map.tiles[s_start[e] + i] = t;
    }
    if (!s_major && part == 0 && rem > 0) {   // position among the partial tiles: more rows first, ties by expert id
      RowTile t;
      t.e = e;
      t.row0 = base + nfull * tile_rows;
      t.nrows = rem;
      t.mates = nfull > 0;
      a.map.tiles[s_nfull + s_rank[e]] = t;
    }
  }
}
// Entry i of a table: Phi(v) or gelu'(v) for the bf16 numbers (layout: gemm.h)
__device__ inline void gelu_table_entry(const TileMapArgs& a, int i) {
  float v = 0.f;
  if (i < 2 * GELU_TAB_NMAG) {
    const uint32_t bits = (uint32_t)((i % GELU_TAB_NMAG) + (GELU_TAB_EXP0 << 7)) | (i >= GELU_TAB_NMAG ? 0x8000u : 0u);
    const float x = __uint_as_float(bits << 16);
    v = a.table == GELU_TAB_PHI ? 0.5f * erfcf(-x * 0.70710678118654752440f) : gelu_grad_f(x);
    // the last magnitude also stands for everything larger: Phi is exactly 1 or 0 there, so that
    // h = a Phi stays a or 0 however large a is
    if (a.table == GELU_TAB_PHI && i % GELU_TAB_NMAG == GELU_TAB_NMAG - 1) v = i >= GELU_TAB_NMAG ? 0.f : 1.f;
  }
  a.map.gelu_tab[i] = v;
}
// Block `b` of the side work (SIDE_THREADS threads): the map first, one thread per table entry, then the gate weight.
__device__ inline void run_side_work(const SideWork& s, int b) {
  if (b == 0) return build_tile_map(s.tm);
  if (b < s.map_blocks) return gelu_table_entry(s.tm, (b - 1) * SIDE_THREADS + threadIdx.x);
  const int n = s.d * s.tm.E, first = (b - s.map_blocks) * SIDE_THREADS * WRT_PER_THREAD + threadIdx.x;
#pragma unroll
  for (int u = 0; u < WRT_PER_THREAD; ++u) {
    const int i = first + u * SIDE_THREADS;
    if (i < n) s.WrT[(size_t)(i % s.tm.E) * s.d + i / s.tm.E] = s.Wr[i];
  }
}
#endif

}  // namespace moe
