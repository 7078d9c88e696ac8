// Launchers of the MFMA grouped GEMM for 16-bit storage, bf16 or fp16 (kernel in gemm_bf16_kernel.h).
#include "gemm_bf16_kernel.h"
#include "gemm_skinny_kernel.h"
#include <algorithm>

namespace moe {

// Block tile 256 x 256 (SwiGLU forward: 256 x 128 for each of its two weight matrices), 2 x 4 waves: two
// waves per SIMD, so one wave's LDS and global traffic hides under the other's MFMAs.  Global loads write LDS
// directly, in 64-wide K stages for all three operand layouts: two of one operand and three of the other.
constexpr int T_BM = 256, T_BN = 256, T_BN_DUAL = 128, T_BN_SEGS = 128, T_WGM = 2, T_WGN = 4;
int gemm_bf16_tile_rows() { return T_BM; }

// blocks of a split launch beyond one per tile
static long long split_blocks(const GemmArgs& g, long long ntn) {
  const long long small = g.split_small ? (long long)g.E * ntn * (SPLIT_K - 1) : 0;
  return g.split_tail && small < TAIL_SLOTS ? TAIL_SLOTS : small;
}
// adds the partial sums of every split tile and writes the 16-bit rows of C [rows][N]
template <typename ST>
static int launch_split_reduce(const GemmArgs& g, long long tiles, hipStream_t s) {
  const long long small = g.split_small ? (long long)g.E * ((SPLIT_ROWS * (g.N / 4) + 255) / 256) : 0;
  const long long tail = g.split_tail ? (tiles < TAIL_SLOTS / 2 ? tiles : TAIL_SLOTS / 2) * (g.tile_rows / TAIL_REDUCE_ROWS) : 0;
  split_reduce_kernel<ST><<<dim3((unsigned)(small > tail ? small : tail)), 256, 0, s>>>(g);
  return launch_status();
}

template <typename ST, int MODE, int EPI, bool DUAL, bool CHAIN, int BM, bool STREAM>
static int launch_rows(const GemmArgs& g, int max_tiles, hipStream_t s) {
  constexpr int BN = DUAL ? T_BN_DUAL : T_BN;
  constexpr int lds = gemm_bf16_lds_bytes<BM, BN, DUAL>();
  // Two matrices of 128 columns: 4 x 2 waves of 64 rows and 64 columns of either, which write whole lines, streamed
  // (2 x 4: 32 columns, half lines).  GEMM1 of SwiGLU, 16 rounds of tiles, us per round, 2 x 4 and plain stores -> 4 x 2:
  // K 512 28.8 -> 25.0, 1024 38.6 -> 35.5, 2048 62.4 -> 60.2, 4096 112 -> 108.5; forward passes: eight experts of 2048 rows,
  // d 1024, f 4096 510 -> 457, 16 of 600, d 2048, f 8192 1149 -> 1112, six of 1200, d 1088, f 2880 194 -> 195.  160 rows
  // have five bands, which four wave rows would share unevenly.
  constexpr int WGM = DUAL && BM == T_BM ? 4 : T_WGM;
  auto kern = gemm_bf16_kernel<ST, MODE, EPI, DUAL, CHAIN, BM, BN, WGM, 8 / WGM, STREAM>;
  // more than 64 KB of dynamic LDS needs the attribute on the current device; set on every launch (a cheap
  // host-side call) rather than remembered, so the library keeps no per-process or per-device state
  {
    hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (err != hipSuccess) return set_hip_error(err);
  }
  const int ntn = (g.N + BN - 1) / BN;
  long long tiles;
  if (MODE == MODE_TN) tiles = dw_blocks(g, T_BM, T_BN);
  else tiles = (long long)ntn * max_tiles;
  const bool split = MODE != MODE_TN && EPI == EPI_STORE && g.split_ws != nullptr;
  kern<<<dim3(gemm_bf16_grid(tiles + (split ? split_blocks(g, ntn) : 0))), T_WGM * T_WGN * 64, lds, s>>>(g);
  int rc = launch_status();
  if (rc != MOE_OK || !split) return rc;
  return launch_split_reduce<ST>(g, tiles, s);
}

template <typename ST, int MODE, int EPI, bool DUAL, bool CHAIN>
static int launch_one(const GemmArgs& g, int max_tiles, hipStream_t s) {
  if constexpr (MODE != MODE_TN) {
    if (g.tile_rows == MID_ROWS && g.stream) return launch_rows<ST, MODE, EPI, DUAL, CHAIN, MID_ROWS, true>(g, max_tiles, s);
    if (g.tile_rows == MID_ROWS) return launch_rows<ST, MODE, EPI, DUAL, CHAIN, MID_ROWS, false>(g, max_tiles, s);
    if (g.stream) return launch_rows<ST, MODE, EPI, DUAL, CHAIN, T_BM, true>(g, max_tiles, s);
  }
  return launch_rows<ST, MODE, EPI, DUAL, CHAIN, T_BM, false>(g, max_tiles, s);
}

// A row-tile GEMM (NT) and a weight-gradient GEMM (TN, one gradient or two of the same A) in one launch; the first one's
// blocks come first.
template <typename ST, int EPI1, bool CHAIN1, int BM1, bool STREAM>
static int launch_pair_rows(const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  constexpr int lds1 = gemm_bf16_lds_bytes<BM1, T_BN, false>();
  constexpr int lds2 = gemm_bf16_lds_bytes<T_BM, T_BN, false>();
  constexpr int lds = lds1 > lds2 ? lds1 : lds2;
  auto kern = gemm_bf16_pair_kernel<ST, MODE_NT, EPI1, CHAIN1, BM1, MODE_TN, EPI_DW, T_BM, T_BN, T_WGM, T_WGN, STREAM>;
  // more than 64 KB of dynamic LDS needs the attribute on the current device; set on every launch (a cheap
  // host-side call) rather than remembered, so the library keeps no per-process or per-device state
  {
    hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (err != hipSuccess) return set_hip_error(err);
  }
  // the first GEMM's block count is a multiple of the XCD count, so that a tile number still tells the
  // XCD its block runs on for the second one (numbers past the last tile return at once)
  // (a plain-store first GEMM may split its smallest row tiles along K: SPLIT_K blocks per column tile, see gemm.h)
  const int ntn1 = (g1.N + T_BN - 1) / T_BN;
  const bool split = EPI1 == EPI_STORE && !CHAIN1 && g1.split_ws != nullptr;
  const long long tiles1 = (long long)ntn1 * max_tiles, t1 = tiles1 + (split ? split_blocks(g1, ntn1) : 0);
  const long long n1 = (t1 + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
  const long long n2 = dw_blocks(g2, T_BM, T_BN);
  if (n1 + n2 > 0x7fffffffll) return MOE_ERR_BAD_SHAPE;
  kern<<<dim3(gemm_bf16_grid(n1 + n2)), T_WGM * T_WGN * 64, lds, s>>>(g1, g2, (int)n1);
  const int rc = launch_status();
  if (rc != MOE_OK || !split) return rc;
  return launch_split_reduce<ST>(g1, tiles1, s);
}

template <typename ST, int EPI1, bool CHAIN1>
static int launch_pair(const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  if (g1.tile_rows == MID_ROWS && g1.stream) return launch_pair_rows<ST, EPI1, CHAIN1, MID_ROWS, true>(g1, max_tiles, g2, s);
  if (g1.tile_rows == MID_ROWS) return launch_pair_rows<ST, EPI1, CHAIN1, MID_ROWS, false>(g1, max_tiles, g2, s);
  if (g1.stream) return launch_pair_rows<ST, EPI1, CHAIN1, T_BM, true>(g1, max_tiles, g2, s);
  return launch_pair_rows<ST, EPI1, CHAIN1, T_BM, false>(g1, max_tiles, g2, s);
}

template <typename ST>
static int dw_segs_for(const GemmArgs& g1, const DwSegs& s1, const GemmArgs& g2, const DwSegs& s2, hipStream_t s) {
  constexpr int BN = T_BN_SEGS, lds = gemm_bf16_lds_bytes<T_BM, BN, false>();
  auto kern = gemm_bf16_dw_segs_kernel<ST, T_BM, BN, 4, 2>;
  hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (err != hipSuccess) return set_hip_error(err);
  const long long n1 = dw_blocks(g1, T_BM, BN), n2 = dw_blocks(g2, T_BM, BN);
  if (n1 + n2 > 0x7fffffffll) return MOE_ERR_BAD_SHAPE;
  kern<<<dim3(gemm_bf16_grid(n1 + n2)), T_WGM * T_WGN * 64, lds, s>>>(DwSegsPair{{g1, g2}, {s1, s2}, (int)n1});
  return launch_status();
}

template <typename ST>
static int pair_for(int epi1, bool chain1, const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  if (epi1 == EPI_GELU_BWD) return launch_pair<ST, EPI_GELU_BWD, false>(g1, max_tiles, g2, s);
  if (epi1 == EPI_SWIGLU_BWD) return launch_pair<ST, EPI_SWIGLU_BWD, false>(g1, max_tiles, g2, s);
  if (epi1 == EPI_STORE && !chain1) return launch_pair<ST, EPI_STORE, false>(g1, max_tiles, g2, s);
  if (epi1 == EPI_STORE && chain1) return launch_pair<ST, EPI_STORE, true>(g1, max_tiles, g2, s);
  return MOE_ERR_BAD_DTYPE;
}

template <typename ST>
static int one_for(int mode, int epi, bool dual, bool chain, const GemmArgs& g, int max_tiles, hipStream_t s) {
  if (mode == MODE_NN && epi == EPI_GELU_FWD) return launch_one<ST, MODE_NN, EPI_GELU_FWD, false, false>(g, max_tiles, s);
  if (mode == MODE_NN && epi == EPI_SWIGLU_FWD && dual) return launch_one<ST, MODE_NN, EPI_SWIGLU_FWD, true, false>(g, max_tiles, s);
  if (mode == MODE_NN && epi == EPI_STORE) return launch_one<ST, MODE_NN, EPI_STORE, false, false>(g, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_GELU_BWD) return launch_one<ST, MODE_NT, EPI_GELU_BWD, false, false>(g, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_SWIGLU_BWD) return launch_one<ST, MODE_NT, EPI_SWIGLU_BWD, false, false>(g, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_STORE && !chain) return launch_one<ST, MODE_NT, EPI_STORE, false, false>(g, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_STORE && chain) return launch_one<ST, MODE_NT, EPI_STORE, false, true>(g, max_tiles, s);
  if (mode == MODE_TN && epi == EPI_DW) return launch_one<ST, MODE_TN, EPI_DW, false, false>(g, max_tiles, s);
  return MOE_ERR_BAD_DTYPE;
}

int launch_gemm_half_dw_segs(int dtype, const GemmArgs& g1, const DwSegs& s1, const GemmArgs& g2, const DwSegs& s2, hipStream_t s) {
  return dtype == MOE_DTYPE_F16 ? dw_segs_for<f16>(g1, s1, g2, s2, s) : dw_segs_for<bf16>(g1, s1, g2, s2, s);
}

int launch_gemm_half_pair(int dtype, int epi1, bool chain1, const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  return dtype == MOE_DTYPE_F16 ? pair_for<f16>(epi1, chain1, g1, max_tiles, g2, s) : pair_for<bf16>(epi1, chain1, g1, max_tiles, g2, s);
}

int launch_gemm_half(int dtype, int mode, int epi, bool dual, bool chain, const GemmArgs& g, int max_tiles, hipStream_t s) {
  return dtype == MOE_DTYPE_F16 ? one_for<f16>(mode, epi, dual, chain, g, max_tiles, s) : one_for<bf16>(mode, epi, dual, chain, g, max_tiles, s);
}

// Few rows per expert (gemm_skinny_kernel.h); the tile map has SKINNY_ROWS rows per tile.
template <typename ST, int EPI, bool DUAL>
static int launch_skinny(const GemmArgs& g, int max_tiles, hipStream_t s) {
  constexpr int lds = skinny_stages<DUAL>() * skinny_stage_bytes<DUAL>();
  auto kern = gemm_skinny_kernel<ST, EPI, DUAL>;
  {
    hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (err != hipSuccess) return set_hip_error(err);
  }
  const int ntn = (g.N + SKINNY_BN - 1) / SKINNY_BN;
  const bool split = EPI == EPI_STORE && g.split_all;
  const long long blocks = (long long)ntn * (split ? std::max(max_tiles * (SPLIT_K / 2), g.E * SPLIT_K) : max_tiles);
  if (blocks > 0x7fffffffll) return MOE_ERR_BAD_SHAPE;
  kern<<<dim3(gemm_bf16_grid(blocks)), 256, lds, s>>>(g);
  const int rc = launch_status();
  if (rc != MOE_OK || !split) return rc;
  split_reduce_kernel<ST><<<dim3((unsigned)(max_tiles * ((SKINNY_ROWS * (g.N / 4) + 255) / 256))), 256, 0, s>>>(g);
  return launch_status();
}
template <typename ST>
static int skinny_for(int epi, bool dual, const GemmArgs& g, int max_tiles, hipStream_t s) {
  if (epi == EPI_GELU_FWD) return launch_skinny<ST, EPI_GELU_FWD, false>(g, max_tiles, s);
  if (epi == EPI_SWIGLU_FWD && dual) return launch_skinny<ST, EPI_SWIGLU_FWD, true>(g, max_tiles, s);
  if (epi == EPI_STORE) return launch_skinny<ST, EPI_STORE, false>(g, max_tiles, s);
  return MOE_ERR_BAD_DTYPE;
}
int launch_gemm_half_skinny(int dtype, int epi, bool dual, const GemmArgs& g, int max_tiles, hipStream_t s) {
  return dtype == MOE_DTYPE_F16 ? skinny_for<f16>(epi, dual, g, max_tiles, s) : skinny_for<bf16>(epi, dual, g, max_tiles, s);
}

}  // namespace moe
