// Row-tile map launch and the fp32 grouped GEMM (fp32 storage, fp32 matrix instructions).
//
// The fp32 path exists for the full-precision configurations, whose tolerance (1e-5) rules out
// reduced-precision matrix instructions.
#include "gemm.h"
#include "tile_map.h"

namespace moe {

__global__ __launch_bounds__(SIDE_THREADS) void tile_map_kernel(SideWork s) { run_side_work(s, blockIdx.x); }
int launch_tile_map(const TileMapArgs& tm, hipStream_t s) {
  const SideWork side = side_work(tm, nullptr, nullptr, 0);
  tile_map_kernel<<<side.blocks(), SIDE_THREADS, 0, s>>>(side);
  return launch_status();
}

// ---- fp32 grouped GEMM on the matrix cores ---------------------------------------------------------------------
// v_mfma_f32_16x16x4_f32 multiplies and accumulates in fp32, at twice the rate of plain fp32 FMAs, and takes its
// operands as one register per lane and matrix, so what is left to do well is to keep it fed: a wave of this kernel
// reads one or two 16-byte LDS words per matrix instruction of 32 cycles.
//
// Block tile 64 x 64, four waves of 16 rows x 64 columns (a wave without valid rows skips its arithmetic), K in stages
// of 32 that buffer loads write straight into a ring of LDS stages.  A small tile on purpose: the matrix instruction
// is slow enough (256 FLOP per cycle and compute unit) that 64 x 64 tiles stay within the L2's rate, 48 KB of LDS let
// three blocks share a compute unit and hide each other's waits, and the small full-precision problems this path
// serves get enough blocks.  It is bound by the matrix cores on large problems and by latency on the smallest.
// T 2000, d 516, f 1540, eight experts, against the LDS-tiled FMA kernel it replaces: SwiGLU
// forward 264 -> 144 us, y 177 -> 90, a weight gradient 139 -> 80, dx 343 -> 175 (42 -> 78 TFLOP/s over the step's GEMMs).
//
// Problems with few tiles take 32 x 64 ones (BM = 32, line in gemm.h): two waves share 16 rows, each with every other run
// of 16 K values, and add their sums through LDS at the end, so twice the blocks walk K at twice the speed.
//
// K order: lane group g = lane / 16 supplies K value 4 g + s of every run of 16 in step s, for both operands, so a
// 16-byte read along K serves four steps.  Columns: lane c = lane % 16 holds columns 4 c .. 4 c + 3 of the wave's 64
// as column tiles j = 0 .. 3, so a 16-byte read across columns serves four tiles and the results leave as 16-byte rows.
constexpr int SB = F32_TILE_COLS;   // tile edge
constexpr int SK = 32;   // K values per stage

// bytes of an operand tile of R rows (or columns); 16-byte chunks of it per thread
constexpr int f32_tile_bytes(int r) { return r * SK * 4; }
constexpr int f32_chunks(int r) { return f32_tile_bytes(r) / (256 * 16); }

// Operand tiles in LDS.  K contiguous in memory: [64][32], 128-byte rows whose eight chunks are XOR-swizzled by the
// row pair (16 lanes reading one chunk of 16 consecutive rows hit 16 different 16-byte bank groups).  K strided:
// [32][64], 256-byte rows whose 64-byte granules are XOR-swizzled by (K row / 4), so the four lane groups, which read
// K rows four apart, use different banks.
__device__ __forceinline__ int f32_kc_off(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }
template <int R>
__device__ __forceinline__ int f32_ks_off(int krow, int col_byte) { return krow * (R * 4) + (col_byte ^ (((krow >> 2) & (R / 16 - 1)) << 6)); }

// Chunk id of a tile (its 16 bytes lie at LDS byte 16 id): the operand's byte offset and its first K index.  PERM: LDS
// row r holds operand row 4 (r % 16) + r / 16, the column order above.
template <bool KC, bool PERM, int R>
__device__ __forceinline__ void f32_chunk(int id, unsigned pitch, unsigned& off, int& k) {
  if constexpr (KC) {
    const int r = id >> 3, c = (id & 7) ^ ((r >> 1) & 7), row = PERM ? 4 * (r & 15) + (r >> 4) : r;
    off = (unsigned)row * pitch + c * 16u;
    k = c * 4;
  } else {
    const int r = id / (R / 4), c = (id % (R / 4)) ^ (((r >> 2) & (R / 16 - 1)) << 2);
    off = (unsigned)r * pitch + c * 16u;
    k = r;
  }
}

template <int EPI>
__device__ __forceinline__ void epilogue_f32x4(const GemmArgs& g, size_t idx, const f32x4& a, const f32x4& a2, const f32x4& s1,
                                               const f32x4& s2, bool second_grad) {
  auto at = [&](void* base) { return reinterpret_cast<f32x4*>(reinterpret_cast<float*>(base) + idx); };
  f32x4 r, q;
  if constexpr (EPI == EPI_STORE) {
    *at(g.C) = a;
  } else if constexpr (EPI == EPI_GELU_FWD) {   // C == NULL: the caller keeps only the hidden activation
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = gelu_f(a[i]);
    if (g.C != nullptr) *at(g.C) = a;
    *at(g.C2) = r;
  } else if constexpr (EPI == EPI_SWIGLU_FWD) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = a[i] * sigmoid_f(a[i]) * a2[i];
    if (g.C != nullptr) { *at(g.C) = a; *at(g.C2) = a2; }
    *at(g.C3) = r;
  } else if constexpr (EPI == EPI_GELU_BWD) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = a[i] * gelu_grad_f(s1[i]);
    *at(g.C) = r;
  } else if constexpr (EPI == EPI_SWIGLU_BWD) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float sg = sigmoid_f(s1[i]);
      r[i] = a[i] * s2[i] * sg * (1.f + s1[i] * (1.f - sg));
      q[i] = a[i] * s1[i] * sg;
    }
    *at(g.C) = r;
    *at(g.C2) = q;
  } else {
    *at(second_grad ? g.C2 : g.C) = g.accumulate ? s1 + a : a;
  }
}

template <bool DUAL, int BM>
constexpr int f32_lds_bytes() { return (f32_tile_bytes(BM) + f32_tile_bytes(SB) * (DUAL ? 2 : 1)) * (DUAL ? 2 : 3); }

// One output tile; vb = its number in dispatch order.
template <int MODE, int EPI, bool DUAL, bool CHAIN, int BM>
__device__ __forceinline__ void gemm_f32_tile(const GemmArgs& g, const int vb, char* smem) {
  constexpr bool A_KC = MODE != MODE_TN, B_KC = MODE == MODE_NT;
  constexpr int BANDS = BM / 16, KH = 4 / BANDS;                        // KH waves share a band, each with every KH-th run of 16 K values
  constexpr int A_TILE = f32_tile_bytes(BM), B_TILE = f32_tile_bytes(SB), CHA = f32_chunks(BM), CHB = f32_chunks(SB);
  constexpr int STAGE = A_TILE + B_TILE * (DUAL ? 2 : 1), NBUF = DUAL ? 2 : 3;   // 48 KB either way (BM 32: 36 and 40 KB)
  constexpr int AHEAD = NBUF - 1;                                       // stages requested ahead of the one in use
  constexpr int L = CHA + CHB * (DUAL ? 2 : 1);                         // loads per thread and stage
  static_assert(NBUF * STAGE == f32_lds_bytes<DUAL, BM>(), "the caller's LDS");
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), band = wave % BANDS, kh = wave / BANDS;
  const int ntn = (g.N + SB - 1) / SB;
  int e, row0, mvalid, klen, m0 = 0, nt;
  bool second_grad = false;
  if constexpr (MODE == MODE_TN) {
    int slot, mt;
    if (!dw_block(vb, (g.M + BM - 1) / BM, ntn, slot, mt, nt)) return;
    if (g.C2 != nullptr) { second_grad = slot & 1; slot >>= 1; }   // the two gradients of an expert follow each other
    e = g.order[slot];
    m0 = mt * BM;
    int l, h;
    share_of(g.lo, g.hi, g.kept[e], e, l, h);
    row0 = g.offsets[e] + l;
    klen = h - l;
    mvalid = min(BM, g.M - m0);
    if (klen == 0 && g.accumulate) return;
  } else {
    RowBlock rb;
    if (!row_tile_block(vb, g.ntiles[0], g.ntiles[1], 0, ntn, false, rb)) return;
    const RowTile t = g.tiles[rb.rt];
    e = t.e;
    row0 = t.row0;
    mvalid = t.nrows;
    klen = g.K;
    nt = rb.nt;
  }
  const int n0 = nt * SB;

  // operand bases, the bytes this tile may read (anything past them arrives as zero), pitch and advance per stage
  size_t aoff, boff, abytes, bbytes;
  unsigned pa, pb, astep, bstep;
  if constexpr (MODE == MODE_TN) {
    aoff = (size_t)row0 * g.M + m0;  abytes = klen > 0 ? ((size_t)klen * g.M - m0) * 4 : 0;
    boff = (size_t)row0 * g.N + n0;  bbytes = klen > 0 ? ((size_t)klen * g.N - n0) * 4 : 0;
    pa = g.M * 4; pb = g.N * 4; astep = SK * pa; bstep = SK * pb;
  } else {
    aoff = (size_t)row0 * g.K;  abytes = (size_t)mvalid * g.K * 4;
    pa = g.K * 4; astep = SK * 4;
    if constexpr (MODE == MODE_NN) {
      boff = (size_t)e * g.K * g.N + n0;  bbytes = ((size_t)g.K * g.N - n0) * 4;
      pb = g.N * 4; bstep = SK * pb;
    } else {
      boff = ((size_t)e * g.N + n0) * g.K;  bbytes = (size_t)(g.N - n0) * g.K * 4;
      pb = g.K * 4; bstep = SK * 4;
    }
  }
  const rsrc_t ra = make_rsrc(reinterpret_cast<const float*>(g.A) + aoff, abytes);
  const rsrc_t rb = make_rsrc(reinterpret_cast<const float*>(second_grad ? g.B2 : g.B) + boff, bbytes);
  const rsrc_t ra2 = make_rsrc(reinterpret_cast<const float*>(CHAIN ? g.A2 : g.A) + aoff, abytes);
  const rsrc_t rb2 = make_rsrc(reinterpret_cast<const float*>(CHAIN || DUAL ? g.B2 : g.B) + boff, bbytes);
  const int KT1 = (klen + SK - 1) / SK, KT = CHAIN ? 2 * KT1 : KT1;   // a chained GEMM runs its two operand pairs back to back
  unsigned a_vo[CHA], b_vo[CHB];
  int a_k[CHA], b_k[CHB];
#pragma unroll
  for (int i = 0; i < CHA; ++i) f32_chunk<A_KC, false, BM>(tid + 256 * i, pa, a_vo[i], a_k[i]);
#pragma unroll
  for (int i = 0; i < CHB; ++i) f32_chunk<B_KC, true, SB>(tid + 256 * i, pb, b_vo[i], b_k[i]);
  const unsigned lds0 = lds_addr(smem) + wave * 1024;   // a wave's load fills 1 KB of the tile
  auto load_stage = [&](int kt, int buf) {
    const bool second = CHAIN && kt >= KT1;
    const unsigned kl = second ? kt - KT1 : kt;
    const int left = klen - (int)kl * SK;   // K values from this stage on; chunks past them must read as zero in both operands
#pragma unroll
    for (int i = 0; i < CHA; ++i)
      load_to_lds16(second ? ra2 : ra, lds0 + buf * STAGE + i * 4096, a_k[i] < left ? a_vo[i] + kl * astep : OUT_OF_RANGE);
#pragma unroll
    for (int i = 0; i < CHB; ++i) {
      const unsigned o = b_k[i] < left ? b_vo[i] + kl * bstep : OUT_OF_RANGE;
      load_to_lds16(second ? rb2 : rb, lds0 + buf * STAGE + A_TILE + i * 4096, o);
      if constexpr (DUAL) load_to_lds16(rb2, lds0 + buf * STAGE + A_TILE + B_TILE + i * 4096, o);
    }
  };

  f32x4 acc[4], acc2[DUAL ? 4 : 1];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (DUAL) acc2[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const bool active = band * 16 < mvalid;
#pragma unroll
  for (int q = 0; q < AHEAD; ++q)
    if (q < KT) load_stage(q, q);
  int buf = 0;
#pragma unroll 1
  for (int kt = 0; kt < KT; ++kt) {
    // own loads of this stage have landed (those of the next may be in flight) and own reads of the last one are done;
    // behind the barrier that holds for every wave, and the buffer of the last stage is free
    constexpr int PEND = (AHEAD - 1) * L;
    static_assert(PEND < 16, "low bits of the wait counter");
    if (kt + 1 < KT) __builtin_amdgcn_s_waitcnt(PEND | 0x70); else __builtin_amdgcn_s_waitcnt(0x70);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + AHEAD < KT) load_stage(kt + AHEAD, buf + AHEAD >= NBUF ? buf + AHEAD - NBUF : buf + AHEAD);
    if (active) {
      const char* sa = smem + buf * STAGE;
      const char* sb = sa + A_TILE;
#pragma unroll
      for (int q = 0; q < SK / 16 / KH; ++q) {
        const int kc = q * KH + kh;
        f32x4 av, bv[4], bv2[DUAL ? 4 : 1];   // bv: K contiguous [tile j][step s], K strided [step s][tile j]
        if constexpr (A_KC) av = *reinterpret_cast<const f32x4*>(sa + f32_kc_off(band * 16 + c, kc * 4 + grp));
        else {
#pragma unroll
          for (int s = 0; s < 4; ++s) av[s] = *reinterpret_cast<const float*>(sa + f32_ks_off<BM>(kc * 16 + grp * 4 + s, (band * 16 + c) * 4));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int o = B_KC ? f32_kc_off(i * 16 + c, kc * 4 + grp) : f32_ks_off<SB>(kc * 16 + grp * 4 + i, c * 16);
          bv[i] = *reinterpret_cast<const f32x4*>(sb + o);
          if constexpr (DUAL) bv2[i] = *reinterpret_cast<const f32x4*>(sb + B_TILE + o);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], B_KC ? bv[j][s] : bv[s][j], acc[j], 0, 0, 0);
            if constexpr (DUAL) acc2[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], bv2[s][j], acc2[j], 0, 0, 0);
          }
      }
    }
    buf = buf + 1 == NBUF ? 0 : buf + 1;
  }
  if constexpr (KH == 2) {   // the second half's sums join the first's through LDS, once every wave has left the ring
    __syncthreads();
    f32x4* sums = reinterpret_cast<f32x4*>(smem) + band * (DUAL ? 8 : 4) * 64 + lane;
    if (kh == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sums[j * 64] = acc[j];
        if constexpr (DUAL) sums[(4 + j) * 64] = acc2[j];
      }
    }
    __syncthreads();
    if (kh == 1) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[j] += sums[j * 64];
      if constexpr (DUAL) acc2[j] += sums[(4 + j) * 64];
    }
  }
  if (!active || n0 + c * 4 >= g.N) return;
  // accumulator register v of a lane: row 4 grp + v of the wave's 16, one column of each of the four column tiles
  size_t idx[4];
  f32x4 s1[4], s2[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int m = band * 16 + grp * 4 + v, mc = min(m, mvalid - 1);
    if constexpr (MODE == MODE_TN) idx[v] = ((size_t)e * g.M + m0 + mc) * g.N + n0 + c * 4;
    else idx[v] = (size_t)(row0 + mc) * g.N + n0 + c * 4;
    if constexpr (EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU_BWD) s1[v] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.S1) + idx[v]);
    if constexpr (EPI == EPI_SWIGLU_BWD) s2[v] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.S2) + idx[v]);
    if constexpr (EPI == EPI_DW)
      if (g.accumulate) s1[v] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(second_grad ? g.C2 : g.C) + idx[v]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (band * 16 + grp * 4 + v < mvalid)
      epilogue_f32x4<EPI>(g, idx[v], f32x4{acc[0][v], acc[1][v], acc[2][v], acc[3][v]},
                          DUAL ? f32x4{acc2[0][v], acc2[DUAL ? 1 : 0][v], acc2[DUAL ? 2 : 0][v], acc2[DUAL ? 3 : 0][v]} : f32x4{}, s1[v], s2[v], second_grad);
}

template <int MODE, int EPI, bool DUAL, bool CHAIN, int BM>
__global__ __launch_bounds__(256, BM == SB ? 3 : 4) void gemm_f32_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) char smem[f32_lds_bytes<DUAL, BM>()];
  gemm_f32_tile<MODE, EPI, DUAL, CHAIN, BM>(g, blockIdx.x, smem);
}

// A row-tile GEMM (NT) and the weight-gradient GEMM(s) that need no result of it in one launch, the row-tile GEMM's
// blocks first: the weight-gradient tiles start where its last round leaves the chip idle.
template <int EPI1, bool CHAIN1, int BM1, int BM2>
__global__ __launch_bounds__(256, BM1 == SB || BM2 == SB ? 3 : 4) void gemm_f32_pair_kernel(GemmArgs g1, GemmArgs g2, int first_blocks) {
  constexpr int lds1 = f32_lds_bytes<false, BM1>(), lds2 = f32_lds_bytes<false, BM2>();
  __shared__ __attribute__((aligned(1024))) char smem[lds1 > lds2 ? lds1 : lds2];
  if ((int)blockIdx.x < first_blocks) gemm_f32_tile<MODE_NT, EPI1, false, CHAIN1, BM1>(g1, blockIdx.x, smem);
  else gemm_f32_tile<MODE_TN, EPI_DW, false, false, BM2>(g2, blockIdx.x - first_blocks, smem);
}

template <int MODE, int EPI, bool DUAL, bool CHAIN, int BM>
static int launch_bm(const GemmArgs& g, int max_tiles, hipStream_t s) {
  const long long ntn = (g.N + SB - 1) / SB, blocks = MODE == MODE_TN ? dw_blocks(g, BM, SB) : ntn * max_tiles;
  if (blocks > 0x7fffffffll) return MOE_ERR_BAD_SHAPE;
  gemm_f32_kernel<MODE, EPI, DUAL, CHAIN, BM><<<dim3((unsigned)blocks), 256, 0, s>>>(g);
  return launch_status();
}
// by one gradient's tiles, also where two share the launch: the height decides how many chains a sum is made of
static int dw_tile_rows(const GemmArgs& g) { return f32_tile_rows((long long)g.M * g.E, 0, g.N); }
// tile_rows: rows per entry of the tile map (row-tile GEMMs)
template <int MODE, int EPI, bool DUAL, bool CHAIN>
static int launch_one(const GemmArgs& g, int tile_rows, int max_tiles, hipStream_t s) {
  if (MODE == MODE_TN) tile_rows = dw_tile_rows(g);
  return tile_rows == SB ? launch_bm<MODE, EPI, DUAL, CHAIN, SB>(g, max_tiles, s)
                         : launch_bm<MODE, EPI, DUAL, CHAIN, SB / 2>(g, max_tiles, s);
}

int launch_gemm_f32(int mode, int epi, bool dual, bool chain, const GemmArgs& g, int tile_rows, int max_tiles, hipStream_t s) {
  if (mode == MODE_NN && epi == EPI_GELU_FWD) return launch_one<MODE_NN, EPI_GELU_FWD, false, false>(g, tile_rows, max_tiles, s);
  if (mode == MODE_NN && epi == EPI_SWIGLU_FWD && dual) return launch_one<MODE_NN, EPI_SWIGLU_FWD, true, false>(g, tile_rows, max_tiles, s);
  if (mode == MODE_NN && epi == EPI_STORE) return launch_one<MODE_NN, EPI_STORE, false, false>(g, tile_rows, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_GELU_BWD) return launch_one<MODE_NT, EPI_GELU_BWD, false, false>(g, tile_rows, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_SWIGLU_BWD) return launch_one<MODE_NT, EPI_SWIGLU_BWD, false, false>(g, tile_rows, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_STORE && !chain) return launch_one<MODE_NT, EPI_STORE, false, false>(g, tile_rows, max_tiles, s);
  if (mode == MODE_NT && epi == EPI_STORE && chain) return launch_one<MODE_NT, EPI_STORE, false, true>(g, tile_rows, max_tiles, s);
  if (mode == MODE_TN && epi == EPI_DW) return launch_one<MODE_TN, EPI_DW, false, false>(g, tile_rows, max_tiles, s);
  return MOE_ERR_BAD_DTYPE;
}

template <int EPI1, bool CHAIN1, int BM1, int BM2>
static int launch_pair_bm(const GemmArgs& g1, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  // a multiple of the XCD count: a tile number still tells the XCD for the second GEMM
  const long long n1 = ((g1.N + SB - 1) / SB * (long long)max_tiles + NUM_XCD - 1) / NUM_XCD * NUM_XCD, n2 = dw_blocks(g2, BM2, SB);
  if (n1 + n2 > 0x7fffffffll) return MOE_ERR_BAD_SHAPE;
  gemm_f32_pair_kernel<EPI1, CHAIN1, BM1, BM2><<<dim3((unsigned)(n1 + n2)), 256, 0, s>>>(g1, g2, (int)n1);
  return launch_status();
}
template <int EPI1, bool CHAIN1>
static int launch_pair(const GemmArgs& g1, int tile_rows, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  const bool low1 = tile_rows != SB, low2 = dw_tile_rows(g2) != SB;
  if (low1) return low2 ? launch_pair_bm<EPI1, CHAIN1, SB / 2, SB / 2>(g1, max_tiles, g2, s) : launch_pair_bm<EPI1, CHAIN1, SB / 2, SB>(g1, max_tiles, g2, s);
  return low2 ? launch_pair_bm<EPI1, CHAIN1, SB, SB / 2>(g1, max_tiles, g2, s) : launch_pair_bm<EPI1, CHAIN1, SB, SB>(g1, max_tiles, g2, s);
}
int launch_gemm_f32_pair(int epi1, bool chain1, const GemmArgs& g1, int tile_rows, int max_tiles, const GemmArgs& g2, hipStream_t s) {
  if (epi1 == EPI_GELU_BWD) return launch_pair<EPI_GELU_BWD, false>(g1, tile_rows, max_tiles, g2, s);
  if (epi1 == EPI_SWIGLU_BWD) return launch_pair<EPI_SWIGLU_BWD, false>(g1, tile_rows, max_tiles, g2, s);
  if (epi1 == EPI_STORE && !chain1) return launch_pair<EPI_STORE, false>(g1, tile_rows, max_tiles, g2, s);
  if (epi1 == EPI_STORE && chain1) return launch_pair<EPI_STORE, true>(g1, tile_rows, max_tiles, g2, s);
  return MOE_ERR_BAD_DTYPE;
}

}  // namespace moe
