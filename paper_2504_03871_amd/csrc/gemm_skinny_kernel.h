// Grouped x W (NN) for 16-bit storage where the experts have few rows each: decode batches and short prompts.
//
// Such a GEMM reads every weight once and does next to no arithmetic with it: HBM bounds it, and what counts is how
// many bytes each compute unit keeps in flight.  The 256-row kernel keeps one block per compute unit with one 32 KB
// stage of weights in flight and drains it at every stage; the 160-row one, with two, is ahead of this kernel in wide layers where it
// streams the weights and fills its rounds (few_rows_streamed).  Here a block owns 64 rows x 128 columns, four waves of 32
// columns each; its K stages of 64 go through a ring of LDS stages that buffer loads fill directly, all but one of
// them in flight, and two blocks share a compute unit: 64 KB of weights on their way per compute unit at any time.
// The weights of an expert with a single row tile are requested as streaming data; row tiles that share weights run
// together (skinny_block) and take them from the L2.  16 tokens, d 4096, f 14336, eight experts, top-2, SwiGLU: both GEMMs
// 606 us with the 256-row kernel (4.65 TB/s), 525 with this one at 64 columns and plain loads, 503 at 128 columns, 465
// at 64 columns with streaming loads, 452 as it is (6.2 TB/s); a third block per compute unit gains nothing.
#pragma once
#include "gemm_bf16_kernel.h"

namespace moe {

constexpr int SKINNY_BN = 128;
template <bool DUAL>
constexpr int skinny_stage_bytes() { return SKINNY_ROWS * BKT * 2 + SKINNY_BN * BKT * 2 * (DUAL ? 2 : 1); }
template <bool DUAL>
constexpr int skinny_stages() { return 80 * 1024 / skinny_stage_bytes<DUAL>(); }   // two blocks per compute unit

template <typename ST, int EPI, bool DUAL>
__global__ __launch_bounds__(256, 2) void gemm_skinny_kernel(GemmArgs g) {
  constexpr int BM = SKINNY_ROWS, BN = SKINNY_BN, A_BYTES = BM * BKT * 2, B_BYTES = BN * BKT * 2;
  constexpr int STAGE = skinny_stage_bytes<DUAL>(), NB = skinny_stages<DUAL>(), AHEAD = NB - 1;
  constexpr int TM = BM / 16, TN = BN / 64;                      // 16 x 16 tiles of a wave: all rows, BN / 4 columns
  constexpr int CHA = BM * BKT / 8 / 256, CHB = BN * BKT / 8 / 256, L = CHA + CHB * (DUAL ? 2 : 1);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int ntn = (g.N + BN - 1) / BN, n_rt = g.ntiles[0];
  constexpr bool CAN_SPLIT = EPI == EPI_STORE;
  const SkinnyOrder so = skinny_order(n_rt, g.ntiles[2] != 0, g.E, CAN_SPLIT && g.split_all);
  const int parts = 1 << so.shift;
  RowBlock rb;
  if (!skinny_block(blockIdx.x, so, ntn, rb)) return;
  const RowTile t = g.tiles[rb.rt];
  const bool shared = __builtin_amdgcn_readfirstlane(t.mates) != 0;
  const int stages = g.K / BKT, k0 = __builtin_amdgcn_readfirstlane((rb.ksplit * stages) >> so.shift), kbase = k0 * BKT;
  const int KT = __builtin_amdgcn_readfirstlane(((rb.ksplit + 1) * stages) >> so.shift) - k0;
  const int n0 = rb.nt * BN, mvalid = t.nrows, ni = (mvalid + 15) / 16;   // ni: row tiles with valid rows

  const rsrc_t ra = make_rsrc(reinterpret_cast<const bf16*>(g.A) + (size_t)t.row0 * g.K + kbase, ((size_t)mvalid * g.K - kbase) * 2);
  const size_t boff = ((size_t)t.e * g.K + kbase) * g.N + n0, bbytes = ((size_t)(g.K - kbase) * g.N - n0) * 2;
  const rsrc_t rw = make_rsrc(reinterpret_cast<const bf16*>(g.B) + boff, bbytes);
  const rsrc_t rw2 = make_rsrc(reinterpret_cast<const bf16*>(DUAL ? g.B2 : g.B) + boff, bbytes);
  const unsigned pa = g.K * 2, pb = g.N * 2;
  unsigned a_vo[CHA], b_vo[CHB];
#pragma unroll
  for (int i = 0; i < CHA; ++i) {
    const int id = tid + 256 * i, r = id >> 3;
    a_vo[i] = (unsigned)r * pa + (unsigned)((id & 7) ^ ((r >> 1) & 7)) * 16u;   // kc_off, inverted
  }
#pragma unroll
  for (int i = 0; i < CHB; ++i) {
    const int id = tid + 256 * i, r = id / (BN / 8), pc = id % (BN / 8);
    b_vo[i] = (unsigned)r * pb + (unsigned)(ks_off<BN>(r, pc * 16) - r * BN * 2);   // ks_off, inverted
  }
  const unsigned lds0 = lds_addr(smem) + wave * 1024;
  auto load_stage = [&](int kt, int buf) {
    const unsigned at = lds0 + buf * STAGE;
    if (shared) {
#pragma unroll
      for (int i = 0; i < CHB; ++i) {
        load_to_lds16(rw, at + A_BYTES + i * 4096, b_vo[i] + kt * (BKT * pb));
        if constexpr (DUAL) load_to_lds16(rw2, at + A_BYTES + B_BYTES + i * 4096, b_vo[i] + kt * (BKT * pb));
      }
    } else {
#pragma unroll
      for (int i = 0; i < CHB; ++i) {
        load_to_lds16_nt(rw, at + A_BYTES + i * 4096, b_vo[i] + kt * (BKT * pb));
        if constexpr (DUAL) load_to_lds16_nt(rw2, at + A_BYTES + B_BYTES + i * 4096, b_vo[i] + kt * (BKT * pb));
      }
    }
#pragma unroll
    for (int i = 0; i < CHA; ++i) load_to_lds16(ra, at + i * 4096, a_vo[i] + kt * (BKT * 2));
  };

  f32x4 acc[TM][TN], acc2[DUAL ? TM : 1][DUAL ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (DUAL) acc2[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  int b_fr[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_fr[j] = A_BYTES + ks_off<BN>(grp * 8 + (c >> 2), (wave * (BN / 4) + j * 16 + (c & 3) * 4) * 2);

#pragma unroll
  for (int q = 0; q < AHEAD; ++q)
    if (q < KT) load_stage(q, q);
  int buf = 0;
#pragma unroll 1
  for (int kt = 0; kt < KT; ++kt) {
    // own loads of this stage have landed (later stages stay in flight) and own reads of the last one are done; behind
    // the barrier that holds for every wave, and the last stage's buffer is free
    constexpr int PEND = (AHEAD - 1) * L;
    static_assert(PEND < 16, "low bits of the wait counter");
    if (kt + AHEAD <= KT) __builtin_amdgcn_s_waitcnt(PEND | 0x70); else __builtin_amdgcn_s_waitcnt(0x70);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + AHEAD < KT) load_stage(kt + AHEAD, buf + AHEAD >= NB ? buf + AHEAD - NB : buf + AHEAD);
    const char* st = smem + buf * STAGE;
#pragma unroll
    for (int ks = 0; ks < BKT / 32; ++ks) {
      bf16x8 b[TN], b2[DUAL ? TN : 1];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const char* p = st + b_fr[j] + ks * 32 * BN * 2;
        b[j] = lds_read_ks2<BN>(p);
        if constexpr (DUAL) b2[j] = lds_read_ks2<BN>(p + B_BYTES);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
        if (i < ni) {
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(st + kc_off(i * 16 + c, ks * 4 + grp));
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc[i][j] = Half16<ST>::mfma(b[j], a, acc[i][j]);
            if constexpr (DUAL) acc2[i][j] = Half16<ST>::mfma(b2[j], a, acc2[i][j]);
          }
        }
    }
    buf = buf + 1 == NB ? 0 : buf + 1;
  }

  // Epilogue straight from the accumulators (layout: gemm_bf16_kernel.h); a wave's 32 columns are all valid or none is
  static_assert(TN == 2, "one pair of column tiles per wave");
  const int c0 = wave * (BN / 4);
  if (n0 + c0 >= g.N) return;
  if (CAN_SPLIT && rb.split_tile >= 0) {   // fp32 partial sums of this block's K part
    const int r8 = lane & 7, right = (lane >> 3) & 1;
    float* sums = g.split_ws + ((size_t)rb.split_tile * parts + rb.ksplit) * SKINNY_ROWS * g.N + n0 + c0 + right * 16 + grp * 4;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if (i < ni) {
        swap8(acc[i][0], acc[i][1]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int m = i * 16 + h * 8 + r8;
          if (m < mvalid) *reinterpret_cast<f32x4*>(sums + (size_t)m * g.N) = acc[i][h];
        }
      }
    return;
  }
  const OutPlanes o = out_planes<ST, EPI>(g, (size_t)t.row0 * g.N + n0, ((size_t)mvalid * g.N - n0) * 2);
#pragma unroll
  for (int i = 0; i < TM; ++i)
    if (i < ni) {
      const int m = i * 16 + c;
      const unsigned off[1] = {m < mvalid ? ((unsigned)m * g.N + c0 + lane_col8(grp)) * 2u : OUT_OF_RANGE};
      epilogue_fwd<ST, EPI, 1, 0>(o, off, acc[i], acc2[DUAL ? i : 0], g.gelu_tab);
    }
}

}  // namespace moe
