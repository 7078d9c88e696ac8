// Dispatch: stable group-by-expert of the T*k assignments and the row gather.
//
// The paper's dispatch all-to-all sends each token embedding to the GPU that holds the target
// expert (Section 2.1); on one GPU this is a permutation.  Order inside an expert is ascending
// token index, so the result is unique and the capacity cut ("first C of the list") is the
// stable rank itself.  Everything here is integer work and deterministic: per-block histograms,
// a scan over blocks, and an in-block stable rank built from wave ballots.
#include "common.h"
#include "prof.h"
#include "tile_map.h"
#include <mutex>

namespace moe {

constexpr int DP_THREADS = 1024;
constexpr int DP_WAVES = DP_THREADS / WAVE;
constexpr int DP_SUB = DP_WAVES;                         // 16 sub-chunks of 64 assignments, ascending
static_assert(DP_THREADS == DISPATCH_CHUNK, "one assignment per thread");
static_assert(MOE_MAX_E == 4 * WAVE, "the rank kernel scans the experts four per lane of one wave");

// The lanes of this wave with the same expert (those with a valid one): one ballot per bit of the id.  `bits`: how many
// bits the ids below E have.
__device__ __forceinline__ unsigned long long same_expert(int e, bool valid, int bits) {
  unsigned long long m = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b)
    if (b < bits) {
      const bool one = (e >> b) & 1;
      const unsigned long long v = __ballot(one);
      m &= one ? v : ~v;
    }
  return m;
}
__device__ __forceinline__ int id_bits(int E) { return 32 - __clz(E - 1); }   // E = 1: 0
// counts[e] += the number of lanes with expert e: one addition per expert present in the wave
__device__ __forceinline__ void count_wave(int* counts, int e, bool valid, int bits, int lane) {
  const unsigned long long m = same_expert(e, valid, bits);
  if (valid && __popcll(m & ((1ull << lane) - 1ull)) == 0) atomicAdd(&counts[e], __popcll(m));
}

__global__ __launch_bounds__(DP_THREADS) void dispatch_hist_kernel(const int32_t* __restrict__ topk_idx, int A, int E,
                                                                  int32_t* __restrict__ blk_cnt) {
  __shared__ int s_cnt[MOE_MAX_E];
  const int a = blockIdx.x * DISPATCH_CHUNK + threadIdx.x, e = a < A ? topk_idx[a] : -1;
  if (threadIdx.x < MOE_MAX_E) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  count_wave(s_cnt, e, e >= 0 && e < E, id_bits(E), threadIdx.x & (WAVE - 1));   // an id outside [0, E) is a dropped assignment
  __syncthreads();
  if (threadIdx.x < E) blk_cnt[(size_t)blockIdx.x * E + threadIdx.x] = s_cnt[threadIdx.x];
}

// Many blocks (more than DP_INLINE_SCAN): the per-block counts are turned into exclusive prefixes over the
// blocks once, in place, one thread per expert, and row nblk receives the totals; the rank kernel then reads
// two rows instead of scanning all of them (which would make the work quadratic in the number of blocks).
constexpr int DP_INLINE_SCAN = 64;
constexpr int DP_SCAN_THREADS = 64, DP_SCAN_BATCH = 32;   // counts in flight per thread
__global__ __launch_bounds__(DP_SCAN_THREADS) void dispatch_scan_kernel(int32_t* __restrict__ blk_cnt, int E, int nblk) {
  const int e = blockIdx.x * DP_SCAN_THREADS + threadIdx.x;
  if (e >= E) return;
  int run = 0;
  for (int b0 = 0; b0 < nblk; b0 += DP_SCAN_BATCH) {
    int c[DP_SCAN_BATCH];
#pragma unroll
    for (int u = 0; u < DP_SCAN_BATCH; ++u) c[u] = b0 + u < nblk ? blk_cnt[(size_t)(b0 + u) * E + e] : 0;
#pragma unroll
    for (int u = 0; u < DP_SCAN_BATCH; ++u) {
      if (b0 + u < nblk) blk_cnt[(size_t)(b0 + u) * E + e] = run;
      run += c[u];
    }
  }
  blk_cnt[(size_t)nblk * E + e] = run;
}

// Where the rank kernel finds the assignments of the other blocks: counts per block (dispatch_hist_kernel), exclusive
// prefixes and a row of totals (dispatch_scan_kernel), or, up to DP_SELF blocks, nowhere: it counts their ids itself.
// A short list is bound by its launches, not by its bytes: 4096 assignments take 4.3 us with the ids counted here (256 experts
// 6.0), 4097 with a histogram 5.9 (7.4); a block's counting grows by 0.3 (0.5) us per 1024, the launch it saves does not.
// One thread per assignment and one ballot per bit of the expert id.  Four assignments per thread and a pass of ballots per
// distinct expert (16 and fewer) or 64 comparisons before, us per call of index work, even ids | all on one expert:
// 1024 assignments, 8 experts 8.7 -> 3.3 | 5.4 -> 3.1, 16 experts 12.4 -> 3.3 | 5.4 -> 3.2, 256 experts 10.5 -> 4.1 | 11.6 -> 3.9; 16384,
// 8 experts 11.1 -> 6.0 | 8.1 -> 5.8; 65536, 256 experts 18.7 -> 9.3; 262144, 16 experts 56.7 -> 18.7 (the scan over blocks had
// one count in flight per thread).
enum RankFrom { FROM_COUNTS, FROM_PREFIXES, FROM_IDS };
constexpr int DP_SELF = 4;

template <RankFrom FROM>
__global__ __launch_bounds__(DP_THREADS) void dispatch_rank_kernel(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ blk_cnt, int A, int E, int capacity, int nblk,
    int32_t* __restrict__ counts, int32_t* __restrict__ kept, int32_t* __restrict__ offsets,
    int32_t* __restrict__ row_of, int32_t* __restrict__ src_of) {
  __shared__ int s_before[MOE_MAX_E];            // assignments of expert e in earlier blocks
  __shared__ int s_kept[MOE_MAX_E];
  __shared__ int s_off[MOE_MAX_E + 1];
  __shared__ int s_sub[DP_SUB][MOE_MAX_E];       // per sub-chunk counts, then exclusive offsets
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;

  // this block's assignments: loaded first, so that their latency runs beside the scan over blocks
  const int a = blockIdx.x * DISPATCH_CHUNK + tid, bits = id_bits(E);
  int my_e = a < A ? topk_idx[a] : -1;
  int id[FROM == FROM_IDS ? DP_SELF : 1];   // the other blocks' ids, all loads in flight together
  if constexpr (FROM == FROM_IDS) {
#pragma unroll
    for (int b = 0; b < DP_SELF; ++b) {
      const int o = b * DISPATCH_CHUNK + tid;
      id[b] = (b != (int)blockIdx.x && o < A) ? topk_idx[o] : -1;
    }
  }
  const bool valid = my_e >= 0 && my_e < E;   // past the end, or an id outside [0, E): dropped, never an index

  // the other blocks: s_before = assignments of e in earlier blocks, s_kept = all of them for now
  if (tid < MOE_MAX_E) { s_before[tid] = 0; s_kept[tid] = 0; }
  for (int i = tid; i < DP_SUB * E; i += DP_THREADS) s_sub[i / E][i % E] = 0;
  __syncthreads();
  if constexpr (FROM == FROM_IDS) {
    // s_before = assignments in earlier blocks, s_kept = those in later ones; the block's own are added below
#pragma unroll
    for (int b = 0; b < DP_SELF; ++b)
      if (b != (int)blockIdx.x && b * DISPATCH_CHUNK < A)
        count_wave(b < (int)blockIdx.x ? s_before : s_kept, id[b], id[b] >= 0 && id[b] < E, bits, lane);
  } else if constexpr (FROM == FROM_PREFIXES) {
    for (int e = tid; e < E; e += DP_THREADS)
      if (nblk > 0) { s_before[e] = blk_cnt[(size_t)blockIdx.x * E + e]; s_kept[e] = blk_cnt[(size_t)nblk * E + e]; }
  } else {
    // few blocks: every block adds up all nblk x E counts itself: all threads load, eight counts each in
    // flight; a thread walks the flat index i = b * E + e in steps of the block size, keeps sums in
    // registers while its expert stays the same (always, when E divides the block size) and adds them to
    // LDS when it changes (integer sums: the order of the additions does not matter)
    const int n = nblk * E;
    const int db = DP_THREADS / E, de = DP_THREADS % E;
    int b = tid / E, e = tid % E;
    int cur = e, tot = 0, bef = 0;
    for (int i0 = tid; i0 < n; i0 += DP_THREADS * 8) {
      int c[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u * DP_THREADS;
        c[u] = i < n ? blk_cnt[i] : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (e != cur) {
          if (tot != 0) atomicAdd(&s_kept[cur], tot);
          if (bef != 0) atomicAdd(&s_before[cur], bef);
          cur = e; tot = 0; bef = 0;
        }
        tot += c[u];
        bef += (b < (int)blockIdx.x) ? c[u] : 0;
        b += db;
        e += de;
        if (e >= E) { e -= E; ++b; }
      }
    }
    if (tot != 0) atomicAdd(&s_kept[cur], tot);
    if (bef != 0) atomicAdd(&s_before[cur], bef);
  }
  // rank among the lanes of this wave with the same expert, and the number of such lanes: one writer per (sub-chunk, expert)
  const unsigned long long same = same_expert(my_e, valid, bits);
  const int my_rank = __popcll(same & ((1ull << lane) - 1ull));
  if (valid && my_rank == 0) s_sub[wave][my_e] = __popcll(same);
  __syncthreads();
  if (tid < E) {
    int c[DP_SUB], run = s_before[tid];
#pragma unroll
    for (int sc = 0; sc < DP_SUB; ++sc) c[sc] = s_sub[sc][tid];
#pragma unroll
    for (int sc = 0; sc < DP_SUB; ++sc) { s_sub[sc][tid] = run; run += c[sc]; }
    if constexpr (FROM == FROM_IDS) s_kept[tid] += run;   // earlier, own and later blocks
  }
  __syncthreads();
  // kept counts and their exclusive scan over the experts: the first wave, four experts per lane
  if (wave == 0) {
    int m[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = lane * 4 + i;
      const int total = s_kept[e];
      m[i] = (capacity > 0) ? min(total, capacity) : total;
      if (blockIdx.x == 0 && e < E) { counts[e] = total; kept[e] = m[i]; }
      sum += m[i];
    }
    const int incl = wave_scan_i(sum);
    int run = incl - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = lane * 4 + i;
      s_kept[e] = m[i];
      s_off[e] = run;
      run += m[i];
    }
    if (lane == WAVE - 1) s_off[MOE_MAX_E] = run;
  }
  __syncthreads();
  // experts past E hold zero counts, so s_off[E] == s_off[MOE_MAX_E] == all kept rows
  if (blockIdx.x == 0)
    for (int e = tid; e <= E; e += DP_THREADS) offsets[e] = s_off[e];

  if (a >= A) return;
  int row = -1;
  if (valid) {
    const int rank = s_sub[wave][my_e] + my_rank;
    if (rank < s_kept[my_e]) { row = s_off[my_e] + rank; src_of[row] = a; }
  }
  row_of[a] = row;
  if (a >= s_off[E]) src_of[a] = -1;   // rows past the end of the kept lists
}

// x_perm[row_of[t*k+j]] = x[t] for the slots that are kept and inside this GPU's shares.  Token-major: a wave
// owns a token, reads its row once (16 bytes per lane, GU column chunks in flight) and writes it to the rows
// of its live slots, so the read traffic is the T*d elements the algorithm needs however large k is.  Every
// in-share row belongs to exactly one slot, so all of them are written and no other row is touched.
// The stores are non-temporal (x_perm is far larger than the caches and is read next by another kernel).
// The first `side_blocks` blocks build what the FFN needs beside the rows (tile_map.h).
constexpr int GU = 8;   // 16-byte column pieces per lane in flight: a row of 4096 16-bit elements in one pass
template <typename T, int KMAX>
__global__ __launch_bounds__(SIDE_THREADS) void dispatch_gather_kernel(
    const T* __restrict__ x, const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ row_of,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ kept, const int32_t* __restrict__ lo,
    const int32_t* __restrict__ hi, T* __restrict__ x_perm, int Tn, int d, int k, SideWork side, int side_blocks) {
  constexpr int VN = Vec16<T>::N;
  if ((int)blockIdx.x < side_blocks) return run_side_work(side, blockIdx.x);
  const int lane = threadIdx.x & (WAVE - 1);
  const int t = ((blockIdx.x - side_blocks) * SIDE_THREADS + threadIdx.x) / WAVE;
  if (t >= Tn) return;
  int rows[KMAX];
  bool any = false;
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    rows[j] = -1;
    if (j < k) {
      const int a = t * k + j, row = row_of[a];
      if (row >= 0) {
        bool mine = true;
        if (lo != nullptr) {   // with no shares given every kept row is ours: skip the expert lookup
          const int e = topk_idx[a];
          int l, h;
          share_of(lo, hi, kept[e], e, l, h);
          const int pos = row - offsets[e];
          mine = pos >= l && pos < h;
        }
        if (mine) { rows[j] = row; any = true; }
      }
    }
  }
  if (!any) return;
  const T* src = x + (size_t)t * d;
  for (int c0 = lane * VN; c0 < d; c0 += WAVE * VN * GU) {
    Vec16<T> v[GU];
#pragma unroll
    for (int u = 0; u < GU; ++u)
      if (c0 + u * WAVE * VN < d) v[u].load_nt(src + c0 + u * WAVE * VN);
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (rows[j] >= 0) {
#pragma unroll
        for (int u = 0; u < GU; ++u)
          if (c0 + u * WAVE * VN < d) v[u].store_nt(x_perm + (size_t)rows[j] * d + c0 + u * WAVE * VN);
      }
  }
}

// ---------------------------------------------------------------- dispatch without a caller workspace
// The per-block histograms of moe_dispatch_static live in this file-scope device array instead of the
// caller's workspace.  Every GPU the library runs on holds its own copy until the process ends.  In host
// code the array's name is only a handle: its device address is asked for once per device
// (hipGetSymbolAddress, with that device current) and kept; kernels and everything else get that pointer.
static __device__ __align__(256) int32_t scratch[MOE_DISPATCH_STATIC_BYTES / 4];

constexpr int MAX_DEVICES = 64;
static int32_t* g_scratch_ptr[MAX_DEVICES] = {};
static std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (MOE_ERR_HIP on failure).
int dispatch_static_scratch(int32_t** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_hip_error(e);
  if (dev < 0 || dev >= MAX_DEVICES) return MOE_ERR_BAD_SHAPE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return set_hip_error(e);
    if (p == nullptr) return set_hip_error(hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = g_scratch_ptr[dev];
  return MOE_OK;
}

int launch_dispatch(const moe_cfg* c, const void* x, const int32_t* idx, const int32_t* lo, const int32_t* hi,
                    int32_t* counts, int32_t* kept, int32_t* offsets, int32_t* row_of, int32_t* src_of, void* x_perm,
                    int32_t* blk_cnt, const SideWork* side, hipStream_t s) {
  const int A = c->T * c->k;
  const int nblk = (A + DISPATCH_CHUNK - 1) / DISPATCH_CHUNK;
  int rc = MOE_OK;
  if (nblk > DP_SELF) {
    dispatch_hist_kernel<<<nblk, DP_THREADS, 0, s>>>(idx, A, c->E, blk_cnt);
    rc = launch_status();
    if (rc != MOE_OK) return rc;
  }
  // with no assignments one block still writes the (all-zero) counts, kept and offsets
  if (nblk > DP_INLINE_SCAN) {
    dispatch_scan_kernel<<<(c->E + DP_SCAN_THREADS - 1) / DP_SCAN_THREADS, DP_SCAN_THREADS, 0, s>>>(blk_cnt, c->E, nblk);
    rc = launch_status();
    if (rc != MOE_OK) return rc;
    dispatch_rank_kernel<FROM_PREFIXES><<<nblk, DP_THREADS, 0, s>>>(idx, blk_cnt, A, c->E, c->capacity, nblk, counts, kept, offsets, row_of, src_of);
  } else if (nblk > DP_SELF) {
    dispatch_rank_kernel<FROM_COUNTS><<<nblk, DP_THREADS, 0, s>>>(idx, blk_cnt, A, c->E, c->capacity, nblk, counts, kept, offsets, row_of, src_of);
  } else {
    dispatch_rank_kernel<FROM_IDS><<<nblk > 0 ? nblk : 1, DP_THREADS, 0, s>>>(idx, blk_cnt, A, c->E, c->capacity, nblk, counts, kept, offsets, row_of, src_of);
  }
  rc = launch_status();
  if (rc != MOE_OK || x_perm == nullptr || A == 0) return rc;
  ProfScope ps(c, MOE_PROF_GATHER, s);
  const int sb = side != nullptr ? side->blocks() : 0, grid = sb + (c->T + SIDE_THREADS / WAVE - 1) / (SIDE_THREADS / WAVE);
  const SideWork sw = side != nullptr ? *side : SideWork{};
#define MOE_GATHER(TY, KM) \
  dispatch_gather_kernel<TY, KM><<<grid, SIDE_THREADS, 0, s>>>((const TY*)x, idx, row_of, offsets, kept, lo, hi, (TY*)x_perm, c->T, c->d_model, c->k, sw, sb)
  if (c->dtype == MOE_DTYPE_BF16) { if (c->k <= 2) MOE_GATHER(bf16, 2); else if (c->k <= 4) MOE_GATHER(bf16, 4); else MOE_GATHER(bf16, 8); }
  else if (c->dtype == MOE_DTYPE_F16) { if (c->k <= 2) MOE_GATHER(f16, 2); else if (c->k <= 4) MOE_GATHER(f16, 4); else MOE_GATHER(f16, 8); }
  else { if (c->k <= 2) MOE_GATHER(float, 2); else if (c->k <= 4) MOE_GATHER(float, 4); else MOE_GATHER(float, 8); }
#undef MOE_GATHER
  return launch_status();
}

}  // namespace moe
