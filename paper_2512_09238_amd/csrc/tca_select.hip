// Online core-context selection and compaction (Alg. 2 lines 1-6; Eq. 5-8).
//
// Three kernels, K is read from HBM exactly once and logits never leave the chip:
//   score_kernel  : one workgroup per (KV head, block of b tokens).  Streams the
//                   block's K rows with 16-byte loads, forms the logits of all G
//                   query heads of the group in fp64 (Eq. 5 numerator), reduces
//                   them to the block statistics max / sum e^x / sum e^2x that
//                   Eq. 6 needs, and emits one 64-bit ranking key per (head,
//                   token).  The rank of a token inside its block does not depend
//                   on the budget, so Eq. 8 becomes "rank < t_j" later.  For
//                   calibration (ranks reused by every candidate) the kernel also
//                   ranks and writes 1 byte per (head, token); for selection the
//                   ranking is left to gather_kernel, which is bound by HBM and
//                   has the vector ALU to spare.
//   assign_kernel : one workgroup per head (one to sixteen waves).  Global softmax normaliser,
//                   h_j (Eq. 6), rank of every block, t_j = Psi[rank] (Eq. 7),
//                   exclusive scan of t_j -> destination row of every block.
//   gather_kernel : one workgroup per (head, block).  Ranks the block's tokens by
//                   counting over their keys (skipped when t_j = b), keeps those
//                   with rank < t_j in position order and copies their K/V rows
//                  and positions into the head's flat region (App. C).  With
//                   few blocks its waves assign the budgets themselves, and
//                   assign_kernel is not launched.
// When the query heads of a group share one selection (an extension for GQA), the
// scores of the group's heads have to be normalised before they can be averaged:
// score_kernel then leaves the fp64 logits in the workspace, group_lse_kernel turns
// the per-head block statistics into each head's normaliser, and group_score_kernel
// merges the G logits of a token into one log-domain score and produces the block
// statistics and ranking keys of that score; assign and gather run once per KV head.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tca_common.h"
#include "tca_device.h"
#include "tca_select.h"

namespace tca {

constexpr int kScoreThreads = 256;
constexpr int kGatherThreads = 256;
constexpr int kGatherRows = 2;        // rows per thread in flight in the copy loop (4 measured the same)
constexpr int kHeadsPerLaunch = 32;
// Blocks, the tail included, that a wave holds one to a lane: up to there the launches between the scores and the copy, which
// are all latency, go into the kernels behind them.  us of the kernels behind the scores, with launches of their own and without:
// 1024 tokens of 4 heads (32 blocks of 32) 10.5 / 6.7; 413 of 32 heads 12.3 / 8.0; 5446 of a shared selection 28.0 / 20.1.
constexpr int kFewBlocks = 64;
constexpr int kBlockStats = 4;        // doubles per (head, block) in SelectWs::stats

// the group's query heads are merged into one score only when there is more than one of them
static bool grouped(const tca_params* prm) { return sel_group(prm) > 1; }

SelectWs carve_select_ws(void* ws, const tca_params* prm, int64_t n_tokens) {
  const int Hq = prm->n_q_heads, Hs = sel_heads(prm), b = prm->block;
  int64_t nb = n_tokens / b, nbt = (n_tokens + b - 1) / b;
  size_t off = 0;
  SelectWs w;
  char* base = (char*)ws;
  w.tokrank = (uint8_t*)(base + off); off = align_up(off + (size_t)Hs * nb * b, 256);
  w.keys = (uint64_t*)(base + off);   off = align_up(off + (size_t)Hs * nb * b * sizeof(uint64_t), 256);
  w.stats = (double*)(base + off);    off = align_up(off + (size_t)Hq * nbt * kBlockStats * sizeof(double), 256);
  w.sel_stats = w.stats;
  w.xlog = nullptr;
  w.lse = nullptr;
  if (grouped(prm)) {
    w.sel_stats = (double*)(base + off); off = align_up(off + (size_t)Hs * nbt * kBlockStats * sizeof(double), 256);
    w.xlog = (double*)(base + off);      off = align_up(off + (size_t)Hq * nbt * b * sizeof(double), 256);
    w.lse = (double*)(base + off);       off = align_up(off + (size_t)Hq * sizeof(double), 256);
  }
  w.blk_t = (int32_t*)(base + off);   off = align_up(off + (size_t)Hs * nb * sizeof(int32_t), 256);
  w.blk_dst = (int32_t*)(base + off); off = align_up(off + (size_t)Hs * nb * sizeof(int32_t), 256);
  w.bytes = off;
  return w;
}

// ---------------------------------------------------------------- scoring --
// Monotone map of a double to an unsigned 64-bit key (larger value -> larger key).
__device__ __forceinline__ uint64_t ordered_key(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Number of keys of a block that beat key ki (higher logit, or the same logit at a lower
// position): the rank of its token.  keys: b 64-bit keys in LDS, 16-byte aligned.
__device__ __forceinline__ int count_greater(const uint64_t* keys, int o_begin, int o_end, uint64_t ki) {
  int cnt = 0;
  for (int o = o_begin; o < o_end; o += 2) {
    const ulonglong2 ko = *reinterpret_cast<const ulonglong2*>(&keys[o]);
    cnt += (ko.x > ki);
    cnt += (ko.y > ki);
  }
  return cnt;
}

// What score_kernel leaves behind besides the block statistics.
constexpr int kEmitKeys = 0;      // ranking keys (selection)
constexpr int kEmitRanks = 1;     // in-block ranks (calibration: reused by every candidate)
constexpr int kEmitLogits = 2;    // the fp64 logits, tail block included (shared selection: merged by group_score_kernel)

// Key that orders the tokens of a block: the ordered image of the score with its 8
// lowest mantissa bits replaced by 255 - position, so that one unsigned compare
// decides "higher score, or the same score at a lower position".  Scores that agree
// in all but those bits (relative distance below 2^-44) count as tied.
__device__ __forceinline__ uint64_t ranking_key(double x, int i) {
  return (ordered_key(x) & ~0xFFull) | (uint64_t)(255 - i);
}

// grid (nbt, Hkv); block 256.  T storage type, D head dim, G query heads per KV head.
template <typename T, int D, int G, int EMIT>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(
    const T* __restrict__ K, const T* __restrict__ q_last, int64_t kv_stride, int64_t pos0,
    int64_t n_tokens, int b, int64_t n_blocks, int64_t nbt, int Hq, double scale,
    uint8_t* __restrict__ tokrank, uint64_t* __restrict__ keys_out, double* __restrict__ stats,
    double* __restrict__ xlog, const int32_t* __restrict__ n_rows, int32_t* __restrict__ fill) {
  constexpr bool RANK = EMIT == kEmitRanks;
  constexpr int EPL = Vec16<T>::N;            // elements per lane per load
  constexpr int LPR = D / EPL;                // lanes per row
  constexpr int RPW = kWave / LPR;            // rows per wave per load
  constexpr int RPI = RPW * (kScoreThreads / kWave);   // rows per workgroup iteration
  constexpr int UNR = 2;                      // 16-byte row loads in flight per lane (more costs occupancy: measured best)
  using GR = GroupReduce<G, LPR>;
  constexpr int GP = GR::GP;
  static_assert(GP <= LPR, "more heads than lanes per row");
  __shared__ double xs[G][256];
  __shared__ __attribute__((aligned(16))) uint64_t keys[G][256];

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t j = blockIdx.x;
  const int kvh = blockIdx.y;
  const int sub = lane % LPR, rsub = lane / LPR;
  if (EMIT == kEmitKeys && fill && j == 0 && tid < G) fill[kvh * G + tid] = n_rows[kvh * G + tid];       // as group_score_kernel

  double qv[GP][EPL];
#pragma unroll
  for (int g = 0; g < GP; ++g) {
    float tmp[EPL];
    if (g < G) Vec16<T>::load(q_last + (size_t)(kvh * G + g) * D + sub * EPL, tmp);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qv[g][e] = g < G ? (double)tmp[e] : 0.0;
  }

  const T* Kb = K + ((size_t)kvh * kv_stride + pos0 + j * b) * D;
  const int64_t left = n_tokens - j * b;                  // tokens from the block start to the end
  const int rows_here = left < b ? (int)left : b;
  const int my_head = GR::head_of(sub);
  const bool writer = my_head < G && (sub & (LPR / GP - 1)) == 0;   // one lane per head holds the row's total
  for (int r0 = 0; r0 < b; r0 += RPI * UNR) {
    raw16_t raw[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int r = r0 + u * RPI + wv * RPW + rsub;
      if (r < rows_here) raw[u] = load_raw16(Kb + (size_t)r * D + sub * EPL);
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int r = r0 + u * RPI + wv * RPW + rsub;
      const bool ok = r < rows_here;
      double acc[GP];
#pragma unroll
      for (int g = 0; g < GP; ++g) acc[g] = 0.0;
      if (ok) {
        float kv[EPL];
        widen_raw16<T>(raw[u], kv);
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const double kd = (double)kv[e];
#pragma unroll
          for (int g = 0; g < GP; ++g)
            if (g < G) acc[g] = fma(kd, qv[g][e], acc[g]);
        }
      }
      const double v = GR::run(acc, sub);
      if (writer && r < b) xs[my_head][r] = ok ? v * scale : -INFINITY;
    }
  }
  __syncthreads();

  // block statistics: one wave per head
  for (int g = wv; g < G; g += kScoreThreads / kWave) {
    double mx = -INFINITY;
    for (int i = lane; i < b; i += kWave) mx = fmax(mx, xs[g][i]);
    mx = wave_max(mx);
    double e1 = 0.0, e2 = 0.0, e3 = 0.0;
    for (int i = lane; i < b; i += kWave) {
      const double dx = xs[g][i] - mx;
      const double e = exp(dx);
      e1 += e;
      e2 += e * e;
      if (e > 0.0) e3 += e * dx;                         // 0 * (-inf) counts as 0
    }
    e1 = wave_sum(e1);
    e2 = wave_sum(e2);
    e3 = wave_sum(e3);
    if (lane == 0) {
      double* st = stats + ((size_t)(kvh * G + g) * nbt + j) * kBlockStats;
      st[0] = mx; st[1] = e1; st[2] = e2; st[3] = e3;
    }
  }
  if constexpr (EMIT == kEmitLogits) {
    for (int pi = tid; pi < G * b; pi += kScoreThreads) {
      const int g = pi / b, i = pi - g * b;
      xlog[((size_t)(kvh * G + g) * nbt + j) * b + i] = xs[g][i];          // -inf past the end of the tail
    }
    return;
  }
  if (j >= n_blocks) return;             // the tail block only feeds the normaliser

  // Rank inside the block = number of tokens that beat token i (higher logit, or
  // the same logit at a lower position): one unsigned compare of ranking keys per pair.
  for (int pi = tid; pi < G * b; pi += kScoreThreads) {
    const int g = pi / b, i = pi - g * b;
    const uint64_t key = ranking_key(xs[g][i], i);
    if constexpr (RANK) keys[g][i] = key;
    else keys_out[(size_t)(kvh * G + g) * (n_blocks * b) + j * b + i] = key;
  }
  if constexpr (RANK) {
    __syncthreads();
    for (int pi = tid; pi < G * b; pi += kScoreThreads) {
      const int g = pi / b, i = pi - g * b;
      tokrank[(size_t)(kvh * G + g) * (n_blocks * b) + j * b + i] = (uint8_t)count_greater(keys[g], 0, b, keys[g][i]);
    }
  }
}

// ----------------------------------------------------------- group score --
// Shared selection: the score of a token is the mean over the group's query heads of their
// Eq. 5 scores, sbar_i = (1/G) sum_g exp(x_gi - lse_g).  It is carried in the log domain,
// y_i = ln sum_g exp(x_gi - lse_g) = ln(G sbar_i), so that the block statistics, ranking keys,
// Eq. 6 and Eq. 7 of the per-head path apply to y unchanged (the factor G cancels in the
// normalised block mass and in both concentration indices).

// grid (Hq); block 256.  lse[h] = ln sum_i e^{x_hi} from the block statistics (tail included).
__global__ __launch_bounds__(256) void group_lse_kernel(const double* __restrict__ stats, int nbt,
                                                        double* __restrict__ lse) {
  __shared__ double red[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const double* st = stats + (size_t)blockIdx.x * nbt * kBlockStats;
  double mx = -INFINITY;
  for (int j = tid; j < nbt; j += 256) mx = fmax(mx, st[(size_t)j * kBlockStats]);
  mx = wave_max(mx);
  if (lane == 0) red[wv] = mx;
  __syncthreads();
  mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  __syncthreads();
  double z = 0.0;
  for (int j = tid; j < nbt; j += 256) z += st[(size_t)j * kBlockStats + 1] * exp(st[(size_t)j * kBlockStats] - mx);
  z = wave_sum(z);
  if (lane == 0) red[wv] = z;
  __syncthreads();
  if (tid == 0) lse[blockIdx.x] = mx + log((red[0] + red[1]) + (red[2] + red[3]));
}

// grid (nbt, Hkv); block 256: thread i owns token i of the block.
// lse == NULL (up to kFewBlocks blocks): the workgroup forms the normalisers of its heads itself, a wave a head and a lane a
// block, the same sums as group_lse_kernel's.  fill != NULL: n_rows as it is before this selection, for gather_kernel.
template <int G, bool RANK>
__global__ __launch_bounds__(256) void group_score_kernel(
    const double* __restrict__ xlog, const double* __restrict__ lse, const double* __restrict__ stats, int b, int64_t n_blocks,
    int64_t nbt, uint8_t* __restrict__ tokrank, uint64_t* __restrict__ keys_out, double* __restrict__ gstats,
    const int32_t* __restrict__ n_rows, int32_t* __restrict__ fill) {
  __shared__ double red[4][3];
  __shared__ double norm[G];
  __shared__ __attribute__((aligned(16))) uint64_t keys[256];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t j = blockIdx.x;
  const int kvh = blockIdx.y;
  if (fill && j == 0 && tid == 0) fill[kvh] = n_rows[kvh];
  double a[G];
#pragma unroll
  for (int g = 0; g < G; ++g) a[g] = tid < b ? xlog[((size_t)(kvh * G + g) * nbt + j) * b + tid] : 0.0;
  if (!lse) {
    for (int g = wv; g < G; g += 4) {
      const double* st = stats + ((size_t)(kvh * G + g) * nbt + lane) * kBlockStats;
      const double bM = lane < nbt ? st[0] : -INFINITY, bE = lane < nbt ? st[1] : 0.0;
      const double mx = wave_max(fmax(-INFINITY, bM));
      const double z = wave_sum(lane < nbt ? bE * exp(bM - mx) : 0.0);
      if (lane == 0) norm[g] = mx + log(z);
    }
    __syncthreads();
  }
  double y = -INFINITY;
  if (tid < b) {
    double top = -INFINITY;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      a[g] -= lse ? lse[kvh * G + g] : norm[g];
      top = fmax(top, a[g]);
    }
    if (top > -INFINITY) {                                 // a token past the end of the tail stays at -inf
      double sum = 0.0;
#pragma unroll
      for (int g = 0; g < G; ++g) sum += exp(a[g] - top);
      y = top + log(sum);
    }
  }
  double mx = wave_max(y);
  if (lane == 0) red[wv][0] = mx;
  __syncthreads();
  mx = fmax(fmax(red[0][0], red[1][0]), fmax(red[2][0], red[3][0]));
  __syncthreads();
  const double dx = y - mx;
  const double e = y > -INFINITY ? exp(dx) : 0.0;
  const double e1 = wave_sum(e), e2 = wave_sum(e * e);
  const double e3 = wave_sum(e > 0.0 ? e * dx : 0.0);
  if (lane == 0) { red[wv][0] = e1; red[wv][1] = e2; red[wv][2] = e3; }
  __syncthreads();
  if (tid == 0) {
    double* st = gstats + ((size_t)kvh * nbt + j) * kBlockStats;
    st[0] = mx;
    st[1] = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
    st[2] = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
    st[3] = (red[0][2] + red[1][2]) + (red[2][2] + red[3][2]);
  }
  if (j >= n_blocks) return;
  const uint64_t key = ranking_key(y, tid);
  if constexpr (RANK) {
    if (tid < b) keys[tid] = key;
    __syncthreads();
    if (tid < b) tokrank[(size_t)kvh * (n_blocks * b) + j * b + tid] = (uint8_t)count_greater(keys, 0, b, key);
  } else {
    if (tid < b) keys_out[(size_t)kvh * (n_blocks * b) + j * b + tid] = key;
  }
}

// ----------------------------------------------------------------- assign --
struct AssignArgs {
  int32_t cum[kHeadsPerLaunch][TCA_MAX_COUNTS];   // cumulative Psi counts: rank < cum[e] -> budget 2^e
  int64_t cap[kHeadsPerLaunch];                   // capacity of the head's region
};

// max / sum over the NT threads of the workgroup, result in every thread; red: one double per wave
template <int NT, bool MAX>
__device__ __forceinline__ double block_reduce(double v, double* red) {
  v = MAX ? wave_max(v) : wave_sum(v);
  if constexpr (NT > kWave) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    v = red[0];
    for (int i = 1; i < NT / kWave; ++i) v = MAX ? fmax(v, red[i]) : v + red[i];
  }
  return v;
}

// Eq. 6: h of a block from its mass in the whole and its statistics (s2: the one that the chosen index needs).  HHI of the
// block, or the entropy of the scores renormalised inside it: t_i = e_i / E1  =>  -sum t_i ln t_i = ln E1 - (sum e_i (x_i - M)) / E1
// A row that is not finite makes every h of its head NaN.  Both sides of a pair decide for themselves in the sort, which
// leaves the blocks a permutation only in a total order: NaN takes the last place, ties by block as ever.
__device__ __forceinline__ double block_index(double mass, double e1, double s2, int b, double alpha, int metric) {
  const double spread = metric == TCA_METRIC_ENTROPY ? (log(e1) - s2 / e1) / log((double)b) : 1.0 - s2 / (e1 * e1);
  const double hj = (1.0 - alpha) * mass + alpha * spread;
  return hj == hj ? hj : INFINITY;
}

// does (ha, ja) come after (hb, jb) in the order: ascending h, ties by lower block
__device__ __forceinline__ bool comes_after(double ha, int ja, double hb, int jb) { return ha > hb || (ha == hb && ja > jb); }

// grid (heads in this launch, or, heads_each > 0, configurations in this launch x heads_each heads that share one); block NT, R
// blocks per thread, m <= NT * R.  Everything is latency: the sort keeps its
// pairs in registers, exchanges at distances below 64 are lane shuffles, those between waves go through LDS
// (barriers), those at NT and beyond stay inside the thread.
template <int NT, int R>
__global__ __launch_bounds__(NT) void assign_kernel(
    AssignArgs args, int head0, int heads_each, int nk, int m, int nbt, int b, double alpha, int metric,
    const double* __restrict__ stats, int32_t* __restrict__ n_rows,
    int32_t* __restrict__ blk_t, int32_t* __restrict__ blk_dst) {
  constexpr int P = NT * R;
  __shared__ double hs[NT > kWave ? P : 1];
  __shared__ uint16_t js[NT > kWave ? P : 1];
  __shared__ uint16_t ts[P];
  __shared__ double red[NT / kWave];
  __shared__ int32_t wave_sum[NT / kWave];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int h = head0 + blockIdx.x, hl = heads_each ? blockIdx.x / heads_each : blockIdx.x;
  const double* st = stats + (size_t)(heads_each ? h % heads_each : h) * nbt * kBlockStats;
  const int32_t fill = n_rows[h];

  // the statistics of this thread's blocks (block j = tid + k * NT, tail block included), read once
  constexpr int KMAX = R + 1;
  double bM[KMAX], bE1[KMAX], bE2[KMAX];              // bE2: the statistic the chosen index needs
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    const int j = tid + k * NT;
    const bool in = j < nbt;
    bM[k] = in ? st[j * kBlockStats] : -INFINITY;
    bE1[k] = in ? st[j * kBlockStats + 1] : 0.0;
    bE2[k] = in ? st[j * kBlockStats + (metric == TCA_METRIC_ENTROPY ? 3 : 2)] : 0.0;
  }
  // global normaliser of Eq. 5 over every scored token, tail included
  double mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) mx = fmax(mx, bM[k]);
  mx = block_reduce<NT, true>(mx, red);
  double z = 0.0;
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    bM[k] = tid + k * NT < nbt ? bE1[k] * exp(bM[k] - mx) : 0.0;   // block mass before normalisation
    z += bM[k];
  }
  z = block_reduce<NT, false>(z, red);

  // Eq. 6
  double key[R];
  int blk[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int j = tid + k * NT;
    key[k] = INFINITY;                                 // padding sorts last
    blk[k] = j;
    // (the wave's test is a branch; its lanes' own becomes a selection, and waves without a block made the divisions and logarithms of
    // all: 281 blocks 16.5 us, now 14.4, 313 of 32 heads 17.5 / 15.2)
    if (__builtin_amdgcn_readfirstlane(j) < m) {
      const double hj = block_index(bM[k] / z, bE1[k], bE2[k], b, alpha, metric);
      if (j < m) key[k] = hj;
    }
  }

  // order the blocks by ascending h (ties: lower block first) with a bitonic sort of (h, block) pairs,
  // then Eq. 7: the block at sorted position r gets Psi[r].  Element e = tid + k * NT.
  int top = 2;
  while (top < m) top <<= 1;                           // what lies beyond is padding, in order already
  for (int kk = 2; kk <= top; kk <<= 1) {
    for (int jj = kk >> 1; jj > 0; jj >>= 1) {
      if (jj >= NT) {
        if constexpr (R > 1) {
          const int dr = jj / NT;
#pragma unroll
          for (int k = 0; k < R; ++k) {
#pragma unroll
            for (int d = 1; d < R; d <<= 1) {          // partners k and k + d, d known to the compiler
              if (d == dr && (k & d) == 0 && k + d < R) {
                const bool ascending = ((tid + k * NT) & kk) == 0;
                if (comes_after(key[k], blk[k], key[k + d], blk[k + d]) == ascending) {
                  const double tk = key[k]; key[k] = key[k + d]; key[k + d] = tk;
                  const int tb = blk[k]; blk[k] = blk[k + d]; blk[k + d] = tb;
                }
              }
            }
          }
        }
      } else if (jj >= kWave) {
        if constexpr (NT > kWave) {
          __syncthreads();                             // the exchange before has been read
#pragma unroll
          for (int k = 0; k < R; ++k) { hs[tid + k * NT] = key[k]; js[tid + k * NT] = (uint16_t)blk[k]; }
          __syncthreads();
#pragma unroll
          for (int k = 0; k < R; ++k) {
            const int e = tid + k * NT, pr = e ^ jj;
            const double ho = hs[pr];
            const int jo = js[pr];
            const bool lower = (e & jj) == 0, ascending = (e & kk) == 0;
            // the lower element of an ascending pair keeps the smaller
            if (comes_after(key[k], blk[k], ho, jo) == (lower == ascending)) { key[k] = ho; blk[k] = jo; }
          }
        }
      } else {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int e = tid + k * NT;
          const double ho = __shfl_xor(key[k], jj, kWave);
          const int jo = __shfl_xor(blk[k], jj, kWave);
          const bool lower = (e & jj) == 0, ascending = (e & kk) == 0;
          if (comes_after(key[k], blk[k], ho, jo) == (lower == ascending)) { key[k] = ho; blk[k] = jo; }
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = tid + k * NT;
    if (r < m) {
      int e = 0;
      while (e < nk - 1 && r >= args.cum[hl][e]) ++e;
      ts[blk[k]] = (uint16_t)(1 << e);
    }
  }
  __syncthreads();

  // exclusive scan of t_j in block order: thread t owns blocks t * R .. t * R + R - 1
  int own[R], local = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    own[k] = tid * R + k < m ? ts[tid * R + k] : 0;
    local += own[k];
  }
  int incl = local;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int v = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += v;
  }
  if (lane == kWave - 1) wave_sum[wv] = incl;
  __syncthreads();
  int before = 0, all = 0;
  for (int i = 0; i < NT / kWave; ++i) {
    if (i < wv) before += wave_sum[i];
    all += wave_sum[i];
  }
  int run = fill + before + incl - local;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int j = tid * R + k;
    if (j < m) {
      blk_t[(size_t)h * m + j] = own[k];
      blk_dst[(size_t)h * m + j] = run;
      run += own[k];
    }
  }
  if (tid == 0) {
    const int64_t total = (int64_t)fill + all;
    n_rows[h] = (int32_t)(total > args.cap[hl] ? args.cap[hl] : total);
  }
}

// ----------------------------------------------------------------- gather --
// offsets of the heads' regions travel in the kernel's argument block: no copy, no extra launch
struct OffsArgs { int64_t offs[TCA_MAX_HEADS + 1]; };
struct NoFew {};
struct FewArgs {                                 // assign_kernel's, for up to kFewBlocks blocks
  uint64_t cum[TCA_MAX_HEADS];                   // byte i: how many blocks get 2^i tokens or fewer
  int nk, nbt, metric;
  double alpha;
  const double* stats;
  const int32_t* fill;                           // n_rows as it was
  int32_t* n_rows;
};

// grid (n_blocks * selection heads); block 256.  G: selection heads per KV head.
// Workgroup ids go round-robin over the 8 XCDs.  The G selection heads of a KV head keep
// overlapping subsets of the same block's rows, so their workgroups are given ids 8 apart:
// same XCD, consecutive in time, and the rows a later one needs are mostly in that L2 already.
// FEW: every wave assigns its head's budgets for itself (the waves of a workgroup run side by side, which costs less than
// sharing), a lane a block: the sums as assign_kernel forms them, a block's place by counting the blocks that precede it.
template <typename T, int D, bool FEW>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(
    const T* __restrict__ K, const T* __restrict__ V, int64_t kv_stride, int64_t pos0, int b,
    int64_t n_blocks, int G, const uint64_t* __restrict__ keys,
    const int32_t* __restrict__ blk_t, const int32_t* __restrict__ blk_dst,
    OffsArgs oa, int32_t* __restrict__ idx, T* __restrict__ Kg, T* __restrict__ Vg, std::conditional_t<FEW, FewArgs, NoFew> few) {
  constexpr int EPL = Vec16<T>::N;
  constexpr int LPR = D / EPL;
  constexpr int RPI = kGatherThreads / LPR;
  __shared__ int32_t sel[256];
  __shared__ int32_t wave_cnt[kGatherThreads / kWave];
  __shared__ __attribute__((aligned(16))) uint64_t bkeys[256];
  __shared__ int32_t rank[256];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int64_t j;
  int h, kvh;
  {
    const int64_t id = blockIdx.x, pairs = (int64_t)gridDim.x / G;       // pairs = n_blocks * KV heads
    if ((pairs & 7) == 0) {
      const int64_t u = id >> 3;                                         // position in the XCD's own sequence
      const int64_t pair = (u / G) * 8 + (id & 7);
      kvh = (int)(pair / n_blocks);
      j = pair - (int64_t)kvh * n_blocks;
      h = kvh * G + (int)(u % G);
    } else {
      h = (int)(id / n_blocks);
      j = id - (int64_t)h * n_blocks;
      kvh = h / G;
    }
  }
  const int64_t base = oa.offs[h], cap = oa.offs[h + 1] - base;
  int t;
  int64_t dst0;
  uint64_t my_key = 0;
  if constexpr (FEW) {
    const double* st = few.stats + ((size_t)h * few.nbt + lane) * kBlockStats;
    const bool in = lane < few.nbt;
    const double bM = in ? st[0] : -INFINITY, bE1 = in ? st[1] : 0.0, bE2 = in ? st[few.metric == TCA_METRIC_ENTROPY ? 3 : 2] : 0.0;
    const int32_t fill = few.fill[h];
    if (tid < b) my_key = keys[(size_t)h * (n_blocks * b) + j * b + tid];
    const double mx = wave_max(fmax(-INFINITY, bM));
    const double own = in ? bE1 * exp(bM - mx) : 0.0, z = wave_sum(own);
    const int m = (int)n_blocks;
    const double hj = lane < m ? block_index(own / z, bE1, bE2, b, few.alpha, few.metric) : INFINITY;
    int r = 0;
    for (int i = 0; i < m; ++i) {
      const double hi = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(hj), i), __builtin_amdgcn_readlane(__double2loint(hj), i));
      r += comes_after(hj, lane, hi, i);
    }
    const uint64_t cum = few.cum[h];
    int e = 0, before = 0, all = 0;
    for (int i = 0; i < few.nk - 1; ++i) e += r >= (int)((cum >> (8 * i)) & 255);
    for (int i = 0; i < few.nk; ++i) {             // tokens of the blocks before this one, and of all
      const uint64_t who = __ballot(lane < m && e == i);
      before += __popcll(who & ((1ull << j) - 1)) << i;
      all += __popcll(who) << i;
    }
    t = min(1 << __builtin_amdgcn_readlane(e, (int)j), b);
    dst0 = (int64_t)fill + before;
    if (j == 0 && tid == 0) few.n_rows[h] = (int32_t)((int64_t)fill + all > cap ? cap : (int64_t)fill + all);
  } else {
    t = min(blk_t[(size_t)h * n_blocks + j], b);                       // sel below has room for b rows, whatever it is told
    dst0 = blk_dst[(size_t)h * n_blocks + j];
  }

  // Eq. 8: rank of every token inside the block, all 256 threads share the b*b comparisons;
  // nothing to rank when the whole block is kept
  bool keep = tid < b;
  if (t < b) {
    if (tid < b) {
      bkeys[tid] = FEW ? my_key : keys[(size_t)h * (n_blocks * b) + j * b + tid];
      rank[tid] = 0;
    }
    __syncthreads();
    // b is a power of two <= 256: thread (i = tid % b, part = tid / b) counts over one even-sized span
    int parts = kGatherThreads / b;
    if (parts > b / 2) parts = b / 2;
    const int i = tid % b, part = tid / b, span = b / parts;
    if (part < parts) {
      const int cnt = count_greater(bkeys, part * span, (part + 1) * span, bkeys[i]);
      if (cnt) atomicAdd(&rank[i], cnt);
    }
    __syncthreads();
    keep = tid < b && rank[tid] < t;
  }
  // compact the kept positions, in ascending position order
  const unsigned long long mask = __ballot(keep);
  if (lane == 0) wave_cnt[wv] = __popcll(mask);
  __syncthreads();
  int before = __popcll(mask & ((1ull << lane) - 1ull));
  for (int w = 0; w < wv; ++w) before += wave_cnt[w];
  if (keep) sel[before] = tid;
  __syncthreads();

  // copy the kept rows, kRows rows per thread in flight (2 * kRows 16-byte loads before the first store)
  constexpr int kRows = kGatherRows;
  const int sub = tid % LPR;
  int n_keep = t;
  if (dst0 + n_keep > cap) n_keep = cap > dst0 ? (int)(cap - dst0) : 0;
  if (!Kg) {                                           // positions only: no compacted copy is kept
    for (int k = tid; k < n_keep; k += kGatherThreads) idx[base + dst0 + k] = (int32_t)(pos0 + j * b + sel[k]);
    return;
  }
  for (int k0 = tid / LPR; k0 < n_keep; k0 += kRows * RPI) {
    uint4 kr[kRows], vr[kRows];
    int64_t pos[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const int k = k0 + u * RPI;
      pos[u] = pos0 + j * b + sel[k < n_keep ? k : k0];
      const size_t src = ((size_t)kvh * kv_stride + pos[u]) * D + sub * EPL;
      kr[u] = *reinterpret_cast<const uint4*>(K + src);
      vr[u] = *reinterpret_cast<const uint4*>(V + src);
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const int k = k0 + u * RPI;
      if (k < n_keep) {
        const size_t dst = (size_t)(base + dst0 + k) * D + sub * EPL;
        *reinterpret_cast<uint4*>(Kg + dst) = kr[u];
        *reinterpret_cast<uint4*>(Vg + dst) = vr[u];
        if (sub == 0) idx[base + dst0 + k] = (int32_t)pos[u];
      }
    }
  }
}

template <typename T, int D, int EMIT>
static void launch_score(int G, dim3 grid, hipStream_t st, const T* K, const T* q, int64_t kv_stride,
                         int64_t pos0, int64_t n_tokens, int b, int64_t nb, int64_t nbt, int Hq,
                         double scale, const SelectWs& w, const int32_t* n_rows, int32_t* fill) {
#define TCA_SCORE_CASE(GG)                                                                           \
  case GG:                                                                                           \
    hipLaunchKernelGGL((score_kernel<T, D, GG, EMIT>), grid, dim3(kScoreThreads), 0, st, K, q,       \
                       kv_stride, pos0, n_tokens, b, nb, nbt, Hq, scale, w.tokrank, w.keys, w.stats, \
                       w.xlog, n_rows, fill);                                                        \
    break;
  switch (G) {
    TCA_SCORE_CASE(1) TCA_SCORE_CASE(2) TCA_SCORE_CASE(3) TCA_SCORE_CASE(4)
    TCA_SCORE_CASE(5) TCA_SCORE_CASE(6) TCA_SCORE_CASE(7) TCA_SCORE_CASE(8)
  }
#undef TCA_SCORE_CASE
}

template <bool RANK>
static void launch_group_score(int G, int Hq, int Hkv, int b, int64_t nb, int64_t nbt, const SelectWs& w,
                               const int32_t* n_rows, int32_t* fill, hipStream_t st) {
  const double* lse = nullptr;
  if (nbt > kFewBlocks) {
    hipLaunchKernelGGL(group_lse_kernel, dim3(Hq), dim3(256), 0, st, w.stats, (int)nbt, w.lse);
    lse = w.lse;
  }
  const dim3 grid((unsigned)nbt, Hkv);
#define TCA_GROUP_CASE(GG)                                                                              \
  case GG:                                                                                              \
    hipLaunchKernelGGL((group_score_kernel<GG, RANK>), grid, dim3(256), 0, st, w.xlog, lse, w.stats, b, nb, nbt, \
                       w.tokrank, w.keys, w.sel_stats, n_rows, fill);                                   \
    break;
  switch (G) {
    TCA_GROUP_CASE(2) TCA_GROUP_CASE(3) TCA_GROUP_CASE(4) TCA_GROUP_CASE(5)
    TCA_GROUP_CASE(6) TCA_GROUP_CASE(7) TCA_GROUP_CASE(8)
  }
#undef TCA_GROUP_CASE
}

// Scores tokens [pos0, pos0 + n_tokens) for every selection head: block statistics in
// w.sel_stats, and in-block ranks in w.tokrank (RANK) or ranking keys in w.keys.  fill: where the heads' n_rows go, or NULL.
template <typename T, int D, bool RANK>
static void score_stage(const tca_params* prm, const T* q_last, const T* K, int64_t kv_stride, int64_t pos0,
                        int64_t n_tokens, const SelectWs& w, const int32_t* n_rows, int32_t* fill, hipStream_t st) {
  const int Hq = prm->n_q_heads, Hkv = prm->n_kv_heads, G = Hq / Hkv, b = prm->block;
  const int64_t nb = n_tokens / b, nbt = (n_tokens + b - 1) / b;
  const dim3 grid((unsigned)nbt, Hkv);
  const double sc = logit_scale(prm);
  if (grouped(prm)) {
    launch_score<T, D, kEmitLogits>(G, grid, st, K, q_last, kv_stride, pos0, n_tokens, b, nb, nbt, Hq, sc, w, nullptr, nullptr);
    launch_group_score<RANK>(G, Hq, Hkv, b, nb, nbt, w, n_rows, fill, st);
  } else {
    launch_score<T, D, RANK ? kEmitRanks : kEmitKeys>(G, grid, st, K, q_last, kv_stride, pos0, n_tokens, b, nb,
                                                      nbt, Hq, sc, w, n_rows, fill);
  }
}

// Stage 1 of selection for callers outside this file (calibration): block statistics
// and in-block ranks of tokens [0, n_tokens) of K scored by q_last.
void select_score_stage(const tca_params* prm, const void* q_last, const void* K, int64_t kv_stride,
                        int64_t n_tokens, const SelectWs& w, hipStream_t st) {
  if (prm->dtype == TCA_BF16) {
    using T = bf16_t;
    if (prm->head_dim == 128) score_stage<T, 128, true>(prm, (const T*)q_last, (const T*)K, kv_stride, 0, n_tokens, w, nullptr, nullptr, st);
    else score_stage<T, 64, true>(prm, (const T*)q_last, (const T*)K, kv_stride, 0, n_tokens, w, nullptr, nullptr, st);
  } else {
    using T = float;
    if (prm->head_dim == 128) score_stage<T, 128, true>(prm, (const T*)q_last, (const T*)K, kv_stride, 0, n_tokens, w, nullptr, nullptr, st);
    else score_stage<T, 64, true>(prm, (const T*)q_last, (const T*)K, kv_stride, 0, n_tokens, w, nullptr, nullptr, st);
  }
}

// One wave where it can hold all blocks (no barrier at all), then four, then sixteen, whose threads take four blocks
// each at most.  us per launch, 32 heads: 64 blocks 12.5 -> 8.6, 3 blocks 8.5 -> 5.3, 1024 blocks 28.3 -> 20.3
// (one shape of 1024 threads, the sort and the scan in LDS, before).
static void launch_assign(const tca_params* prm, const AssignArgs& aa, int grid, int head0, int heads_each, int64_t n_tokens,
                          const double* stats, int32_t* n_rows, int32_t* blk_t, int32_t* blk_dst, hipStream_t st) {
  const int b = prm->block, nk = block_log2(b) + 1;
  const int64_t nb = n_tokens / b, nbt = (n_tokens + b - 1) / b;
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, aa, head0, heads_each, nk, (int)nb, (int)nbt, b, prm->alpha,
                       prm->metric, stats, n_rows, blk_t, blk_dst);
  };
  if (nb <= 64) launch(assign_kernel<64, 1>, 64);
  else if (nb <= 256) launch(assign_kernel<256, 1>, 256);
  else if (nb <= 1024) launch(assign_kernel<1024, 1>, 1024);
  else launch(assign_kernel<1024, 4>, 1024);
}

static void fill_cum(AssignArgs& aa, int i, int nk, int64_t nb, const double* p, int64_t cap) {
  int64_t c[TCA_MAX_COUNTS], run = 0;
  psi_counts(nk, nb, p, c);
  for (int e = 0; e < nk; ++e) aa.cum[i][e] = (int32_t)(run += c[e]);
  aa.cap[i] = cap;
}

// Stage 2: block metric, ranking and budgets for one configuration per selection head.
// blk_t / blk_dst: [Hs][nb]; n_rows: [Hs] fill counters (in/out); cap: per-head capacity.
void select_assign_stage(const tca_params* prm, int64_t n_tokens, const double* p, const int64_t* cap,
                         const double* stats, int32_t* n_rows, int32_t* blk_t, int32_t* blk_dst,
                         hipStream_t st) {
  const int Hs = sel_heads(prm), nk = block_log2(prm->block) + 1;
  for (int h0 = 0; h0 < Hs; h0 += kHeadsPerLaunch) {
    const int nh = Hs - h0 < kHeadsPerLaunch ? Hs - h0 : kHeadsPerLaunch;
    AssignArgs aa;
    for (int hl = 0; hl < nh; ++hl) fill_cum(aa, hl, nk, n_tokens / prm->block, p + (size_t)(h0 + hl) * nk, cap[h0 + hl]);
    launch_assign(prm, aa, nh, h0, 0, n_tokens, stats, n_rows, blk_t, blk_dst, st);
  }
}

// One launch for up to 32 of calibration's candidates (14 launches of 7 us before, 9 us now, 32 heads and 64 blocks).
void select_assign_all(const tca_params* prm, int64_t n_tokens, int n, const double* p, const double* stats, int32_t* n_rows,
                       int32_t* blk_t, int32_t* blk_dst, hipStream_t st) {
  const int Hs = sel_heads(prm), nk = block_log2(prm->block) + 1;
  for (int i0 = 0; i0 < n; i0 += kHeadsPerLaunch) {
    const int ni = n - i0 < kHeadsPerLaunch ? n - i0 : kHeadsPerLaunch;
    AssignArgs aa;
    for (int i = 0; i < ni; ++i) fill_cum(aa, i, nk, n_tokens / prm->block, p + (size_t)(i0 + i) * nk, INT32_MAX);
    const size_t off = (size_t)i0 * Hs;
    launch_assign(prm, aa, ni * Hs, 0, Hs, n_tokens, stats, n_rows + off, blk_t + off * (n_tokens / prm->block),
                  blk_dst + off * (n_tokens / prm->block), st);
  }
}

template <typename T, int D>
static int run_select(const tca_params* prm, const T* q_last, const T* K, const T* V,
                      int64_t kv_stride, int64_t pos0, int64_t n_tokens, const double* p,
                      const int64_t* offs, int32_t* n_rows, int32_t* idx, T* Kg, T* Vg, void* ws,
                      hipStream_t st) {
  const int Hs = sel_heads(prm), Hkv = prm->n_kv_heads, b = prm->block;
  const int64_t nb = n_tokens / b;
  SelectWs w = carve_select_ws(ws, prm, n_tokens);
  OffsArgs oa;
  for (int h = 0; h <= Hs; ++h) oa.offs[h] = offs[h];

  const bool few = nb > 0 && (n_tokens + b - 1) / b <= kFewBlocks;
  int32_t* const fill = few ? w.blk_t : nullptr;                       // [Hs], in a place that such a call has no other use for
  score_stage<T, D, false>(prm, q_last, K, kv_stride, pos0, n_tokens, w, n_rows, fill, st);
  if (nb == 0) return TCA_OK;

  auto gather = [&](auto few_tag, const auto& args) {
    hipLaunchKernelGGL((gather_kernel<T, D, decltype(few_tag)::value>), dim3((unsigned)(nb * Hs)), dim3(kGatherThreads), 0, st, K, V,
                       kv_stride, pos0, b, nb, Hs / Hkv, w.keys, w.blk_t, w.blk_dst, oa, idx, Kg, Vg, args);
  };
  if (few) {
    const int nk = block_log2(b) + 1;
    FewArgs fa;
    for (int h = 0; h < Hs; ++h) {
      int64_t c[TCA_MAX_COUNTS], run = 0;
      psi_counts(nk, nb, p + (size_t)h * nk, c);
      fa.cum[h] = 0;
      for (int e = 0; e < nk - 1; ++e) fa.cum[h] |= (uint64_t)(run += c[e]) << (8 * e);
    }
    fa.nk = nk;
    fa.nbt = (int)((n_tokens + b - 1) / b);
    fa.metric = prm->metric;
    fa.alpha = prm->alpha;
    fa.stats = w.sel_stats;
    fa.fill = fill;
    fa.n_rows = n_rows;
    gather(std::true_type{}, fa);
    return TCA_OK;
  }
  int64_t cap[TCA_MAX_HEADS];
  for (int h = 0; h < Hs; ++h) cap[h] = offs[h + 1] - offs[h];
  select_assign_stage(prm, n_tokens, p, cap, w.sel_stats, n_rows, w.blk_t, w.blk_dst, st);
  gather(std::false_type{}, NoFew{});
  return TCA_OK;
}

}  // namespace tca

using namespace tca;

extern "C" size_t tca_select_workspace_bytes(const tca_params* prm, int64_t n_tokens) {
  if (check_params(prm) != TCA_OK || n_tokens < 0) return 0;
  SelectWs w = carve_select_ws(nullptr, prm, n_tokens);
  return w.bytes;
}

extern "C" int tca_select(const tca_params* prm, const void* q_last, const void* K, const void* V,
                          int64_t kv_stride, int64_t pos0, int64_t n_tokens, const double* p,
                          const int64_t* offs, int32_t* n_rows, int32_t* idx, void* Kg, void* Vg,
                          void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!q_last || !K || !V || !p || !offs || !n_rows || !idx || !ws)
    return fail(TCA_ERR_INVALID, "tca_select: NULL pointer argument");
  if ((Kg == nullptr) != (Vg == nullptr))
    return fail(TCA_ERR_INVALID, "tca_select: Kg and Vg must both be given, or both be NULL (positions only)");
  const int b = prm->block, Hs = sel_heads(prm);
  if (n_tokens < 0 || pos0 < 0 || pos0 % b != 0 || pos0 + n_tokens > kv_stride)
    return fail(TCA_ERR_INVALID, "tca_select: pos0=%lld n_tokens=%lld kv_stride=%lld (pos0 must be a "
                "multiple of b and the range must fit)", (long long)pos0, (long long)n_tokens,
                (long long)kv_stride);
  if (pos0 + n_tokens > INT32_MAX) return fail(TCA_ERR_UNSUPPORTED, "positions beyond int32");
  if (n_tokens / b > TCA_MAX_BLOCKS)
    return fail(TCA_ERR_UNSUPPORTED, "tca_select: %lld blocks exceed the limit of %d per call",
                (long long)(n_tokens / b), TCA_MAX_BLOCKS);
  const int nk = block_log2(b) + 1;
  for (int h = 0; h < Hs; ++h) {
    if (!valid_config(p + (size_t)h * nk, nk))
      return fail(TCA_ERR_INVALID, "tca_select: p[%d] is not a distribution", h);
    if (offs[h + 1] < offs[h]) return fail(TCA_ERR_INVALID, "tca_select: offs not ascending at %d", h);
  }
  if (offs[0] != 0) return fail(TCA_ERR_INVALID, "tca_select: offs[0] must be 0");
  if (ws_bytes < tca_select_workspace_bytes(prm, n_tokens) || ((uintptr_t)ws & 255))
    return fail(TCA_ERR_WORKSPACE, "tca_select: workspace needs %zu bytes, 256-byte aligned",
                tca_select_workspace_bytes(prm, n_tokens));
  if (n_tokens == 0) return TCA_OK;
  hipStream_t st = (hipStream_t)stream;
  const int D = prm->head_dim;
  if (prm->dtype == TCA_BF16) {
    using T = bf16_t;
    rc = D == 128 ? run_select<T, 128>(prm, (const T*)q_last, (const T*)K, (const T*)V, kv_stride, pos0,
                                       n_tokens, p, offs, n_rows, idx, (T*)Kg, (T*)Vg, ws, st)
                  : run_select<T, 64>(prm, (const T*)q_last, (const T*)K, (const T*)V, kv_stride, pos0,
                                      n_tokens, p, offs, n_rows, idx, (T*)Kg, (T*)Vg, ws, st);
  } else {
    using T = float;
    rc = D == 128 ? run_select<T, 128>(prm, (const T*)q_last, (const T*)K, (const T*)V, kv_stride, pos0,
                                       n_tokens, p, offs, n_rows, idx, (T*)Kg, (T*)Vg, ws, st)
                  : run_select<T, 64>(prm, (const T*)q_last, (const T*)K, (const T*)V, kv_stride, pos0,
                                      n_tokens, p, offs, n_rows, idx, (T*)Kg, (T*)Vg, ws, st);
  }
  if (rc) return rc;
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}
