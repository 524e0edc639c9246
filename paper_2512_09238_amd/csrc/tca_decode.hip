// Single-token decode over the compacted KV cache, and selection of blocks
// completed while decoding (Sec. IV-B, "Online Token Selection in Decoding Stage").
//
// One step = two launches on the caller's stream:
//   partial : split-K attention.  grid (units of a sequence, sequences), numbered through: the units of
//             all rings first.  A unit is a chunk of rows of one head's global region, or of one KV
//             head's ring, and there is one for every chunk of the region's capacity (heads keep
//             different numbers of rows; a grid of heads x longest head had two workgroups of three
//             find nothing to do).  The host does not know
//             how full a region is: in a cache with room for far more than it holds, units behind
//             the last row return at once, and the chunk length is chosen as for a full one.
//             The rows that have left the window (idx <= T-w; idx is ascending, so a prefix of the
//             chunk) are found by a 64-way search, one load as a rule.  The unit that holds the new
//             row's ring slot writes the row there first.  The 256 threads form sixteen 16-lane
//             groups (or 32 of eight: kWideRows), each streaming whole rows and keeping its own online
//             softmax; groups are merged into one (max, sum, acc[D]) partial per unit and query head.
//             HBM-bound: every K/V row is read once per selection head - once per query head,
//             or, when the group shares one selection, once per KV head with every row scored
//             against the group's G queries.
//   merge   : log-sum-exp merge of a head's partials -> O.  If the new token completes a
//             block, the same workgroup scores the block's b rows with this step's query in
//             fp64 (Eq. 5 restricted to the block), ranks them and appends the top t =
//             floor(sum k p_k) to the head's global region in position order.  Shared
//             selection: the group's first workgroup ranks by the sum over the group's heads
//             of their block-normalised scores and appends once per KV head.  The first
//             head's workgroup of a sequence advances its length.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cfloat>
#include <functional>
#include <type_traits>

#include "tca_common.h"
#include "tca_device.h"

namespace tca {

constexpr int kPartThreads = 256;                 // threads of a split-K workgroup (64 with 256-row slots measured 8-14 % slower)
constexpr int kPartWaves = kPartThreads / 64;
constexpr int kChunk = 4 * kPartThreads;          // rows per split-K unit of a long step: 64 per 16-lane group
constexpr int kChunkShared = 2048;                // the same when every row is scored against a group of queries (1024: 507, 2048: 480, 4096: 540 us per step)
constexpr int kMinChunk = 128;                    // of a short step: see choose_chunk
constexpr int kDecThreads = 256;                  // the other kernels
constexpr int kMaxSlots = 4096;       // split-K units per head that a step is taken for (4M rows per head): far inside the 24 bits order_units has for them

struct DecodeHeads {
  int64_t offs[TCA_MAX_HEADS + 1];
  int32_t t_dec[TCA_MAX_HEADS];
  int32_t unit0[TCA_MAX_HEADS + 1];   // first unit of each head's region; unit0[Hs]: their number
  int32_t first[TCA_MAX_HEADS];       // the order of the regions' workgroups: see order_units
  uint8_t by_units[TCA_MAX_HEADS];    // the heads, those with the most units first
  int32_t chunk;                      // rows per unit
  int32_t ring_units;                 // units of one ring
  int32_t units;                      // of a sequence: those of its rings and regions
};

// Partials of a sequence: region [selection head][its query heads][its units], then ring [query head][ring_units];
// D + 2 floats each.
struct DecodeWs {
  uint32_t* pos;     // [B] low half of the step's position (written by the partial kernel: see decode_merge_kernel)
  float* part;
  size_t bytes;
};

static DecodeWs carve_decode_ws(void* ws, int B, int Hq, int D, int64_t partials_per_seq) {
  DecodeWs w;
  char* base = (char*)ws;
  size_t off = 0;
  w.pos = (uint32_t*)(base + off); off = align_up(off + (size_t)B * Hq * sizeof(int32_t), 256);
  w.part = (float*)(base + off);   off = align_up(off + (size_t)B * partials_per_seq * (D + 2) * sizeof(float), 256);
  w.bytes = off;
  return w;
}

static int long_chunk(const tca_params* prm) { return sel_group(prm) > 1 ? kChunkShared : kChunk; }
static int64_t chunks_of(int64_t rows, int chunk) { return (rows + chunk - 1) / chunk; }

// Bytes every call must have: the partials of chunks of the full length, every head as long as the longest.
static size_t decode_ws_need(const tca_params* prm, int batch, int64_t max_head_rows) {
  const int c = long_chunk(prm);
  return carve_decode_ws(nullptr, batch, prm->n_q_heads, prm->head_dim,
                         prm->n_q_heads * (chunks_of(max_head_rows, c) + chunks_of(prm->window, c))).bytes;
}

// A step whose chunks of full length would leave CUs without work takes shorter ones, down to kMinChunk rows, as long as
// they come to at most this many workgroups.  us per step (32 query heads, one selection each, d = 128, bf16) with full chunks,
// and up to 512 / 1536 / 3072 / 4096 workgroups: 1 x 8000 tokens 44 / 18 / 19 / 18 / 17; 4 x 30000 95 / 96 / 87 / 84 /
// 83; 8 x 30011 fp8 107 / 108 / 112 / 95 / 93; shared selection 4 x 30000 107 / 66 / 53 / 59 / 59, 64 heads 3 x 110000 128 / 127
// / 118 / 125 / 125 (2048: 115).
static int64_t short_units(const tca_params* prm) { return sel_group(prm) > 1 ? 2048 : 3072; }
// Bytes a caller is told to bring: the same, or what a step of short chunks can need (each unit serves at most a
// group of queries).
static size_t decode_ws_bytes(const tca_params* prm, int batch, int64_t max_head_rows) {
  const int G = prm->n_q_heads / prm->n_kv_heads;
  int64_t few = (int64_t)batch * prm->n_q_heads * (chunks_of(max_head_rows, kMinChunk) + chunks_of(prm->window, kMinChunk));
  if (few > short_units(prm) * G) few = short_units(prm) * G;
  const size_t need = decode_ws_need(prm, batch, max_head_rows);
  const size_t with_short = carve_decode_ws(nullptr, batch, prm->n_q_heads, prm->head_dim, 0).bytes +
                            align_up((size_t)few * (prm->head_dim + 2) * sizeof(float), 256);
  return need > with_short ? need : with_short;
}

// max over the 16 lanes of a row, result in every lane
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_f32<kDppXor1>(v));
  v = fmaxf(v, dpp_f32<kDppXor2>(v));
  v = fmaxf(v, dpp_f32<kDppHalfMirror>(v));
  v = fmaxf(v, dpp_f32<kDppMirror>(v));
  return v;
}

// sum over the 16 lanes of a row, or over each half of them
template <int LPR, typename V> __device__ __forceinline__ V row_sum(V v) {
  if constexpr (LPR == 16) {
    return row16_sum(v);
  } else {
    static_assert(LPR == 8 && sizeof(V) == 4, "");
    v += dpp_f32<kDppXor1>(v);
    v += dpp_f32<kDppXor2>(v);
    return v + dpp_f32<kDppHalfMirror>(v);
  }
}

// Scale of an FP8 row from the largest magnitude of its elements, and its reciprocal use: the codes are
// RNE_e4m3(x / scale) with both divisions in float32 (the rule stated with TCA_KV_FP8).
__device__ __forceinline__ float fp8_row_scale(float amax) { return amax > 0.f ? amax / 448.f : 1.f; }

// One 16-lane group stores one row of D elements (a lane's slice: D/16 consecutive elements, 4 or 8)
// into a cache row of storage type KV: a plain conversion-free copy for the native types, codes and a
// scale for FP8.  x: the lane's slice widened to float.  Called by all 16 lanes of the group.
template <typename KV, int EL>
__device__ __forceinline__ void store_cache_slice(const float (&x)[EL], KV* dst_row, float* scale_slot, int sub) {
  static_assert(sizeof(KV) == 1, "native rows are copied as stored");
  float amax = 0.f;
#pragma unroll
  for (int e = 0; e < EL; ++e) amax = fmaxf(amax, fabsf(x[e]));
  amax = row16_max(amax);
  const float scale = fp8_row_scale(amax);
  uint32_t* out = reinterpret_cast<uint32_t*>(dst_row + sub * EL);
  // One division a row and a step of Newton's iteration per element: the quotient y = x inv is off by little more than a
  // unit in its last place, x - y scale is exact in one fused operation, and y + that times inv rounds to what the
  // division gives (Markstein), as long as nothing on the way is subnormal or infinite; outside that range, and for a row
  // that holds an infinity, the divisions are made (ten instructions each).  Handover of 32768 tokens, 32 heads: 45.1 -> 42.9 us.
  if (scale > 0x1p-60f && scale < 0x1p60f) {
    const float inv = 1.f / scale;
    float y[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      y[e] = x[e] * inv;
      y[e] = copysignf(fmaf(fmaf(-y[e], scale, x[e]), inv, y[e]), x[e]);       // (of zero the sign went in the sum)
    }
#pragma unroll
    for (int e = 0; e < EL; e += 4) out[e / 4] = f32x4_to_fp8(y[e], y[e + 1], y[e + 2], y[e + 3]);
  } else {
#pragma unroll
    for (int e = 0; e < EL; e += 4) out[e / 4] = f32x4_to_fp8(x[e] / scale, x[e + 1] / scale, x[e + 2] / scale, x[e + 3] / scale);
  }
  if (sub == 0) *scale_slot = scale;
}

// Copies a row of T into a cache row of storage type KV: as stored, or as codes and a scale (called by the 16 lanes of a
// group).  ALIGNED: slices of up to 16 bytes at a time; otherwise element by element.
template <typename T, typename KV, int D, bool ALIGNED>
struct RowCopy {
  static constexpr int EL = D / 16;
  static constexpr bool kSame = std::is_same<T, KV>::value;
  RawSlice<T, EL> raw;
  __device__ __forceinline__ void load(const T* row, int sub) {
    if constexpr (ALIGNED) {
      raw.load(row + sub * EL);
    } else if constexpr (sizeof(T) == 2) {
      const uint16_t* p = reinterpret_cast<const uint16_t*>(row) + sub * EL;
#pragma unroll
      for (int i = 0; i < EL / 2; ++i) raw.w[i] = p[2 * i] | ((uint32_t)p[2 * i + 1] << 16);
    } else {
      const uint32_t* p = reinterpret_cast<const uint32_t*>(row) + sub * EL;
#pragma unroll
      for (int i = 0; i < EL; ++i) raw.w[i] = p[i];
    }
  }
  __device__ __forceinline__ void store(KV* row, float* scale_slot, int sub) const {
    if constexpr (!kSame) {
      float x[EL];
      raw.widen(x);
      store_cache_slice<KV, EL>(x, row, scale_slot, sub);
    } else if constexpr (ALIGNED) {
      constexpr int W = RawSlice<T, EL>::W;
      if constexpr (W == 2) {
        *reinterpret_cast<uint2*>(row + sub * EL) = make_uint2(raw.w[0], raw.w[1]);
      } else {
#pragma unroll
        for (int i = 0; i < W / 4; ++i)
          reinterpret_cast<uint4*>(row + sub * EL)[i] = make_uint4(raw.w[4 * i], raw.w[4 * i + 1], raw.w[4 * i + 2], raw.w[4 * i + 3]);
      }
    } else if constexpr (sizeof(T) == 2) {
      uint16_t* p = reinterpret_cast<uint16_t*>(row) + sub * EL;
#pragma unroll
      for (int i = 0; i < EL; ++i) p[i] = (uint16_t)(raw.w[i >> 1] >> (16 * (i & 1)));
    } else {
      uint32_t* p = reinterpret_cast<uint32_t*>(row) + sub * EL;
#pragma unroll
      for (int i = 0; i < EL; ++i) p[i] = raw.w[i];
    }
  }
};

// Writes the new row (k_new, v_new: D elements each) into row `row` of the ring; called by a whole workgroup, which may
// read it back after the barrier inside (KV = T: the row as it is; KV = fp8_t: as codes and a scale).
template <typename T, typename KV, int D>
__device__ __forceinline__ void store_new_row(const tca_cache& c, size_t row, const T* __restrict__ k_new, const T* __restrict__ v_new) {
  if (threadIdx.x < 32) {                              // one 16-lane group for K, one for V
    const int sub = threadIdx.x & 15;
    const bool is_v = threadIdx.x >= 16;
    const T* src = is_v ? v_new : k_new;
    RowCopy<T, KV, D, true> x;
    if ((((uintptr_t)k_new | (uintptr_t)v_new) & 15) == 0) {
      x.load(src, sub);
    } else {                                           // the caller's rows may start at any element
      RowCopy<T, KV, D, false> y;
      y.load(src, sub);
      x.raw = y.raw;
    }
    x.store((KV*)(is_v ? c.ringV : c.ringK) + row * D, (is_v ? c.ringV_scale : c.ringK_scale) + row, sub);
    __threadfence_block();
    __builtin_amdgcn_s_waitcnt(0x0F70);                // the stores have reached the cache the workgroup reads through
  }
  __syncthreads();
}

// Tail of the split-K kernels: every group of LPR lanes of the workgroup holds, for each of NQ
// queries, an online-softmax state (reference m in base-2 units, sum l, acc over the lane's
// slice of d).  Merges the groups of each wave, then the 4 waves through LDS, and writes one
// (reference, sum, acc[D]) partial per query at out + g * out_head, the reference still in
// base-2 units (integer references, as the fp32 path keeps them, stay exact through every merge).
template <int D, int NQ, int LPR>
__device__ __forceinline__ void merge_partials(float (&m)[NQ], float (&l)[NQ], float (&acc)[NQ][D / LPR],
                                               float* __restrict__ out, size_t out_head, float* red) {
  constexpr int EL = D / LPR;
  constexpr int PW = EL + 2;                          // floats of one lane's share of a partial
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
    // Through LDS these exchanges took a fourth of a short unit of 128 elements a row.  With 64 elements, where a unit has half as many
    // lines to wait for, the swaps' instructions cost more: 4096 sequences of 200 tokens 90.7 us through LDS, 93.9 by swaps.
    auto across = [&](auto o_tag) {
      constexpr int O = decltype(o_tag)::value;
      auto pair = [&](float v, float& a, float& b) {
        if constexpr (D == 64) { a = v; b = __shfl_xor(v, O, kWave); }
        else lane_pair<O>(v, a, b);
      };
      float ma, mb, x, y;
      pair(m[g], ma, mb);
      const float mn = fmaxf(ma, mb);
      const float ca = (ma == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ma - mn);
      const float cb = (mb == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mb - mn);
      pair(l[g], x, y);
      l[g] = x * ca + y * cb;
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        pair(acc[g][e], x, y);
        acc[g][e] = x * ca + y * cb;
      }
      m[g] = mn;
    };
    if constexpr (LPR == 8) across(std::integral_constant<int, 8>{});
    across(std::integral_constant<int, 16>{});
    across(std::integral_constant<int, 32>{});
    if (lane < LPR) {
      red[(wv * LPR + lane) * (NQ * PW) + g * PW] = m[g];
      red[(wv * LPR + lane) * (NQ * PW) + g * PW + 1] = l[g];
#pragma unroll
      for (int e = 0; e < EL; ++e) red[(wv * LPR + lane) * (NQ * PW) + g * PW + 2 + e] = acc[g][e];
    }
  }
  __syncthreads();
  for (int pi = tid; pi < LPR * NQ; pi += kPartThreads) {
    const int g = pi / LPR, ln = pi % LPR;
    float M = -INFINITY;
    for (int x = 0; x < kPartWaves; ++x) M = fmaxf(M, red[(x * LPR + ln) * (NQ * PW) + g * PW]);
    float L = 0.f, a[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) a[e] = 0.f;
    for (int x = 0; x < kPartWaves; ++x) {
      const float mx = red[(x * LPR + ln) * (NQ * PW) + g * PW];
      const float cf = (mx == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mx - M);
      L += red[(x * LPR + ln) * (NQ * PW) + g * PW + 1] * cf;
#pragma unroll
      for (int e = 0; e < EL; ++e) a[e] += red[(x * LPR + ln) * (NQ * PW) + g * PW + 2 + e] * cf;
    }
    float* og = out + g * out_head;
    if (ln == 0) { og[0] = M; og[1] = L; }
#pragma unroll
    for (int e = 0; e < EL; ++e) og[2 + ln * EL + e] = a[e];
  }
}

// Split-K attention of NQ queries (consecutive heads, q0 = the first one's row) over rows
// [r_begin, r_end) of one K/V buffer: every row is read once and scored against all NQ queries.
// Writes one (max, sum, acc[D]) partial per query at out + g * out_head.  red: LDS scratch of
// kPartWaves * LPR * NQ * (D/LPR + 2) floats.  Called by a whole workgroup.
// T: type of the queries; KV: storage type of the rows (T itself, or fp8_t with one float scale per
// row in kscale / vscale, indexed like the rows).
// LPR: lanes that share a row, 16 or (FP8, 16 bytes each) 8: see kWideRows.
template <typename T, typename KV, int D, int NQ, int LPR, typename Visible>
__device__ __forceinline__ void partial_rows(const KV* __restrict__ kbase, const KV* __restrict__ vbase,
                                             const float* __restrict__ kscale, const float* __restrict__ vscale,
                                             int r_begin, int r_cap, Visible visible, const T* __restrict__ q0, double scale,
                                             float* __restrict__ out, size_t out_head, float* red) {
  constexpr int EL = D / LPR, GROUPS = kPartThreads / LPR;
  const int tid = threadIdx.x;
  const int grp = tid / LPR, sub = tid % LPR;
  int r_end = r_cap;                                  // until the first rows are requested
  // logits are carried in base-2 units (scale * log2 e) so that the exponential is one v_exp_f32.
  // bf16 storage: q.k over a lane's slice is EL/2 two-element bf16 dot products with fp32
  // accumulation straight from the loaded words, and the factor is applied to the row's sum.
  // fp32 storage: q.k is accumulated in fp64 and the reference of the exponentials is kept at an
  // integer (exact in fp32, and exact through every later merge), so that x - reference is formed
  // without cancellation error even for logits in the hundreds.
  // FP8 storage: the codes are widened to float, q.k is the fp32 dot product with the codes times the
  // row's scale, and p.v takes the V row's scale into the weight.
  constexpr double kLog2e = 1.4426950408889634;
  constexpr bool kDot2 = sizeof(KV) == 2;
  constexpr bool kFp8 = sizeof(KV) == 1;
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  using logit_t = typename std::conditional<sizeof(KV) == 4, double, float>::type;
  const logit_t qk_factor = (logit_t)(scale * kLog2e);
  float qv[kDot2 ? 1 : NQ][EL];
  RawSlice<T, EL> qraw[kDot2 ? NQ : 1];
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
    if constexpr (kDot2) {
      qraw[g].load(q0 + (size_t)g * D + sub * EL);
    } else {
      constexpr int E = EL < 8 ? EL : 8;
#pragma unroll
      for (int e = 0; e < EL; e += E) load_slice<T, E>(q0 + (size_t)g * D + sub * EL + e, *reinterpret_cast<float(*)[E]>(&qv[g][e]));
    }
  }

  float m[NQ], l[NQ], acc[NQ][EL];
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
    m[g] = -FLT_MAX;                                   // finite: a first logit of -inf has the term 0, not NaN
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EL; ++e) acc[g][e] = 0.f;
  }

  // Online softmax with a lazy reference: m[g] is raised (and l, acc rescaled) only when a
  // logit exceeds it by more than kSlack, so the common row costs one subtract, one exp and
  // the multiply-adds.  Terms are then at most 2^kSlack; the result is exact because l and
  // acc share the reference, which the merge steps below carry along.
  constexpr float kSlack = 8.f;
  // Rows are fetched one iteration ahead of their use (kUnr rows of K and of V per group,
  // kept as loaded until then), so that a lane has 2*kUnr loads in flight while it computes.
  constexpr int kUnr = 2;
  using Raw = RawSlice<KV, EL>;
  Raw kr[kUnr], vr[kUnr];
  float ksc[kUnr], vsc[kUnr];                          // row scales (FP8 rows only)
  bool ok[kUnr];
  auto fetch = [&](int r0, Raw (&kk)[kUnr], Raw (&vq)[kUnr], float (&ks)[kUnr], float (&vs)[kUnr], bool (&okk)[kUnr]) {
#pragma unroll
    for (int u = 0; u < kUnr; ++u) {
      const int r = r0 + u * GROUPS + grp;
      okk[u] = r < r_end;
      ks[u] = vs[u] = 1.f;
      if (okk[u]) {
        kk[u].load(kbase + (size_t)r * D + sub * EL);
        vq[u].load(vbase + (size_t)r * D + sub * EL);
        if constexpr (kFp8) { ks[u] = kscale[r]; vs[u] = vscale[r]; }
      }
    }
  };
  fetch(r_begin, kr, vr, ksc, vsc, ok);
  r_end = visible();
  if (r_begin >= r_end) {
    if (tid < NQ) { out[tid * out_head] = -INFINITY; out[tid * out_head + 1] = 0.f; }
    return;
  }
#pragma unroll
  for (int u = 0; u < kUnr; ++u) ok[u] = r_begin + u * GROUPS + grp < r_end;
  for (int r0 = r_begin; r0 < r_end; r0 += GROUPS * kUnr) {
    Raw kn[kUnr], vn[kUnr];
    float ksn[kUnr], vsn[kUnr];
    bool okn[kUnr];
    fetch(r0 + GROUPS * kUnr, kn, vn, ksn, vsn, okn);          // nothing is loaded past r_end
#pragma unroll
    for (int u = 0; u < kUnr; ++u) {
      float kv[EL], vv[EL];
      if (ok[u]) {
        if constexpr (!kDot2) kr[u].widen(kv);
        vr[u].widen(vv);
      }
#pragma unroll
      for (int g = 0; g < NQ; ++g) {
        logit_t sc = 0;
        if (ok[u]) {
          if constexpr (kDot2) {
#pragma unroll
            for (int i = 0; i < EL / 2; ++i)
              sc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kr[u].w[i]),
                                                   __builtin_bit_cast(bf16x2_t, qraw[g].w[i]), sc, false);
          } else {
#pragma unroll
            for (int e = 0; e < EL; ++e) {
              if constexpr (sizeof(logit_t) == 4) sc = fmaf(qv[g][e], kv[e], sc);
              else sc = fma((double)qv[g][e], (double)kv[e], sc);
            }
          }
        }
        sc = row_sum<LPR>(sc) * qk_factor;
        if constexpr (kFp8) sc *= ksc[u];
        if (ok[u]) {
          if (sc > (logit_t)m[g] + (logit_t)kSlack) {
            const float m_new = sizeof(KV) == 4 ? ceilf((float)sc) : (float)sc;
            const float corr = __builtin_amdgcn_exp2f(m[g] - m_new);    // 0 on the first row (m = -FLT_MAX)
            l[g] *= corr;
#pragma unroll
            for (int e = 0; e < EL; ++e) acc[g][e] *= corr;
            m[g] = m_new;
          }
          const float pr = __builtin_amdgcn_exp2f((float)(sc - (logit_t)m[g]));
          l[g] += pr;
          const float pw = kFp8 ? pr * vsc[u] : pr;                   // the V row's scale rides on the weight
#pragma unroll
          for (int e = 0; e < EL; ++e) acc[g][e] = fmaf(pw, vv[e], acc[g][e]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kUnr; ++u) { kr[u] = kn[u]; vr[u] = vn[u]; ksc[u] = ksn[u]; vsc[u] = vsn[u]; ok[u] = okn[u]; }
  }
  merge_partials<D, NQ, LPR>(m, l, acc, out, out_head, red);
}

// The same for bf16 rows of 128 elements and NQ > 1 queries, and FP8 rows and NQ > 2, with q.k on the matrix cores.
// A wave takes 16 rows per iteration (its 16-lane group kb the rows 4kb .. 4kb+3).  K rows go
// from registers into a wave-private LDS tile and come back in MFMA operand order (lane
// (n, kb) = 8 consecutive elements of row n), so that four 16x16x32 MFMAs against the queries
// (operand B, columns >= NQ zero) leave S[row 4kb+i][query n] in lane (n, kb): the NQ*4 lanes
// with n < NQ hold every score once, and only they do the softmax arithmetic.  Their terms p
// return through LDS to the lanes that hold the V rows, which accumulate p.v on the vector ALU
// as before.  The reference m[g] is common to the wave and lazy (raised only when a score
// exceeds it by more than kSlack, decided by a wave-wide vote).  Against partial_rows this
// removes, per (row, query), the dot products, the 16-lane reductions and 15 of the 16 copies
// of the exponential.  FP8 rows come this way too (8 sequences of 30K tokens, the rings' rows scored against 4 queries: the
// step 89.0 -> 85.6 us).  tiles: LDS, kMfmaTileBytes per wave, then 256 bytes per query.
constexpr int kMfmaTileBytes = 16 * 256 + 16 * 8 * 4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 dec_bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float dec_f32x4_t;

template <typename KV, int NQ, typename Visible>
__device__ __forceinline__ void partial_rows_mfma(const KV* __restrict__ kbase, const KV* __restrict__ vbase,
                                                  const float* __restrict__ kscale, const float* __restrict__ vscale,
                                                  int r_begin, int r_cap, Visible visible, const bf16_t* __restrict__ q0,
                                                  double scale, float* __restrict__ out, size_t out_head, float* red,
                                                  unsigned char* tiles) {
  constexpr int D = 128, EL = 8;
  constexpr float kLog2e = 1.4426950408889634f;
  constexpr float kSlack = 8.f;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int kb = lane >> 4, n = lane & 15;            // group inside the wave; lane inside the group
  int r_end = r_cap;                                  // until the first rows are requested
  unsigned char* kt = tiles + wv * kMfmaTileBytes;    // [16 rows][16 chunks of 16 B], chunk index xor row
  float* pt = reinterpret_cast<float*>(kt + 16 * 256); // [16 rows][8 queries]: scores, then terms p
  const bool holder = n < NQ;                         // this lane owns the scores of query n

  // The queries sit in LDS (chunk index xor query, like the K tile) and are read as operand B
  // of MFMA j (elements (4j + kb) * 8 .. + 7 of query n) every iteration: 4 registers instead of 16.
  unsigned char* qt = tiles + kPartWaves * kMfmaTileBytes;       // [NQ][16 chunks of 16 B]
  static_assert(NQ * 16 <= kPartThreads, "one chunk a thread");
  uint4 q_chunk;
  if (tid < NQ * 16) q_chunk = *reinterpret_cast<const uint4*>(q0 + (size_t)(tid >> 4) * D + (tid & 15) * 8);
  const float factor = (float)(scale * (double)kLog2e);

  float m[NQ], l[NQ], acc[NQ][EL];
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EL; ++e) acc[g][e] = 0.f;
  }
  float m_mine = -INFINITY, l_mine = 0.f;             // holder lanes: reference and sum of query n over rows 4kb .. 4kb+3

  // K rows are requested one iteration ahead (they are needed first, for the tile); V rows at the
  // end of the iteration before, so that they travel while the next scores are formed.
  // FP8 rows: the codes are bf16 numbers, so the products on the matrix cores are those of the codes; the K row's scale
  // multiplies the score, the V row's the term (both in the lanes of group kb, whose rows they are).
  constexpr bool kFp8 = sizeof(KV) == 1;
  using Raw = RawSlice<KV, EL>;
  Raw kn[4], vn[4];
  float ks[4], ksn[4], vs[4];
  bool okk[4], okv[4];
  auto fetch_k = [&](int r0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + 16 * wv + 4 * kb + u;
      okk[u] = r < r_end;                              // nothing is loaded past r_end
      if (okk[u]) kn[u].load(kbase + (size_t)r * D + n * EL);
      if constexpr (kFp8) ksn[u] = okk[u] ? kscale[r] : 0.f;
    }
  };
  auto fetch_v = [&](int r0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + 16 * wv + 4 * kb + u;
      okv[u] = r < r_end;
      if (okv[u]) vn[u].load(vbase + (size_t)r * D + n * EL);
      if constexpr (kFp8) vs[u] = okv[u] ? vscale[r] : 0.f;
    }
  };
  fetch_k(r_begin);
  fetch_v(r_begin);
  if (tid < NQ * 16) *reinterpret_cast<uint4*>(qt + (tid >> 4) * 256 + (((tid & 15) ^ (tid >> 4)) & 15) * 16) = q_chunk;
  __syncthreads();
  r_end = visible();
  if (r_begin >= r_end) {
    if (tid < NQ) { out[tid * out_head] = -INFINITY; out[tid * out_head + 1] = 0.f; }
    return;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) okk[u] = okv[u] = r_begin + 16 * wv + 4 * kb + u < r_end;
  for (int r0 = r_begin; r0 < r_end; r0 += 16 * kPartWaves) {
    // this iteration's K rows into the tile, the next ones requested
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = 4 * kb + u;
      uint4 chunk;
      if constexpr (kFp8) {
        float x[EL];
        kn[u].widen(x);
        auto pair = [&](int i) { return __builtin_amdgcn_perm(__float_as_uint(x[i + 1]), __float_as_uint(x[i]), 0x07060302u); };
        chunk = make_uint4(pair(0), pair(2), pair(4), pair(6));
        ks[u] = ksn[u];
      } else {
        chunk = make_uint4(kn[u].w[0], kn[u].w[1], kn[u].w[2], kn[u].w[3]);
      }
      if (okk[u]) *reinterpret_cast<uint4*>(kt + row * 256 + ((n ^ row) & 15) * 16) = chunk;
    }
    fetch_k(r0 + 16 * kPartWaves);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // S[row 4kb+i][query n] = sum over d; operand A of MFMA j: chunk 4j + kb of row n
    dec_f32x4_t sv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 a = *reinterpret_cast<const uint4*>(kt + n * 256 + (((4 * j + kb) ^ n) & 15) * 16);
      uint4 bq = make_uint4(0, 0, 0, 0);               // columns >= NQ of operand B are zero
      if (holder) bq = *reinterpret_cast<const uint4*>(qt + n * 256 + (((4 * j + kb) ^ n) & 15) * 16);
      sv = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8_t, a),
                                                   __builtin_bit_cast(dec_bf16x8_t, bq), sv, 0, 0, 0);
    }
    float s2[4];
    bool raise = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool valid = r0 + 16 * wv + 4 * kb + i < r_end;      // rows past the end hold stale tile data
      s2[i] = valid ? (kFp8 ? sv[i] * factor * ks[i] : sv[i] * factor) : -INFINITY;
      raise |= holder && s2[i] > m_mine + kSlack;
    }
    if (__any(raise)) {
      // raise the references: every lane learns the largest score of each query over the 16 rows
      float top = fmaxf(fmaxf(s2[0], s2[1]), fmaxf(s2[2], s2[3])), x, y;
      lane_pair<16>(top, x, y);
      lane_pair<32>(fmaxf(x, y), x, y);
      top = fmaxf(x, y);
#pragma unroll
      for (int g = 0; g < NQ; ++g) {
        const float mx = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(top), g));
        const float m_new = fmaxf(m[g], mx);
        const float corr = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m[g] - m_new);   // 0 while m[g] = -inf
#pragma unroll
        for (int e = 0; e < EL; ++e) acc[g][e] *= corr;
        if (n == g) { l_mine *= corr; m_mine = m_new; }
        m[g] = m_new;
      }
    }
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {                    // (a score that is NaN has a term, NaN: only those of -inf, rows past the end among them, have none)
      p[i] = (holder && s2[i] != -INFINITY) ? __builtin_amdgcn_exp2f(s2[i] - m_mine) : 0.f;
      l_mine += p[i];
    }
    if (holder) {
#pragma unroll
      for (int i = 0; i < 4; ++i) pt[(4 * kb + i) * 8 + n] = kFp8 ? p[i] * vs[i] : p[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (okv[u]) {
        float pr[8];                                   // terms of row 4kb+u for every query
        *reinterpret_cast<float4*>(&pr[0]) = *reinterpret_cast<const float4*>(pt + (4 * kb + u) * 8);
        if constexpr (NQ > 4) *reinterpret_cast<float4*>(&pr[4]) = *reinterpret_cast<const float4*>(pt + (4 * kb + u) * 8 + 4);
        float vv[EL];
        vn[u].widen(vv);
#pragma unroll
        for (int g = 0; g < NQ; ++g) {
#pragma unroll
          for (int e = 0; e < EL; ++e) acc[g][e] = fmaf(pr[g], vv[e], acc[g][e]);
        }
      }
    }
    fetch_v(r0 + 16 * kPartWaves);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the tile and pt are rewritten by the next iteration
  }
  // the sum of query g over this group's rows sits in lane g of the group
#pragma unroll
  for (int g = 0; g < NQ; ++g) l[g] = __shfl(l_mine, (lane & 48) + g, kWave);
  merge_partials<D, NQ, 16>(m, l, acc, out, out_head, red);
}

// Unit u of all sequences' rings (Hkv * ring_units each), and the position of its sequence's step.  Where the first 64 sequences'
// rings are full: sequence by sequence and ring by ring; else all rings' first units, then all their second ones, .., so that those
// without rows come last.  Uniform; called by whole waves.
// (The second order for full rings reads the same places of power-of-two strides at once: 8 x 12000 tokens 66.5 / 72.6.  The units
// with rows of each sequence counted, and those without put behind them: one round of loads and a scan for every 64 sequences,
// 4096 of them 111 us, now 94; 128 x 1000 190 / 153, 2 x 16000 29.5 / 29.3, 8 x 30011 141 / 140.)
struct RingUnit {
  int s, kvh, slot;
  int64_t T;
};
__device__ __forceinline__ RingUnit ring_unit(int u, const int64_t* __restrict__ length, int batch, int Hkv, int ring_units, int w) {
  if (batch == 1) {                                  // without vector loads: 0.3 us of a small step
    const int64_t T1 = length[0];
    if (T1 >= w) return {0, u / ring_units, u % ring_units, T1};
    return {0, u % Hkv, u / Hkv, T1};
  }
  const int lane = threadIdx.x & 63;
  int64_t T = w;
  if (lane < batch) T = length[lane];
  // both, while the lengths are on their way
  const int seq = Hkv * ring_units, s_f = u / seq, in_f = u - s_f * seq, kvh_f = in_f / ring_units;
  const int turn = batch * Hkv, slot_p = u / turn, in_p = u - slot_p * turn, s_p = in_p / Hkv;
  RingUnit r;
  if (__all(T >= w)) r = {s_f, kvh_f, in_f - kvh_f * ring_units, 0};
  else r = {s_p, in_p - s_p * Hkv, slot_p, 0};
  if (r.s < kWave) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)T, r.s), hi = __builtin_amdgcn_readlane((int)(T >> 32), r.s);
    r.T = (int64_t)((uint64_t)hi << 32 | lo);
  } else {
    r.T = length[r.s];
  }
  return r;
}

// grid (units, B); block kPartThreads.  Selection head hs serves the GQ query heads hs*GQ .. hs*GQ+GQ-1 (GQ = 1: one
// selection per query head).  The ring belongs to the KV head, so its units score each row against all GW query heads of
// the group.  Workgroups are numbered through (one dimension would leave them 2^24: 65535 sequences of 257), and in their order
// the rings' units of all sequences come first: they take the longest (FP8, four
// queries a row: 32 us where a region's takes 18), and with each sequence's in front of its regions the last one's ended 15 us
// behind everything else: FP8, 8 x 30011 tokens 90 / 85 us, 64 heads 169 / 154.  Rings that are half full, their empty units
// among the others, left half of the CUs, which are served in turn, without work: 32 x 2000 68 / 45.
// Then the regions', sequence by sequence, all heads' first chunks, then all heads' second ones, ..: in
// a cache with room to spare those that hold rows are neighbours, which the chip deals to its XCDs and CUs in turn, and the
// empty ones follow.  (Head after head, the first chunks of all heads may be on one or two XCDs.  us per step of 32 heads with
// room for 40000 rows each, head after head / this: 4 sequences of 1500 rows 91 / 53, 16 of 1500 286 / 162, 16 of 10000 618 /
// 518, 16 of 3000 with a shared selection 222 / 135; full caches, 16 x 128K tokens 1088 / 1066, 5 x 112K 790 / 768.)
template <typename T, typename KV, int D, int GQ, int GW, int LPR>
__global__ __launch_bounds__(kPartThreads) void decode_partial_kernel(
    tca_cache c, DecodeHeads dh, int Hq, int Hkv, int w, double scale, const T* __restrict__ q,
    const T* __restrict__ k_new, const T* __restrict__ v_new, uint32_t* __restrict__ pos, float* __restrict__ part) {
  constexpr int EL = D / 16;
  constexpr int NMAX = GQ > GW ? GQ : GW;
  __shared__ float red[kPartWaves * 16 * NMAX * (EL + 2)];
  // Rows that partial_rows_mfma takes.  FP8 rows that meet two queries are faster without: us on vector units / on the matrix cores,
  // rings only 1 x 8000 tokens 14.4 / 14.6, 4 x 12000 26.2 / 27.9, 8 x 30000 85.8 / 89.7, shared selection 1 x 100000 32.3 /
  // 36.8, 8 x 30000 51.4 / 53.2, 16 x 60000 180 / 178; three queries, shared, 8 x 30000 67.5 / 56.6.
  constexpr bool kMfma = D == 128 && (sizeof(KV) == 2 || (sizeof(KV) == 1 && GW > 2));
  __shared__ __attribute__((aligned(16))) unsigned char tiles[kMfma && NMAX > 1 ? kPartWaves * kMfmaTileBytes + NMAX * 256 : 16];
  const int Hs = Hq / GQ;
  const int all_ring_units = Hkv * dh.ring_units, region_units = dh.units - all_ring_units;
  // (dh.units, not gridDim.x or from unit0: those are lines of their own to wait for, 0.5 us of a step)
  const int number = blockIdx.y * dh.units + blockIdx.x;
  const int id = number - c.batch * all_ring_units;                   // < 0: a ring's
  RingUnit ru = {};
  if (id < 0) ru = ring_unit(number, c.length, c.batch, Hkv, dh.ring_units, w);
  const int s = id >= 0 ? id / region_units : ru.s;
  const int64_t Tpos = id >= 0 ? c.length[s] : ru.T;
  float* const seq_part = part + (size_t)s * ((size_t)GQ * region_units + (size_t)Hq * dh.ring_units) * (D + 2);
  if (id < 0 && ru.kvh == 0 && ru.slot == 0 && threadIdx.x == 0) pos[s] = (uint32_t)Tpos;       // for the merge that follows

  if (id >= 0) {
    // The lanes read the tables at once and they are looked up in registers: in memory, one lookup behind the other and each
    // line a miss at first, it cost the smallest steps 0.6 us of 17.
    const int r = id - s * region_units, lane = threadIdx.x & 63;
    auto in_regs = [&](auto table) {
      const int lo = lane < Hs ? table(lane) : INT32_MAX, hi = lane + 64 < Hs ? table(lane + 64) : INT32_MAX;
      return [=](int i) { return i < 64 ? __builtin_amdgcn_readlane(lo, i) : __builtin_amdgcn_readlane(hi, i - 64); };
    };
    const int f0 = lane < Hs ? dh.first[lane] : INT32_MAX, f1 = lane + 64 < Hs ? dh.first[lane + 64] : INT32_MAX;
    const auto by_units = in_regs([&](int i) { return (int)dh.by_units[i]; });
    const auto unit0 = in_regs([&](int i) { return dh.unit0[i]; });
    const auto unit1 = in_regs([&](int i) { return dh.unit0[i + 1]; });
    const auto rows = in_regs([&](int i) { return c.n_rows[s * Hs + i]; });
    // 2^32 / heads rounded up: its high product with a number below 2^25 is the quotient (heads <= 128; 1 has no such number)
    const auto magic = in_regs([&](int i) { return (int)(0xFFFFFFFFu / (uint32_t)(Hs - i) + 1); });
    const int i = __popcll(__ballot(f0 <= r)) + __popcll(__ballot(f1 <= r)) - 1, heads = Hs - i;
    const int in = r - (i < 64 ? __builtin_amdgcn_readlane(f0, i) : __builtin_amdgcn_readlane(f1, i - 64));
    const int turn = heads == 1 ? in : (int)__umulhi((uint32_t)in, (uint32_t)magic(i));
    const int hs = by_units(in - turn * heads), above = by_units(i ? heads : 0);
    const int u0 = unit0(hs), ns = unit1(hs) - u0, slot = turn + (i ? unit1(above) - unit0(above) : 0);
    const int r_begin = slot * dh.chunk;
    const size_t base = (size_t)s * c.cap_rows + dh.offs[hs];
    int len = rows(hs) - r_begin;
    if (len > dh.chunk) len = dh.chunk;
    // the rows that have left the window: looked up while the first ones are on their way
    auto visible = [&] { return r_begin + (len > 0 ? count_le_wave(c.idx + base + r_begin, len, Tpos - w) : 0); };
    float* out = seq_part + ((size_t)GQ * u0 + slot) * (D + 2);              // query g: + g * ns * (D+2)
    const size_t out_head = (size_t)ns * (D + 2);
    const T* q0 = q + ((size_t)s * Hq + hs * GQ) * D;
    if constexpr (kMfma && GQ > 1)
      partial_rows_mfma<KV, GQ>((const KV*)c.Kg + base * D, (const KV*)c.Vg + base * D, c.Kg_scale + base, c.Vg_scale + base,
                                r_begin, r_begin + len, visible, q0, scale, out, out_head, red, tiles);
    else
      partial_rows<T, KV, D, GQ, LPR>((const KV*)c.Kg + base * D, (const KV*)c.Vg + base * D, c.Kg_scale + base,
                                 c.Vg_scale + base, r_begin, r_begin + len, visible, q0, scale, out, out_head, red);
  } else {
    const int kvh = ru.kvh, slot = ru.slot, h0 = kvh * GW;
    const int r_begin = slot * dh.chunk;
    const size_t base = ((size_t)s * Hkv + kvh) * w;
    // Slot r of the ring holds the latest position congruent to r mod w that is <= Tpos.  Once
    // Tpos >= w every slot is filled; before that only slots 0 .. Tpos are.
    const int filled = Tpos >= w ? w : (int)Tpos + 1;
    const int r_end = min(filled, r_begin + dh.chunk);
    auto visible = [&] { return r_end; };
    const int newest = (int)(Tpos % w);
    if (newest >= r_begin && newest < r_begin + dh.chunk)
      store_new_row<T, KV, D>(c, base + newest, k_new + ((size_t)s * Hkv + kvh) * D, v_new + ((size_t)s * Hkv + kvh) * D);
    float* out = seq_part + ((size_t)GQ * region_units + (size_t)h0 * dh.ring_units + slot) * (D + 2);
    const size_t out_head = (size_t)dh.ring_units * (D + 2);
    const T* q0 = q + ((size_t)s * Hq + h0) * D;
    if constexpr (kMfma && GW > 1)
      partial_rows_mfma<KV, GW>((const KV*)c.ringK + base * D, (const KV*)c.ringV + base * D, c.ringK_scale + base,
                                c.ringV_scale + base, r_begin, r_end, visible, q0, scale, out, out_head, red, tiles);
    else
      partial_rows<T, KV, D, GW, 16>((const KV*)c.ringK + base * D, (const KV*)c.ringV + base * D, c.ringK_scale + base,
                                 c.ringV_scale + base, r_begin, r_end, visible, q0, scale, out, out_head, red);
  }
}

// grid (Hq, B); block 256.  A thread merges four columns over its share of the head's partials, reference and sum carried
// along, so that one round of loads stands between the launch and the sums in LDS (a pass for the references, one for the
// weights and one for the columns, and the workgroups of a sequence counted through an atomic before its length could
// advance: 6.7 us for 35 partials a head, now 4.6; 132 partials, 16 sequences: 12.3 / 7.7; 27 partials, 32 sequences: 15.8 / 7.6).
template <typename T, typename KV, int D>
__global__ __launch_bounds__(kDecThreads) void decode_merge_kernel(
    tca_cache c, DecodeHeads dh, int Hq, int Hkv, int GS, int w, int b, double scale,
    const T* __restrict__ q, const float* __restrict__ part, const uint32_t* __restrict__ pos, T* __restrict__ O) {
  constexpr int EL = D / 16;
  __shared__ double xs[256];
  __shared__ double gred[kDecThreads / kWave];
  __shared__ int32_t sel[256];
  __shared__ int32_t wave_cnt[kDecThreads / kWave];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int h = blockIdx.x, s = blockIdx.y;
  const int G = Hq / Hkv, kvh = h / G;
  const int hs = h / GS, Hs = Hq / GS;
  // the head's partials: those of its region, then those of its ring
  const int ns = dh.unit0[hs + 1] - dh.unit0[hs], n_slots = ns + dh.ring_units;
  const float* const seq_part = part + (size_t)s * ((size_t)GS * dh.unit0[Hs] + (size_t)Hq * dh.ring_units) * (D + 2);
  const float* const p_region = seq_part + ((size_t)GS * dh.unit0[hs] + (size_t)(h - hs * GS) * ns) * (D + 2);
  const float* const p_ring = seq_part + ((size_t)GS * dh.unit0[Hs] + (size_t)h * dh.ring_units) * (D + 2);
  auto partial_at = [&](int x) { return x < ns ? p_region + (size_t)x * (D + 2) : p_ring + (size_t)(x - ns) * (D + 2); };
  // The first head's workgroup advances the sequence's length while others may still read it: the low half the partial
  // kernel left tells which of the two values they saw.
  const int64_t len = __hip_atomic_load(&c.length[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t Tpos = len - ((uint32_t)len != pos[s] ? 1 : 0);

  constexpr int CQ = D / 4;                              // column quads of a partial
  constexpr int SPLIT = kDecThreads / CQ;                // threads per column quad
  constexpr int UN = 4;                                  // partials of a thread in flight
  __shared__ __attribute__((aligned(16))) float colsum[SPLIT][D];
  // fp32 rows: the sum in fp64, for a thread adds its partials one behind the other and in fp32 a small one behind a large one
  // is rounded away.  Error against 64 bits, mean of 40 calls: 1.24e-7, with fp64 1.09e-7, in the same time.
  using sum_t = std::conditional_t<sizeof(T) == 4, double, float>;
  __shared__ float refs[SPLIT];
  __shared__ sum_t sums[SPLIT];
  {
    const int cq = tid % CQ, mine = tid / CQ;
    // the columns of an empty partial were never written: read all the same where there are few, so that they do not
    // wait for the sums
    const bool few = n_slots <= 2 * UN * SPLIT;
    float M = -INFINITY, a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    sum_t L = 0;
    for (int x0 = mine; x0 < n_slots; x0 += UN * SPLIT) {
      const float* src[UN];
      float2 ml[UN], lo[UN], hi[UN];                     // partials are 8-byte aligned
      auto columns = [&](int u) {
        lo[u] = *reinterpret_cast<const float2*>(src[u] + 2 + 4 * cq);
        hi[u] = *reinterpret_cast<const float2*>(src[u] + 4 + 4 * cq);
      };
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int x = x0 + u * SPLIT;
        src[u] = partial_at(min(x, n_slots - 1));
        ml[u] = *reinterpret_cast<const float2*>(src[u]);
        if (x >= n_slots) ml[u] = make_float2(-INFINITY, 0.f);
        lo[u] = hi[u] = make_float2(0.f, 0.f);
        if (few) columns(u);
      }
      float m_new = M;
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        if (!few && ml[u].y != 0.f) columns(u);
        if (ml[u].y != 0.f) m_new = fmaxf(m_new, ml[u].x);             // (a NaN sum is no empty partial)
      }
      const float corr = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(M - m_new);   // references are in base-2 units
      L *= corr; a0 *= corr; a1 *= corr; a2 *= corr; a3 *= corr;
      M = m_new;
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        if (ml[u].y != 0.f) {
          const float wx = __builtin_amdgcn_exp2f(ml[u].x - M);
          L += (sum_t)ml[u].y * wx;
          a0 += lo[u].x * wx; a1 += lo[u].y * wx; a2 += hi[u].x * wx; a3 += hi[u].y * wx;
        }
      }
    }
    *reinterpret_cast<float4*>(&colsum[mine][4 * cq]) = make_float4(a0, a1, a2, a3);
    if (cq == 0) { refs[mine] = M; sums[mine] = L; }
    __syncthreads();
    if (tid < D) {
      float R = -INFINITY, t = 0.f;
      sum_t Lt = 0;
#pragma unroll
      for (int x = 0; x < SPLIT; ++x) R = fmaxf(R, refs[x]);
#pragma unroll
      for (int x = 0; x < SPLIT; ++x) {
        const float wx = sums[x] == 0 ? 0.f : __builtin_amdgcn_exp2f(refs[x] - R);
        Lt += sums[x] * wx;
        t += colsum[x][tid] * wx;
      }
      store_f32(O + ((size_t)s * Hq + h) * D + tid, (float)(t / Lt));
    }
  }
  if (h == 0 && tid == 0) __hip_atomic_store(&c.length[s], Tpos + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // block completed by this token?
  // (one workgroup per selection head ranks the block)
  if ((Tpos + 1) % b != 0 || h % GS != 0) return;
  const int64_t p0 = Tpos + 1 - b;                     // first position of the block
  const int slot0 = (int)(p0 % w);                     // contiguous in the ring: w is a multiple of b
  const size_t ring_row0 = ((size_t)s * Hkv + kvh) * w + slot0;
  const KV* kb = (const KV*)c.ringK + ring_row0 * D;
  const KV* vb = (const KV*)c.ringV + ring_row0 * D;
  const int grp = tid >> 4, sub = tid & 15;
  // score of row i: the logit of the head's query, or, for a shared selection, the sum over the
  // group's heads of exp(logit - log-sum-exp over the block) (G times the mean score)
  double score = 0.0;
  for (int g = 0; g < GS; ++g) {
    float qf[EL];
    load_slice<T, EL>(q + ((size_t)s * Hq + h + g) * D + sub * EL, qf);
    __syncthreads();                                   // xs of the previous head has been consumed
    for (int r0 = 0; r0 < b; r0 += 16) {
      const int r = r0 + grp;
      double a = 0.0;
      if (r < b) {
        float kf[EL];
        RawSlice<KV, EL> raw;
        raw.load(kb + (size_t)r * D + sub * EL);
        raw.widen(kf);
#pragma unroll
        for (int e = 0; e < EL; ++e) a = fma((double)kf[e], (double)qf[e], a);
        if constexpr (sizeof(KV) == 1) a *= (double)c.ringK_scale[ring_row0 + r];   // the row read back: code * scale
      }
      a = group_sum(a, 16);
      if (r < b && sub == 0) xs[r] = a * scale;
    }
    __syncthreads();
    if (GS == 1) {
      if (tid < b) score = xs[tid];
    } else {
      const double xi = tid < b ? xs[tid] : -INFINITY;
      double mx = group_max(xi, kWave);
      if (lane == 0) gred[wv] = mx;
      __syncthreads();
      mx = fmax(fmax(gred[0], gred[1]), fmax(gred[2], gred[3]));
      __syncthreads();
      const double e = tid < b ? exp(xi - mx) : 0.0;
      const double zs = group_sum(e, kWave);
      if (lane == 0) gred[wv] = zs;
      __syncthreads();
      score += e / ((gred[0] + gred[1]) + (gred[2] + gred[3]));
    }
  }
  __syncthreads();
  if (tid < b) xs[tid] = score;
  __syncthreads();
  const int t = dh.t_dec[hs];
  bool keep = false;
  if (tid < b) {
    const double xi = xs[tid];
    int cnt = 0;
    for (int o = 0; o < b; ++o) {
      const double xo = xs[o];
      cnt += (xo > xi) || (xo == xi && o < tid);
    }
    keep = cnt < t;
  }
  const unsigned long long mask = __ballot(keep);
  if (lane == 0) wave_cnt[wv] = __popcll(mask);
  __syncthreads();
  int before = __popcll(mask & ((1ull << lane) - 1ull));
  for (int x = 0; x < wv; ++x) before += wave_cnt[x];
  if (keep) sel[before] = tid;
  __syncthreads();
  const int64_t cap = dh.offs[hs + 1] - dh.offs[hs];
  const int32_t fill = c.n_rows[s * Hs + hs];
  const size_t base = (size_t)s * c.cap_rows + dh.offs[hs];
  KV* Kg = (KV*)c.Kg;
  KV* Vg = (KV*)c.Vg;
  for (int k = grp; k < t; k += 16) {
    const int64_t row = (int64_t)fill + k;
    if (row >= cap) break;
    const int src = sel[k];
    for (int e = 0; e < EL; ++e) {                     // rows are copied as stored
      Kg[(base + row) * D + sub * EL + e] = kb[(size_t)src * D + sub * EL + e];
      Vg[(base + row) * D + sub * EL + e] = vb[(size_t)src * D + sub * EL + e];
    }
    if (sub == 0) {
      c.idx[base + row] = (int32_t)(p0 + src);
      if constexpr (sizeof(KV) == 1) {
        c.Kg_scale[base + row] = c.ringK_scale[ring_row0 + src];
        c.Vg_scale[base + row] = c.ringV_scale[ring_row0 + src];
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    int64_t nf = (int64_t)fill + t;
    c.n_rows[s * Hs + hs] = (int32_t)(nf > cap ? cap : nf);
  }
}

// Both handover kernels are HBM-bound copies: one 16-lane group per row, kCopyRows (kWinRows) rows of K and of V per
// group requested before the first is stored.  The two launches of a sequence of 32768 tokens and 32 heads that keeps a third of
// its rows, into the FP8 cache, take 54.6 us (58.5 on rows that are not in the caches); with four rows of the regions at a time
// 56.8 (63.4), two of the window 54.7 (58.7).  8192 tokens 22.1; 24.6 and 23.1.
constexpr int kCopyRows = 2, kWinRows = 1;

// grid (ceil(rows / (16 kWinRows)), Hkv); block 256
template <typename T, typename KV, int D, bool ALIGNED>
__global__ __launch_bounds__(256) void load_window_kernel(tca_cache c, int seq, int Hkv, int w, const T* __restrict__ K,
                                                          const T* __restrict__ V, int64_t kv_stride, int64_t L) {
  const int kvh = blockIdx.y, sub = threadIdx.x & 15;
  const int64_t first = L - w > 0 ? L - w : 0;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) c.length[seq] = L;
  const int64_t pos0 = first + (int64_t)blockIdx.x * (16 * kWinRows) + (threadIdx.x >> 4);
  RowCopy<T, KV, D, ALIGNED> k[kWinRows], v[kWinRows];
#pragma unroll
  for (int u = 0; u < kWinRows; ++u) {
    const int64_t pos = pos0 + u * 16;
    if (pos < L) {
      k[u].load(K + ((size_t)kvh * kv_stride + pos) * D, sub);
      v[u].load(V + ((size_t)kvh * kv_stride + pos) * D, sub);
    }
  }
#pragma unroll
  for (int u = 0; u < kWinRows; ++u) {
    const int64_t pos = pos0 + u * 16;
    if (pos < L) {                                     // (all 16 lanes of a group alike)
      const size_t row = ((size_t)seq * Hkv + kvh) * w + (int)(pos % w);
      k[u].store((KV*)c.ringK + row * D, c.ringK_scale + row, sub);
      v[u].store((KV*)c.ringV + row * D, c.ringV_scale + row, sub);
    }
  }
}

// grid (ceil(cap_rows / (16 kCopyRows))); block 256
template <typename T, typename KV, int D, bool ALIGNED>
__global__ __launch_bounds__(256) void load_global_kernel(tca_cache c, int seq, DecodeHeads dh, int Hs,
                                                          const int32_t* __restrict__ idx, const T* __restrict__ Kg,
                                                          const T* __restrict__ Vg, const int32_t* __restrict__ n_rows) {
  const int sub = threadIdx.x & 15;
  if (blockIdx.x == 0 && threadIdx.x < Hs) c.n_rows[(size_t)seq * Hs + threadIdx.x] = n_rows[threadIdx.x];
  // The heads whose regions hold the workgroup's first and last row, found by all lanes at once.  As a rule they are one:
  // then its rows are counted once for all, and two rounds of loads stand in front of the rows' own (a search and a count for
  // every row were ten: the handover of 32768 tokens 42.9 us, now 40.8).
  const int64_t first = (int64_t)blockIdx.x * (16 * kCopyRows);
  const int lane = threadIdx.x & 63;
  const int64_t end0 = lane < Hs ? dh.offs[lane + 1] : INT64_MAX, end1 = lane + 64 < Hs ? dh.offs[lane + 65] : INT64_MAX;
  auto head_of = [&](int64_t r) { return __popcll(__ballot(end0 <= r)) + __popcll(__ballot(end1 <= r)); };
  const int h0 = head_of(first);
  const bool one = h0 == head_of(first + 16 * kCopyRows - 1);
  int64_t filled = 0;                              // one: rows from the workgroup's first one on
  if (one) filled = dh.offs[h0] + n_rows[h0] - first;
  RowCopy<T, KV, D, ALIGNED> k[kCopyRows], v[kCopyRows];
  int32_t at[kCopyRows];
  bool ok[kCopyRows];
#pragma unroll
  for (int u = 0; u < kCopyRows; ++u) {
    const int64_t r = first + u * 16 + (threadIdx.x >> 4);
    if (one) {
      ok[u] = r - first < filled;                  // not the capacity beyond the filled rows
    } else {
      int h = h0;
      while (h + 1 < Hs && dh.offs[h + 1] <= r) ++h;
      ok[u] = r < c.cap_rows && r - dh.offs[h] < n_rows[h];
    }
    if (ok[u]) {
      at[u] = idx[r];
      k[u].load(Kg + (size_t)r * D, sub);
      v[u].load(Vg + (size_t)r * D, sub);
    }
  }
#pragma unroll
  for (int u = 0; u < kCopyRows; ++u) {
    if (ok[u]) {
      const size_t dst = (size_t)seq * c.cap_rows + first + u * 16 + (threadIdx.x >> 4);
      if (sub == 0) c.idx[dst] = at[u];
      k[u].store((KV*)c.Kg + dst * D, c.Kg_scale + dst, sub);
      v[u].store((KV*)c.Vg + dst * D, c.Vg_scale + dst, sub);
    }
  }
}

// May rows be copied 16 bytes at a time?  (rows are multiples of 64 bytes)
static bool aligned16(const void* a, const void* b, const void* c, const void* d) {
  return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)d) & 15) == 0;
}

static int check_cache(const tca_params* prm, const tca_cache* c) {
  if (!c) return fail(TCA_ERR_INVALID, "cache is NULL");
  if (c->batch < 1 || c->cap_rows < 0) return fail(TCA_ERR_INVALID, "cache: batch=%d cap_rows=%lld", c->batch,
                                                   (long long)c->cap_rows);
  if (!c->idx || !c->Kg || !c->Vg || !c->n_rows || !c->ringK || !c->ringV || !c->length)
    return fail(TCA_ERR_INVALID, "cache: NULL pointer member");
  if (c->kv_format != TCA_KV_NATIVE && c->kv_format != TCA_KV_FP8)
    return fail(TCA_ERR_UNSUPPORTED, "cache: kv_format=%d", c->kv_format);
  if (c->kv_format == TCA_KV_FP8) {
    if (prm->dtype != TCA_BF16) return fail(TCA_ERR_UNSUPPORTED, "cache: TCA_KV_FP8 requires dtype TCA_BF16");
    if (!c->Kg_scale || !c->Vg_scale || !c->ringK_scale || !c->ringV_scale)
      return fail(TCA_ERR_INVALID, "cache: NULL scale pointer with TCA_KV_FP8");
  }
  return TCA_OK;
}

// Fills dh.chunk, dh.ring_units and dh.unit0 for chunks of `chunk` rows; the workgroups per sequence.
static int64_t set_chunk(DecodeHeads& dh, const tca_params* prm, int chunk) {
  const int Hs = sel_heads(prm);
  int64_t run = 0;
  for (int h = 0; h < Hs; ++h) {
    dh.unit0[h] = (int32_t)run;
    run += chunks_of(dh.offs[h + 1] - dh.offs[h], chunk);
  }
  dh.unit0[Hs] = (int32_t)run;
  dh.chunk = chunk;
  dh.ring_units = (int32_t)chunks_of(prm->window, chunk);
  run += (int64_t)prm->n_kv_heads * dh.ring_units;
  dh.units = (int32_t)run;
  return run;
}

static size_t ws_of(const DecodeHeads& dh, const tca_params* prm, int batch) {
  return carve_decode_ws(nullptr, batch, prm->n_q_heads, prm->head_dim,
                         (int64_t)sel_group(prm) * dh.unit0[sel_heads(prm)] + (int64_t)prm->n_q_heads * dh.ring_units).bytes;
}

// The chunk length of a step: the shortest that stays within short_units workgroups (and the workspace), the full one
// from there on.
static int64_t choose_chunk(DecodeHeads& dh, const tca_params* prm, int batch, size_t ws_bytes) {
  for (int c = kMinChunk; c < long_chunk(prm); c *= 2) {
    const int64_t units = set_chunk(dh, prm, c);
    if (units * batch <= short_units(prm) && ws_of(dh, prm, batch) <= ws_bytes) return units;
  }
  return set_chunk(dh, prm, long_chunk(prm));
}

// The order of the regions' workgroups, all heads' first chunks first: heads sorted by their number of units, most first; the
// chunks in which the same heads take part form a piece.  Piece i holds the first Hs - i heads, and the chunks from the
// number of units of head Hs - i of that order (0 for i = 0) to that of the one before it; its workgroups start at number
// first[i], chunk by chunk.
static void order_units(DecodeHeads& dh, int Hs) {
  auto units = [&](int h) { return dh.unit0[h + 1] - dh.unit0[h]; };
  uint32_t key[TCA_MAX_HEADS];                         // units, then the head (there are at most kMaxSlots units per head)
  for (int h = 0; h < Hs; ++h) key[h] = (uint32_t)units(h) << 8 | (uint32_t)(255 - h);
  std::sort(key, key + Hs, std::greater<uint32_t>());
  for (int h = 0; h < Hs; ++h) dh.by_units[h] = (uint8_t)(255 - (key[h] & 255u));
  int32_t run = 0, before = 0;
  for (int i = 0; i < Hs; ++i) {
    const int32_t upto = units(dh.by_units[Hs - 1 - i]);
    dh.first[i] = run;
    run += (upto - before) * (Hs - i);
    before = upto;
  }
}

// FP8 rows of 128 elements that meet one query: eight lanes a row, 16 bytes each, which halves the reductions and exponentials per
// byte, where chunks are this long; in shorter ones, of two or four rounds of 64 rows, sixteen lanes of 8 bytes have twice the loads to start
// with (and with groups of one or two queries six and five waves a SIMD instead of four).  us per step with sixteen / with eight, chunks of
// 1024 rows: 32 heads, 16 x 60000 tokens 278 / 272; of 512: 2 x 100000 72.9 / 63.7, 8 x 30011 86.2 / 83.3, 64 heads 164 / 154, 16 KV heads
// 104 / 96, 32 KV heads 123 / 119; of 256: 4 x 30000 43.1 / 43.4, 16 KV heads 44.0 / 46.3; of 128: 2 x 16000 23.9 / 24.6, 4 x 12000
// 29.9 / 30.5, 16 KV heads 2 x 16000 25.1 / 26.6, 32 KV heads 2 x 8000 23.0 / 25.4.  (Two rows ahead in both.  Four with eight lanes: 64
// heads, 8 x 8000 52.9 instead of 52.2, 4 x 12000 39.2 instead of 38.6; with sixteen, 2 x 16000 37.5 instead of 37.1.)
constexpr int kWideRows = 512;

template <typename T, typename KV, int D>
static int run_decode(const tca_params* prm, const tca_cache* c, const DecodeHeads& dh, int64_t units, const T* q,
                      const T* k_new, const T* v_new, T* O, void* ws, hipStream_t st) {
  const int Hq = prm->n_q_heads, Hkv = prm->n_kv_heads, B = c->batch, w = prm->window;
  const int GS = sel_group(prm);
  const DecodeWs dw = carve_decode_ws(ws, B, Hq, D, 0);
  const double sc = logit_scale(prm);
  // (queries per region row, queries per ring row): (G, G) for a shared selection, else (1, G)
  const int G = Hq / Hkv;
  constexpr int kWideLpr = sizeof(KV) == 1 && D == 128 ? 8 : 16;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)units, B), dim3(kPartThreads), 0, st, *c, dh, Hq, Hkv, w, sc, q, k_new, v_new,
                       dw.pos, dw.part);
  };
#define TCA_PARTIAL_CASE(GG)                                                                  \
  case GG:                                                                                    \
    if (GS > 1) launch(decode_partial_kernel<T, KV, D, GG, GG, 16>);                          \
    else if (dh.chunk >= kWideRows) launch(decode_partial_kernel<T, KV, D, 1, GG, kWideLpr>); \
    else launch(decode_partial_kernel<T, KV, D, 1, GG, 16>);                                  \
    break;
  switch (G) {
    TCA_PARTIAL_CASE(1) TCA_PARTIAL_CASE(2) TCA_PARTIAL_CASE(3) TCA_PARTIAL_CASE(4)
    TCA_PARTIAL_CASE(5) TCA_PARTIAL_CASE(6) TCA_PARTIAL_CASE(7) TCA_PARTIAL_CASE(8)
  }
#undef TCA_PARTIAL_CASE
  hipLaunchKernelGGL((decode_merge_kernel<T, KV, D>), dim3(Hq, B), dim3(kDecThreads), 0, st, *c, dh, Hq, Hkv, GS, w,
                     prm->block, sc, q, dw.part, dw.pos, O);
  return TCA_OK;
}

}  // namespace tca

using namespace tca;

extern "C" size_t tca_decode_workspace_bytes(const tca_params* prm, int batch, int64_t max_head_rows) {
  if (check_params(prm) != TCA_OK || batch < 1 || max_head_rows < 0) return 0;
  return decode_ws_bytes(prm, batch, max_head_rows);
}

extern "C" int tca_cache_load_window(const tca_params* prm, const tca_cache* cache, int seq, const void* K,
                                     const void* V, int64_t kv_stride, int64_t L, void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  rc = check_cache(prm, cache);
  if (rc) return rc;
  if (!K || !V || seq < 0 || seq >= cache->batch || L < 0 || L > kv_stride)
    return fail(TCA_ERR_INVALID, "tca_cache_load_window: seq=%d L=%lld kv_stride=%lld", seq, (long long)L,
                (long long)kv_stride);
  const int w = prm->window;
  const int64_t rows = L < w ? L : w;
  const int64_t blocks = (rows + 16 * kWinRows - 1) / (16 * kWinRows);
  dim3 grid((unsigned)(blocks > 0 ? blocks : 1), prm->n_kv_heads);
  const bool wide = aligned16(K, V, cache->ringK, cache->ringV);
  hipStream_t st = (hipStream_t)stream;
  const bool d128 = prm->head_dim == 128;
  auto go = [&](auto kernel, auto tag) {
    using TT = decltype(tag);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, *cache, seq, prm->n_kv_heads, w, (const TT*)K, (const TT*)V, kv_stride, L);
  };
#define TCA_LOAD_WINDOW(TT, KK, DD)                                      \
  do {                                                                   \
    if (wide) go(load_window_kernel<TT, KK, DD, true>, TT{});            \
    else go(load_window_kernel<TT, KK, DD, false>, TT{});                \
  } while (0)
  if (cache->kv_format == TCA_KV_FP8) { if (d128) TCA_LOAD_WINDOW(bf16_t, fp8_t, 128); else TCA_LOAD_WINDOW(bf16_t, fp8_t, 64); }
  else if (prm->dtype == TCA_BF16) { if (d128) TCA_LOAD_WINDOW(bf16_t, bf16_t, 128); else TCA_LOAD_WINDOW(bf16_t, bf16_t, 64); }
  else { if (d128) TCA_LOAD_WINDOW(float, float, 128); else TCA_LOAD_WINDOW(float, float, 64); }
#undef TCA_LOAD_WINDOW
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}

extern "C" int tca_cache_load_global(const tca_params* prm, const tca_cache* cache, int seq, const int32_t* idx,
                                     const void* Kg, const void* Vg, const int64_t* offs, const int32_t* n_rows,
                                     void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  rc = check_cache(prm, cache);
  if (rc) return rc;
  const int Hs = sel_heads(prm);
  if (!idx || !Kg || !Vg || !offs || !n_rows || seq < 0 || seq >= cache->batch)
    return fail(TCA_ERR_INVALID, "tca_cache_load_global: NULL pointer argument or seq=%d outside the batch", seq);
  if (offs[0] != 0 || offs[Hs] != cache->cap_rows)
    return fail(TCA_ERR_INVALID, "tca_cache_load_global: offs[0] must be 0 and offs[Hs] must equal cap_rows");
  DecodeHeads dh;
  for (int h = 0; h < Hs; ++h) {
    if (offs[h + 1] < offs[h]) return fail(TCA_ERR_INVALID, "tca_cache_load_global: offs not ascending at %d", h);
    dh.offs[h] = offs[h];
    dh.t_dec[h] = 0;
  }
  dh.offs[Hs] = offs[Hs];
  if (cache->cap_rows == 0) return TCA_OK;
  hipStream_t st = (hipStream_t)stream;
  dim3 grid((unsigned)((cache->cap_rows + 16 * kCopyRows - 1) / (16 * kCopyRows)));
  const bool wide = aligned16(Kg, Vg, cache->Kg, cache->Vg);
  const bool d128 = prm->head_dim == 128;
  auto go = [&](auto kernel, auto tag) {
    using TT = decltype(tag);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, *cache, seq, dh, Hs, idx, (const TT*)Kg, (const TT*)Vg, n_rows);
  };
#define TCA_LOAD_GLOBAL(TT, KK, DD)                                      \
  do {                                                                   \
    if (wide) go(load_global_kernel<TT, KK, DD, true>, TT{});            \
    else go(load_global_kernel<TT, KK, DD, false>, TT{});                \
  } while (0)
  if (cache->kv_format == TCA_KV_FP8) { if (d128) TCA_LOAD_GLOBAL(bf16_t, fp8_t, 128); else TCA_LOAD_GLOBAL(bf16_t, fp8_t, 64); }
  else if (prm->dtype == TCA_BF16) { if (d128) TCA_LOAD_GLOBAL(bf16_t, bf16_t, 128); else TCA_LOAD_GLOBAL(bf16_t, bf16_t, 64); }
  else { if (d128) TCA_LOAD_GLOBAL(float, float, 128); else TCA_LOAD_GLOBAL(float, float, 64); }
#undef TCA_LOAD_GLOBAL
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}

// Argument checks and the two launches of a step, on a caller-visible scratch buffer.
static int decode_step(const tca_params* prm, const tca_cache* cache, const int64_t* offs, const void* q,
                       const void* k_new, const void* v_new, const double* p, void* O, void* ws, size_t ws_bytes,
                       void* stream, const char* who) {
  int rc = check_params(prm);
  if (rc) return rc;
  rc = check_cache(prm, cache);
  if (rc) return rc;
  if (!offs || !q || !k_new || !v_new || !p || !O || !ws)
    return fail(TCA_ERR_INVALID, "%s: NULL pointer argument", who);
  const int Hs = sel_heads(prm), b = prm->block, nk = block_log2(b) + 1;
  if (offs[0] != 0 || offs[Hs] != cache->cap_rows)
    return fail(TCA_ERR_INVALID, "%s: offs[0] must be 0 and offs[Hs] must equal cap_rows", who);
  DecodeHeads dh;
  int64_t max_rows = 0;
  for (int h = 0; h < Hs; ++h) {
    if (offs[h + 1] < offs[h]) return fail(TCA_ERR_INVALID, "%s: offs not ascending at %d", who, h);
    if (offs[h + 1] - offs[h] > INT32_MAX) return fail(TCA_ERR_UNSUPPORTED, "head region beyond int32 rows");
    if (offs[h + 1] - offs[h] > max_rows) max_rows = offs[h + 1] - offs[h];
    if (!valid_config(p + (size_t)h * nk, nk))
      return fail(TCA_ERR_INVALID, "%s: p[%d] is not a distribution", who, h);
    dh.offs[h] = offs[h];
    dh.t_dec[h] = tca_decode_budget(b, p + (size_t)h * nk);
  }
  dh.offs[Hs] = offs[Hs];
  if (chunks_of(max_rows, long_chunk(prm)) + chunks_of(prm->window, long_chunk(prm)) > kMaxSlots)
    return fail(TCA_ERR_UNSUPPORTED, "%s: more than %d split-K slots per head", who, kMaxSlots);
  const size_t need = decode_ws_need(prm, cache->batch, max_rows);
  if (ws_bytes < need || ((uintptr_t)ws & 255))
    return fail(TCA_ERR_WORKSPACE, "%s: scratch needs %zu bytes, 256-byte aligned; %zu available", who, need,
                ws_bytes);
  const int64_t units = choose_chunk(dh, prm, cache->batch, ws_bytes);
  order_units(dh, Hs);
  // (a unit's partial takes 264 bytes or more: 2^31 of them have no place on a GPU)
  if (units * cache->batch > INT32_MAX || cache->batch > 65535) return fail(TCA_ERR_UNSUPPORTED, "%s: batch=%d", who, cache->batch);
  hipStream_t st = (hipStream_t)stream;
#define TCA_RUN_DECODE(TT, KK)                                                                                         \
  (prm->head_dim == 128                                                                                                \
       ? run_decode<TT, KK, 128>(prm, cache, dh, units, (const TT*)q, (const TT*)k_new, (const TT*)v_new, (TT*)O, ws, st) \
       : run_decode<TT, KK, 64>(prm, cache, dh, units, (const TT*)q, (const TT*)k_new, (const TT*)v_new, (TT*)O, ws, st))
  if (cache->kv_format == TCA_KV_FP8) rc = TCA_RUN_DECODE(bf16_t, fp8_t);
  else if (prm->dtype == TCA_BF16) rc = TCA_RUN_DECODE(bf16_t, bf16_t);
  else rc = TCA_RUN_DECODE(float, float);
#undef TCA_RUN_DECODE
  if (rc) return rc;
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}

extern "C" int tca_decode(const tca_params* prm, const tca_cache* cache, const int64_t* offs, const void* q,
                          const void* k_new, const void* v_new, const double* p, void* O, void* ws,
                          size_t ws_bytes, void* stream) {
  return decode_step(prm, cache, offs, q, k_new, v_new, p, O, ws, ws_bytes, stream, "tca_decode");
}

// ---- tca_decode_static: the same step for callers that cannot provide scratch memory.
// The split-K partials live in an array that is part of the library's code object: every GPU the
// library runs on holds its own copy, at its own address, from the moment the code object is
// loaded until the process ends.  `scratch` below is only a host-side handle of that array; the
// device address is asked for once per device and kept.
static __device__ __align__(256) unsigned char scratch[TCA_DECODE_STATIC_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_addr[kMaxDevices];
}  // namespace

extern "C" int tca_decode_static(const tca_params* prm, const tca_cache* cache, const int64_t* offs, const void* q,
                                 const void* k_new, const void* v_new, const double* p, void* O, void* stream) {
  int dev = -1;
  TCA_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(TCA_ERR_UNSUPPORTED, "tca_decode_static: device %d", dev);
  void* ptr = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (!ptr) {                                          // first call on this device (it is the current one)
    TCA_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(TCA_ERR_HIP, "tca_decode_static: no device address for the scratch array");
    g_scratch_addr[dev].store(ptr, std::memory_order_release);   // racing first calls store the same address
  }
  return decode_step(prm, cache, offs, q, k_new, v_new, p, O, ptr, (size_t)TCA_DECODE_STATIC_BYTES, stream,
                     "tca_decode_static");
}
