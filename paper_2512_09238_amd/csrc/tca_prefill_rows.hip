// fp32 prefill attention (Eq. 2; Alg. 2 line 7): the TCA_F32 path.
//
// Logits (in units of ln 2) and the running maximum are fp64 (the products of fp32 inputs are exact in it), so that the exponent
// x - max carries no cancellation error even when the logits are in the hundreds; exponentials, sums and P.V are
// fp32.  Both products run on the matrix cores: S^T = K Q^T with v_mfma_f64_16x16x4_f64 on operands widened in
// registers, O^T = V^T P^T with v_mfma_f32_16x16x4_f32.  The bound is the fp64 product: 64 cycles per 16 x 16 x 4
// block and SIMD against 32 for the fp32 one.
//
// A wave owns 16 queries; lane (kb = lane / 16, c = lane % 16) holds, of every 16-key block, the scores of the
// keys kb + 4 r (r = 0 .. 3) against query c, which is where P^T must lie as operand B of the second product if
// its step r takes those keys: no exchange between the two.  The order of the head's elements inside the first
// product is free as long as K and Q agree: lane kb takes the kb-th quarter of a row, so that K is read from LDS
// 16 bytes at a time (chunk index xor row, conflict-free); in the second, row i of block s is element
// (D / 16) i + s, so that V is too, and a lane ends up with D / 4 consecutive elements of its query.
//
// KG = 1: four waves (64 queries) share tiles of 16 keys.  KG = 4, 8: four or eight waves take the same 16 queries and
// every fourth or eighth tile each, and are merged at the end: four times the workgroups, and a chain of tiles a
// fourth or an eighth as long, for calls that would not fill the chip.
//
// 1024 tokens of 4 heads, d = 64 (256 workgroups of eight waves): 15 us, 25 with the search of the region in front of everything
// and a test per 16 bytes of a tile.  A step of two waves on a SIMD takes 2 us, 1.4 of them the products.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "tca_common.h"
#include "tca_device.h"
#include "tca_prefill.h"

namespace tca {

constexpr int row_threads(int kg) { return kg == 8 ? 512 : 256; }

// 2^d for a difference of logits: the whole part taken off in fp64, so that nothing is lost of the fraction.  (-inf and what
// lies below 2^31 give zero, a NaN a NaN.)  Seven instructions where expf of the rounded difference takes fifteen.
__device__ __forceinline__ float exp2_diff(double d) {
  int n;
  asm("v_cvt_i32_f64 %0, %1" : "=v"(n) : "v"(d));                    // (saturates)
  return ldexpf(__builtin_amdgcn_exp2f((float)(d - (double)n)), n);
}

struct HeadOffs { int64_t offs[TCA_MAX_HEADS + 1]; };

// grid (query tiles * Hq), longest query tiles first, heads inside; block 256, 512 with KG = 8
template <int D, int KG>
__global__ __launch_bounds__(row_threads(KG), D == 64 && KG == 1 ? 4 : 2) void prefill_f32_kernel(
    const float* __restrict__ Q, int64_t q_pos0, int64_t n_queries, const float* __restrict__ K,
    const float* __restrict__ V, int64_t kv_stride, const int32_t* __restrict__ idx,
    const float* __restrict__ Kg, const float* __restrict__ Vg, HeadOffs ho,
    const int32_t* __restrict__ n_rows, int Hq, int G, int GS, int w, double scale, float* __restrict__ O,
    float* __restrict__ lse, int part) {
  typedef double f64x4_t __attribute__((ext_vector_type(4)));
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  constexpr int TK = 16;                           // keys per tile
  constexpr double kLn2 = 0.693147180559945309417;
  constexpr int GW = row_threads(KG) / 64 / KG, GT = GW * 64;      // waves, threads that share a tile
  constexpr int QT = GW * 16;                      // queries per workgroup
  constexpr int C4 = D / 4;                        // 16-byte chunks of a row
  constexpr int SB = D / 16;                       // blocks of O^T; chunks of a quarter row
  constexpr int NL = TK * C4 / GT;                 // chunks a thread stages, of K and of V
  // KG > 1 shares nothing of V: at d = 128, where the registers are short, V goes from memory to its operands (at d = 64
  // requesting it a tile ahead and keeping it in LDS is faster: 1024 tokens, 4 heads, 23 against 28 us).
  constexpr bool kStageV = KG == 1 || D == 64;
  __shared__ f32x4_t kt[KG][TK][C4], vt[kStageV ? KG : 1][TK][C4];
  constexpr int kSpan = KG == 1 ? 256 : 512;       // of the search
  __shared__ int seen_ahead[KG == 1 ? GW : 1][KG == 1 ? kSpan + QT : 1];     // its positions; KG > 1: in the place of the wave's tile
  static_assert(KG == 1 || sizeof(kt) / KG >= (kSpan + QT) * 4, "room for the search");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kb = lane >> 4, c = lane & 15;
  const int grp = wv / GW, gt = tid - grp * GT;    // key group, thread inside it
  const int h = blockIdx.x % Hq;
  const int qtile = gridDim.x / Hq - 1 - blockIdx.x / Hq;
  const int kvh = h / G, hs = h / GS;              // hs: the selection this query head reads
  const int64_t base = ho.offs[hs];
  const int64_t r0 = (int64_t)qtile * QT;
  int64_t qrow = r0 + (wv - grp * GW) * 16 + c;    // this lane's query
  const bool stored = qrow < n_queries;
  if (!stored) qrow = n_queries - 1;               // computes a duplicate
  const int qpos = (int)(q_pos0 + qrow);
  const int wg_first = (int)(q_pos0 + r0);
  const int wg_last = (int)(q_pos0 + (r0 + QT < n_queries ? r0 + QT : n_queries) - 1);

  // (part: both key subsets, or one of them alone, normalised by itself and merged later through lse)
  const int nr = part == TCA_PART_WINDOW ? 0 : n_rows[hs];
  const int win_lo = wg_first - w + 1 > 0 ? wg_first - w + 1 : 0;
  // tiles of the window, which are known, before those of the region, which have to be looked for
  const int n_wt = part == TCA_PART_GLOBAL ? 0 : (wg_last - win_lo) / TK + 1;
  int n_tiles = n_wt, nv_hi = 0, nvis = 0;         // rows of the region visible to some query of the workgroup, to this lane's

  // Where the rows of tile t lie (gather-free call, Kg = NULL: the kept rows are read where they are).  Past the last key its row is
  // read once more: no query sees it.  (A test per 16 bytes, for zeros there, made up half of a step: 4 us with
  // eight waves and d = 64, 2 now.)
  const float* const k_reg = Kg ? Kg + base * D : K + (size_t)kvh * kv_stride * D;
  const float* const v_reg = Kg ? Vg + base * D : V + (size_t)kvh * kv_stride * D;
  const float* const k_win = K + ((size_t)kvh * kv_stride + win_lo) * D;
  const float* const v_win = V + ((size_t)kvh * kv_stride + win_lo) * D;
  const int32_t* const gather = Kg ? nullptr : idx + base;
  auto rows_of = [&](int t, auto use) {            // use(K rows, V rows, the row that row r of the tile is)
    const bool region = t >= n_wt;
    const int first = (region ? t - n_wt : t) * TK, last = region ? nv_hi - 1 : wg_last - win_lo;
    if (region && gather) use(k_reg, v_reg, [&](int r) { return gather[min(first + r, last)]; });
    else use(region ? k_reg : k_win, region ? v_reg : v_win, [&](int r) { return min(first + r, last); });
  };
  // the next tile, on its way (where V is not staged: its K)
  f32x4_t kr[NL], vr[kStageV ? NL : 1];
  auto fetch = [&](int t) {
    rows_of(t, [&](const float* k, const float* v, auto row) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int ci = i * GT + gt, r = ci / C4, ch = ci - r * C4;
        const size_t at = (size_t)row(r) * D + 4 * ch;
        kr[i] = *reinterpret_cast<const f32x4_t*>(k + at);
        if constexpr (kStageV) vr[i] = *reinterpret_cast<const f32x4_t*>(v + at);
      }
    });
  };
  auto sync = [&] {                                // the threads that share a tile
    if constexpr (KG == 1) {
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };

  double q[D / 4];                                 // element kb D/4 + t of the query
  {
    f32x4_t v[SB];
#pragma unroll
    for (int t = 0; t < SB; ++t) v[t] = *reinterpret_cast<const f32x4_t*>(Q + ((size_t)h * n_queries + qrow) * D + kb * (D / 4) + 4 * t);
    const bool early = grp < n_wt;                 // (uniform where the tiles are shared)
    if (early) fetch(grp);
    // The rows of the region that the workgroup's first query sees are counted, by every wave for itself and while the first
    // tile is on its way: kSpan / 64 positions a lane at a time, of 496 (KG = 1: 192) rows in one round of loads.  Each query behind
    // it can see one more than the query before (positions ascend, as a rule strictly): the next QT decide.
    if (nr > 0 && wg_last >= w) {
      int* const ahead = KG == 1 ? seen_ahead[wv] : reinterpret_cast<int*>(&kt[grp][0][0]);
      const int32_t* const at = idx + base;
      const int64_t bound = (int64_t)wg_first - w;
      int lo = 0, len = nr;                        // the count lies in [lo, lo + len]
      while (len > kSpan - QT) {
        const int step = (len + kSpan - 1) / kSpan;
        int32_t last[kSpan / 64];                  // of each piece
#pragma unroll
        for (int i = 0; i < kSpan / 64; ++i) last[i] = at[lo + min((i * 64 + lane + 1) * step, len) - 1];
        int below = 0;
#pragma unroll
        for (int i = 0; i < kSpan / 64; ++i) below += __popcll(__ballot((i * 64 + lane) * step < len && (int64_t)last[i] <= bound));
        const int skip = min(below * step, len);
        lo += skip;
        len = min(len - skip, step - 1);           // (the last row of the piece is above the bound)
      }
      int32_t pos[kSpan / 64];
#pragma unroll
      for (int i = 0; i < kSpan / 64; ++i) pos[i] = at[min(lo + i * 64 + lane, nr - 1)];
      int count = 0;
#pragma unroll
      for (int i = 0; i < kSpan / 64; ++i) {
        if (lo + i * 64 + lane >= nr) pos[i] = 0x7FFFFFFF;
        count += __popcll(__ballot((int64_t)pos[i] <= bound));
        ahead[i * 64 + lane] = pos[i];
      }
      if (lane < QT) ahead[kSpan + lane] = 0x7FFFFFFF;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int next = ahead[count + (lane & (QT - 1))];         // row lo + count + lane
      count += lo;
      const int mine = qpos - w;
      int more = 0;
      if constexpr (QT <= 16) {
#pragma unroll
        for (int i = 0; i < QT; ++i) more += __builtin_amdgcn_readlane(next, i) <= mine;
      } else {
        for (int step = QT / 2; step > 0; step >>= 1) more += __shfl(next, more + step - 1, kWave) <= mine ? step : 0;
        more += __shfl(next, more, kWave) <= mine;
      }
      nvis = count + more;
      nv_hi = count + __popcll(__ballot(lane < QT && next <= wg_last - w));
      // all of them, so that there may be more: a position held more than once
      if (__builtin_expect(nv_hi == count + QT, 0)) {
        nv_hi = count_le_wave(at, nr, (int64_t)wg_last - w);
        int a = 0, b = nv_hi;
        while (a < b) {
          const int mid = (a + b) >> 1;
          if (at[mid] <= mine) a = mid + 1; else b = mid;
        }
        nvis = a;
      }
      n_tiles += (nv_hi + TK - 1) / TK;
    }
    if (!early && grp < n_tiles) fetch(grp);
#pragma unroll
    for (int t = 0; t < SB; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) q[4 * t + e] = (double)v[t][e];
  }

  double m;                                        // the same in the four lanes of a query
  float l;                                         // over this lane's keys
  f32x4_t o[SB];
  // The product gives a masked key the weight 0, which an infinity or a NaN in its V row turns into NaN for queries that do
  // not see the row.  Such a value always shows in the sums of all queries of the wave: where it does, the walk is made again
  // with PLAIN = false, which adds V key by key to the queries that see the key.  (Looking for it per tile, with the second
  // way of adding beside the first: 43 against 31 us at 4 heads and 1024 tokens.)
  auto walk = [&](auto plain_tag) {
    constexpr bool PLAIN = decltype(plain_tag)::value;
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int s = 0; s < SB; ++s) o[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (!PLAIN && grp < n_tiles) fetch(grp);
    for (int t = grp; t < n_tiles; t += KG) {
      sync();                                        // the tile before has been consumed
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int ci = i * GT + gt, r = ci / C4, ch = ci - r * C4;
        kt[grp][r][ch ^ (r & 15)] = kr[i];
        if constexpr (kStageV) vt[grp][r][ch] = vr[i];
      }
      sync();
      f32x4_t vd[kStageV ? 1 : 4][SB / 4];           // this lane's chunks of the rows kb + 4 r
      if constexpr (!kStageV) {
        rows_of(t, [&](const float*, const float* v, auto row) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float* const at = v + (size_t)row(kb + 4 * r) * D;
#pragma unroll
            for (int u = 0; u < SB / 4; ++u) vd[r][u] = *reinterpret_cast<const f32x4_t*>(at + 4 * (c * (SB / 4) + u));
          }
        });
      }
      if (t + KG < n_tiles) fetch(t + KG);

      f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        const f32x4_t kf = kt[grp][c][(kb * SB + u) ^ c];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kf[e], q[4 * u + e], acc, 0, 0, 0);
      }
      // visible <=> lo <= key inside the tile < hi
      int lo = 0, hi;
      if (t >= n_wt) {
        hi = nvis - (t - n_wt) * TK;
      } else {
        const int j0 = win_lo + t * TK;
        lo = qpos - w + 1 - j0;
        hi = qpos + 1 - j0;
      }
      auto seen = [&](int r) { return kb + 4 * r >= lo && kb + 4 * r < hi; };
      double x[4], mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[r] = seen(r) ? acc[r] * scale : -INFINITY;
        mx = fmax(mx, x[r]);
      }
      mx = fmax(mx, __shfl_xor(mx, 16, kWave));
      mx = fmax(mx, __shfl_xor(mx, 32, kWave));
      const double mn = fmax(m, mx);
      const float corr = mn > m ? exp2_diff(m - mn) : 1.f;         // 0 on the first keys (m = -inf)
      m = mn;
      float p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = seen(r) ? exp2_diff(x[r] - m) : 0.f;       // by the mask: a NaN logit is no masked key
      l = fmaf(l, corr, (p[0] + p[1]) + (p[2] + p[3]));
      // The tile's part is summed from zero and added to the rest once: a quarter of the roundings at the size of the
      // whole sum (error against 64 bits at 1500 tokens 2e-7; 4e-7 with every product added to the whole).
      f32x4_t ot[SB];
#pragma unroll
      for (int s = 0; s < SB; ++s) ot[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (PLAIN) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int u = 0; u < SB / 4; ++u) {
            f32x4_t vf;
            if constexpr (kStageV) vf = vt[grp][kb + 4 * r][c * (SB / 4) + u];
            else vf = vd[r][u];
#pragma unroll
            for (int e = 0; e < 4; ++e) ot[4 * u + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e], p[r], ot[4 * u + e], 0, 0, 0);
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll 1
          for (int k = 0; k < 4; ++k) {
            const int from = k * 16, key = k + 4 * r;                // the lanes that hold the key
            const float pk = __shfl(p[r], from + c, kWave);          // its weight for this lane's query
            const bool sees = key >= lo && key < hi;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int u = 0; u < SB / 4; ++u)                       // elements SB (4 kb + j) + 4 u ..
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  float v;
                  if constexpr (kStageV) v = vt[grp][key][(4 * kb + j) * (SB / 4) + u][e];
                  else v = __shfl(vd[r][u][e], from + 4 * kb + j, kWave);
                  if (sees) ot[4 * u + e][j] = fmaf(pk, v, ot[4 * u + e][j]);
                }
          }
        }
      }
#pragma unroll
      for (int s = 0; s < SB; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[s][e] = fmaf(o[s][e], corr, ot[s][e]);
    }
  };
  walk(std::true_type{});
  float odd = 0.f;                                 // 0 times every sum: not 0 if one is an infinity or a NaN
#pragma unroll
  for (int s = 0; s < SB; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) odd = fmaf(o[s][e], 0.f, odd);
  // (a wave of KG > 1 shares nothing with the others; with KG = 1 the barriers of the walk are the whole workgroup's)
  if (__builtin_expect(KG == 1 ? __syncthreads_or(odd != 0.f) : __any(odd != 0.f), 0)) walk(std::false_type{});
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);

  // o[s][r] is element SB (4 kb + r) + s of query c
  if constexpr (KG == 1) {
    if (!stored) return;
    const float inv = l > 0.f ? 1.f / l : 0.f;     // an empty part: zeros, lse = -inf
    float* orow = O + ((size_t)h * n_queries + qrow) * D + kb * (D / 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int u = 0; u < SB / 4; ++u) {
        const f32x4_t v = {o[4 * u][r] * inv, o[4 * u + 1][r] * inv, o[4 * u + 2][r] * inv, o[4 * u + 3][r] * inv};
        *reinterpret_cast<f32x4_t*>(orow + r * SB + 4 * u) = v;
      }
    if (lse && kb == 0) lse[(size_t)h * n_queries + qrow] = l > 0.f ? (float)(m * kLn2 + log((double)l)) : -INFINITY;
  } else {
    __shared__ double ms[KG][16];
    __shared__ float ls[KG][16];
    static_assert(sizeof(kt) >= sizeof(float) * KG * 16 * D, "the tiles' place holds the waves' results");
    f32x4_t* const po = &kt[0][0][0];              // [wave][query][D]
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int u = 0; u < SB / 4; ++u)             // (chunk xor query: the queries of a chunk lie on different banks)
        po[(wv * 16 + c) * C4 + (((kb * 4 + r) * (SB / 4) + u) ^ c)] = f32x4_t{o[4 * u][r], o[4 * u + 1][r], o[4 * u + 2][r], o[4 * u + 3][r]};
    if (kb == 0) { ms[wv][c] = m; ls[wv][c] = l; }
    __syncthreads();
    // In fp64: added in fp32, eight parts put the error against 64 bits at 1.2e-7 and four at 1.1e-7; in fp64 it is 9e-8.
    __shared__ double weight[KG][16];               // of a part in a query's result
    if (tid < KG * 16) {
      const int g = tid >> 4, qi = tid & 15;
      double M = ms[0][qi];
#pragma unroll
      for (int k = 1; k < KG; ++k) M = fmax(M, ms[k][qi]);
      double wgt = 0;                              // no keys: a sum of 0 (or of NaN, which stays)
      if (ms[g][qi] != -INFINITY) wgt = exp2(ms[g][qi] - M);
      weight[g][qi] = wgt;
    }
    __syncthreads();
    const int qi = tid >> 4, sub = tid & 15;       // 16 threads per query, D / 16 elements each
    if (qi >= 16 || r0 + qi >= n_queries) return;
    double L = 0, a[SB];
#pragma unroll
    for (int e = 0; e < SB; ++e) a[e] = 0;
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      const double wgt = weight[g][qi];
      L += ls[g][qi] * wgt;
#pragma unroll
      for (int u = 0; u < SB / 4; ++u) {
        const f32x4_t v = po[(g * 16 + qi) * C4 + ((sub * (SB / 4) + u) ^ qi)];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * u + e] += v[e] * wgt;
      }
    }
    const double inv = L > 0 ? 1 / L : 0;
    float* orow = O + ((size_t)h * n_queries + r0 + qi) * D + sub * SB;
#pragma unroll
    for (int u = 0; u < SB / 4; ++u) {
      const f32x4_t v = {(float)(a[4 * u] * inv), (float)(a[4 * u + 1] * inv), (float)(a[4 * u + 2] * inv), (float)(a[4 * u + 3] * inv)};
      *reinterpret_cast<f32x4_t*>(orow + 4 * u) = v;
    }
    double M = ms[0][qi];
#pragma unroll
    for (int g = 1; g < KG; ++g) M = fmax(M, ms[g][qi]);
    if (lse && sub == 0) lse[(size_t)h * n_queries + r0 + qi] = L > 0 ? (float)(M * kLn2 + log((double)L)) : -INFINITY;
  }
}

int launch_prefill_f32(const tca_params* prm, const float* Q, int64_t q_pos0, int64_t n_queries, const float* K,
                       const float* V, int64_t kv_stride, const int32_t* idx, const float* Kg, const float* Vg,
                       const int64_t* offs, const int32_t* n_rows, float* O, float* lse, hipStream_t st, int part) {
  HeadOffs ho;
  for (int h = 0; h <= sel_heads(prm); ++h) ho.offs[h] = offs[h];
  const int Hq = prm->n_q_heads;
  const double scale = logit_scale(prm) * 1.44269504088896340736;      // log2 e
  // Few workgroups of 64 queries for 256 CUs: 16 each.  us with 64 / with 16, on inputs in the caches: 4 heads, d = 64, 4096
  // tokens (256 workgroups of 64) 149 / 69, 8000 (500) 319 / 185; 32 heads, d = 128, 700 tokens (352) 124 / 84, 1000 (512)
  // 189 / 150, 1500 (768) 298 / 298 (not in the caches 313 / 326); 64 heads, 500 tokens (512) 99 / 92.  (One wave per query, keys
  // read from L2 by each, took 95 us at 4 heads and 1024 tokens where this takes 15.)
  const bool few = (n_queries + 63) / 64 * Hq < 640;
  const int64_t n_wg = (n_queries + (few ? 15 : 63)) / (few ? 16 : 64) * Hq;
  if (n_wg > INT32_MAX) return fail(TCA_ERR_UNSUPPORTED, "tca_prefill (fp32): %lld queries", (long long)n_queries);
  // And of those, few enough that no CU has two, and with keys for twice the waves: eight share the walk.  us with four / with
  // eight, on inputs in the caches and not: 4 heads, d = 64, 64 tokens (4 tiles of keys) 8.5 / 8.4 and 8.3 / 9.1, 96 (6) 8.5 / 8.4 and
  // 9.8 / 10.3, 1024 (256 workgroups) 15.8 / 14.8 and 19.0 / 18.0, 1024 behind 8192 77 / 64 and 80 / 68, 2048 (512 workgroups)
  // 29.3 / 30.5 and 32.6 / 33.8; 32 heads, d = 128, 128 tokens (8 tiles) 10.6 / 11.9 and 13.8 / 14.7, 64 behind 200 (17) 17.9 / 17.0
  // and 22.2 / 20.2, 64 behind 4096 235 / 186 and 265 / 200.
  int64_t region = 0;                              // keys the last query may see
  for (int h = 0; h < sel_heads(prm); ++h) region = std::max(region, offs[h + 1] - offs[h]);
  const int64_t seen = q_pos0 + n_queries, old = std::max<int64_t>(0, seen - prm->window);
  const int64_t keys = (part == TCA_PART_GLOBAL ? 0 : seen - old) + (part == TCA_PART_WINDOW ? 0 : std::min(region, old));
  const bool fewest = few && n_wg <= 256 && keys > 8 * 16;
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_wg), dim3(threads), 0, st, Q, q_pos0, n_queries, K, V, kv_stride, idx,
                       Kg, Vg, ho, n_rows, Hq, Hq / prm->n_kv_heads, sel_group(prm), prm->window, scale, O, lse, part);
  };
  auto choose = [&](auto d_tag) {
    constexpr int D = decltype(d_tag)::value;
    if (fewest) launch(prefill_f32_kernel<D, 8>, row_threads(8));
    else if (few) launch(prefill_f32_kernel<D, 4>, row_threads(4));
    else launch(prefill_f32_kernel<D, 1>, row_threads(1));
  };
  if (prm->head_dim == 128) choose(std::integral_constant<int, 128>{});
  else choose(std::integral_constant<int, 64>{});
  return TCA_OK;
}

}  // namespace tca
