// Offline head-specific sparsity determination (Alg. 1; Eq. 3, Eq. 4).
//
// Runs once per model, and everything is fp64: the decisions a_i >= tau then agree with an fp64 reference
// except at exact ties.  The dense causal attention matrix A is never materialised:
//   rows      : per query row j, max and sum of exp of the causal logits        (softmax denominators)
//   columns   : per key column k, sum_{j>=k} exp(x_jk - max_j) / sum_j, divided
//               by the structural column count L-k                              (Eq. 4 inner term)
// Samples in bf16 take their products in int8 digits (below).  fp32 samples, and calls whose workspace has no room for the
// digits: both are passes of one kernel over Q K^T on the matrix cores (v_mfma_f64_16x16x4_f64, operands widened in
// registers): a wave keeps 32 rows of one operand (the queries of its row statistics, the keys of its column sums) in
// registers and streams the other through LDS.  The order of the head's elements inside a product is free as long as
// both operands agree: lane kb takes the kb-th quarter of a row, so that LDS is read 16 bytes at a time (chunk index
// xor row, conflict-free).  The bound is the fp64 matrix product, 64 cycles per 16 x 16 x 4 block and SIMD, and the exponentials
// (24 fp64 instructions) on top of it: fp64 instructions of the vector ALU do not run beside it (8 multiply-adds and one block
// 102 cycles, 36 and 64 alone).  8192 tokens, 32 heads, bf16: 3.6 ms of products per pass at 2.4 GHz, measured 5.1 and 4.9 ms; on the vector ALU (dot products of 16 lanes and a
// butterfly) the passes took 16.5 and 18.9 ms.
// The selection of every candidate reuses the online-selection stages (scores
// and in-block ranks once, budgets per candidate); cand_score sums the column
// means of the tokens a candidate keeps (Eq. 4).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "tca_common.h"
#include "tca_device.h"
#include "tca_select.h"

namespace tca {

constexpr int kCalThreads = 256;

// grid (ceil(L / 128) * Hq), the longest walks first, heads inside (head by head, the last head's longest walks start when
// the others are done: 16.0 against 10.1 ms for both passes); block 256: wave = 32 fixed rows, lane (kb = lane / 16, c = lane % 16)
// holds, of every 16 streamed rows, the logits of the rows kb + 4 r against the fixed rows c and c + 16.
// COL = false: the queries are fixed, keys 0 .. j stream by, stats are written.  COL = true: the keys are
// fixed, queries k .. L-1 stream by, abar is written.
template <typename T, int D, bool COL>
__global__ __launch_bounds__(kCalThreads, 2) void cal_pass_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, int64_t L, int Hq, int G, double scale, double2* __restrict__ stats,
    double* __restrict__ abar, const int32_t* __restrict__ only) {
  typedef double f64x4_t __attribute__((ext_vector_type(4)));
  constexpr int EPC = Vec16<T>::N;                 // elements of a 16-byte chunk
  constexpr int CPR = D / EPC, CPQ = CPR / 4;      // chunks of a row, of a quarter row
  constexpr int TS = 32;                           // streamed rows per tile
  constexpr int NL = TS * CPR / kCalThreads;       // chunks a thread stages
  constexpr int SWZ = (CPR < 16 ? CPR : 16) - 1;
  static_assert(NL >= 1 && NL * kCalThreads == TS * CPR, "shape");
  __shared__ raw16_t tile[TS][CPR];
  __shared__ double rmx[COL ? TS : 1], rinv[COL ? TS : 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, kb = lane >> 4, c = lane & 15;
  const int h = blockIdx.x % Hq, kvh = h / G, turn = blockIdx.x / Hq;
  if (only && !only[h]) return;
  const int64_t f0 = (int64_t)(COL ? turn : gridDim.x / Hq - 1 - turn) * 128;
  const T* fixed = COL ? K + (size_t)kvh * L * D : Q + (size_t)h * L * D;
  const T* stream = COL ? Q + (size_t)h * L * D : K + (size_t)kvh * L * D;
  const double2* const rows = stats + (size_t)h * L;                 // (maximum, sum)

  int64_t frow[2];
  double f[2][D / 4];                              // elements kb D/4 .. of the fixed rows
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    frow[b] = f0 + wv * 32 + b * 16 + c;
    const int64_t r = frow[b] < L ? frow[b] : L - 1;                 // rows past the end compute a duplicate, never stored
#pragma unroll
    for (int u = 0; u < CPQ; ++u) {
      float v[EPC];
      Vec16<T>::load(fixed + (size_t)r * D + kb * (D / 4) + u * EPC, v);
#pragma unroll
      for (int e = 0; e < EPC; ++e) f[b][u * EPC + e] = (double)v[e];
    }
  }
  const int64_t s_begin = COL ? f0 : 0, s_end = COL ? L : (f0 + 128 < L ? f0 + 128 : L);
  raw16_t nxt[NL];
  double nrm = 0.0, nri = 0.0;
  auto fetch = [&](int64_t s0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int ci = i * kCalThreads + tid, r = ci / CPR, ch = ci - r * CPR;
      nxt[i] = raw16_t{0, 0, 0, 0};
      if (s0 + r < s_end) nxt[i] = load_raw16(stream + (size_t)(s0 + r) * D + ch * EPC);
    }
    if (COL && tid < TS && s0 + tid < s_end) {
      const double2 st = rows[s0 + tid];
      nrm = st.x;
      nri = 1.0 / st.y;
    }
  };
  double m[2] = {-INFINITY, -INFINITY}, l[2] = {0.0, 0.0};          // COL: l alone, the sum
  fetch(s_begin);
  for (int64_t s0 = s_begin; s0 < s_end; s0 += TS) {
    __syncthreads();                               // the tile before has been consumed
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int ci = i * kCalThreads + tid, r = ci / CPR, ch = ci - r * CPR;
      tile[r][ch ^ (r & SWZ)] = nxt[i];
    }
    if (COL && tid < TS) { rmx[tid] = nrm; rinv[tid] = nri; }
    __syncthreads();
    if (s0 + TS < s_end) fetch(s0 + TS);
#pragma unroll
    for (int sub = 0; sub < TS / 16; ++sub) {
      f64x4_t acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
      for (int u = 0; u < CPQ; ++u) {
        float v[EPC];
        widen_raw16<T>(tile[sub * 16 + c][(kb * CPQ + u) ^ (c & SWZ)], v);
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
          const double a = (double)v[e];
          acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, f[0][u * EPC + e], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, f[1][u * EPC + e], acc[1], 0, 0, 0);
        }
      }
      // A block of rows that every fixed row of the wave may see takes no tests: its exponentials are independent of
      // each other (under a test each, they ran one after the other: 17.8 against 16.4 ms for the call).
      const int64_t si0 = s0 + sub * 16;
      const int64_t wave0 = f0 + wv * 32;
      const bool full = COL ? si0 >= wave0 + 31 && si0 + 16 <= L : si0 + 15 <= wave0 && si0 + 16 <= s_end;
      auto take = [&](auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          auto sees = [&](int r) {                 // by position, not by the logit: a NaN is no masked one
            const int64_t si = si0 + kb + 4 * r;
            return FULL || (COL ? si >= frow[b] && si < L : si <= frow[b] && si < s_end);
          };
          double x[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = sees(r) ? acc[b][r] * scale : -INFINITY;
          if constexpr (COL) {
            double e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int sl = sub * 16 + kb + 4 * r;
              e[r] = sees(r) ? exp(x[r] - rmx[sl]) * rinv[sl] : 0.0;
            }
            l[b] += (e[0] + e[1]) + (e[2] + e[3]);
          } else {
            const double mx = fmax(m[b], fmax(fmax(x[0], x[1]), fmax(x[2], x[3])));
            if (mx > m[b]) {                       // this lane's rows: the four lanes of a query are merged at the end
              l[b] *= exp(m[b] - mx);              // 0 on the first rows (m = -inf)
              m[b] = mx;
            }
            double e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) e[r] = sees(r) ? exp(x[r] - mx) : 0.0;
            l[b] += (e[0] + e[1]) + (e[2] + e[3]);
          }
        }
      };
      if (full) take(std::true_type{});
      else take(std::false_type{});
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    for (int o = 16; o < 64; o <<= 1) {
      const double lo = __shfl_xor(l[b], o, kWave);
      if constexpr (COL) {
        l[b] += lo;
      } else {
        const double mo = __shfl_xor(m[b], o, kWave);
        const double mn = fmax(m[b], mo);
        const double wa = (m[b] == -INFINITY) ? 0.0 : exp(m[b] - mn);
        const double wb = (mo == -INFINITY) ? 0.0 : exp(mo - mn);
        l[b] = l[b] * wa + lo * wb;
        m[b] = mn;
      }
    }
    if (kb == 0 && frow[b] < L) {
      const size_t at = (size_t)h * L + frow[b];
      if constexpr (COL) abar[at] = l[b] / (double)(L - frow[b]);
      else stats[at] = make_double2(m[b], l[b]);
    }
  }
}

// ------------------------------------------------------------------------------------------------ bf16 samples --
// A bf16 element is an 8-bit integer times a power of two, so 16 rows that share an exponent are integers of 32 bits, and
// these four signed digits of 8 bits: a logit is then the sum of sixteen int8 matrix products, each exact (128 products of
// 2^14, four sums of them: at most 2^23), added up by weight in fp64.  One int8 product takes a 64th of the fp64 one, and
// the lowest digit is seldom there.  An element whose bits would fall off the end, below 2^-24 of the group's largest, is left
// out of the digits and added by itself; a group with several, or with one that is not finite, has its products in fp64 (and a head
// with many such groups takes the fp64 passes: cal_heads_kernel).  What the sample holds decides the time: 8192 tokens of 32 heads,
// Gaussian elements 2.8 ms, with references far from zero 4.3, with channels 2^4, 2^8 and 2^12 times the others 4.3, 4.8 and 10.2, in
// fp64 throughout 10.1.
constexpr int kDigits = 4;
constexpr int kGroupRows = 16;                     // rows that share an exponent
constexpr int kDigitBias = 127 + 7 + 23;           // a group of exponent e holds its elements times 2^(kDigitBias - e)
// In a group's word beside its exponent (9 bits): not to be had in digits; with a lowest digit; rows whose reference is far from
// zero; an element left out
constexpr int kOddGroup = 1 << 20, kLowGroup = 1 << 21, kFarGroup = 1 << 22, kRestGroup = 1 << 23;
struct GroupInfo {
  int32_t word;
  float norm;          // no row is longer (infinite: one is not finite)
  int32_t rest_at;     // the element left out: 256 row + column,
  float rest;          // and its value
};
constexpr int kExpTable = 256;
typedef int i32x4_t __attribute__((ext_vector_type(4)));
// 2^(i / 256) as its bits, less i where the exponent's lower neighbours lie: adding n << 12 to the upper half then gives
// 2^(n / 256) for any n = i modulo 256
struct ExpTable { uint64_t t[kExpTable]; };

static int64_t digit_groups(int64_t L) { return (L + 127) / 128 * (128 / kGroupRows); }       // per head, whole workgroups of the passes

// grid (groups of all heads of Q, then of K, / 4); block 256, a wave per group.  Lane (kb, c) holds of row c the elements 64 s + 16 kb .. + 15
// of every step s, which is its operand of v_mfma_i32_16x16x64_i8 either way round; a group lies as [digit][step][lane][16
// bytes], lowest digit first.
template <int D>
__global__ __launch_bounds__(256) void cal_digits_kernel(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, int64_t L,
                                                         int64_t groups, int64_t q_groups, int64_t all, i32x4_t* __restrict__ Qd,
                                                         i32x4_t* __restrict__ Kd, GroupInfo* __restrict__ q_info,
                                                         GroupInfo* __restrict__ k_info) {
  constexpr int KS = D / 64;
  const int lane = threadIdx.x & 63, kb = lane >> 4, c = lane & 15;
  int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= all) return;
  const bool of_k = g >= q_groups;
  if (of_k) g -= q_groups;
  const bf16_t* const X = of_k ? K : Q;
  i32x4_t* const digits = of_k ? Kd : Qd;
  GroupInfo* const info = of_k ? k_info : q_info;
  const int64_t row = (g % groups) * kGroupRows + c;
  const bf16_t* x = X + ((size_t)(g / groups) * L + row) * D + kb * 16;
  uint32_t w[KS][8];
  uint32_t top = 0;
  float len = 0.f;
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      raw16_t v = {0, 0, 0, 0};
      if (row < L) v = load_raw16(x + s * 64 + i * 8);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float lo = __uint_as_float(v[j] << 16), hi = __uint_as_float(v[j] & 0xffff0000u);
        w[s][4 * i + j] = v[j];
        top = max(top, max(v[j] & 0x7fffu, (v[j] >> 16) & 0x7fffu));
        len = fmaf(lo, lo, fmaf(hi, hi, len));
      }
    }
  top = group_max(top, kWave);
  len += __shfl_xor(len, 16, kWave);
  len += __shfl_xor(len, 32, kWave);
  len = group_max(len, 16);
  // (255 as the leading digits of the largest element would round up to a 33rd bit)
  const int e_top = max((int)(top >> 7), 1) + ((top & 0x7f) == 0x7f ? 1 : 0);
  int rests = 0, rest_at = 0, low = 0;
  float rest = 0.f;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    i32x4_t out[kDigits];
#pragma unroll
    for (int q = 0; q < 4; ++q) {                  // four elements: a dword of each digit
      uint32_t n[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t u = (w[s][2 * q + (j >> 1)] >> (16 * (j & 1))) & 0xffffu;
        const int e = (u >> 7) & 255;
        const uint32_t m = ((u & 0x7fu) | (e ? 0x80u : 0u)) << 23;
        const int fall = min(e_top - max(e, 1), 31);
        uint32_t a = m >> fall;
        if ((a << fall) != m) {
          ++rests;
          rest_at = 256 * c + 64 * s + 16 * kb + 4 * q + j;
          rest = __uint_as_float(u << 16);
          a = 0;
        }
        n[j] = ((u & 0x8000u ? 0u - a : a) + 0x80808080u) ^ 0x80808080u;
      }
      const uint32_t l01 = __builtin_amdgcn_perm(n[1], n[0], 0x05010400u), h01 = __builtin_amdgcn_perm(n[1], n[0], 0x07030602u);
      const uint32_t l23 = __builtin_amdgcn_perm(n[3], n[2], 0x05010400u), h23 = __builtin_amdgcn_perm(n[3], n[2], 0x07030602u);
      out[0][q] = (int)__builtin_amdgcn_perm(l23, l01, 0x05040100u);
      out[1][q] = (int)__builtin_amdgcn_perm(l23, l01, 0x07060302u);
      out[2][q] = (int)__builtin_amdgcn_perm(h23, h01, 0x05040100u);
      out[3][q] = (int)__builtin_amdgcn_perm(h23, h01, 0x07060302u);
      low |= out[0][q];
    }
#pragma unroll
    for (int p = 0; p < kDigits; ++p) digits[((size_t)g * kDigits * KS + p * KS + s) * 64 + lane] = out[p];
  }
  const bool finite = (top >> 7) != 255, any_low = __any(low != 0);
  const uint64_t who = __ballot(rests != 0);
  const bool odd = !finite || __popcll(who) > 1 || __any(rests > 1);
  if (who ? lane == __ffsll((long long)who) - 1 : lane == 0)
    info[g] = GroupInfo{e_top + (odd ? kOddGroup : who ? kRestGroup : 0) + (any_low ? kLowGroup : 0),
                        finite ? sqrtf(len) * 1.001f : INFINITY, rest_at, rest};
}

// The two passes on digits; the walk and the order of the workgroups are cal_pass_kernel's.  Lane (kb, c) holds, of every 16
// streamed rows, the logits of the rows 4 kb + r against the fixed rows c and c + 16.  Logits are carried in units of
// ln 2 / 256, `unit` being the scale in them: an exponential is then a whole number and a fraction away, 2^(n / 256) from a
// table and a polynomial of degree four (Tang's method).  A row's exponentials are taken against a reference, a multiple of
// 256, so that moving it costs a power of two; stats holds it and the inverse of the row's sum.
// Where no logit can be further than kFar from zero (by the norms, Cauchy and Schwarz) any reference as near will do, and
// nothing can leave its range: adding kMagic rounds, and the whole number lies in the lower half of the sum.  Elsewhere and on
// the diagonal the reference follows the maximum, step by step.
//
// 8192 tokens, 32 heads, d = 128: 1.38 and 1.46 ms, where the passes above take 5.05 and 4.92.  The bound is instruction issue: per
// 16 x 16 block 18 products of 16 cycles (32 with a lowest digit), 7 (10) instructions an element to put the sums together, 11
// for the exponential, at 4 to 5.4 cycles each; the matrix cores are busy 40 % of the time.  Three waves a SIMD, although some
// registers of the uncommon paths spill for it, against two: 1.38 / 1.48.  A tile's two halves are written out in one block so that
// the second's products run under the first's exponentials.  One element left out of a group: with its products in fp64
// instead the few workgroups that have one end last, 1.83 ms.
template <int D, bool COL>
__global__ __launch_bounds__(kCalThreads, 3) void cal_digit_pass_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const i32x4_t* __restrict__ Qd, const i32x4_t* __restrict__ Kd,
    GroupInfo* __restrict__ q_info, const GroupInfo* __restrict__ k_info, int64_t L, int64_t groups, int Hq, int G, double unit,
    double2* __restrict__ stats, double* __restrict__ abar, const int32_t* __restrict__ fp64_head, ExpTable table) {
  typedef double f64x4_t __attribute__((ext_vector_type(4)));
  constexpr int KS = D / 64;
  constexpr int TS = 2 * kGroupRows;               // streamed rows per tile
  constexpr int GB = kGroupRows * D * kDigits;     // bytes of a group
  constexpr int NL = 2 * GB / (kCalThreads * 16);  // copies of 16 bytes a thread makes of a tile
  constexpr double kMagic = 0x1.8p52;
  constexpr float kFar = 120000.f;                 // two of it and 256 stay above 2^-1022
  __shared__ __attribute__((aligned(16))) unsigned char tile[2][2 * GB];
  __shared__ __attribute__((aligned(16))) double2 rstat[COL ? 2 : 1][COL ? 64 : 1];       // 32 rows, and what the upper half of the wave leaves
  __shared__ i32x4_t f_low[4][2][KS][64];          // the fixed rows' lowest digit
  __shared__ uint64_t exp2_frac[kExpTable];
  const int tid = threadIdx.x, lane = tid & 63, kb = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % Hq, kvh = h / G, turn = blockIdx.x / Hq;
  if (fp64_head[h]) return;
  const int64_t f0 = (int64_t)(COL ? turn : gridDim.x / Hq - 1 - turn) * 128;
  const int64_t wave0 = f0 + wv * 32;
  const bf16_t* const fixed = COL ? K + (size_t)kvh * L * D : Q + (size_t)h * L * D;
  const bf16_t* const stream = COL ? Q + (size_t)h * L * D : K + (size_t)kvh * L * D;
  const i32x4_t* const fixed_d = COL ? Kd + (size_t)kvh * groups * (GB / 16) : Qd + (size_t)h * groups * (GB / 16);
  const i32x4_t* const stream_d = COL ? Qd + (size_t)h * groups * (GB / 16) : Kd + (size_t)kvh * groups * (GB / 16);
  const GroupInfo* const fixed_info = (COL ? k_info + (size_t)kvh * groups : q_info + (size_t)h * groups) + wave0 / kGroupRows;
  const GroupInfo* const stream_info = COL ? q_info + (size_t)h * groups : k_info + (size_t)kvh * groups;
  exp2_frac[tid] = table.t[tid];

  i32x4_t f[2][kDigits - 1][KS];                   // the others
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int p = 0; p < kDigits; ++p)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const i32x4_t v = fixed_d[((wave0 / kGroupRows + b) * kDigits * KS + p * KS + s) * 64 + lane];
        if (p) f[b][p - 1][s] = v;
        else f_low[wv][b][s][lane] = v;            // (read by the lane that wrote it)
      }
  const GroupInfo f_info[2] = {fixed_info[0], fixed_info[1]};
  const int f_word = f_info[0].word | f_info[1].word;
  const float f_far = fmaxf(f_info[0].norm, f_info[1].norm) * fabsf((float)unit);
  bool far = false;                                // ROW: some reference is far from zero
  const int64_t s_begin = COL ? f0 : 0, s_end = COL ? L : (f0 + 128 < L ? f0 + 128 : L);
  constexpr int kRsrcFlags = 0x00020000;           // raw buffer, 32-bit data format
  const __amdgpu_buffer_rsrc_t rs_d = __builtin_amdgcn_make_buffer_rsrc((void*)stream_d, 0, (int)(groups * GB), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rs_s = __builtin_amdgcn_make_buffer_rsrc((void*)(stats + (size_t)h * L), 0, (int)(L * 16), kRsrcFlags);
  auto copy = [&](int64_t s0, int to) {
    const int off = (int)(s0 / kGroupRows) * GB;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int at = (i * 4 + wv) * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_d, (__attribute__((address_space(3))) void*)(tile[to] + at), 16, lane * 16, off + at, 0, 0);
    }
    if constexpr (COL)
      if (wv == 0)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_s, (__attribute__((address_space(3))) void*)&rstat[to][0], 16, lane * 16, (int)s0 * 16, 0, 0);
  };

  double m[2] = {0.0, 0.0}, l[2] = {0.0, 0.0};     // COL: l alone, the sum
  copy(s_begin, 0);
  int cur = 0;
  // The sixteen products of 16 streamed rows with the fixed ones, by weight; nine without lowest digits.
  auto products = [&](auto low, const unsigned char* at, i32x4_t (&acc)[2][2 * kDigits - 1]) {
    constexpr int first = decltype(low)::value ? 0 : 1;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 2 * kDigits - 1; ++i) acc[b][i] = i32x4_t{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int p = first; p < kDigits; ++p) {
        const i32x4_t a = *reinterpret_cast<const i32x4_t*>(at + ((p * KS + s) * 64 + lane) * 16);
#pragma unroll
        for (int q = first; q < kDigits; ++q)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[b][p + q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, q ? f[b][q ? q - 1 : 0][s] : f_low[wv][b][s][lane], acc[b][p + q], 0, 0, 0);
      }
  };
  auto combine = [&](auto low, const i32x4_t (&acc)[2][2 * kDigits - 1], double (&u)[2][4]) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {                // two neighbouring weights fit 32 bits
        const int z = (acc[b][6][r] << 8) + acc[b][5][r], y = (acc[b][4][r] << 8) + acc[b][3][r];
        double v = fma((double)z, 65536.0, (double)y);
        if constexpr (decltype(low)::value) v = fma(fma(v, 65536.0, (double)((acc[b][2][r] << 8) + acc[b][1][r])), 256.0, (double)acc[b][0][r]);
        else v = fma(v, 256.0, (double)acc[b][2][r]);
        u[b][r] = v;
      }
  };
  auto unit_of = [&](auto low, const GroupInfo& s_info, int b) {
    return ldexp(unit, (s_info.word & 511) + (f_info[b].word & 511) - 2 * (decltype(low)::value ? kDigitBias : kDigitBias - 8));
  };
  // e^x - 1 over a fraction of a unit
  auto poly = [](double x) {
    constexpr double k1 = 0x1.62e42fefa39efp-9, k2 = k1 * k1 / 2, k3 = k1 * k1 * k1 / 6, k4 = k1 * k1 * k1 * k1 / 24;
    return x * fma(fma(fma(k4, x, k3), x, k2), x, k1);
  };
  auto near_tail = [&](int sub, const double (&u)[2][4], const double (&ch)[2], double (&lt)[2]) {
    double e[2][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double2 st = {};
      if constexpr (COL) st = rstat[cur][sub * 16 + 4 * kb + r];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const double magic = kMagic - (COL ? st.x : m[b]), a = fma(u[b][r], ch[b], magic), x = fma(u[b][r], ch[b], magic - a);
        const uint32_t n = (uint32_t)__double_as_longlong(a);
        const uint2 t = *reinterpret_cast<const uint2*>(&exp2_frac[n & (kExpTable - 1)]);
        uint32_t hi;                               // (written out: the compiler makes five instructions of it)
        asm("v_lshl_add_u32 %0, %1, 12, %2" : "=v"(hi) : "v"(n), "v"(t.y));
        const double T = __hiloint2double((int)hi, (int)t.x);
        e[b][r] = fma(T, poly(x), T);
        if constexpr (COL) lt[b] = fma(e[b][r], st.y, lt[b]);
      }
    }
    if constexpr (!COL) {
#pragma unroll
      for (int b = 0; b < 2; ++b) lt[b] += (e[b][0] + e[b][1]) + (e[b][2] + e[b][3]);
    }
  };
  GroupInfo next_info[2] = {stream_info[s_begin / kGroupRows], stream_info[s_begin / kGroupRows + 1]};
  for (int64_t s0 = s_begin; s0 < s_end; s0 += TS, cur ^= 1) {
    __builtin_amdgcn_s_waitcnt(0x0F70);            // this wave's copies of the tile have landed
    __syncthreads();                               // everybody's; and the other place has been consumed
    if (s0 + TS < s_end) copy(s0 + TS, cur ^ 1);
    const unsigned char* const tl = tile[cur];
    double lt[2] = {0.0, 0.0};                     // the tile's part, added to the rest once
    const GroupInfo t_info[2] = {next_info[0], next_info[1]};
    if (s0 + TS < s_end) {
      next_info[0] = stream_info[s0 / kGroupRows + 2];
      next_info[1] = stream_info[s0 / kGroupRows + 3];
    }
    const int t_word = t_info[0].word | t_info[1].word | f_word;
    const bool t_near = !far && !(t_word & kFarGroup) && fmaxf(t_info[0].norm, t_info[1].norm) * f_far < kFar;
    if (__builtin_expect(t_near && !(t_word & (kOddGroup | kRestGroup)) && (COL ? s0 >= wave0 + 31 && s0 + TS <= L : s0 + TS - 1 <= wave0), 1)) {      // all is seen by all
      auto both = [&](auto low) {
        i32x4_t acc[2][2][2 * kDigits - 1];
        double u[2][2][4];
        const double ch[2][2] = {{unit_of(low, t_info[0], 0), unit_of(low, t_info[0], 1)}, {unit_of(low, t_info[1], 0), unit_of(low, t_info[1], 1)}};
        products(low, tl, acc[0]);
        combine(low, acc[0], u[0]);
        __builtin_amdgcn_sched_barrier(0);
        products(low, tl + GB, acc[1]);
        near_tail(0, u[0], ch[0], lt);
        constexpr int kMfma = 0x008, kValu = 0x002;
        constexpr int n_mfma = 2 * KS * (decltype(low)::value ? 16 : 9);
#pragma unroll
        for (int i = 0; i < n_mfma; ++i) {
          __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kValu, decltype(low)::value ? 2 : 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        combine(low, acc[1], u[1]);
        near_tail(1, u[1], ch[1], lt);
      };
      if (t_word & kLowGroup) both(std::true_type{});
      else both(std::false_type{});
#pragma unroll
      for (int b = 0; b < 2; ++b) l[b] += lt[b];
      continue;
    }
#pragma unroll 1
    for (int sub = 0; sub < 2; ++sub) {
      const int64_t si0 = s0 + sub * kGroupRows;
      if (COL ? si0 + 15 < wave0 : si0 > wave0 + 31) continue;       // nothing of it is seen
      const GroupInfo s_info = sub ? t_info[1] : t_info[0];
      const int word = s_info.word | f_word;
      double u[2][4], ch[2];
      {
        i32x4_t acc[2][2 * kDigits - 1];
        products(std::true_type{}, tl + sub * GB, acc);
        combine(std::true_type{}, acc, u);
#pragma unroll
        for (int b = 0; b < 2; ++b) ch[b] = unit_of(std::true_type{}, s_info, b);
      }
      if (word & kRestGroup) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
          for (int r = 0; r < 4; ++r) u[b][r] *= ch[b];
          if (f_info[b].word & kRestGroup) {       // times the streamed rows, put together from their digits
            const int col = f_info[b].rest_at & 255;
            const double v = f_info[b].rest_at >> 8 == c ? ldexp((double)f_info[b].rest * unit, (s_info.word & 511) - kDigitBias) : 0.0;
            const signed char* const at = reinterpret_cast<const signed char*>(tl) + sub * GB + ((col >> 6) * 64 + ((col >> 4) & 3) * 16 + 4 * kb) * 16 + (col & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              int n = 0;
#pragma unroll
              for (int p = kDigits - 1; p >= 0; --p) n = (n << 8) + at[p * KS * 1024 + r * 16];
              u[b][r] = fma(v, (double)n, u[b][r]);
            }
          }
          if (s_info.word & kRestGroup) {          // times the fixed rows
            const int64_t row = wave0 + b * 16 + c;
            const double v = (double)load_f32(fixed + (size_t)(row < L ? row : L - 1) * D + (s_info.rest_at & 255)) * (double)s_info.rest;
#pragma unroll
            for (int r = 0; r < 4; ++r) u[b][r] = fma(s_info.rest_at >> 8 == 4 * kb + r ? v : 0.0, unit, u[b][r]);
          }
          ch[b] = 1.0;
        }
      }
      if (__builtin_expect((word & kOddGroup) != 0, 0)) {
        // row 4 (c % 4) + c / 4 as the c-th, so that the products lie as above
        const int64_t ar = si0 + 4 * (c & 3) + (c >> 2);
        const bf16_t* const arow = stream + (size_t)(ar < L ? ar : L - 1) * D + kb * (D / 4);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          if (!((s_info.word | f_info[b].word) & kOddGroup)) continue;
          const int64_t br = wave0 + b * 16 + c;
          const bf16_t* const brow = fixed + (size_t)(br < L ? br : L - 1) * D + kb * (D / 4);
          raw16_t ra[D / 32], rb[D / 32];
#pragma unroll
          for (int t = 0; t < D / 32; ++t) {
            ra[t] = load_raw16(arow + t * 8);
            rb[t] = load_raw16(brow + t * 8);
          }
          f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int t = 0; t < D / 32; ++t) {
            float av[8], bv[8];
            widen_raw16<bf16_t>(ra[t], av);
            widen_raw16<bf16_t>(rb[t], bv);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[e], (double)bv[e], acc, 0, 0, 0);
          }
          ch[b] = unit;
#pragma unroll
          for (int r = 0; r < 4; ++r) u[b][r] = acc[r];
        }
      }
      if (t_near && (COL ? si0 >= wave0 + 31 && si0 + 16 <= L : si0 + 15 <= wave0)) {
        near_tail(sub, u, ch, lt);
      } else {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int64_t frow = wave0 + b * 16 + c;
          auto sees = [&](int r) {                 // by position, not by the logit: a NaN is no masked one
            const int64_t si = si0 + 4 * kb + r;
            return COL ? si >= frow && si < L : si <= frow && si < s_end;
          };
          auto power = [&](int r, double ref) {
            const double t = fma(u[b][r], ch[b], -ref), n = rint(t);
            int i;
            asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(n));          // (saturates)
            const uint64_t f0 = exp2_frac[i & (kExpTable - 1)] + ((uint64_t)(i & (kExpTable - 1)) << 44);
            const double T = __longlong_as_double((long long)f0), e = ldexp(fma(T, poly(t - n), T), i >> 8);
            return !sees(r) || t == -INFINITY ? 0.0 : e;
          };
          if constexpr (COL) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const double2 st = rstat[cur][sub * 16 + 4 * kb + r];
              const double e = power(r, st.x);
              lt[b] = sees(r) ? fma(e, st.y, lt[b]) : lt[b];
            }
          } else {
            double x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = sees(r) ? u[b][r] * ch[b] : -INFINITY;
            const double mx = fmax(fmax(x[0], x[1]), fmax(x[2], x[3]));
            l[b] += lt[b];
            lt[b] = 0.0;
            if (mx > m[b] || (l[b] == 0.0 && mx > -INFINITY)) {      // this lane's rows: the four lanes of a query are merged at the end
              const double to = 256.0 * ceil(mx * 0x1p-8);
              l[b] = ldexp(l[b], (int)fmax((m[b] - to) * 0x1p-8, -4096.0));
              m[b] = to;
            }
            far = __any(far || !(fabs(m[b]) <= (double)kFar));
            double e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) e[r] = power(r, m[b]);
            lt[b] += (e[0] + e[1]) + (e[2] + e[3]);
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) l[b] += lt[b];
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int64_t frow = wave0 + b * 16 + c;
    for (int o = 16; o < 64; o <<= 1) {
      const double lo = __shfl_xor(l[b], o, kWave);
      if constexpr (COL) {
        l[b] += lo;
      } else {
        // A lane that has seen no key (of the first queries) has no say in the reference: its zero may lie far above the others'.
        const double mo = __shfl_xor(m[b], o, kWave), mn = l[b] == 0.0 ? mo : lo == 0.0 ? m[b] : fmax(m[b], mo);
        auto scaled = [&](double sum, double ref) { return ldexp(sum, (int)fmax(fmin((ref - mn) * 0x1p-8, 0.0), -4096.0)); };
        l[b] = scaled(l[b], m[b]) + scaled(lo, mo);
        m[b] = mn;
      }
    }
    if constexpr (!COL) {                          // for the second pass
      if (__any(frow < L && !(fabs(m[b]) <= (double)kFar)) && lane == 0)
        q_info[(size_t)h * groups + wave0 / kGroupRows + b].word = f_info[b].word | kFarGroup;
    }
    if (kb == 0 && frow < L) {
      if constexpr (COL) abar[(size_t)h * L + frow] = l[b] / (double)(L - frow);
      else stats[(size_t)h * L + frow] = make_double2(m[b], 1.0 / l[b]);
    }
  }
}

// grid (M, Hs); block 256.  a[h][i] = sum of abar over tokens with rank < t_block (Eq. 4).
// Selection head h serves query heads h*GS .. h*GS+GS-1; with GS > 1 the importance of a
// key is the mean of their column means.
__global__ __launch_bounds__(kCalThreads) void cal_cand_score_kernel(
    const uint8_t* __restrict__ tokrank, const int32_t* __restrict__ blk_t, const double* __restrict__ abar,
    int64_t L, int b, int64_t nb, int Hs, int GS, int M, double* __restrict__ a_out, int64_t* __restrict__ n_out) {
  __shared__ double red[kCalThreads];
  __shared__ long long redn[kCalThreads];
  const int i = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const int32_t* bt = blk_t + ((size_t)i * Hs + h) * nb;
  const uint8_t* tr = tokrank + (size_t)h * (nb * b);
  double acc = 0.0;
  long long cnt = 0;
  // (loads without regard to the rank, several tokens ahead: 26 -> 16 us for 14 candidates of 32 heads and 8192 tokens)
  const int lb = __builtin_ctz(b);
#pragma unroll 4
  for (int64_t k = tid; k < nb * b; k += kCalThreads) {
    double v = 0.0;
    for (int g = 0; g < GS; ++g) v += abar[(size_t)(h * GS + g) * L + k];
    const bool kept = tr[k] < bt[k >> lb];
    acc += kept ? (GS > 1 ? v / (double)GS : v) : 0.0;
    cnt += kept;
  }
  red[tid] = acc;
  redn[tid] = cnt;
  __syncthreads();
  for (int o = kCalThreads / 2; o > 0; o >>= 1) {
    if (tid < o) { red[tid] += red[tid + o]; redn[tid] += redn[tid + o]; }
    __syncthreads();
  }
  if (tid == 0) {
    a_out[(size_t)h * M + i] = red[0];
    n_out[(size_t)h * M + i] = redn[0];
  }
}

__global__ void cal_zero_kernel(int32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

struct CalWs {
  void* select_ws;      // tokrank + stats (+ one blk_t/blk_dst pair, unused here)
  double2* stats;       // [Hq][L] of a query's row: reference and sum, or (digits) its inverse
  double* abar;         // [Hq][L]
  int32_t* blk_t;       // [M][Hs][nb]   (Hs selection heads <= Hq; sized for Hq)
  int32_t* blk_dst;     // [M][Hs][nb]
  int32_t* n_rows;      // [M][Hs]
  double* a_dev;        // [Hs][M]
  int64_t* n_dev;       // [Hs][M]
  void* q_last;         // [Hq][D] contiguous copy of the last query rows
  size_t need;          // bytes up to here: what a call must be given
  i32x4_t *Qd, *Kd;     // bf16: [Hq], [Hkv] x [groups][digit][step][64 lanes] (what lies from here on may be missing)
  GroupInfo *q_info, *k_info;     // [Hq][groups], [Hkv][groups]
  size_t bytes;
};

static CalWs carve_cal_ws(void* ws, const tca_params* prm, int64_t L, int M) {
  CalWs c;
  char* base = (char*)ws;
  size_t off = 0;
  const int Hq = prm->n_q_heads;
  const int64_t nb = L / prm->block;
  const size_t sel = carve_select_ws(nullptr, prm, L).bytes;
  c.select_ws = base + off;          off = align_up(off + sel, 256);
  c.stats = (double2*)(base + off);  off = align_up(align_up(off + (size_t)Hq * L * 8, 256) + (size_t)Hq * L * 8, 256);
  c.abar = (double*)(base + off);    off = align_up(off + (size_t)Hq * L * 8, 256);
  c.blk_t = (int32_t*)(base + off);  off = align_up(off + (size_t)M * Hq * nb * 4, 256);
  c.blk_dst = (int32_t*)(base + off); off = align_up(off + (size_t)M * Hq * nb * 4, 256);
  c.n_rows = (int32_t*)(base + off); off = align_up(off + (size_t)M * Hq * 4, 256);
  c.a_dev = (double*)(base + off);   off = align_up(off + (size_t)Hq * M * 8, 256);
  c.n_dev = (int64_t*)(base + off);  off = align_up(off + (size_t)Hq * M * 8, 256);
  c.q_last = base + off;             off = align_up(off + (size_t)Hq * prm->head_dim * 4, 256);
  c.need = off;
  if (prm->dtype == TCA_BF16) {
    const size_t groups = digit_groups(L), gb = (size_t)kGroupRows * prm->head_dim * kDigits;
    c.Qd = (i32x4_t*)(base + off);     off = align_up(off + Hq * groups * gb, 256);
    c.Kd = (i32x4_t*)(base + off);     off = align_up(off + prm->n_kv_heads * groups * gb, 256);
    c.q_info = (GroupInfo*)(base + off); off = align_up(off + Hq * groups * sizeof(GroupInfo), 256);
    c.k_info = (GroupInfo*)(base + off); off = align_up(off + prm->n_kv_heads * groups * sizeof(GroupInfo), 256);
  }
  c.bytes = off;
  return c;
}

// grid Hq; block 128
template <typename T>
__global__ void cal_gather_qlast_kernel(const T* __restrict__ Q, int64_t L, int D, T* __restrict__ out) {
  const int h = blockIdx.x;
  for (int e = threadIdx.x; e < D; e += blockDim.x) out[(size_t)h * D + e] = Q[((size_t)h * L + (L - 1)) * D + e];
}

// The same for bf16 samples, cal_zero_kernel's work, and which heads take the fp64 passes: those of whose pairs of groups more than half are not to be
// had in digits.  Such a pair costs the digit passes 1.6 times what the fp64 ones take for it, any other a fourth.  8192 tokens, 32
// heads, keys with channels 2^8, 2^12 and 2^16 times the others (a few, most, all of the pairs): ms with digits 4.8, 10.2 and 16.6, in
// fp64 10.1.  grid Hq; block 256
__global__ __launch_bounds__(256) void cal_heads_kernel(const bf16_t* __restrict__ Q, int64_t L, int D, bf16_t* __restrict__ out,
                                                        int64_t groups, int G, const GroupInfo* __restrict__ q_info,
                                                        const GroupInfo* __restrict__ k_info, int32_t* __restrict__ fp64_head,
                                                        int32_t* __restrict__ zeros, int n_zeros) {
  __shared__ int odd[2];
  const int h = blockIdx.x, tid = threadIdx.x;
  if (tid < 2) odd[tid] = 0;
  for (int i = h * 256 + tid; i < n_zeros; i += gridDim.x * 256) zeros[i] = 0;
  if (tid < D) out[(size_t)h * D + tid] = Q[((size_t)h * L + (L - 1)) * D + tid];
  int q = 0, k = 0;
#pragma unroll 4
  for (int64_t g = tid; g < groups; g += 256) {
    q += (q_info[(size_t)h * groups + g].word & kOddGroup) != 0;
    k += (k_info[(size_t)(h / G) * groups + g].word & kOddGroup) != 0;
  }
  __syncthreads();
  if (q) atomicAdd(&odd[0], q);
  if (k) atomicAdd(&odd[1], k);
  __syncthreads();
  if (tid == 0) fp64_head[h] = 2 * (groups - odd[0]) * (groups - odd[1]) < groups * groups;
}

template <int D>
static void run_digit_passes(const tca_params* prm, const bf16_t* Q, const bf16_t* K, int64_t L, int M, const CalWs& c, hipStream_t st) {
  const int Hq = prm->n_q_heads, Hkv = prm->n_kv_heads;
  const int64_t groups = digit_groups(L);
  const dim3 grid((unsigned)((L + 127) / 128 * Hq));
  static const ExpTable table = [] {
    ExpTable t;
    for (uint64_t i = 0; i < kExpTable; ++i) {
      const double v = (double)exp2l(i / (long double)kExpTable);
      std::memcpy(&t.t[i], &v, 8);
      t.t[i] -= i << 44;
    }
    return t;
  }();
  const double unit = (double)(logit_scale(prm) * (kExpTable * 1.44269504088896340735992468100189214L));
  const int G = Hq / Hkv;
  const int64_t q_groups = groups * Hq, all = q_groups + groups * Hkv;
  hipLaunchKernelGGL((cal_digits_kernel<D>), dim3((unsigned)((all + 3) / 4)), dim3(256), 0, st, Q, K, L, groups, q_groups, all, c.Qd, c.Kd,
                     c.q_info, c.k_info);
  int32_t* const fp64_head = (int32_t*)c.n_dev;                      // [Hq], where the candidates' sizes come later
  hipLaunchKernelGGL(cal_heads_kernel, dim3(Hq), dim3(256), 0, st, Q, L, D, (bf16_t*)c.q_last, groups, G, c.q_info, c.k_info, fp64_head,
                     c.n_rows, M * sel_heads(prm));
  auto pass = [&](auto kernel, auto fp64_kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kCalThreads), 0, st, Q, K, c.Qd, c.Kd, c.q_info, c.k_info, L, groups, Hq, G, unit, c.stats,
                       c.abar, fp64_head, table);
    hipLaunchKernelGGL(fp64_kernel, grid, dim3(kCalThreads), 0, st, Q, K, L, Hq, G, logit_scale(prm), c.stats, c.abar, fp64_head);
  };
  pass(cal_digit_pass_kernel<D, false>, cal_pass_kernel<bf16_t, D, false>);
  pass(cal_digit_pass_kernel<D, true>, cal_pass_kernel<bf16_t, D, true>);
}

template <typename T, int D>
static void run_passes(const tca_params* prm, const T* Q, const T* K, int64_t L, int M, const CalWs& c, bool digits, hipStream_t st) {
  const int Hq = prm->n_q_heads, G = Hq / prm->n_kv_heads;
  const dim3 grid((unsigned)((L + 127) / 128 * Hq));
  const double sc = logit_scale(prm);
  if constexpr (sizeof(T) == 2) {
    if (digits) {
      run_digit_passes<D>(prm, Q, K, L, M, c, st);
      return;
    }
  }
  hipLaunchKernelGGL((cal_pass_kernel<T, D, false>), grid, dim3(kCalThreads), 0, st, Q, K, L, Hq, G, sc, c.stats, c.abar, nullptr);
  hipLaunchKernelGGL((cal_pass_kernel<T, D, true>), grid, dim3(kCalThreads), 0, st, Q, K, L, Hq, G, sc, c.stats, c.abar, nullptr);
  hipLaunchKernelGGL((cal_gather_qlast_kernel<T>), dim3(Hq), dim3(128), 0, st, Q, L, D, (T*)c.q_last);
}

}  // namespace tca

using namespace tca;

extern "C" size_t tca_calibrate_workspace_bytes(const tca_params* prm, int64_t L_cal, int M) {
  if (check_params(prm) != TCA_OK || L_cal < 1 || M < 1) return 0;
  return carve_cal_ws(nullptr, prm, L_cal, M).bytes;
}

extern "C" int tca_calibrate_budgets(const tca_params* prm, const void* Qcal, const void* Kcal, int64_t L_cal,
                                     int M, double sigma, double tau, double* p_star, int32_t* cand_idx,
                                     double* a_out, int64_t* n_out, int32_t* fallback, void* ws, size_t ws_bytes,
                                     void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!Qcal || !Kcal || !p_star || !cand_idx || !ws)
    return fail(TCA_ERR_INVALID, "tca_calibrate_budgets: NULL pointer argument");
  if (L_cal < 1 || M < 1 || M > 256 || !(sigma > 0.0))
    return fail(TCA_ERR_INVALID, "tca_calibrate_budgets: L_cal=%lld M=%d sigma=%g", (long long)L_cal, M, sigma);
  const int Hs = sel_heads(prm), b = prm->block, nk = block_log2(b) + 1;
  const int64_t nb = L_cal / b;
  if (nb > TCA_MAX_BLOCKS)
    return fail(TCA_ERR_UNSUPPORTED, "tca_calibrate_budgets: %lld blocks exceed the limit of %d", (long long)nb,
                TCA_MAX_BLOCKS);
  CalWs c = carve_cal_ws(ws, prm, L_cal, M);
  const size_t need = c.need;
  if (ws_bytes < need || ((uintptr_t)ws & 255))
    return fail(TCA_ERR_WORKSPACE, "tca_calibrate_budgets: workspace needs %zu bytes, 256-byte aligned", need);
  hipStream_t st = (hipStream_t)stream;
  const bool digits = prm->dtype == TCA_BF16 && ws_bytes >= c.bytes;

  std::vector<double> cands((size_t)M * nk);
  rc = tca_make_candidates(b, M, sigma, cands.data());
  if (rc) return rc;

  // column means of the dense causal attention matrix (Alg. 1 line 1, Eq. 4)
  if (prm->dtype == TCA_BF16) {
    using T = bf16_t;
    if (prm->head_dim == 128) run_passes<T, 128>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, M, c, digits, st);
    else run_passes<T, 64>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, M, c, digits, st);
  } else {
    using T = float;
    if (prm->head_dim == 128) run_passes<T, 128>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, M, c, digits, st);
    else run_passes<T, 64>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, M, c, digits, st);
  }

  // selection of every candidate (Alg. 1 line 4): scores and ranks once, budgets per candidate
  SelectWs sw = carve_select_ws(c.select_ws, prm, L_cal);
  select_score_stage(prm, c.q_last, Kcal, L_cal, L_cal, sw, st);
  std::vector<double> a_host((size_t)Hs * M, 0.0);
  std::vector<int64_t> n_host((size_t)Hs * M, 0);
  if (nb > 0) {
    const int64_t nz = (int64_t)M * Hs;
    if (!digits) hipLaunchKernelGGL(cal_zero_kernel, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, st, c.n_rows, nz);
    select_assign_all(prm, L_cal, M, cands.data(), sw.sel_stats, c.n_rows, c.blk_t, c.blk_dst, st);
    hipLaunchKernelGGL(cal_cand_score_kernel, dim3(M, Hs), dim3(kCalThreads), 0, st, sw.tokrank, c.blk_t, c.abar,
                       L_cal, b, nb, Hs, sel_group(prm), M, c.a_dev, c.n_dev);
    TCA_HIP_CHECK(hipGetLastError());
    TCA_HIP_CHECK(hipMemcpyAsync(a_host.data(), c.a_dev, a_host.size() * 8, hipMemcpyDeviceToHost, st));
    TCA_HIP_CHECK(hipMemcpyAsync(n_host.data(), c.n_dev, n_host.size() * 8, hipMemcpyDeviceToHost, st));
  }
  TCA_HIP_CHECK(hipStreamSynchronize(st));
  TCA_HIP_CHECK(hipGetLastError());

  // Alg. 1 lines 6-8: the valid candidate with the fewest kept tokens (ties: lower index)
  for (int h = 0; h < Hs; ++h) {
    int best = -1;
    for (int i = 0; i < M; ++i) {
      if (a_host[(size_t)h * M + i] >= tau &&
          (best < 0 || n_host[(size_t)h * M + i] < n_host[(size_t)h * M + best]))
        best = i;
    }
    const bool fb = best < 0;
    if (fb) best = M - 1;
    cand_idx[h] = best;
    if (fallback) fallback[h] = fb ? 1 : 0;
    for (int e = 0; e < nk; ++e) p_star[(size_t)h * nk + e] = cands[(size_t)best * nk + e];
    if (a_out) for (int i = 0; i < M; ++i) a_out[(size_t)h * M + i] = a_host[(size_t)h * M + i];
    if (n_out) for (int i = 0; i < M; ++i) n_out[(size_t)h * M + i] = n_host[(size_t)h * M + i];
  }
  return TCA_OK;
}

// Alg. 1 for every layer of a model (Sec. IV-A: the determination is made once per model and
// covers all heads of all layers): one tca_calibrate_budgets pass per layer on that layer's
// sample, on the same workspace, results laid out layer-major.
extern "C" int tca_calibrate_layers(const tca_params* prm, int n_layers, const void* const* Qcal,
                                    const void* const* Kcal, int64_t L_cal, int M, double sigma, double tau,
                                    double* p_star, int32_t* cand_idx, double* a_out, int64_t* n_out,
                                    int32_t* fallback, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (n_layers < 1 || !Qcal || !Kcal || !p_star || !cand_idx)
    return fail(TCA_ERR_INVALID, "tca_calibrate_layers: n_layers=%d or NULL pointer argument", n_layers);
  const int Hs = sel_heads(prm), nk = block_log2(prm->block) + 1;
  for (int l = 0; l < n_layers; ++l) {
    if (!Qcal[l] || !Kcal[l]) return fail(TCA_ERR_INVALID, "tca_calibrate_layers: NULL sample of layer %d", l);
    rc = tca_calibrate_budgets(prm, Qcal[l], Kcal[l], L_cal, M, sigma, tau, p_star + (size_t)l * Hs * nk,
                               cand_idx + (size_t)l * Hs, a_out ? a_out + (size_t)l * Hs * M : nullptr,
                               n_out ? n_out + (size_t)l * Hs * M : nullptr,
                               fallback ? fallback + (size_t)l * Hs : nullptr, ws, ws_bytes, stream);
    if (rc) return rc;
  }
  return TCA_OK;
}
