// Offline head-specific sparsity determination (Alg. 1; Eq. 3, Eq. 4).
//
// Runs once per model, and everything is fp64: the decisions a_i >= tau then agree with an fp64 reference
// except at exact ties.  The dense causal attention matrix A is never materialised:
//   rows      : per query row j, max and sum of exp of the causal logits        (softmax denominators)
//   columns   : per key column k, sum_{j>=k} exp(x_jk - max_j) / sum_j, divided
//               by the structural column count L-k                              (Eq. 4 inner term)
// Both are passes of one kernel over Q K^T on the matrix cores (v_mfma_f64_16x16x4_f64, operands widened in
// registers): a wave keeps 32 rows of one operand (the queries of its row statistics, the keys of its column sums) in
// registers and streams the other through LDS.  The order of the head's elements inside a product is free as long as
// both operands agree: lane kb takes the kb-th quarter of a row, so that LDS is read 16 bytes at a time (chunk index
// xor row, conflict-free).  The bound is the fp64 matrix product, 64 cycles per 16 x 16 x 4 block and SIMD: 8192 tokens,
// 32 heads, 3.6 ms per pass at 2.4 GHz, measured 5.1 and 4.9 ms; on the vector ALU (dot products of 16 lanes and a
// butterfly) the passes took 16.5 and 18.9 ms.
// The selection of every candidate reuses the online-selection stages (scores
// and in-block ranks once, budgets per candidate); cand_score sums the column
// means of the tokens a candidate keeps (Eq. 4).
#include <hip/hip_runtime.h>

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
// COL = false: the queries are fixed, keys 0 .. j stream by, row_max / row_sum are written.  COL = true: the keys are
// fixed, queries k .. L-1 stream by, abar is written.
template <typename T, int D, bool COL>
__global__ __launch_bounds__(kCalThreads, 2) void cal_pass_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, int64_t L, int Hq, int G, double scale,
    double* __restrict__ row_max, double* __restrict__ row_sum, double* __restrict__ abar) {
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
  const int64_t f0 = (int64_t)(COL ? turn : gridDim.x / Hq - 1 - turn) * 128;
  const T* fixed = COL ? K + (size_t)kvh * L * D : Q + (size_t)h * L * D;
  const T* stream = COL ? Q + (size_t)h * L * D : K + (size_t)kvh * L * D;
  const double* rm = row_max + (size_t)h * L;
  const double* rs = row_sum + (size_t)h * L;

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
      nrm = rm[s0 + tid];
      nri = 1.0 / rs[s0 + tid];
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
      else { row_max[at] = m[b]; row_sum[at] = l[b]; }
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
  for (int64_t k = tid; k < nb * b; k += kCalThreads) {
    if (tr[k] < bt[k / b]) {
      double v = 0.0;
      for (int g = 0; g < GS; ++g) v += abar[(size_t)(h * GS + g) * L + k];
      acc += GS > 1 ? v / (double)GS : v;
      ++cnt;
    }
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
  double* row_max;      // [Hq][L]
  double* row_sum;      // [Hq][L]
  double* abar;         // [Hq][L]
  int32_t* blk_t;       // [M][Hs][nb]   (Hs selection heads <= Hq; sized for Hq)
  int32_t* blk_dst;     // [M][Hs][nb]
  int32_t* n_rows;      // [M][Hs]
  double* a_dev;        // [Hs][M]
  int64_t* n_dev;       // [Hs][M]
  void* q_last;         // [Hq][D] contiguous copy of the last query rows
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
  c.row_max = (double*)(base + off); off = align_up(off + (size_t)Hq * L * 8, 256);
  c.row_sum = (double*)(base + off); off = align_up(off + (size_t)Hq * L * 8, 256);
  c.abar = (double*)(base + off);    off = align_up(off + (size_t)Hq * L * 8, 256);
  c.blk_t = (int32_t*)(base + off);  off = align_up(off + (size_t)M * Hq * nb * 4, 256);
  c.blk_dst = (int32_t*)(base + off); off = align_up(off + (size_t)M * Hq * nb * 4, 256);
  c.n_rows = (int32_t*)(base + off); off = align_up(off + (size_t)M * Hq * 4, 256);
  c.a_dev = (double*)(base + off);   off = align_up(off + (size_t)Hq * M * 8, 256);
  c.n_dev = (int64_t*)(base + off);  off = align_up(off + (size_t)Hq * M * 8, 256);
  c.q_last = base + off;             off = align_up(off + (size_t)Hq * prm->head_dim * 4, 256);
  c.bytes = off;
  return c;
}

template <typename T>
__global__ void cal_gather_qlast_kernel(const T* __restrict__ Q, int64_t L, int D, T* __restrict__ out) {
  const int h = blockIdx.x;
  for (int e = threadIdx.x; e < D; e += blockDim.x) out[(size_t)h * D + e] = Q[((size_t)h * L + (L - 1)) * D + e];
}

template <typename T, int D>
static void run_passes(const tca_params* prm, const T* Q, const T* K, int64_t L, const CalWs& c, hipStream_t st) {
  const int Hq = prm->n_q_heads, G = Hq / prm->n_kv_heads;
  const dim3 grid((unsigned)((L + 127) / 128 * Hq));
  const double sc = logit_scale(prm);
  hipLaunchKernelGGL((cal_pass_kernel<T, D, false>), grid, dim3(kCalThreads), 0, st, Q, K, L, Hq, G, sc, c.row_max, c.row_sum, c.abar);
  hipLaunchKernelGGL((cal_pass_kernel<T, D, true>), grid, dim3(kCalThreads), 0, st, Q, K, L, Hq, G, sc, c.row_max, c.row_sum, c.abar);
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
  const size_t need = tca_calibrate_workspace_bytes(prm, L_cal, M);
  if (ws_bytes < need || ((uintptr_t)ws & 255))
    return fail(TCA_ERR_WORKSPACE, "tca_calibrate_budgets: workspace needs %zu bytes, 256-byte aligned", need);
  hipStream_t st = (hipStream_t)stream;
  CalWs c = carve_cal_ws(ws, prm, L_cal, M);

  std::vector<double> cands((size_t)M * nk);
  rc = tca_make_candidates(b, M, sigma, cands.data());
  if (rc) return rc;

  // column means of the dense causal attention matrix (Alg. 1 line 1, Eq. 4)
  if (prm->dtype == TCA_BF16) {
    using T = bf16_t;
    if (prm->head_dim == 128) run_passes<T, 128>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, c, st);
    else run_passes<T, 64>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, c, st);
  } else {
    using T = float;
    if (prm->head_dim == 128) run_passes<T, 128>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, c, st);
    else run_passes<T, 64>(prm, (const T*)Qcal, (const T*)Kcal, L_cal, c, st);
  }

  // selection of every candidate (Alg. 1 line 4): scores and ranks once, budgets per candidate
  SelectWs sw = carve_select_ws(c.select_ws, prm, L_cal);
  select_score_stage(prm, c.q_last, Kcal, L_cal, L_cal, sw, st);
  std::vector<double> a_host((size_t)Hs * M, 0.0);
  std::vector<int64_t> n_host((size_t)Hs * M, 0);
  if (nb > 0) {
    const int64_t nz = (int64_t)M * Hs;
    hipLaunchKernelGGL(cal_zero_kernel, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, st, c.n_rows, nz);
    std::vector<double> p_all((size_t)Hs * nk);
    int64_t cap[TCA_MAX_HEADS];
    for (int h = 0; h < Hs; ++h) cap[h] = INT32_MAX;
    for (int i = 0; i < M; ++i) {
      for (int h = 0; h < Hs; ++h)
        for (int e = 0; e < nk; ++e) p_all[(size_t)h * nk + e] = cands[(size_t)i * nk + e];
      select_assign_stage(prm, L_cal, p_all.data(), cap, sw.sel_stats, c.n_rows + (size_t)i * Hs,
                          c.blk_t + (size_t)i * Hs * nb, c.blk_dst + (size_t)i * Hs * nb, st);
    }
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
