// tca_prefill entry point (Eq. 2; Alg. 2 line 7): argument checks and dispatch.
#include <hip/hip_runtime.h>

#include "tca_common.h"
#include "tca_device.h"
#include "tca_prefill.h"

using namespace tca;

extern "C" size_t tca_prefill_workspace_bytes(const tca_params* prm, int64_t n_queries, int64_t cap_rows) {
  if (check_params(prm) != TCA_OK || n_queries < 0 || cap_rows < 0) return 0;
  if (prm->dtype != TCA_BF16) return 0;
  return prefill_mfma_workspace_bytes(prm, n_queries, cap_rows);
}

namespace tca {

// Merge of two attention results over disjoint key sets, each normalised by itself, through their
// log-sum-exp (Eq. 2 is one softmax over the union): O = (e^{lse_a} O_a + e^{lse_b} O_b) / (e^{lse_a} + e^{lse_b}).
// grid (ceil(rows/4)); block 256: one wave per row, each lane D/64 columns.  O_a is overwritten.
template <typename T>
__global__ __launch_bounds__(256) void merge_parts_kernel(T* __restrict__ Oa, const float* __restrict__ lse_a,
                                                          const T* __restrict__ Ob, const float* __restrict__ lse_b,
                                                          float* __restrict__ lse_out, int64_t rows, int D) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int lane = threadIdx.x & 63;
  const float la = lse_a[r], lb = lse_b[r];
  const float mx = fmaxf(la, lb);
  const float wa = la == -INFINITY ? 0.f : expf(la - mx), wb = lb == -INFINITY ? 0.f : expf(lb - mx);
  const float inv = 1.f / (wa + wb);                   // every query sees itself: at least one part is not empty
  for (int e = lane; e < D; e += 64) {
    const float a = wa > 0.f ? load_f32(Oa + r * D + e) * wa : 0.f;
    const float b = wb > 0.f ? load_f32(Ob + r * D + e) * wb : 0.f;
    store_f32(Oa + r * D + e, (a + b) * inv);
  }
  if (lse_out && lane == 0) lse_out[r] = mx + logf(wa + wb);
}

// Merge of the chunks of a split call: O = sum_s e^{m_s - M} O_s / sum_s e^{m_s - M} l_s per query (references m in
// score units, as the kernel keeps them).  grid (query tiles, Hq, D / 32); block 256: wave = 32 queries, lane =
// (half, query) with 4 x 4 of the D / 32 slice's columns, the layout the accumulators were left in: coalesced reads.
// Bound by latency: 27 MB of parts for 413 queries of 32 heads behind 64K tokens (6 us at the copy
// rate).  The references, eight at a time, and the first two chunks are requested together, two more ahead of every two; a
// place behind the last chunk is the last one again with the weight zero, so that no chunk's loads wait for another's.  us, a loop with
// a remainder and four chunks in flight / this / four at a time, whose 217 registers leave two waves a SIMD instead of three: there
// 11.1 / 7.4 / 8.7; 413 of 64 heads 18.6 / 13.1 / 14.3; 9000 tokens of 4 heads of 64 elements (568 workgroups) 8.6 / 8.0 / 9.4; 1 behind
// 8192, 32 heads, 9.5 / 4.9 / 4.7.
// A chunk is empty if its sum l is 0; one whose sum is NaN (a key or a query that is not finite) takes part.  (The file of
// the attention kernel is compiled without regard for NaN, this one is not.)
template <int D>
__global__ __launch_bounds__(256) void merge_split_kernel(SplitPlan sp, int64_t n_queries, float scale,
                                                          uint16_t* __restrict__ O, float* __restrict__ lse) {
  typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
  const int qtile = blockIdx.x, n_qt = gridDim.x, h = blockIdx.y, sl = blockIdx.z;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, hh = lane >> 5, c = lane & 31;
  const int n_ch = (sp.item_start[h + 1] - sp.item_start[h]) / n_qt;
  const size_t stride = (size_t)n_qt * split_floats<D>();
  const float* base = sp.part + (size_t)(sp.item_start[h] + qtile) * split_floats<D>();
  const float sl2e = scale * 1.4426950408889634f;
  const int q = wv * 32 + c;
  const int64_t r = (int64_t)qtile * 128 + q;
  if (r >= n_queries) return;
  constexpr int kAhead = 2, kRef = 8;
  f32x4_t v[2][kAhead][4];
  float m[2][kAhead], l[2][kAhead], ref[kRef];
  auto load = [&](int b, int s0) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const float* po = base + min(s0 + i, n_ch - 1) * stride;
      m[b][i] = po[128 * D + q];
      l[b][i] = po[128 * D + 128 + q];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) v[b][i][q4] = *reinterpret_cast<const f32x4_t*>(po + (((sl * 4 + q4) * 4 + wv) * 64 + lane) * 4);
    }
  };
  auto load_refs = [&](int s0) {
#pragma unroll
    for (int i = 0; i < kRef; ++i) ref[i] = base[min(s0 + i, n_ch - 1) * stride + 128 * D + q];
  };
  load_refs(0);
  load(0, 0);
  float M = -INFINITY;
  for (int s = 0;;) {
#pragma unroll
    for (int i = 0; i < kRef; ++i) M = fmaxf(M, ref[i]);
    s += kRef;
    if (s >= n_ch) break;
    load_refs(s);
  }
  f32x4_t acc[4];
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) acc[q4] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float L = 0.f;
  auto add = [&](int b, int s0) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const float li = s0 + i < n_ch ? l[b][i] : 0.f;
      const float wgt = li != 0.f ? __builtin_amdgcn_exp2f((m[b][i] - M) * sl2e) : 0.f;
      L += li * wgt;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[q4][j] += li != 0.f ? v[b][i][q4][j] * wgt : 0.f;   // an empty chunk's accumulators were never written
    }
  };
  for (int s0 = 0; s0 < n_ch; s0 += 2 * kAhead) {
    if (s0 + kAhead < n_ch) load(1, s0 + kAhead);
    add(0, s0);
    if (s0 + kAhead >= n_ch) break;
    if (s0 + 2 * kAhead < n_ch) load(0, s0 + 2 * kAhead);
    add(1, s0 + kAhead);
  }
  const float inv = L != 0.f ? 1.f / L : 0.f;
  uint16_t* orow = O + ((size_t)h * n_queries + r) * D;
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    bf16x4_t pk;
#pragma unroll
    for (int j = 0; j < 4; ++j) pk[j] = (__bf16)(acc[q4][j] * inv);
    *reinterpret_cast<bf16x4_t*>(orow + sl * 32 + 8 * q4 + 4 * hh) = pk;
  }
  if (lse && sl == 0 && hh == 0) lse[(size_t)h * n_queries + r] = L > 0.f ? M * scale + __logf(L) : -INFINITY;
}

void launch_merge_split(const tca_params* prm, const SplitPlan& sp, int64_t n_queries, uint16_t* O, float* lse, hipStream_t st) {
  const int D = prm->head_dim;
  const dim3 grid((unsigned)((n_queries + 127) / 128), prm->n_q_heads, D / 32);
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, sp, n_queries, (float)logit_scale(prm), O, lse); };
  if (D == 128) launch(merge_split_kernel<128>);
  else launch(merge_split_kernel<64>);
}

static int prefill_checked(const tca_params* prm, const void* Q, int64_t q_pos0, int64_t n_queries, const void* K,
                           const void* V, int64_t kv_stride, const int32_t* idx, const void* Kg, const void* Vg,
                           const int64_t* offs, const int32_t* n_rows, void* O, float* lse, void* ws,
                           size_t ws_bytes, void* stream, int part, const char* who) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!Q || !K || !V || !idx || !offs || !n_rows || !O)
    return fail(TCA_ERR_INVALID, "%s: NULL pointer argument", who);
  if ((Kg == nullptr) != (Vg == nullptr))
    return fail(TCA_ERR_INVALID, "%s: Kg and Vg must both be given, or both be NULL (gather-free call)", who);
  if (part != TCA_PART_ALL && part != TCA_PART_WINDOW && part != TCA_PART_GLOBAL)
    return fail(TCA_ERR_INVALID, "%s: part=%d", who, part);
  if (part != TCA_PART_ALL && !lse) return fail(TCA_ERR_INVALID, "%s: a part needs lse to be merged", who);
  if (n_queries < 0 || q_pos0 < 0 || q_pos0 + n_queries > kv_stride)
    return fail(TCA_ERR_INVALID, "%s: q_pos0=%lld n_queries=%lld kv_stride=%lld", who, (long long)q_pos0,
                (long long)n_queries, (long long)kv_stride);
  if (q_pos0 + n_queries > INT32_MAX) return fail(TCA_ERR_UNSUPPORTED, "positions beyond int32");
  if (offs[0] != 0) return fail(TCA_ERR_INVALID, "%s: offs[0] must be 0", who);
  for (int h = 0; h < sel_heads(prm); ++h)
    if (offs[h + 1] < offs[h]) return fail(TCA_ERR_INVALID, "%s: offs not ascending at %d", who, h);
  const size_t need = prm->dtype == TCA_BF16 ? prefill_mfma_workspace_need(prm, n_queries, offs[sel_heads(prm)]) : 0;
  if (need && (!ws || ws_bytes < need || ((uintptr_t)ws & 255)))
    return fail(TCA_ERR_WORKSPACE, "%s: workspace needs %zu bytes, 256-byte aligned", who, need);
  if (n_queries == 0) return TCA_OK;
  hipStream_t st = (hipStream_t)stream;
  if (prm->dtype == TCA_F32) {
    rc = launch_prefill_f32(prm, (const float*)Q, q_pos0, n_queries, (const float*)K,
                            (const float*)V, kv_stride, idx, (const float*)Kg, (const float*)Vg, offs, n_rows,
                            (float*)O, lse, st, part);
  } else {
    rc = launch_prefill_mfma(prm, (const bf16_t*)Q, q_pos0, n_queries, (const bf16_t*)K, (const bf16_t*)V,
                             kv_stride, idx, (const bf16_t*)Kg, (const bf16_t*)Vg, offs, n_rows,
                             (bf16_t*)O, lse, ws, ws_bytes, st, part);
  }
  if (rc) return rc;
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}

}  // namespace tca

extern "C" int tca_prefill(const tca_params* prm, const void* Q, int64_t q_pos0, int64_t n_queries,
                           const void* K, const void* V, int64_t kv_stride, const int32_t* idx,
                           const void* Kg, const void* Vg, const int64_t* offs, const int32_t* n_rows,
                           void* O, float* lse, void* ws, size_t ws_bytes, void* stream) {
  return prefill_checked(prm, Q, q_pos0, n_queries, K, V, kv_stride, idx, Kg, Vg, offs, n_rows, O, lse, ws, ws_bytes,
                         stream, TCA_PART_ALL, "tca_prefill");
}

extern "C" int tca_prefill_part(const tca_params* prm, int part, const void* Q, int64_t q_pos0, int64_t n_queries,
                                const void* K, const void* V, int64_t kv_stride, const int32_t* idx,
                                const void* Kg, const void* Vg, const int64_t* offs, const int32_t* n_rows,
                                void* O, float* lse, void* ws, size_t ws_bytes, void* stream) {
  return prefill_checked(prm, Q, q_pos0, n_queries, K, V, kv_stride, idx, Kg, Vg, offs, n_rows, O, lse, ws, ws_bytes,
                         stream, part, "tca_prefill_part");
}

extern "C" int tca_prefill_merge(const tca_params* prm, int64_t n_queries, void* O_a, const float* lse_a,
                                 const void* O_b, const float* lse_b, float* lse_out, void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!O_a || !lse_a || !O_b || !lse_b || n_queries < 0)
    return fail(TCA_ERR_INVALID, "tca_prefill_merge: NULL pointer argument or n_queries=%lld", (long long)n_queries);
  const int64_t rows = (int64_t)prm->n_q_heads * n_queries;
  if (rows == 0) return TCA_OK;
  hipStream_t st = (hipStream_t)stream;
  const dim3 grid((unsigned)((rows + 3) / 4));
  if (prm->dtype == TCA_BF16)
    hipLaunchKernelGGL((merge_parts_kernel<bf16_t>), grid, dim3(256), 0, st, (bf16_t*)O_a, lse_a, (const bf16_t*)O_b,
                       lse_b, lse_out, rows, prm->head_dim);
  else
    hipLaunchKernelGGL((merge_parts_kernel<float>), grid, dim3(256), 0, st, (float*)O_a, lse_a, (const float*)O_b, lse_b,
                       lse_out, rows, prm->head_dim);
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}

// Alg. 2 with the window part of the attention started before the selection (App. C, the
// overlap named there as a further optimisation): on `side_stream` the attention of every query
// over its window alone, which needs nothing the selection produces; on `stream` the selection,
// then the attention over the selected rows alone; then the merge of the two through their lse.
extern "C" int tca_select_prefill_overlapped(const tca_params* prm, const void* q_last, const void* Q,
                                             const void* K, const void* V, int64_t kv_stride, int64_t pos0,
                                             int64_t n_tokens, const double* p, const int64_t* offs,
                                             int32_t* n_rows, int32_t* idx, void* Kg, void* Vg, void* O,
                                             void* O_part, float* lse_parts, void* ws_select,
                                             size_t ws_select_bytes, void* ws_prefill, size_t ws_prefill_bytes,
                                             void* stream, void* side_stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!O_part || !lse_parts || !side_stream || side_stream == stream)
    return fail(TCA_ERR_INVALID, "tca_select_prefill_overlapped: needs O_part, lse_parts and a second stream");
  const int64_t n_lse = (int64_t)prm->n_q_heads * n_tokens;
  hipStream_t st = (hipStream_t)stream, side = (hipStream_t)side_stream;
  hipEvent_t ready = nullptr, window_done = nullptr;
  auto finish = [&](int code) {                   // the events go on every way out
    if (ready) (void)hipEventDestroy(ready);
    if (window_done) (void)hipEventDestroy(window_done);
    return code;
  };
  auto hip_ok = [&](hipError_t e, const char* what) {
    return e == hipSuccess ? TCA_OK : fail(TCA_ERR_HIP, "tca_select_prefill_overlapped: %s: %s", what, hipGetErrorString(e));
  };
  if ((rc = hip_ok(hipEventCreateWithFlags(&ready, hipEventDisableTiming), "event"))) return finish(rc);
  if ((rc = hip_ok(hipEventCreateWithFlags(&window_done, hipEventDisableTiming), "event"))) return finish(rc);
  // the inputs are ready where `stream` stands now
  if ((rc = hip_ok(hipEventRecord(ready, st), "record"))) return finish(rc);
  if ((rc = hip_ok(hipStreamWaitEvent(side, ready, 0), "wait"))) return finish(rc);
  rc = prefill_checked(prm, Q, pos0, n_tokens, K, V, kv_stride, idx, Kg, Vg, offs, n_rows, O_part, lse_parts,
                       ws_prefill, ws_prefill_bytes, side, TCA_PART_WINDOW, "tca_select_prefill_overlapped (window)");
  if (rc) return finish(rc);
  if ((rc = hip_ok(hipEventRecord(window_done, side), "record"))) return finish(rc);
  rc = tca_select(prm, q_last, K, V, kv_stride, pos0, n_tokens, p, offs, n_rows, idx, Kg, Vg, ws_select,
                  ws_select_bytes, stream);
  if (rc) return finish(rc);
  rc = prefill_checked(prm, Q, pos0, n_tokens, K, V, kv_stride, idx, Kg, Vg, offs, n_rows, O, lse_parts + n_lse,
                       ws_prefill, ws_prefill_bytes, stream, TCA_PART_GLOBAL, "tca_select_prefill_overlapped (global)");
  if (rc) return finish(rc);
  if ((rc = hip_ok(hipStreamWaitEvent(st, window_done, 0), "wait"))) return finish(rc);
  rc = tca_prefill_merge(prm, n_tokens, O, lse_parts + n_lse, O_part, lse_parts, nullptr, stream);
  return finish(rc);
}
