// Layer integration in front of the path (extensions; the paper takes Q and K as given, after
// position encoding): rotary position embedding of Q / K rows, in place.
//
// The pair (x_a, x_b) of a row at position t is turned by the angle t * base^(-2i/d),
// i = 0 .. d/2-1 (the RoFormer rotation); pair i is (i, i + d/2) or (2i, 2i+1).  Angles, sines and
// cosines are fp64 (a position of 10^5 times a frequency near 1 leaves fp32 no fraction digits
// to speak of), one per (row, pair), shared by the heads; the products are fp64 and rounded once
// to the storage type, so the result is the correctly rounded rotation up to the last fp64 digit.
#include <hip/hip_runtime.h>

#include "tca_common.h"
#include "tca_device.h"

namespace tca {

constexpr int kRopeRows = 8;                       // rows per workgroup: 8 x d/2 angles, one or less per thread
constexpr int kRopeThreads = 64 * kRopeRows;

// grid (ceil(n_rows / 8)).  First the workgroup's angles, one (row, pair) per thread, into LDS; then all heads' rows, N pairs
// (two 16-byte chunks) per thread.  HBM-bound: 32 heads x 8192 rows (134 MB read and written) 27.1 -> 25.9 us, x 32768 138 ->
// 126, x 1000 13.8 -> 9.6, one row 13.2 -> 2.5 us of kernel time (one thread per pair looping over the heads in 2-byte accesses
// before).  Four rows per workgroup: 25 us at 8000 rows but 33 at 8192, where the heads lie a power of two apart and the
// shorter pieces of each meet on the same channels; several turns requested ahead: no faster.  ALIGNED: X is 16-byte
// aligned; otherwise the chunks are read and written element by element.
template <typename T, bool INTERLEAVED, bool ALIGNED>
__global__ __launch_bounds__(kRopeThreads) void rope_kernel(T* __restrict__ X, int n_heads, int64_t n_rows, int d, int64_t pos0,
                                                            double log2_base) {
  constexpr int N = Vec16<T>::N;                   // elements of a chunk = pairs per thread and turn
  __shared__ double2 turn[kRopeRows][64];          // (cos, sin); the N of a thread apart, so that its neighbours' lie beside them
  const int half = d >> 1, per_row = half / N;     // threads per row
  const int64_t r0 = (int64_t)blockIdx.x * kRopeRows;
  const int rows = n_rows - r0 < kRopeRows ? (int)(n_rows - r0) : kRopeRows;
  {
    const int r = threadIdx.x >> 6, i = threadIdx.x & 63;
    if (r < rows && i < half) {
      const double inv_freq = exp2(-2.0 * (double)i / (double)d * log2_base);
      const double ang = (double)(pos0 + r0 + r) * inv_freq;
      double sn, cs;
      sincos(ang, &sn, &cs);
      turn[r][i % N * per_row + i / N] = make_double2(cs, sn);
    }
  }
  __syncthreads();
  const int per_head = rows * per_row, items = n_heads * per_head;
  for (int it = threadIdx.x; it < items; it += kRopeThreads) {
    const int h = it / per_head, in = it - h * per_head;
    const int row = in / per_row, k = in - row * per_row;            // this thread's pairs: k N .. k N + N - 1
    T* const at0 = X + ((size_t)h * n_rows + r0 + row) * d + (INTERLEAVED ? 2 * k * N : k * N);
    T* const at[2] = {at0, at0 + (INTERLEAVED ? N : half)};
    float x[2][N], y[2][N];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if constexpr (ALIGNED) {
        Vec16<T>::load(at[c], x[c]);
      } else {
#pragma unroll
        for (int e = 0; e < N; ++e) x[c][e] = load_f32(at[c] + e);
      }
    }
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const double2 t = turn[row][e * per_row + k];
      // pair e: element e of both chunks, or neighbours
      const int ca = INTERLEAVED ? 2 * e / N : 0, ea = INTERLEAVED ? 2 * e % N : e;
      const int cb = INTERLEAVED ? ca : 1, eb = INTERLEAVED ? ea + 1 : e;
      const double a = (double)x[ca][ea], b = (double)x[cb][eb];
      y[ca][ea] = (float)(a * t.x - b * t.y);
      y[cb][eb] = (float)(b * t.x + a * t.y);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if constexpr (ALIGNED) {
        uint32_t w[4];
        if constexpr (sizeof(T) == 4) {
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(y[c][e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = f32_to_bf16(y[c][2 * e]) | ((uint32_t)f32_to_bf16(y[c][2 * e + 1]) << 16);
        }
        *reinterpret_cast<uint4*>(at[c]) = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
#pragma unroll
        for (int e = 0; e < N; ++e) store_f32(at[c] + e, y[c][e]);
      }
    }
  }
}

template <typename T>
static void launch_rope(T* X, int n_heads, int64_t n_rows, int d, int64_t pos0, double l2b, bool interleaved, hipStream_t st) {
  const dim3 grid((unsigned)((n_rows + kRopeRows - 1) / kRopeRows));
  const bool aligned = ((uintptr_t)X & 15) == 0;   // rows are 128 bytes and more
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kRopeThreads), 0, st, X, n_heads, n_rows, d, pos0, l2b); };
  if (interleaved) { if (aligned) go(rope_kernel<T, true, true>); else go(rope_kernel<T, true, false>); }
  else { if (aligned) go(rope_kernel<T, false, true>); else go(rope_kernel<T, false, false>); }
}

}  // namespace tca

using namespace tca;

extern "C" int tca_rope(const tca_params* prm, void* X, int n_heads, int64_t n_rows, int64_t pos0, double base,
                        int pairing, void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!X || n_heads < 1 || n_rows < 0 || pos0 < 0 || !(base > 1.0))
    return fail(TCA_ERR_INVALID, "tca_rope: X=%p n_heads=%d n_rows=%lld pos0=%lld base=%g", X, n_heads,
                (long long)n_rows, (long long)pos0, base);
  if (pairing != TCA_ROPE_HALF && pairing != TCA_ROPE_INTERLEAVED)
    return fail(TCA_ERR_UNSUPPORTED, "tca_rope: pairing=%d", pairing);
  if (n_rows == 0) return TCA_OK;
  hipStream_t st = (hipStream_t)stream;
  const double l2b = __builtin_log2(base);
  const bool interleaved = pairing == TCA_ROPE_INTERLEAVED;
  if (prm->dtype == TCA_BF16) launch_rope((bf16_t*)X, n_heads, n_rows, prm->head_dim, pos0, l2b, interleaved, st);
  else launch_rope((float*)X, n_heads, n_rows, prm->head_dim, pos0, l2b, interleaved, st);
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}
