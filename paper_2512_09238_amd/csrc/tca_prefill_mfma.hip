// bf16 MFMA flash-attention prefill over the global and local subsets (Eq. 2;
// Alg. 2 line 7) for gfx950.
//
// Work decomposition.  One workgroup = NW wavefronts = one tile of BM = 32 NW
// consecutive queries of one query head; wave v owns 32 of them (NW = 8, 256
// queries, for long calls; NW = 4 when a call has few query tiles).  The
// workgroup walks 64-key tiles: first the head's compacted global rows (tiles
// of the head's region of Kg), then the dense keys of the sliding window
// (absolute 64-key tiles of K).  Visibility is a prefix test in both parts:
//   global row g of the region : g  < nvis(i) = #{idx <= i-w}   (idx ascends)
//   dense key j                : i-w < j <= i
// so only boundary tiles evaluate a mask.
//
// MFMA mapping (v_mfma_f32_32x32x16_bf16, 64 lanes; lane = (hh = lane/32, c = lane%32)):
//   S^T = K Q^T  : A = K rows (key = c, 8 consecutive d), B = Q (query = c, same 8 d),
//                  C[key = 8*(r/4)+4*hh+r%4][query = c].  A lane therefore holds 16
//                  keys of ONE query per 32-key sub-tile: the softmax max/sum are
//                  in-register reductions plus one exchange between the two halves.
//   O^T = V^T P^T: B = P^T taken straight from the C registers of S^T (registers
//                  8g..8g+7 -> one bf16x8), A = V^T (d = c, the same 8 keys: 4 hh .. 4 hh + 3 and
//                  the four 8 further on).  Four waves: V lies in LDS as it does in memory, a row per
//                  key, and ds_read_b64_tr_b16 transposes on the way out: 16 lanes address 4 keys x 16
//                  columns, and lane i receives column i of the four keys, half an operand.  Eight waves:
//                  V^T tiles are produced once per call by a transposing pre-pass into the workspace, the 64
//                  keys of a tile in the order the C registers hold them, so that the operand is one
//                  16-byte LDS read (uses_transposed_v).
//   O^T accumulators: C[d = 32*s + 8*(r/4)+4*hh+r%4][query = c]: every register of
//                  a lane belongs to the same query, so rescaling is a per-lane scalar.
//
// LDS holds a ring of K tiles [64][D] and a ring of V ([64][D]) or V^T ([D][64]) tiles (two tiles each; three
// in the two-blocks-per-wave shape) with XOR-swizzled 16-byte chunks (conflict-free
// reads without padding), filled by direct global -> LDS loads.  The loop is
// software-pipelined by one tile (see the kernel); one barrier per tile.
//
// Softmax bookkeeping.  One block per wave (the shapes the library launches by itself): the
// reference m of a query's exponentials is the running maximum of its visible scores; the
// state is rescaled, before a tile's exponentials, only when some query's maximum moved.
// Two blocks per wave (a diagnostic shape): the reference is lazy - any earlier maximum of
// visible scores, raised only when a tile's terms would come near the top of the fp32 range
// (row sum of the tile >= kRaise); terms, sum and accumulators share the reference, so the
// quotient is the same, and the common tile needs no maximum at all.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "tca_prefill.h"

namespace tca {
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int kBN = 64;              // keys per tile
constexpr int kFragAhead = 4;        // LDS fragment reads in flight ahead of the MFMA that uses them
constexpr float kRaise = 0x1p60f;    // a tile whose terms sum to this much raises the softmax reference

struct PrefillHeads {
  int64_t offs[TCA_MAX_HEADS + 1];      // row offsets of the heads' regions
  int32_t tile_off[TCA_MAX_HEADS + 1];  // V^T tile offsets of the heads' regions
  int32_t xcd_start[9];                 // the range of the (head, query tile) sequence each XCD works through
  int32_t order;                        // how an XCD walks its range: see the ids in prefill_mfma_kernel
  uint8_t perm[TCA_MAX_HEADS];          // order 1 and 2: the heads in the sequence
};

struct NoSplit {};

// Where the V^T operand comes from.  The transposing reads take twice the instructions of plain ones, and the eight-wave
// step, whose order is pinned to the instruction, pays for them: 3.7 % more cycles, 72.7 -> 73.7 ms at 128K tokens with
// the pre-pass (0.31 ms) already taken off, 16.20 -> 16.15 for 8192 tokens behind 112K (64 heads).  The four-wave shapes take
// the calls of few query tiles, which read a tile a few times: there the pre-pass is a launch and two passes over V for
// nothing (413 tokens behind 64K: 231 -> 193 us, 41 of them the pre-pass; on inputs that are not in the caches 330 -> 251
// together with the fenced order of the steps).
constexpr bool uses_transposed_v(int nw) { return nw == 8; }

// position p (0..63) inside a stored V^T tile -> key (0..63) of the tile
__host__ __device__ inline int vt_key_of_pos(int p) {
  const int sub = p >> 5, q = p & 31;
  const int g = q >> 4, hh = (q >> 3) & 1, e = q & 7;
  return sub * 32 + 16 * g + 8 * (e >> 2) + 4 * hh + (e & 3);
}

// ---------------------------------------------------------------- pre-pass --
// Transposes 64-row tiles of row-major [rows, D] bf16 matrices into [D][64] tiles (keys permuted by
// vt_key_of_pos); rows past the last become zero, tiles past it are left alone (nobody reads them).  HBM-bound: no
// LDS, a thread loads 16 bytes of the eight keys of one output chunk, transposes the 8 x 8 block in registers and
// stores eight 16-byte chunks; of a wave's loads and stores every eight lanes cover 128 consecutive bytes.
// The loads are non-temporal: nothing else reads these rows, and what they would push out of the caches is what the
// attention kernel starts with.  us per call, staged through LDS in two launches / plain loads / this: 64 heads behind 112K
// tokens (2.4 GB moved) 420 / 438 / 417, 32 heads and 128K tokens 326 / 341 / 314, 64 heads behind 64K 159 / 165 / 151,
// 5446 tokens 14.3 / 11.1 / 11.0.  (Non-temporal stores, or a wave over whole rows and half the keys: 459 and 500 at 112K.)
// The first region_tiles tiles are those of the regions (head by ph.tile_off; gather_idx != NULL: row r of a region
// is row gather_idx[ph.offs[g] + r] of the dense matrix of KV head g / sel_per_kv, no compacted copy exists), the
// others dense rows (tiles_per_group per KV head, from row first_row on, valid below valid_all).
// grid (ceil(tiles / (256 / D))): D threads per tile; block 256.
template <int D>
__global__ __launch_bounds__(256) void transpose_tiles_kernel(
    const uint16_t* __restrict__ Vg, const uint16_t* __restrict__ V, int64_t kv_stride, const int32_t* __restrict__ n_rows,
    const int32_t* __restrict__ gather_idx, int sel_per_kv, int Hs, int region_tiles, int tiles, int tiles_per_group,
    int64_t first_row, int64_t valid_all, uint16_t* __restrict__ region_dst, uint16_t* __restrict__ dense_dst,
    PrefillHeads ph) {
  constexpr int TPT = D;                           // threads per tile: 8 chunks of keys x D / 8 chunks of columns
  const int tid = threadIdx.x;
  const int t = __builtin_amdgcn_readfirstlane(blockIdx.x * (256 / TPT) + tid / TPT);      // uniform: a wave has one tile
  if (t >= tiles) return;
  const int in = tid % TPT;
  const int part = (in >> 3) & 7, cg = (in & 7) + 8 * (in >> 6);       // chunk of keys, chunk of columns
  const uint16_t* src;
  const int32_t* gi = nullptr;
  int64_t row0, n_valid;
  uint16_t* out;
  if (t < region_tiles) {
    int g = 0;
    for (int step = 64; step > 0; step >>= 1)
      if (g + step < Hs && ph.tile_off[g + step] <= t) g += step;
    const int64_t r = (int64_t)(t - ph.tile_off[g]) * kBN;
    n_valid = n_rows[g] - r;
    row0 = r;
    if (gather_idx) {
      gi = gather_idx + ph.offs[g] + r;
      src = V + (size_t)(g / sel_per_kv) * kv_stride * D;
    } else {
      src = Vg + (size_t)ph.offs[g] * D;
    }
    out = region_dst + (size_t)t * (D * kBN);
  } else {
    const int dt = t - region_tiles, g = dt / tiles_per_group;
    row0 = first_row + (int64_t)(dt - g * tiles_per_group) * kBN;
    n_valid = valid_all - row0;
    src = V + (size_t)g * kv_stride * D;
    out = dense_dst + (size_t)dt * (D * kBN);
  }
  if (n_valid <= 0) return;
  uint4 v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = vt_key_of_pos(part * 8 + e);
    v[e] = make_uint4(0, 0, 0, 0);
    if (k < n_valid) {
      const size_t row = gi ? (size_t)gi[k] : (size_t)(row0 + k);
      const raw16_t x = __builtin_nontemporal_load(reinterpret_cast<const raw16_t*>(src + row * D + cg * 8));
      v[e] = make_uint4(x.x, x.y, x.z, x.w);
    }
  }
  const uint32_t* w = reinterpret_cast<const uint32_t*>(v);            // [key][pair of columns]
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint4 lo, hi;                                  // columns 2 j and 2 j + 1 over the eight keys
    uint32_t* l = reinterpret_cast<uint32_t*>(&lo);
    uint32_t* h = reinterpret_cast<uint32_t*>(&hi);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      l[k] = __builtin_amdgcn_perm(w[(2 * k + 1) * 4 + j], w[2 * k * 4 + j], 0x05040100u);
      h[k] = __builtin_amdgcn_perm(w[(2 * k + 1) * 4 + j], w[2 * k * 4 + j], 0x07060302u);
    }
    uint16_t* o = out + (size_t)(cg * 8 + 2 * j) * kBN + part * 8;
    *reinterpret_cast<uint4*>(o) = lo;
    *reinterpret_cast<uint4*>(o + kBN) = hi;
  }
}

// The cycle counters of a call (diagnostics only), cleared in front of the kernel that adds to them.
__global__ void clear_clocks_kernel(unsigned long long* clk) { clk[threadIdx.x] = 0; }

// ------------------------------------------------------------- main kernel --
__device__ __forceinline__ int64_t i64min(int64_t a, int64_t b) { return a < b ? a : b; }

// O^T += V^T P^T step.  With two query blocks per wave the O^T accumulators (128 registers for
// d = 128) are pinned to the accumulation registers, which only the matrix pipe touches, so that
// the scores and the exponentials' terms keep the vector registers.  The instruction is written
// out because the register file of an operand cannot be chosen through the builtin; what the
// compiler then cannot see is that o is being written for 8 passes after issue: every vector
// ALU read of o goes through settle_acc() first.
template <bool ACC>
__device__ __forceinline__ void pv_mfma(f32x16_t& o, const bf16x8_t& a, const bf16x8_t& b) {
  if constexpr (ACC) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
  else o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, o, 0, 0, 0);
}
// S^T = K Q^T steps for two query blocks per wave: scores in vector registers, Q fragments in
// accumulation registers.  FIRST starts a chain from zero.
template <bool FIRST>
__device__ __forceinline__ void s_mfma(f32x16_t& s, const bf16x8_t& k, const bf16x8_t& q) {
  if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "a"(q));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "a"(q));
}
// The last step of the four chains of a tile (two blocks x two 32-key sub-tiles), followed by the
// wait states the vector ALU needs before it may touch their results (19 at most; the compiler
// inserts them for the builtin, not for a written-out instruction).
__device__ __forceinline__ void s_mfma_last(f32x16_t& s00, f32x16_t& s10, f32x16_t& s01, f32x16_t& s11,
                                            const bf16x8_t& k0, const bf16x8_t& k1, const bf16x8_t& q0,
                                            const bf16x8_t& q1) {
  asm volatile(
      "v_mfma_f32_32x32x16_bf16 %0, %4, %6, %0\n\t"
      "v_mfma_f32_32x32x16_bf16 %1, %4, %7, %1\n\t"
      "v_mfma_f32_32x32x16_bf16 %2, %5, %6, %2\n\t"
      "v_mfma_f32_32x32x16_bf16 %3, %5, %7, %3\n\t"
      "s_nop 15\n\ts_nop 7"
      : "+v"(s00), "+v"(s10), "+v"(s01), "+v"(s11)
      : "v"(k0), "v"(k1), "a"(q0), "a"(q1));
}
// Marks the accumulators as living in the accumulation registers at this point (no instruction):
// placed after every vector-ALU update of o, so that the value the loop carries has one home and
// is not shuttled between the two register files on every iteration.
template <int N>
__device__ __forceinline__ void home_acc(f32x16_t (&o)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+a"(o[i]));
}
// Waits out the matrix pipe's pending writes to accumulators before the vector ALU reads them.
template <int N>
__device__ __forceinline__ void settle_acc(f32x16_t (&o)[N]) {
  static_assert(N == 2 || N == 4, "one statement per supported slice count");
  if constexpr (N == 4)
    asm volatile("s_nop 15\n\ts_nop 7" : "+a"(o[0]), "+a"(o[1]), "+a"(o[2]), "+a"(o[3]));
  else
    asm volatile("s_nop 15\n\ts_nop 7" : "+a"(o[0]), "+a"(o[1]));
}

// Two four-wave workgroups share a CU, and an XCD deals its ids to its 32 CUs in turn: every second run of 32 ids is
// taken backwards, so that of a sequence sorted by length the longest and the shortest meet on a CU.
__host__ __device__ __forceinline__ int pair_up(int u, int n) {
  const int b = u & ~31, len = n - b < 32 ? n - b : 32;
  return (u & 32) ? b + len - 1 - (u - b) : u;
}

// Cross-half exchange: returns max over the two 32-lane halves, in every lane.
__device__ __forceinline__ float half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// XOR swizzle of a row's 16-byte chunks.  K, V^T: the 32 lanes of a half read one chunk column of 32 rows.  V: a half of a
// transposing read takes 64 bytes, four chunks, of rows 0 .. 3 or 4 .. 7, which fill the 64 banks once if the four chunks
// move together by the row (by two at a time, so that eight rows of 32 bytes fill them, every read took twice as long:
// SQ_LDS_BANK_CONFLICT).
template <int D> __device__ __forceinline__ int k_swz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D> __device__ __forceinline__ int v_swz(int r) { return D == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; }
// LDS byte offset of 16-byte chunk `ch` of K row r, of V^T row dd
template <int D> __device__ __forceinline__ int k_off(int r, int ch) { return r * (D * 2) + ((ch ^ k_swz<D>(r)) << 4); }
__device__ __forceinline__ int vt_off(int dd, int ch) { return dd * (kBN * 2) + ((ch ^ ((dd >> 1) & 7)) << 4); }

// Four keys of this lane's column (see vfa).  Without the __restrict__ the compiler takes the read for one that may meet
// the tile copies in flight and waits for them first, in the middle of every step (128K tokens: 7 % more cycles).  No such wait
// is needed: the tile read has landed by the wait and the barrier of the step before, and the copies in flight go to
// other places of the ring.
__device__ __forceinline__ bf16x4_t read_transposed(const unsigned char* __restrict__ lds_src) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4_t*)lds_src);
}

// Tile copies go global -> LDS directly (buffer loads with the LDS modifier: no
// staging registers, no ds_write).  Every lane of a wave-load deposits 16 bytes at
// consecutive LDS addresses, so the lane that fills LDS chunk position p of a row
// fetches the global chunk the XOR swizzle assigns to p: a per-lane byte offset
// inside the tile that never changes.  The tile itself is selected by the scalar
// offset of the load, and rows past the end of a buffer read as zero (range check of
// the buffer descriptor), so a copy costs no vector ALU work at all.  A K or V tile is
// CPR wave-loads; each wave issues its share one load at a time, spread
// between the MFMAs instead of queueing up behind the barrier.
template <int D, int NW>
struct TileCopy {
  static constexpr int CPR = D / 8;
  static constexpr int NK = CPR / NW;               // K wave-loads per wave
  static constexpr int NV = CPR / NW;               // V wave-loads per wave
  static constexpr int N = NK + NV;
  static_assert(NK >= 1 && NV >= 1 && N <= D / 16, "too many or too few waves for this tile");
  // byte offset inside a K tile of the chunk this lane fetches in wave-load q
  static __device__ __forceinline__ int k_lane_offset(int q, int lane) {
    const int cid = q * 64 + lane;                  // 16-byte chunk of the LDS tile this lane fills
    const int r = cid / CPR, pch = cid % CPR;
    return (r * D + (pch ^ k_swz<D>(r)) * 8) * 2;
  }
  static __device__ __forceinline__ int v_lane_offset(int q, int lane) {
    const int cid = q * 64 + lane;
    const int r = cid / CPR, pch = cid % CPR;
    return (r * D + (pch ^ v_swz<D>(r)) * 8) * 2;
  }
  static __device__ __forceinline__ int vt_lane_offset(int q, int lane) {
    const int cid = q * 64 + lane;
    const int dd = cid >> 3, pch = cid & 7;
    return (dd * kBN + (pch ^ ((dd >> 1) & 7)) * 8) * 2;
  }
};

__device__ __forceinline__ void copy16_to_lds(__amdgpu_buffer_rsrc_t rsrc, int lane_off, int tile_off,
                                              unsigned char* lds_dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds_dst, 16, lane_off,
                                           tile_off, 0, 0);
}

// Software pipeline over the tiles of a workgroup (tile t = 0 .. n_tiles-1: first the
// n_gt tiles of the head's compacted region, then the dense tiles of the window).  A wave
// owns QB blocks of 32 queries.  With QB = 1, iteration t is
//   slot A :  S(t+1) = K(t+1) Q^T          (MFMA)  }  one basic block: the MFMAs of the next
//             P(t)   = exp step on S(t)    (VALU)  }  tile run under this tile's exponentials
//   slot B :  O     += V(t)^T P(t)         (MFMA)
// With QB = 2 every K / V^T fragment read from LDS feeds two MFMAs (one per block; the LDS
// port moves 128 bytes per clock and CU, which with one fragment per MFMA is as much of a
// limit as the matrix pipe itself), the wave has a SIMD to itself (512 registers), and the
// second block's softmax runs half an iteration late so that both slots pair 32 MFMAs with
// one block's exponentials, neither depending on the other:
//   slot A :  S_a(t+1), S_b(t+1)           (MFMA)  |  P_a(t)   from S_a(t)     (VALU)
//   slot B :  O_a += V(t)^T P_a(t), O_b += V(t)^T P_b(t)  |  P_b(t+1) from S_b(t+1)
// K(t+RING) and V(t+RING-1) are copied global -> LDS during iteration t, into the places
// of K(t) and V(t-1); the rings hold RING = 2 or 3 tiles each; one barrier per iteration.
// Positions and byte offsets are 32-bit here: the host checks (q_pos0 + n_queries) * D * 2 < 2^31.
// GATHER: no compacted copy exists; the K and V rows of a region tile are fetched from the dense K and V
// through idx (the position of every row is read one iteration ahead and becomes the lane's offset of the
// tile copies: V's tile is the one whose K was copied an iteration before, its positions are still there;
// V^T tiles were built through idx by the pre-pass).
// SPLIT: the workgroup walks one chunk of the item's tiles and leaves its accumulators, m and l to the merge.
template <int D, int NW, int QB, bool GATHER, bool SPLIT = false>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2 / QB, 2 / QB)))
void prefill_mfma_kernel(
    const uint16_t* __restrict__ Q, int64_t q_pos0, int64_t n_queries, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, int64_t kv_stride, const int32_t* __restrict__ idx,
    const uint16_t* __restrict__ Kg, const uint16_t* __restrict__ Vg, const int32_t* __restrict__ n_rows,
    int64_t dense_tile0, int dense_tiles, PrefillHeads ph, int Hq, int G, int GS, int w, float scale,
    uint16_t* __restrict__ O, float* __restrict__ lse, unsigned long long* __restrict__ clk, int part,
    std::conditional_t<SPLIT, SplitPlan, NoSplit> sp) {
  // part: TCA_PART_ALL, or one of the two key subsets alone (TCA_PART_WINDOW: the dense window;
  // TCA_PART_GLOBAL: the region), each normalised by itself, to be merged through lse
  // V, Vg: the rows as the caller has them, or (uses_transposed_v) the pre-pass's tiles: of the dense rows from tile
  // dense_tile0 on, dense_tiles per KV head, and of the regions
  constexpr bool VT = uses_transposed_v(NW);
  constexpr int KK = D / 16;             // MFMA k-steps over the head dimension
  constexpr int DS = D / 32;             // 32-row slices of O^T
  constexpr int WQ = QB * 32;            // queries per wave
  constexpr int BM = NW * WQ;            // queries per workgroup
  const unsigned long long clk_c0 = __builtin_readcyclecounter(), clk_r0 = __builtin_amdgcn_s_memrealtime();
  constexpr int KBYTES = kBN * D * 2;    // K tile
  constexpr int VBYTES = kBN * D * 2;    // V tile
  // Rows are not padded; the 16-byte chunk index is XOR-swizzled with the row so that
  // the b128 reads of 16 consecutive rows at one chunk column fall into distinct banks.
  // Tiles in flight: rings of two K and two V tiles, a copy has one iteration to arrive (with two
  // waves per SIMD a third tile measured no faster); the one-wave-per-SIMD shape, where nothing else
  // covers a late copy, keeps three.
  constexpr int RING = QB == 2 ? 3 : 2;
  __shared__ __attribute__((aligned(16))) unsigned char lds[RING * (KBYTES + VBYTES)];
  unsigned char* const kring = lds;
  unsigned char* const vring = lds + RING * KBYTES;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave index, scalar
  const int hh = lane >> 5, c = lane & 31;
  const int n_qt = (int)((n_queries + BM - 1) / BM);
  const int bid = blockIdx.x;
  // Workgroup ids go round-robin over the 8 XCDs, each with an L2 of its own.  With Hq a multiple
  // of 8, XCD x is given the heads x*Hq/8 .. (x+1)*Hq/8 - 1 and works through them one at a time:
  // the query tiles in flight on an XCD then belong to one head and stream the same K / V^T tiles
  // through its L2 (and the heads of a KV group, which share the dense tiles - with a shared
  // selection all tiles - follow each other on the same XCD).
  // Heads differ in the rows they keep, so whole heads per XCD leave the XCDs unevenly loaded: the
  // sequence (head-major, a head's query tiles longest first) is cut instead into eight ranges of equal
  // estimated work (xcd_start, from the host).  An XCD takes the piece of the head its range ends in
  // first (that head's longest tiles) and the rest in order, so that it ends on a head's shortest tiles.
  // That is order 0.  With few rounds of workgroups the order matters more than the L2: order 1 takes the query
  // tiles longest first and the XCD's heads inside, order 2 the heads longest first (plan_xcds chooses).
  int h, qtile;
  int t_first = 0;                                 // the first tile this workgroup walks
  [[maybe_unused]] int item = 0;
  if constexpr (SPLIT) {
    // The order is chunk-major inside a head, so that the query tiles that read the same keys are neighbours; runs
    // of them are dealt to the XCDs in turn: a run shares an L2, and the chunks that are short or empty (where the
    // queries see less than the longest one does) spread over all XCDs.
    const int u = bid >> 3, turn = u / sp.run;
    item = (turn * 8 + (bid & 7)) * sp.run + (u - turn * sp.run);
    if (item >= sp.item_start[Hq]) return;
    h = 0;
    for (int step = 64; step > 0; step >>= 1)
      if (h + step < Hq && sp.item_start[h + step] <= item) h += step;
    const int in = item - sp.item_start[h], ch = in / n_qt;
    qtile = in - ch * n_qt;
    t_first = ch * sp.chunk;
  } else if ((Hq & 7) == 0) {
    const int x = bid & 7;                         // XCD
    int u = bid >> 3;                              // position in the XCD's own sequence
    const int s = ph.xcd_start[x], e = ph.xcd_start[x + 1];
    if (u >= e - s) return;                        // the grid is sized for the longest range
    if (NW == 4 && ph.order == 1) u = pair_up(u, e - s);
    if (ph.order == 0) {
      const int he = e / n_qt * n_qt;              // where the head begins in which the range ends
      const int len_e = he > s ? e - he : 0;
      const int g = u < len_e ? he + u : s + (u - len_e);
      h = g / n_qt;
      qtile = n_qt - 1 - g % n_qt;
    } else {                                       // whole heads per XCD, Hq / 8 each
      const int nh = Hq >> 3, hp = ph.order == 1 ? u % nh : u / n_qt;
      h = ph.perm[x * nh + hp];
      qtile = n_qt - 1 - (ph.order == 1 ? u / nh : u - hp * n_qt);
    }
  } else {
    // longest query tiles first, all heads of each; the heads are shifted from turn to turn so that an XCD (which
    // gets every eighth id) does not always meet the same ones
    const int x = bid & 7, mine = (n_qt * Hq - x + 7) >> 3;       // XCD, and how many ids it gets
    const int g = NW == 4 ? pair_up(bid >> 3, mine) * 8 + x : bid;
    const int k = g / Hq, period = 8 / ((Hq & 1) ? 1 : (Hq & 2) ? 2 : 4);
    h = (g - k * Hq + k / period) % Hq;
    qtile = n_qt - 1 - k;
  }
  const int kvh = h / G;
  const int64_t r0 = (int64_t)qtile * BM;          // first query row of the workgroup
  const int64_t last_row = n_queries - 1;
  const float sl2e = scale * 1.4426950408889634f;

  // ---- per-lane query state (lane column c = one query of each block)
  const int hs = h / GS;                           // the selection this query head reads (GS query heads share it)
  const int64_t base = ph.offs[hs];
  const int nr = part == TCA_PART_WINDOW ? 0 : n_rows[hs];     // without the region nothing below sees a global row
  int qpos[QB], nvis[QB];
  bf16x8_t qf[QB][KK];
#pragma unroll
  for (int blk = 0; blk < QB; ++blk) {
    int64_t qrow_i = r0 + wv * WQ + blk * 32 + c;
    if (qrow_i > last_row) qrow_i = last_row;       // clamped rows compute a duplicate; never stored
    qpos[blk] = (int)(q_pos0 + qrow_i);
    const uint16_t* qrow = Q + ((size_t)h * n_queries + qrow_i) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[blk][kk] = *reinterpret_cast<const bf16x8_t*>(qrow + kk * 16 + hh * 8);
  }
  // wave-level visibility bounds (queries ascend with block and lane column; clamped rows repeat the last)
  const int wave_first = (int)(q_pos0 + i64min(r0 + wv * WQ, last_row));
  const int wave_last = (int)(q_pos0 + i64min(r0 + wv * WQ + WQ - 1, last_row));
  const int wg_last = (int)(q_pos0 + i64min(r0 + BM - 1, last_row));
  const int wg_first = (int)(q_pos0 + r0);
  const int last_pos = (int)(q_pos0 + last_row);
  // Global rows visible to every query of the wave, to some query of the workgroup, to each lane's query.  A
  // workgroup has the CU to itself (or shares it with one other), so what its prologue waits for is lost: one
  // search with a wave-uniform bound, done by the wave together (three dependent loads for 2^18 rows; a binary
  // search per lane was 17), then one round more: positions are distinct and ascending and the workgroup's last
  // query lies at most BM - 1 behind the wave's first, so only the next BM rows can make the differences.
  // While the window reaches back to the start there is nothing to count.
  int nv_wave_lo = 0, nv_wg_hi = 0;
#pragma unroll
  for (int blk = 0; blk < QB; ++blk) nvis[blk] = 0;
  if (wg_last >= w && nr > 0) {
    nv_wave_lo = __builtin_amdgcn_readfirstlane(count_le_wave(idx + base, nr, (int64_t)wave_first - w));
    int nxt[BM / 64];                              // lane j of nxt[i]: the position of row nv_wave_lo + 64 i + j
#pragma unroll
    for (int i = 0; i < BM / 64; ++i) {
      const int r = nv_wave_lo + i * 64 + lane;
      nxt[i] = r < nr ? idx[base + r] : 0x7FFFFFFF;
    }
    nv_wg_hi = nv_wave_lo;
#pragma unroll
    for (int i = 0; i < BM / 64; ++i) nv_wg_hi += __builtin_popcountll(__ballot(nxt[i] <= wg_last - w));
#pragma unroll
    for (int blk = 0; blk < QB; ++blk) nvis[blk] = nv_wave_lo;
#pragma unroll
    for (int j = 0; j < WQ - 1; ++j) {
      const int pj = __builtin_amdgcn_readlane(nxt[0], j);
#pragma unroll
      for (int blk = 0; blk < QB; ++blk) nvis[blk] += (int64_t)pj <= (int64_t)qpos[blk] - w;
    }
  }
  const int n_gt = (nv_wg_hi + kBN - 1) / kBN;
  const int win_lo = wg_first - w + 1 > 0 ? wg_first - w + 1 : 0;
  const int wt0 = win_lo / kBN, wt1 = wg_last / kBN;                      // absolute dense tiles [wt0, wt1]
  int n_tiles = n_gt + (part == TCA_PART_GLOBAL ? 0 : wt1 - wt0 + 1);       // SPLIT: up to the end of the chunk
  if constexpr (SPLIT) {
    if (t_first >= n_tiles) {                      // nothing left for this chunk: the merge skips it by its l
      float* const ml = sp.part + (size_t)item * split_floats<D>() + 128 * D;
      if (tid < 128) { ml[tid] = -INFINITY; ml[128 + tid] = 0.f; }
      return;
    }
    if (t_first + sp.chunk < n_tiles) n_tiles = t_first + sp.chunk;
  }
  const int last = n_tiles - 1;
  if (n_tiles == 0) {                              // TCA_PART_GLOBAL with no visible global row: an empty part
#pragma unroll
    for (int blk = 0; blk < QB; ++blk) {
      const int64_t r = r0 + wv * WQ + blk * 32 + c;
      if (r <= last_row) {
        uint16_t* orow = O + ((size_t)h * n_queries + r) * D;
#pragma unroll
        for (int sl = 0; sl < DS; ++sl)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) *reinterpret_cast<uint2*>(orow + sl * 32 + 8 * q4 + 4 * hh) = make_uint2(0u, 0u);
        if (lse && hh == 0) lse[(size_t)h * n_queries + r] = -INFINITY;
      }
    }
    return;
  }
  const int dshift = wt0 - n_gt;                   // tile t >= n_gt is the dense tile t + dshift

  // ---- sources of the tile copies: one descriptor per buffer, the tile chosen by a scalar byte offset
  using Copy = TileCopy<D, NW>;
  constexpr int kRsrcFlags = 0x00020000;           // raw buffer, 32-bit data format
  const __amdgpu_buffer_rsrc_t krs_g = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(GATHER ? K : Kg + (size_t)base * D), 0, GATHER ? 0 : nr * (D * 2), kRsrcFlags);   // GATHER: never read
  const __amdgpu_buffer_rsrc_t krs_d = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(K + (size_t)kvh * kv_stride * D), 0, (last_pos + 1) * (D * 2), kRsrcFlags);
  constexpr bool VGATHER = GATHER && !VT;
  const __amdgpu_buffer_rsrc_t vrs_g = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(VT ? Vg + (size_t)ph.tile_off[hs] * (D * kBN) : VGATHER ? V : Vg + (size_t)base * D), 0,
      VT ? n_gt * VBYTES : VGATHER ? 0 : nr * (D * 2), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t vrs_d = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(V + (VT ? (size_t)kvh * dense_tiles * (D * kBN) : (size_t)kvh * kv_stride * D)), 0,
      VT ? dense_tiles * VBYTES : (last_pos + 1) * (D * 2), kRsrcFlags);
  const int vdshift = VT ? dshift - (int)dense_tile0 : dshift;       // tile t >= n_gt is tile t + vdshift of the dense V or V^T buffer
  int klo[Copy::NK], vlo[VT ? Copy::NV : 1];       // this lane's byte offsets inside a tile, per wave-load (V: 1024 more for the next)
  int krow[Copy::NK];                              // the tile row this lane copies a chunk of, per wave-load of K or V
#pragma unroll
  for (int j = 0; j < Copy::NK; ++j) {
    klo[j] = Copy::k_lane_offset(wv * Copy::NK + j, lane);
    krow[j] = ((wv * Copy::NK + j) * 64 + lane) / Copy::CPR;
  }
#pragma unroll
  for (int j = 0; j < (VT ? Copy::NV : 1); ++j)
    vlo[j] = VT ? Copy::vt_lane_offset(wv * Copy::NV + j, lane) : Copy::v_lane_offset(wv * Copy::NV + j, lane);
  // One K tile and one V tile to copy: descriptors and scalar offsets chosen once, then
  // load(j) issues wave-load j of the K tile (j < NK) or of the V tile (j >= NK)
  struct CopyJob {
    __amdgpu_buffer_rsrc_t krs, vrs;
    int koff, voff;
    unsigned char* kdst;
    unsigned char* vdst;
    bool k_through_idx, v_through_idx;       // GATHER: a region tile, its rows fetched from the dense K, V
    int kgo[Copy::NK], vgo[VGATHER ? Copy::NV : 1];  // GATHER: this lane's byte offset into the dense K, V, per wave-load
  };
  // GATHER: positions of the rows this lane copies from region tile t (rows past the region's end get
  // an offset beyond the buffer, which the descriptor's range check turns into zeros)
  struct TileRows { int pos[Copy::NK]; };
  auto load_tile_rows = [&](int t) {
    TileRows tr;
#pragma unroll
    for (int j = 0; j < Copy::NK; ++j) {
      const int r = t * kBN + krow[j];
      tr.pos[j] = (t < n_gt && r < nr) ? idx[base + r] : -1;
    }
    return tr;
  };
  auto copy_job = [&](int tk, int tv, unsigned char* kstage, unsigned char* vstage, const TileRows& rows_k,
                      const TileRows& rows_v) {
    CopyJob j;
    const bool kg = tk < n_gt, vg = tv < n_gt;
    j.krs = (kg && !GATHER) ? krs_g : krs_d;
    j.vrs = (vg && !VGATHER) ? vrs_g : vrs_d;
    j.koff = (tk + (kg ? 0 : dshift)) * KBYTES;
    j.voff = (tv + (vg ? 0 : vdshift)) * VBYTES;
    j.kdst = kstage + wv * (Copy::NK * 1024);
    j.vdst = vstage + wv * (Copy::NV * 1024);
    j.k_through_idx = GATHER && kg;
    j.v_through_idx = VGATHER && vg;
    if constexpr (GATHER) {
      static_assert(Copy::NK == Copy::NV, "a lane copies the same rows of K and of V");
#pragma unroll
      for (int q = 0; q < Copy::NK; ++q) {     // the chunk inside the row stays the swizzled one of klo, vlo
        j.kgo[q] = rows_k.pos[q] >= 0 ? rows_k.pos[q] * (D * 2) + (klo[q] - krow[q] * (D * 2)) : 0x7FFFFFF0;
        if constexpr (VGATHER) j.vgo[q] = rows_v.pos[q] >= 0 ? rows_v.pos[q] * (D * 2) + (vlo[0] + q * 1024 - krow[q] * (D * 2)) : 0x7FFFFFF0;
      }
    }
    return j;
  };
  auto copy_load = [&](const CopyJob& job, int j) {
    if (j < Copy::NK) {
      if (GATHER && job.k_through_idx) copy16_to_lds(job.krs, job.kgo[j], 0, job.kdst + j * 1024);
      else copy16_to_lds(job.krs, klo[j], job.koff, job.kdst + j * 1024);
    } else {
      if (VGATHER && job.v_through_idx) copy16_to_lds(job.vrs, job.vgo[j - Copy::NK], 0, job.vdst + (j - Copy::NK) * 1024);
      else if (VT) copy16_to_lds(job.vrs, vlo[VT ? j - Copy::NK : 0], job.voff, job.vdst + (j - Copy::NK) * 1024);
      else copy16_to_lds(job.vrs, vlo[0], job.voff + (j - Copy::NK) * 1024, job.vdst + (j - Copy::NK) * 1024);
    }
  };

  f32x16_t o[QB][DS];
  float m[QB], l[QB];
#pragma unroll
  for (int blk = 0; blk < QB; ++blk) {
    m[blk] = -INFINITY;
    l[blk] = 0.f;
#pragma unroll
    for (int sl = 0; sl < DS; ++sl)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[blk][sl][r] = 0.f;
    if constexpr (QB == 2) home_acc(o[blk]);
  }

  // per-lane LDS byte offsets of the MFMA fragments inside a tile (the rest is compile-time constant):
  // K fragment (sub, kk) sits at kfa[kk] + sub * 32 rows; V^T fragment (sl, sg) at vfa[sg] + sl * 32 rows, or its halves in
  // V at vfa[sl] + sg * 16 rows and 8 rows behind; the swizzles depend on the row only through c (K, V^T), vr (V)
  int kfa[KK], vfa[4];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) kfa[kk] = k_off<D>(c, 2 * kk + hh);
  if constexpr (VT) {
#pragma unroll
    for (int sg = 0; sg < 4; ++sg) vfa[sg] = vt_off(c, 2 * sg + hh);
  } else {
    const int vr = 4 * hh + ((c >> 2) & 3);        // what a lane addresses: 4 columns of a key; what it receives: a column of 4 keys
#pragma unroll
    for (int sl = 0; sl < DS; ++sl)
      vfa[sl] = vr * (D * 2) + (((4 * sl + 2 * (c >> 4) + ((c >> 1) & 1)) ^ v_swz<D>(vr)) << 4) + (c & 1) * 8;
  }

  // S^T = K Q^T for the 64 keys of the tile at kb and every query block of the wave (two 32-key
  // sub-tiles per block = 2 QB accumulation chains that alternate; fragments read kFragAhead
  // ahead and used once per block); between_pairs(kk) runs after the kk-th pair of fragments
  // (the place where the tile copies are issued)
  auto s_tile = [&](const unsigned char* kb, f32x16_t (&s)[QB][2], auto after_fragment) {
    auto kfrag = [&](int i) {
      return *reinterpret_cast<const bf16x8_t*>(kb + kfa[i >> 1] + (i & 1) * (32 * D * 2));
    };
    bf16x8_t fr[kFragAhead];
#pragma unroll
    for (int i = 0; i < kFragAhead; ++i) fr[i] = kfrag(i);
    if constexpr (QB == 1) {
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[0][sub][r] = 0.f;
#pragma unroll
      for (int i = 0; i < 2 * KK; ++i) {
        const int sub = i & 1, kk = i >> 1;
        s[0][sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % kFragAhead], qf[0][kk], s[0][sub], 0, 0, 0);
        if (i + kFragAhead < 2 * KK) fr[i % kFragAhead] = kfrag(i + kFragAhead);
        after_fragment(i);
      }
    } else {
      // the Q fragments (64 registers for d = 128) sit in the accumulation registers as well; the
      // last MFMA of every chain and the wait for their results share one statement
#pragma unroll
      for (int i = 0; i < 2 * KK - 2; ++i) {
        const int sub = i & 1, kk = i >> 1;
#pragma unroll
        for (int blk = 0; blk < QB; ++blk) {
          if (kk == 0) s_mfma<true>(s[blk][sub], fr[i % kFragAhead], qf[blk][kk]);
          else s_mfma<false>(s[blk][sub], fr[i % kFragAhead], qf[blk][kk]);
        }
        if (i + kFragAhead < 2 * KK) fr[i % kFragAhead] = kfrag(i + kFragAhead);
        after_fragment(i);
      }
      s_mfma_last(s[0][0], s[1][0], s[0][1], s[1][1], fr[(2 * KK - 2) % kFragAhead], fr[(2 * KK - 1) % kFragAhead],
                  qf[0][KK - 1], qf[1][KK - 1]);
      after_fragment(2 * KK - 2);
      after_fragment(2 * KK - 1);
    }
  };

  // maximum over the 32 scores a lane holds of its query, then over the two lanes of the query
  auto lane_max = [&](const f32x16_t (&s)[2]) {
    float m8[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) m8[r] = fmaxf(fmaxf(s[0][r], s[0][r + 8]), fmaxf(s[1][r], s[1][r + 8]));
    return half_max(fmaxf(fmaxf(fmaxf(m8[0], m8[1]), fmaxf(m8[2], m8[3])), fmaxf(fmaxf(m8[4], m8[5]), fmaxf(m8[6], m8[7]))));
  };

  // exponentials of the scores s against the reference mb (already in base-2 units): bf16 terms in
  // operand order, and their sum over the lane's 32 keys.  With the running maximum as reference
  // (QB = 1) the largest term of a query is exactly 1, which bf16 holds exactly, and the sum takes
  // the fp32 terms; summing the bf16-rounded ones instead (one v_dot2_f32_bf16 per pair), so that
  // numerator and denominator carry the same rounding, was measured: 1.2 % slower, and 8.3e-3
  // instead of 9.7e-3 worst error on logits in the hundreds, both far inside the 2e-2 the outputs
  // are held to.  With the lazy reference (QB = 2) the largest term is an arbitrary number whose
  // rounding (2^-9 relative) goes straight into the output of a query that attends to one key:
  // there the sum must take the rounded terms, so that the quotient cancels that rounding.
  auto exp_tile = [&](const f32x16_t (&s)[2], float mb, bf16x8_t (&pf)[2][2]) {
    float ls[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        bf16x8_t pk;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[sub][8 * g + e], sl2e, -mb));
          pk[e] = (__bf16)p;
          ls[e & 3] += QB == 2 ? (float)pk[e] : p;
        }
        pf[sub][g] = pk;
      }
    return (ls[0] + ls[1]) + (ls[2] + ls[3]);
  };

  // The same work cut into NCH pieces for the two-block schedule, where the written-out MFMAs pin
  // the instruction order and the pieces are placed between them by hand: piece i forms the
  // exponentials of elements i*EPC .. i*EPC+EPC-1 and rounds, stores and sums those of piece i-1
  // (one piece later, so that no instruction waits on the exponential it has just issued);
  // piece NCH only finishes piece NCH-1.  ls must start at zero; the tile's sum is ls[0..3] added up.
  constexpr int NCH = 2 * KK;            // = fragments of a K tile = fragments of a V^T tile
  constexpr int EPC = 32 / NCH;          // elements of a lane's 32 per piece: 2 (d = 128) or 4 (d = 64)
  auto exp_piece = [&](int i, const f32x16_t (&s)[2], float mb, bf16x8_t (&pf)[2][2], float (&ls)[4], float (&pend)[EPC]) {
    const bf16x2_t ones = {(__bf16)1.f, (__bf16)1.f};
    if (i >= 1) {
#pragma unroll
      for (int k = 0; k < EPC; k += 2) {                 // the sum takes the rounded terms (see exp_tile)
        const int n = (i - 1) * EPC + k;                 // even element of a pair
        const bf16x2_t pr = {(__bf16)pend[k], (__bf16)pend[k + 1]};
        pf[n >> 4][(n >> 3) & 1][n & 7] = pr[0];
        pf[n >> 4][(n >> 3) & 1][(n & 7) + 1] = pr[1];
        ls[(n >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, ls[(n >> 1) & 3], false);
      }
    }
    if (i < NCH) {
#pragma unroll
      for (int k = 0; k < EPC; ++k) {
        const int n = i * EPC + k;
        pend[k] = __builtin_amdgcn_exp2f(fmaf(s[n >> 4][n & 15], sl2e, -mb));
      }
    }
  };

  // And for the four-wave shape, whose steps the scheduler gives up ordering by itself (all exponentials between the MFMAs of S
  // and those of P V): one slot of it behind every MFMA of the step (t = 0 .. 2 KK - 1: of S, from 2 KK on: of P V), the order
  // written out and fenced.  Exponentials at an even pace, done two slots before the last of them are needed (the last
  // quarter of P V), rounded and summed one slot behind; the terms' sum in the order of exp_tile.  413 tokens behind 64K: 193
  // -> 183.6 us.  The eight-wave shape is 1.1 % slower this way than in the order pinned below, and with rows fetched through
  // idx there are no registers left for it.  With 64 elements only chunks take it (us pinned / fenced: 8192 tokens of 4 heads
  // 64.3 / 60.0, 6363 of 8 heads behind 64K 510 / 467); calls that walk their tiles whole are as fast or faster in the pinned
  // order: 4 heads, 12000 tokens 82 / 90, 20000 on inputs that are not in the caches 144 / 168, 40000 behind 64K 1693 / 1790.
  constexpr bool kFenced = NW == 4 && QB == 1 && !GATHER && (D == 128 || SPLIT);
  constexpr int kSlots = 2 * KK + 4 * DS;
  auto exp_slot = [&](int t, const f32x16_t (&s)[2], float mb, bf16x8_t (&pf)[2][2], float (&ls)[4], float (&p)[32]) {
    auto done = [](int u) {                          // elements formed by the end of slot u
      constexpr int span = kSlots * 13 / 16;
      const int n = u < 0 ? 0 : ((u + 1) * 16 + span - 1) / span * 2;
      return n < 32 ? n : 32;
    };
    for (int n = done(t - 2); n < done(t - 1); ++n) {
      pf[n >> 4][(n >> 3) & 1][n & 7] = (__bf16)p[n];
      ls[n & 3] += p[n];
      asm volatile("" : "+v"(ls[n & 3]));            // added here: left to itself the compiler keeps all 32 terms to the end
    }
    for (int n = done(t - 1); n < done(t); ++n) p[n] = __builtin_amdgcn_exp2f(fmaf(s[n >> 4][n & 15], sl2e, -mb));
  };

  // Does every query of the wave see every key of tile t?  (wave-uniform)
  auto mask_tile_is_clear = [&](int t) {
    const bool is_glob = t < n_gt;
    const int key0 = (t + (is_glob ? 0 : dshift)) * kBN;
    return t <= last && (is_glob ? (key0 + kBN <= nv_wave_lo) : (key0 + kBN - 1 <= wave_first && key0 > wave_last - w));
  };
  // Mask of tile t on the scores s of block blk (boundary tiles only; a tile this wave sees nothing
  // of, or past the last one, is fully masked).  Returns whether this lane's query sees any key of it.
  auto mask_tile = [&](int t, int blk, f32x16_t (&s)[2]) {
    const bool is_glob = t < n_gt;
    const int key0 = (t + (is_glob ? 0 : dshift)) * kBN;
    const bool beyond = t > last;
    const bool masked = beyond || (is_glob ? (key0 + kBN > nv_wave_lo)
                                           : !(key0 + kBN - 1 <= wave_first && key0 > wave_last - w));
    bool sees = true;
    if (masked) {
      // visible <=> lo <= key - key0 < hi, with one unsigned compare per element
      int lo, hi;
      if (is_glob) {
        lo = 0;
        hi = nvis[blk] - key0 < kBN ? nvis[blk] - key0 : kBN;
      } else {
        const int l32 = qpos[blk] - w + 1 - key0, h32 = qpos[blk] + 1 - key0;
        lo = l32 < 0 ? 0 : (l32 > kBN ? kBN : l32);
        hi = h32 < 0 ? 0 : (h32 > kBN ? kBN : h32);
      }
      const unsigned span = (hi > lo && !beyond) ? (unsigned)(hi - lo) : 0u;
      sees = span != 0u;
      const int rel0 = 4 * hh - lo;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const unsigned kr = (unsigned)(rel0 + sub * 32 + 8 * (r >> 2) + (r & 3));
          s[sub][r] = kr < span ? s[sub][r] : -INFINITY;
        }
    }
    return sees;
  };

  // The uncommon tile: the query's first visible keys, or terms too large for the reference.
  // The reference becomes the maximum over the visible scores so far (the same in both lanes of
  // a query), the state is rescaled and the tile's terms are formed again.
  auto softmax_fixup = [&](int blk, const f32x16_t (&s)[2], bool cold, bool sees, float& lt, bf16x8_t (&pf)[2][2]) {
    if (__any(lt >= kRaise || (cold && sees))) {
      const float m_new = fmaxf(m[blk], lane_max(s));
      const float alpha = (m_new > m[blk]) ? __builtin_amdgcn_exp2f((m[blk] - m_new) * sl2e) : 1.f;   // 0 when m was -inf
      l[blk] *= alpha;
      if constexpr (QB == 2) settle_acc(o[blk]);
#pragma unroll
      for (int sl = 0; sl < DS; ++sl)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[blk][sl][r] *= alpha;
      if constexpr (QB == 2) home_acc(o[blk]);
      m[blk] = m_new;
      lt = exp_tile(s, (m_new == -INFINITY) ? 0.f : m_new * sl2e, pf);
    }
  };

  bf16x8_t pf[QB][2][2];                 // P of block 0: formed and used inside a step; of block 1: formed one step ahead

  int rpos = 0;                          // it % RING of the step about to run
  float mx_pre = -INFINITY;              // QB = 1: unmasked maximum of the scores the next step starts from
  TileRows rows_ahead = {}, rows_before = {};        // GATHER: row positions of tile it + RING, read during step it - 1, and of it + RING - 1
  static_assert((RING - 2) * Copy::N < 16, "the wait below encodes its count in four bits");

  // One pipeline step: tile `it` (scores in sc; with QB = 2 those of block 1 are already in pf[1])
  // goes through softmax and P V; the scores of tile it+1 go to sn.
  // clear_tag: std::true_type when the caller knows that this wave sees every key of tile `it` (the
  // stretches of the loop below where no tile needs a mask), which saves the test per step
  auto step = [&](int it, f32x16_t (&sc)[QB][2], f32x16_t (&sn)[QB][2], auto clear_tag) {
    constexpr bool kKnownClear = decltype(clear_tag)::value;
    // K(it+1) and V(it) have landed for this wave (only the copies of the previous step may still
    // be on their way when the rings hold three tiles); after the barrier for every wave, and every
    // wave is done reading K(it) and V(it-1).  With one block per wave this wait and barrier sit
    // inside the previous step, before its last P V MFMAs (see there).
    if constexpr (QB != 1) {
      __builtin_amdgcn_s_waitcnt(0x0F70 | ((RING - 2) * Copy::N));     // vmcnt((RING - 2) * N)
      __syncthreads();
    }
    const int tk = it + RING < last ? it + RING : last, tv = it + RING - 1 < last ? it + RING - 1 : last;   // past the end: a harmless reload
    // ring places (it - 1, it, it + 1) % RING; with two places they follow from the parity of `it`, which the
    // twice-unrolled loop makes a constant of each copy of the step (LDS offsets fold into the instructions)
    const int r_cur = RING == 2 ? (it & 1) : rpos;
    const int r_next = RING == 2 ? ((it + 1) & 1) : (rpos + 1 == RING ? 0 : rpos + 1);
    const int r_prev = RING == 2 ? r_next : (rpos == 0 ? RING - 1 : rpos - 1);
    const CopyJob job = copy_job(tk, tv, kring + r_cur * KBYTES, vring + r_prev * VBYTES, rows_ahead, rows_before);
    // GATHER: the positions for the copies of the next step are requested before this step's copies,
    // so that the wait at the top of the next step, which lets only the newest copies pass, covers them
    if constexpr (GATHER) {
      rows_before = rows_ahead;
      rows_ahead = load_tile_rows(it + 1 + RING < last ? it + 1 + RING : last);
    }
    const unsigned char* kb = kring + r_next * KBYTES;
    const unsigned char* vb = vring + r_cur * VBYTES;
    if constexpr (RING != 2) rpos = r_next;

    // ---- slot A: scores of the next tile (MFMA) under the exponentials of this one (VALU), taken
    // against the reference as it stands
    // With 64 elements, whose steps are short, V is asked for before K: the step's end waits for both.  us K / V first, pinned
    // steps, 4 heads: 20000 tokens on inputs that are not in the caches 144 / 141, 40000 behind 64K 1693 / 1618; with 128
    // elements neither is better.
    constexpr bool kVFirst = D == 64 && NW == 4 && QB == 1 && !GATHER;
    auto issue_copies = [&](int i) {     // copies spread as evenly as the counts allow: load j after fragment pair j * KK / N
      const int kk = i >> 1, j = kk * Copy::N / KK;
      if ((i & 1) && (kk * Copy::N) % KK == 0 && j < Copy::N) copy_load(job, kVFirst ? (j + Copy::NK) % Copy::N : j);
    };
    auto vfrag = [&](int j) {
      if constexpr (VT) return *reinterpret_cast<const bf16x8_t*>(vb + vfa[j / DS] + (j % DS) * (32 * kBN * 2));
      const unsigned char* at = vb + vfa[j % DS] + (j / DS) * (16 * D * 2);
      const bf16x4_t lo = read_transposed(at), hi = read_transposed(at + 8 * D * 2);
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    bf16x8_t vfr[kFragAhead];
    float ls_slot[4] = {0.f, 0.f, 0.f, 0.f}, p_slot[32], m2[2], mb_slot = 0.f;
    if constexpr (QB == 1) {
      // One block per wave, two waves per SIMD: the reference is the running maximum of the visible
      // scores.  The maximum of this tile was taken under the previous step's P V MFMAs (again after
      // masking on a boundary tile); the state is rescaled, before the exponentials, only when some
      // query's maximum moved.  Everything from here to the end of the step is one basic block, so
      // that the first P V MFMAs can start while the later exponentials are still being formed.
      const bool masked = !kKnownClear && !mask_tile_is_clear(it);
      float mx = mx_pre;
      if (masked) {
        mask_tile(it, 0, sc[0]);
        mx = lane_max(sc[0]);
      }
      const float m_new = fmaxf(m[0], mx);
      if (__any(m_new > m[0])) {
        const float alpha = (m_new > m[0]) ? __builtin_amdgcn_exp2f((m[0] - m_new) * sl2e) : 1.f;   // 0 when m was -inf
        l[0] *= alpha;
#pragma unroll
        for (int sl = 0; sl < DS; ++sl)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[0][sl][r] *= alpha;
        m[0] = m_new;
      }
      const float mb = mb_slot = (m_new == -INFINITY) ? 0.f : m_new * sl2e;
      if constexpr (kFenced) {
        __builtin_amdgcn_sched_barrier(0);
        s_tile(kb, sn, [&](int i) {
          issue_copies(i);
          if (i >= 2 * KK - kFragAhead) vfr[i - (2 * KK - kFragAhead)] = vfrag(i - (2 * KK - kFragAhead));
          exp_slot(i, sc[0], mb, pf[0], ls_slot, p_slot);
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
        s_tile(kb, sn, issue_copies);
        l[0] += exp_tile(sc[0], mb, pf[0]);
      }
    } else {
      const bool sees = mask_tile(it, 0, sc[0]);
      const bool cold = m[0] == -INFINITY;          // no reference yet: no key seen so far
      const float mb = cold ? 0.f : m[0] * sl2e;
      float ls[4] = {0.f, 0.f, 0.f, 0.f}, pend[EPC];
      __builtin_amdgcn_sched_barrier(0);
      s_tile(kb, sn, [&](int i) {
        issue_copies(i);
        exp_piece(i, sc[0], mb, pf[0], ls, pend);
        __builtin_amdgcn_sched_barrier(0);
      });
      exp_piece(NCH, sc[0], mb, pf[0], ls, pend);
      float lt = (ls[0] + ls[1]) + (ls[2] + ls[3]);
      softmax_fixup(0, sc[0], cold, sees, lt, pf[0]);
      l[0] += lt;
    }

    // ---- slot B: O^T += V^T P^T for every block (the accumulation chains alternate; V^T fragments
    // are read ahead and used once per block), under the exponentials of block 1's next tile
    bool sees1 = true, cold1 = false;
    float mb1 = 0.f, ls1[4] = {0.f, 0.f, 0.f, 0.f}, pend1[EPC];
    bf16x8_t pn[2][2];
    if constexpr (QB == 2) {
      sees1 = mask_tile(it + 1, 1, sn[1]);
      cold1 = m[1] == -INFINITY;
      mb1 = cold1 ? 0.f : m[1] * sl2e;
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!kFenced) {
#pragma unroll
      for (int j = 0; j < kFragAhead; ++j) vfr[j] = vfrag(j);
    }
#pragma unroll
    for (int j = 0; j < 4 * DS; ++j) {
      const int sl = j % DS, sg = j / DS;           // sg = sub*2 + g: 16 keys
      if constexpr (QB == 1) {
        // The barrier of the next step, taken as soon as the last V fragment of this tile has been
        // requested (the reads run kFragAhead ahead): the MFMAs still to come work from registers and
        // cover the first fragment reads of the next tile, which cannot start before the barrier.
        if (j == 4 * DS - kFragAhead) {
          __builtin_amdgcn_s_waitcnt(0x0F70);          // this wave's copies of K(it+2), V(it+1) have landed
          __syncthreads();
        }
      }
#pragma unroll
      for (int blk = 0; blk < QB; ++blk) pv_mfma<QB == 2>(o[blk][sl], vfr[j % kFragAhead], pf[blk][sg >> 1][sg & 1]);
      if (j + kFragAhead < 4 * DS) vfr[j % kFragAhead] = vfrag(j + kFragAhead);
      if constexpr (kFenced) {
        exp_slot(2 * KK + j, sc[0], mb_slot, pf[0], ls_slot, p_slot);
        const int r = 2 * (j - (4 * DS - 8) / 2);    // the next tile's maximum over the lane's keys
        if (r >= 0 && r < 16) {
          m2[0] = fmaxf(fmaxf(r ? m2[0] : sn[0][0][0], sn[0][0][r]), sn[0][0][r + 1]);
          m2[1] = fmaxf(fmaxf(r ? m2[1] : sn[0][1][0], sn[0][1][r]), sn[0][1][r + 1]);
          asm volatile("" : "+v"(m2[0]), "+v"(m2[1]));         // formed here, as the sums
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (QB == 2) {
        exp_piece(j, sn[1], mb1, pn, ls1, pend1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (kFenced) {
      l[0] += (ls_slot[0] + ls_slot[1]) + (ls_slot[2] + ls_slot[3]);
      mx_pre = half_max(fmaxf(m2[0], m2[1]));
    } else if constexpr (QB == 1) {
      mx_pre = lane_max(sn[0]);                        // vector ALU work for the shadow of the MFMAs above
      // The order of the step's instructions, spelled out for the scheduler (the step is one scheduling
      // region): behind every MFMA one fragment read and an even share of the plain vector ALU work, the
      // exponentials left to fall where they may, which is two per MFMA of the S half.  Left to itself the
      // scheduler starts the step with eight bare MFMAs and crowds the exponentials into the middle;
      // measured 2 - 2.5 % faster than that (2 .. 6 instructions behind an MFMA of S and 3 .. 6 behind
      // one of P V tried: within 1 % of each other).  Pinning the exponentials or the scalar
      // instructions as well measured 8 % slower.
      constexpr int kMfma = 0x008, kValu = 0x002, kDsRead = 0x100, kVmemRead = 0x020;
      constexpr int kVReads = VT ? 1 : 2;              // of a V^T fragment
      constexpr int VA = 384 / D, VB = 640 / D;        // plain vector ALU instructions behind an MFMA of S, of P V
      __builtin_amdgcn_sched_group_barrier(kDsRead, kFragAhead, 0);
#pragma unroll
      for (int i = 0; i < 2 * KK; ++i) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
        if (!VT && i >= 2 * KK - kFragAhead) __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
        if ((i & 1) && ((i >> 1) * Copy::N) % KK == 0 && (i >> 1) * Copy::N / KK < Copy::N)
          __builtin_amdgcn_sched_group_barrier(kVmemRead, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kValu, VA, 0);
      }
#pragma unroll
      for (int j = 0; j < 4 * DS; ++j) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
        if (j + kFragAhead < 4 * DS) __builtin_amdgcn_sched_group_barrier(kDsRead, kVReads, 0);
        __builtin_amdgcn_sched_group_barrier(kValu, VB, 0);
      }
    }
    if constexpr (QB == 2) {
      exp_piece(NCH, sn[1], mb1, pn, ls1, pend1);
      float lt = (ls1[0] + ls1[1]) + (ls1[2] + ls1[3]);
      softmax_fixup(1, sn[1], cold1, sees1, lt, pn);
      l[1] += lt;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int g = 0; g < 2; ++g) pf[1][a][g] = pn[a][g];
    }
  };

  // ---- prologue: everything the steps do not copy themselves - K(0) .. K(RING-1), V(0) ..
  // V(RING-2) - is requested here, oldest first; S(0) is formed as soon as K(0) is in
  f32x16_t sa[QB][2], sb[QB][2];
  {
    auto tile_or_last = [&](int t) { return t < last ? t : last; };
    const TileRows rows_first = load_tile_rows(t_first), rows_second = load_tile_rows(tile_or_last(t_first + 1));
    const CopyJob first = copy_job(t_first, t_first, kring, vring, rows_first, rows_first);
#pragma unroll
    for (int j = 0; j < Copy::N; ++j) copy_load(first, j);
    const CopyJob second = copy_job(tile_or_last(t_first + 1), 0, kring + KBYTES, vring, rows_second, rows_first);
#pragma unroll
    for (int j = 0; j < Copy::NK; ++j) copy_load(second, j);
    if constexpr (RING == 3) {
      const CopyJob third = copy_job(tile_or_last(2), tile_or_last(1), kring + 2 * KBYTES, vring + VBYTES,
                                     load_tile_rows(tile_or_last(2)), rows_second);
#pragma unroll
      for (int j = 0; j < Copy::N; ++j) copy_load(third, j);
    }
    if constexpr (GATHER) {                        // for the copies of step 0
      rows_before = rows_second;
      rows_ahead = load_tile_rows(tile_or_last(t_first + RING));
    }
    // A wave without a query (of a last query tile, four waves) makes its copies and meets the barriers of every step, and
    // nothing else: what the matrix cores are spared raises the clock.  413 queries behind 64K tokens, of whose sixteen waves a
    // head three have none: 1.81 -> 1.90 GHz, 150 -> 143 us.
    if constexpr (NW == 4 && QB == 1) {
      if (r0 + wv * WQ > last_row) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        __syncthreads();
        for (int it = t_first; it < n_tiles; ++it) {
          const CopyJob job = copy_job(tile_or_last(it + 2), tile_or_last(it + 1), kring + (it & 1) * KBYTES, vring + ((it + 1) & 1) * VBYTES,
                                       rows_ahead, rows_before);
          if constexpr (GATHER) {
            rows_before = rows_ahead;
            rows_ahead = load_tile_rows(tile_or_last(it + 3));
          }
#pragma unroll
          for (int j = 0; j < Copy::N; ++j) copy_load(job, j);
          __builtin_amdgcn_s_waitcnt(0x0F70);
          __syncthreads();
        }
        return;                                        // (the merge of chunks reads no row without a query)
      }
    }
    // K(0), V(0) are in (GATHER: the positions just requested count among the newest as well)
    __builtin_amdgcn_s_waitcnt(0x0F70 | (Copy::NK + (RING - 2) * Copy::N + (GATHER ? Copy::NK : 0)));
    __syncthreads();
    s_tile(kring, sa, [&](int) {});
    if constexpr (QB == 1) mx_pre = lane_max(sa[0]);
    if constexpr (QB == 2) {            // block 1 runs half a step ahead with its exponentials
      const bool sees = mask_tile(0, 1, sa[1]);
      float lt = exp_tile(sa[1], 0.f, pf[1]);
      softmax_fixup(1, sa[1], true, sees, lt, pf[1]);
      l[1] += lt;
    }
  }
  const unsigned long long clk_loop = __builtin_readcyclecounter();
  if constexpr (QB == 1) {
    __builtin_amdgcn_s_waitcnt(0x0F70);              // K(1) is in: the barrier of step 0 (every later one sits in the step before)
    __syncthreads();
  }
  // (the stretches below pay off with eight waves; with four the scheduler no longer follows the order
  // pinned in the step for the test-free copies of it, and the plain loop is faster)
  if constexpr (QB == 1 && NW == 8) {
    // The tiles this wave sees all of form two stretches: the region tiles below the rows visible to its
    // first query, and the window tiles between its last query's window start and its first query.  Their
    // ends are moved to even steps (a clear tile may always take the masked path), so that every stretch
    // is a run of the twice-unrolled loop.
    const int a0 = nv_wave_lo / kBN;                                         // region tiles [0, a0) are clear
    const int t_lo = wave_last - w < 0 ? 0 : (wave_last - w) / kBN + 1;       // dense tiles [t_lo, t_hi] are clear
    const int t_hi = wave_first - (kBN - 1) < 0 ? -1 : (wave_first - (kBN - 1)) / kBN;
    int b0 = t_lo - dshift, c0 = t_hi + 1 - dshift;                           // as steps: [b0, c0)
    if (b0 < n_gt) b0 = n_gt;
    if (c0 > n_tiles) c0 = n_tiles;
    const int a = a0 & ~1;
    int b = (b0 + 1) & ~1, c = c0 & ~1;
    if (b < a) b = a;
    if (c < b) c = b;
    if (b > n_tiles) b = c = n_tiles & ~1;
    for (int it = 0; it < a; it += 2) {
      step(it, sa, sb, std::true_type{});
      step(it + 1, sb, sa, std::true_type{});
    }
    for (int it = a; it < b; it += 2) {
      step(it, sa, sb, std::false_type{});
      if (it + 1 < n_tiles) step(it + 1, sb, sa, std::false_type{});
    }
    for (int it = b; it < c; it += 2) {
      step(it, sa, sb, std::true_type{});
      step(it + 1, sb, sa, std::true_type{});
    }
    for (int it = c; it < n_tiles; it += 2) {
      step(it, sa, sb, std::false_type{});
      if (it + 1 < n_tiles) step(it + 1, sb, sa, std::false_type{});
    }
  } else {
    for (int it = t_first; it < n_tiles; it += 2) {
      step(it, sa, sb, std::false_type{});
      if (it + 1 < n_tiles) step(it + 1, sb, sa, std::false_type{});
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);             // no copy into this workgroup's LDS may outlive it
  if (clk && tid == 0) {                          // diagnostics only: elapsed shader-clock cycles and 100 MHz ticks of this workgroup
    atomicAdd(clk, (unsigned long long)__builtin_readcyclecounter() - clk_c0);
    atomicAdd(clk + 1, (unsigned long long)__builtin_amdgcn_s_memrealtime() - clk_r0);
    atomicAdd(clk + 2, clk_loop - clk_c0);        // of which before the first step
    atomicAdd(clk + 3, (unsigned long long)(n_tiles - t_first));
  }

  if constexpr (SPLIT) {                           // the lanes' accumulators as they lie: the merge reads them the same way
    static_assert(NW == 4 && QB == 1, "128 queries per workgroup");
    float* const po = sp.part + (size_t)item * split_floats<D>();
    typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
#pragma unroll
    for (int sl = 0; sl < DS; ++sl)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4_t v = {o[0][sl][4 * q4], o[0][sl][4 * q4 + 1], o[0][sl][4 * q4 + 2], o[0][sl][4 * q4 + 3]};
        *reinterpret_cast<f32x4_t*>(po + (((sl * 4 + q4) * NW + wv) * 64 + lane) * 4) = v;
      }
    const float lt = half_sum(l[0]);
    if (hh == 0) { po[128 * D + wv * 32 + c] = m[0]; po[128 * D + 128 + wv * 32 + c] = lt; }
    return;
  }

  // ---- normalise and store
#pragma unroll
  for (int blk = 0; blk < QB; ++blk) {
    const int64_t r = r0 + wv * WQ + blk * 32 + c;
    const float lt = half_sum(l[blk]);
    if constexpr (QB == 2) settle_acc(o[blk]);
    if (r <= last_row) {
      const float inv = lt > 0.f ? 1.f / lt : 0.f;    // a query that sees nothing of this part: zeros, lse = -inf
      uint16_t* orow = O + ((size_t)h * n_queries + r) * D;
#pragma unroll
      for (int sl = 0; sl < DS; ++sl)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          bf16x4_t pk;
#pragma unroll
          for (int j = 0; j < 4; ++j) pk[j] = (__bf16)(o[blk][sl][4 * q4 + j] * inv);
          *reinterpret_cast<bf16x4_t*>(orow + sl * 32 + 8 * q4 + 4 * hh) = pk;
        }
      if (lse && hh == 0) lse[(size_t)h * n_queries + r] = lt > 0.f ? m[blk] * scale + __logf(lt) : -INFINITY;
    }
  }
}

// ------------------------------------------------------------------ host side --
struct MfmaWs {
  unsigned long long* clk;   // sums over the workgroups of the last call: {shader-clock cycles, 100 MHz ticks, cycles before the first step, tiles}
  uint16_t* Vgt;       // [g_tiles][D][64]
  uint16_t* Vt;        // [Hkv][dense_tiles][D][64]
  float* part;         // split calls: [workgroups][split_floats]; what lies behind it may be missing
  size_t need;         // bytes without it: what a call must be given
  size_t bytes;        // bytes with it
};

static int64_t max_region_tiles(int Hq, int64_t cap_rows) { return (cap_rows + kBN - 1) / kBN + Hq; }
static int64_t max_dense_tiles(int64_t n_queries, int w) { return (n_queries + w) / kBN + 2; }

// Workgroups of a split call, at most: two rounds of what the chip holds at a time, and no more than the tiles there
// are in chunks of kMinChunk.  Grows with both arguments, so that a workspace sized for the largest call of a
// program serves its smaller ones.
constexpr int kSplitSlots = 512;       // four-wave workgroups the chip runs at a time: two per CU
constexpr int kMinChunk = 8;           // tiles: below that a workgroup's prologue and its partial results outweigh the walk
static int64_t max_split_items(const tca_params* prm, int64_t n_queries, int64_t cap_rows) {
  const int64_t tiles = (cap_rows + kBN - 1) / kBN + max_dense_tiles(n_queries, prm->window);
  const int64_t all = prm->n_q_heads * ((n_queries + 127) / 128) * ((tiles + kMinChunk - 1) / kMinChunk);
  return all < 2 * kSplitSlots ? all : 2 * kSplitSlots;
}

static MfmaWs carve_mfma_ws(void* ws, const tca_params* prm, int64_t g_tiles, int64_t d_tiles, int64_t split_items) {
  MfmaWs m;
  char* b = (char*)ws;
  size_t off = 0;
  const size_t tile_bytes = (size_t)prm->head_dim * kBN * 2;
  m.clk = (unsigned long long*)(b + off); off = align_up(off + 4 * sizeof(unsigned long long), 256);
  m.Vgt = (uint16_t*)(b + off); off = align_up(off + (size_t)g_tiles * tile_bytes, 256);      // (room a four-wave call leaves alone)
  m.Vt = (uint16_t*)(b + off);  off = align_up(off + (size_t)prm->n_kv_heads * d_tiles * tile_bytes, 256);
  m.need = off;
  m.part = (float*)(b + off);
  off += (size_t)split_items * (prm->head_dim == 128 ? split_floats<128>() : split_floats<64>()) * sizeof(float);
  m.bytes = off;
  return m;
}

static MfmaWs mfma_ws(void* ws, const tca_params* prm, int64_t n_queries, int64_t cap_rows) {
  return carve_mfma_ws(ws, prm, max_region_tiles(sel_heads(prm), cap_rows), max_dense_tiles(n_queries, prm->window),
                       max_split_items(prm, n_queries, cap_rows));
}
size_t prefill_mfma_workspace_bytes(const tca_params* prm, int64_t n_queries, int64_t cap_rows) {
  return mfma_ws(nullptr, prm, n_queries, cap_rows).bytes;
}
size_t prefill_mfma_workspace_need(const tca_params* prm, int64_t n_queries, int64_t cap_rows) {
  return mfma_ws(nullptr, prm, n_queries, cap_rows).need;
}

// Tile steps of query tile qt (BM queries) of a head with a region of cap rows: the dense tiles of the window,
// exactly; the visible part of the region as if its rows were spread evenly over the positions seen so far (the
// host does not know idx).
static int64_t tile_steps(const tca_params* prm, int64_t cap, int64_t q_pos0, int64_t n_queries, int BM, int64_t qt, int part) {
  const int w = prm->window;
  const int64_t L_end = q_pos0 + n_queries;
  const int64_t first = q_pos0 + qt * BM, lastq = first + BM - 1 < L_end - 1 ? first + BM - 1 : L_end - 1;
  int64_t c = 0;
  if (part != TCA_PART_GLOBAL) c += lastq / kBN - (first - w + 1 > 0 ? first - w + 1 : 0) / kBN + 1;
  if (part != TCA_PART_WINDOW && lastq >= w && cap) c += (cap * (lastq - w + 1) / L_end + kBN - 1) / kBN;
  return c;
}

// The workgroup places of one XCD, items taken in order by the first free one: when the slowest ends.  A tournament over the
// times the places are free: an item costs one path to the root and no branch.  The XCDs are played side by side (plan_xcds), so
// that their paths, each a chain of a dozen dependent instructions, overlap: 3.6 ns an item (64 places), a binary heap 19.
template <int SLOTS>
struct Places {
  int32_t worst = 0, node[2 * SLOTS];              // 64 time + place; node[1] the earliest, node[SLOTS + i] place i
  Places() {
    for (int i = 0; i < SLOTS; ++i) node[SLOTS + i] = i;
    for (int i = SLOTS - 1; i > 0; --i) node[i] = std::min(node[2 * i], node[2 * i + 1]);
  }
  void take(int32_t cost) {                        // (times stay below 2^25: 16 rounds of an item's steps, which are 2^18 at most)
    int32_t k = node[1] + (cost << 6);
    int i = SLOTS + (k & 63);
    worst = std::max(worst, k >> 6);
    node[i] = k;
    for (int level = 1; level < SLOTS; level *= 2) {
      k = std::min(k, node[i ^ 1]);
      i >>= 1;
      node[i] = k;
    }
  }
};

// Chooses which items an XCD takes and in which order (PrefillHeads: xcd_start, order, perm), and returns the
// length of the longest range.  *makespan: the estimated end of the call in tile steps.
// Candidates: the (head, query tile) sequence, a head at a time, cut into eight ranges of equal estimated work
// (heads keep different numbers of rows) or of whole heads; and whole heads dealt out so that the XCDs' sums come
// close, walked by query tile (longest first, the heads inside) or by head (longest first).  Where there are many
// rounds of workgroups, equal work ends evenly by itself and one head at a time is the order that the L2 likes
// (a late start of a long head costs little): no other is looked at from 16 rounds on.  Otherwise each is played
// through (`slots` workgroups at a time per XCD, the next item to the first free slot).  The estimate is in tile steps
// (tile_steps), and a constant for what a workgroup does before and after its loop; a poor one costs balance, never
// correctness.  It knows nothing of what the order costs besides: several heads at a time (by query tile) share the L2
// where one had it alone, and heads dealt by cost leave their KV group.  So by head must promise 2.5 % more than the
// ranges and by query tile 5 % more than either.  Estimated and measured end against the better of the two ranges (calls
// on inputs in turn; 32 or 64 heads):
//   by head        8192 behind 112K .988 -> 1.008, .960 -> .986; 8192 behind 64K .968 -> .992; 4096 behind 64K .890 -> .967;
//                  4000 behind 64K .805 -> .907; 3000 behind 40K .792 -> .928; 12000 tokens .985 -> 1.004
//   by query tile  4096 tokens .844 -> .925; 2700 .844 -> .937; 5000 .890 -> .962; 8192 .949 -> 1.000 and .961 -> 1.010;
//                  12000 .954 -> 1.024; 16000 .976 -> 1.040; 20000 .965 -> 1.104; 32000 .993 -> 1.096
constexpr int64_t kFixedSteps = 4;
static int64_t plan_xcds(PrefillHeads& ph, const tca_params* prm, const int64_t* offs, int64_t q_pos0,
                         int64_t n_queries, int BM, int part, int slots, int64_t* makespan = nullptr) {
  const int Hq = prm->n_q_heads, GS = sel_group(prm), nh = Hq / 8;
  const int64_t n_qt = (n_queries + BM - 1) / BM, n_items = Hq * n_qt;
  ph.order = 0;
  int32_t by_head[9], by_work[9];
  for (int x = 0; x <= 8; ++x) by_head[x] = (int32_t)(x * nh * n_qt);
  const bool few_rounds = n_items < (int64_t)8 * slots * 16;
  if (few_rounds) {
    // whole heads dealt out, the costliest (by its last query tile) first, each to the XCD with the smallest sum that
    // has room; with a shared selection the heads stay with their group, whose tiles they share
    int64_t last_cost[TCA_MAX_HEADS], sum[8] = {};
    int by_cost[TCA_MAX_HEADS], have[8] = {};
    for (int h = 0; h < Hq; ++h) {
      ph.perm[h] = (uint8_t)h;
      by_cost[h] = h;
      last_cost[h] = h % GS ? last_cost[h - 1] : tile_steps(prm, offs[h / GS + 1] - offs[h / GS], q_pos0, n_queries, BM, n_qt - 1, part);
    }
    if (GS == 1) {
      std::stable_sort(by_cost, by_cost + Hq, [&](int a, int b) { return last_cost[a] > last_cost[b]; });
      for (int i = 0; i < Hq; ++i) {
        int to = -1;
        for (int xc = 0; xc < 8; ++xc)
          if (have[xc] < nh && (to < 0 || sum[xc] < sum[to])) to = xc;
        ph.perm[to * nh + have[to]++] = (uint8_t)by_cost[i];
        sum[to] += last_cost[by_cost[i]];
      }
    }
  }
  if (!makespan && n_items <= (int64_t)8 * slots) {            // all at once: the order only decides who shares a CU
    ph.order = 1;
    for (int x = 0; x <= 8; ++x) ph.xcd_start[x] = by_head[x];
    return nh * n_qt;
  }
  // item g of the sequence: head g / n_qt, its query tiles longest first
  std::vector<int32_t> c((size_t)n_items);
  std::vector<int64_t> head_cost((size_t)Hq, 0);
  int64_t total = 0;
  for (int h = 0; h < Hq; ++h) {
    if (h % GS) {                                  // the heads of a shared selection cost the same
      for (int64_t i = 0; i < n_qt; ++i) c[h * n_qt + i] = c[(h - 1) * n_qt + i];
      head_cost[h] = head_cost[h - 1];
    } else {
      const int64_t cap = offs[h / GS + 1] - offs[h / GS];
      for (int64_t i = 0; i < n_qt; ++i)
        head_cost[h] += c[h * n_qt + i] = (int32_t)(kFixedSteps + tile_steps(prm, cap, q_pos0, n_queries, BM, n_qt - 1 - i, part));
    }
    total += head_cost[h];
  }
  int64_t acc = 0;
  int x = 0;
  by_work[0] = 0;
  for (int64_t g = 0; g < n_items; ++g) {
    acc += c[g];
    while (x < 7 && acc * 8 >= total * (x + 1)) by_work[++x] = (int32_t)(g + 1);
  }
  while (x < 8) by_work[++x] = (int32_t)n_items;
  const int32_t* best = by_work;
  if (few_rounds) {
    auto played = [&](auto walk) {                 // walk(take): take(xcd, cost) in every XCD's order
      auto with = [&](auto slots_tag) {
        Places<decltype(slots_tag)::value> pl[8];
        walk([&](int xc, int32_t cost) { pl[xc].take(cost); });
        int32_t t = 0;
        for (const auto& p : pl) t = std::max(t, p.worst);
        return (int64_t)t;
      };
      return slots == 64 ? with(std::integral_constant<int, 64>{}) : with(std::integral_constant<int, 32>{});      // (xcd_slots)
    };
    auto ranges = [&](const int32_t* st) {
      return played([&](auto take) {
        int32_t at[8], most = 0;                   // an XCD takes the piece of the head its range ends in first
        for (int xc = 0; xc < 8; ++xc) {
          at[xc] = std::max(st[xc], st[xc + 1] / (int32_t)n_qt * (int32_t)n_qt);
          most = std::max(most, st[xc + 1] - st[xc]);
        }
        for (int32_t u = 0; u < most; ++u)
          for (int xc = 0; xc < 8; ++xc)
            if (u < st[xc + 1] - st[xc]) {
              if (at[xc] == st[xc + 1]) at[xc] = st[xc];
              take(xc, c[at[xc]++]);
            }
      });
    };
    auto dealt = [&](int order) {
      return played([&](auto take) {
        auto all = [&](int i, int64_t qt) {
          for (int xc = 0; xc < 8; ++xc) take(xc, c[ph.perm[xc * nh + i] * n_qt + qt]);
        };
        if (order == 1) {
          for (int64_t qt = 0; qt < n_qt; ++qt)
            for (int i = 0; i < nh; ++i) all(i, qt);
        } else {
          for (int i = 0; i < nh; ++i)
            for (int64_t qt = 0; qt < n_qt; ++qt) all(i, qt);
        }
      });
    };
    // (what the sum of its fullest XCD rules out is not played)
    int64_t sum_head = 0, sum_dealt = 0;
    for (int xc = 0; xc < 8; ++xc) {
      int64_t a = 0, b = 0;
      for (int i = xc * nh; i < (xc + 1) * nh; ++i) {
        a += head_cost[i];
        b += head_cost[ph.perm[i]];
      }
      sum_head = std::max(sum_head, a / slots);
      sum_dealt = std::max(sum_dealt, b / slots);
    }
    const int64_t t_work = ranges(by_work), t_head = sum_head > t_work ? sum_head : ranges(by_head);
    const bool too_full = sum_dealt >= std::min(t_head, t_work);
    const int64_t t_one = too_full ? sum_dealt : dealt(1), t_two = too_full ? sum_dealt : dealt(2);
    int64_t t = std::min(t_head, t_work);
    best = t_head <= t_work ? by_head : by_work;
    if (t_two * 40 < t * 39) {
      t = t_two;
      ph.order = 2;
    }
    if (t_one * 20 < t * 19) ph.order = 1;
    if (ph.order) best = by_head;
    if (makespan) *makespan = std::min(std::min(t_head, t_work), std::min(t_one, t_two));
  } else if (makespan) {
    *makespan = total / (8 * slots);
  }
  int64_t longest = 0;
  for (x = 0; x <= 8; ++x) ph.xcd_start[x] = best[x];
  for (x = 0; x < 8; ++x)
    if (best[x + 1] - best[x] > longest) longest = best[x + 1] - best[x];
  return longest;
}

// What a tile step takes, us with the chip full (two four-wave workgroups to a CU), and of that with one workgroup to a CU:
// measured over calls of 257 to 512 workgroups, whole and in chunks (4 to 64 heads behind 0 to 64K tokens).
static double step_us(const tca_params* prm) { return prm->head_dim == 128 ? 1.8 : 1.25; }
static double alone(const tca_params* prm) { return prm->head_dim == 128 ? 0.6 : 0.69; }

// When a call of up to kSplitSlots four-wave workgroups, all resident at once, would end, in full steps: that of the CU whose
// two (by the ids of prefill_mfma_kernel, an XCD's 32 CUs served in turn) take longest, the longer one alone once the other
// has ended.  A call whose long heads meet on a CU runs to the end at the full chip's pace: 6363 queries of 8 heads (d = 64,
// one to an XCD) behind 64K 562 us whole and 474 in chunks, 4000 of 12 heads behind 32768 293 and 250; one whose long heads
// meet short ones does not: 859 of 64 heads (d = 128) 796 and 880.  (A call cut for 5 % is still worth it: in chunks two
// workgroups to a CU hide each other's waits for inputs that are not in the caches.  8192 queries of 4 heads, d = 64, behind
// 32768 236 us whole, 218 in chunks; 249 and 205 on such inputs.)
static double whole_steps(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part) {
  const int Hq = prm->n_q_heads, GS = sel_group(prm), nh = Hq / 8;
  const int n_qt = (int)((n_queries + 127) / 128), n_items = Hq * n_qt;
  double share[kSplitSlots], window[kSplitSlots];  // of a query tile: of a region's rows, in tiles, and its steps without them
  for (int qt = 0; qt < n_qt; ++qt) {
    const int64_t lastq = std::min<int64_t>(q_pos0 + 128 * qt + 127, q_pos0 + n_queries - 1);
    window[qt] = (double)(kFixedSteps + tile_steps(prm, 0, q_pos0, n_queries, 128, qt, part));
    share[qt] = part == TCA_PART_WINDOW || lastq < prm->window ? 0.0 : (double)(lastq - prm->window + 1) / (double)((q_pos0 + n_queries) * kBN);
  }
  double cap[TCA_MAX_HEADS];
  for (int h = 0; h < Hq; ++h) cap[h] = (double)(offs[h / GS + 1] - offs[h / GS]);
  auto cost = [&](int h, int qt) {                 // as tile_steps, which divides for every item
    return window[qt] + (double)(int32_t)(cap[h] * share[qt] + (kBN - 1.0) / kBN);
  };
  double end = 0.0;
  if (n_items <= kSplitSlots / 2) {                // nobody shares a CU: the longest, a head's last query tile
    for (int h = 0; h < Hq; h += GS) end = std::max(end, alone(prm) * cost(h, n_qt - 1));
    return end;
  }
  double c[8][kSplitSlots / 8];                    // of the XCDs' items, in the order in which prefill_mfma_kernel counts them
  if ((Hq & 7) == 0) {
    PrefillHeads ph;
    plan_xcds(ph, prm, offs, q_pos0, n_queries, 128, part, 64);
    for (int x = 0; x < 8; ++x)
      for (int k = 0, v = 0; k < n_qt; ++k)
        for (int i = 0; i < nh; ++i) c[x][v++] = cost(ph.perm[x * nh + i], n_qt - 1 - k);
  } else {
    const int period = 8 / ((Hq & 1) ? 1 : (Hq & 2) ? 2 : 4);
    for (int k = 0, g = 0; k < n_qt; ++k)
      for (int i = 0, h = k / period % Hq; i < Hq; ++i, ++g, h = h + 1 < Hq ? h + 1 : 0) c[g & 7][g >> 3] = cost(h, n_qt - 1 - k);
  }
  for (int x = 0; x < 8; ++x) {
    const int mine = (Hq & 7) == 0 ? nh * n_qt : (n_items - x + 7) >> 3;
    for (int u = 0; u < 32 && u < mine; ++u) {
      const double a = c[x][pair_up(u, mine)], b = u + 32 < mine ? c[x][pair_up(u + 32, mine)] : 0.0;
      end = std::max(end, alone(prm) * std::fabs(a - b) + std::min(a, b));
    }
  }
  return end;
}

// Whether a call's items are cut into chunks, and how long: fills sp (all but part) and returns the number of
// workgroups, or 0 for the plain launch.  plain_steps: when the plain launch would end, in tile steps of the full chip.
// Measured, whole and in chunks: 413 queries behind 64K tokens (32 heads) 539 -> 218 us, behind 112K 949 -> 344 us; 128 behind
// 16K 164 -> 62 us; 2048 behind 30K (4 heads, d = 64) 304 -> 93 us; from 512 items of equal length on nothing is gained.
static int64_t plan_split(SplitPlan& sp, const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries,
                          size_t ws_left, double plain_steps) {
  const int Hq = prm->n_q_heads, GS = sel_group(prm);
  const int64_t n_qt = (n_queries + 127) / 128, n_items = Hq * n_qt;
  const size_t item_bytes = (prm->head_dim == 128 ? split_floats<128>() : split_floats<64>()) * sizeof(float);
  const int64_t fit = (int64_t)(ws_left / item_bytes);
  const int64_t most = fit < 2 * kSplitSlots ? fit : 2 * kSplitSlots;
  if (n_items >= most) return 0;
  int64_t total = 0, longest = 0, bound[TCA_MAX_HEADS];
  for (int h = 0; h < Hq; ++h) {
    if (h % GS) {
      bound[h] = bound[h - 1];
    } else {
      const int64_t cap = offs[h / GS + 1] - offs[h / GS];
      bound[h] = 0;
      for (int64_t qt = 0; qt < n_qt; ++qt) {
        total += GS * tile_steps(prm, cap, q_pos0, n_queries, 128, qt, TCA_PART_ALL);
        // an upper bound, wherever the region's rows lie: the chunks must cover every tile
        const int64_t last = q_pos0 + (qt + 1 < n_qt ? qt * 128 + 127 : n_queries - 1);
        const int64_t seen = last - prm->window + 1 < 0 ? 0 : last - prm->window + 1;
        const int64_t b = tile_steps(prm, 0, q_pos0, n_queries, 128, qt, TCA_PART_ALL) + ((seen < cap ? seen : cap) + kBN - 1) / kBN;
        if (b > bound[h]) bound[h] = b;
      }
    }
    if (bound[h] > longest) longest = bound[h];
  }
  // Chunk lengths: the shortest that keeps one round of the chip, and two.  Their cost in us: the steps; the merge a launch,
  // 0.3 us per chunk of an item, and the partial results written and read at 4 TB/s.
  const double step = step_us(prm);
  double best = 0.95 * plain_steps * step;
  int64_t best_items = 0, best_chunk = 0;
  for (const int64_t room : {(int64_t)kSplitSlots / 2, (int64_t)kSplitSlots, (int64_t)2 * kSplitSlots}) {
    const int64_t lim = room < most ? room : most;
    if (n_items > lim) continue;
    int64_t chunk = (total + lim - 1) / lim, items = 0;
    for (chunk = chunk < kMinChunk ? kMinChunk : chunk;; chunk += (chunk + 15) / 16) {
      chunk = (chunk + 1) & ~(int64_t)1;
      items = 0;
      for (int h = 0; h < Hq; ++h) items += n_qt * ((bound[h] + chunk - 1) / chunk);
      if (items <= lim) break;
    }
    const double walk = items <= kSplitSlots / 2 ? alone(prm) * (chunk + kFixedSteps)
                        : items <= kSplitSlots   ? (double)(chunk + kFixedSteps)
                                                 : 1.1 * (total + kFixedSteps * items) / kSplitSlots + 0.3 * chunk;
    const double t = walk * step + 5.0 + 0.3 * ((longest + chunk - 1) / chunk) + items * (double)item_bytes * 2e-6 / 4.0;
    if (t < best) { best = t; best_items = items; best_chunk = chunk; }
  }
  if (!best_items) return 0;
  int64_t run = 0;
  for (int h = 0; h < Hq; ++h) {
    sp.item_start[h] = (int32_t)run;
    run += n_qt * ((bound[h] + best_chunk - 1) / best_chunk);
  }
  sp.item_start[Hq] = (int32_t)run;
  sp.chunk = (int32_t)best_chunk;
  // Few query tiles: an eighth of the sequence per XCD (64 heads, 413 queries behind 64K tokens: 423 us, against 468
  // with runs of one chunk's query tiles).  Many: their chunks end at different places, and runs of 8 spread
  // the short ones (4 heads, 17000 tokens: an eighth each left XCDs with a quarter of the others' work).
  sp.run = n_qt <= 16 ? (int32_t)((run + 7) / 8) : 8;
  return run;
}

// The workgroup shape of a call: waves, and blocks of 32 queries per wave.  The size of the call chooses
// between eight and four waves of 32 queries; the diagnostics switch can force a shape.
struct WgShape { int nw, qb; };
// workgroups of it an XCD runs at a time: 32 CUs, one eight-wave workgroup, one of four waves with a SIMD each, or two of four waves
static int xcd_slots(WgShape sh) { return sh.nw == 8 || sh.qb == 2 ? 32 : 64; }
// v_aligned: V and Vg are 16-byte aligned.  Where they are not (the entry points take any element for a start) the direct
// copies into LDS cannot be relied on, which the four-wave shapes make of V itself: such a call takes eight waves, whose
// pre-pass reads V with plain loads.
static WgShape choose_shape(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, bool gather, bool v_aligned) {
  if (!v_aligned) return {8, 1};
  const int variant = prefill_variant();
  // With rows fetched through idx eight waves from 1024 items of 256 queries on.  Otherwise they must also pay for the pre-pass
  // (uses_transposed_v), for their coarser last round of workgroups and for prologues that nothing covers: by many query
  // tiles, or by a long walk of each.  us with four / with eight, the attention alone, 64 heads, region rows 0.2 to 0.5 of the
  // tokens: 4096 tokens 291 / 300, 5446 476 / 503, 6144 (24 tiles) 593 / 589, 6656 672 / 658, 7900 917 / 871; 4096 behind 8192
  // (about 110 steps an item) 792 / 820, behind 16384 (150) 1119 / 1131, behind 30000 (220) 1680 / 1657, behind 64K (430)
  // 3050 / 2998; 5446 behind 6000 1000 / 1061; 5888 behind 30000 2477 / 2412, behind 64K 4490 / 4380.  With a shared selection
  // 5446 tokens 471 / 487, 6656 661 / 651, 4096 behind 8192 796 / 809, behind 16384 1150 / 1150 and 1170 / 1127, behind 64K
  // 3156 / 3118.  On inputs that are not in the caches the same within 1 %.
  const int64_t tiles = (n_queries + 255) / 256;
  bool many = tiles * prm->n_q_heads >= 1024;
  if (many && !gather && tiles < 24) {
    const int Hs = sel_heads(prm);
    int64_t steps = 0, most = 0;                   // of all query tiles; of a head's last, and what another may have more of the window
    for (int h = 0; h < Hs; ++h) most += 6 + tile_steps(prm, offs[h + 1] - offs[h], q_pos0, n_queries, 256, tiles - 1, TCA_PART_ALL);
    if (most >= 130 * Hs)
      for (int h = 0; h < Hs; ++h)
        for (int64_t qt = 0; qt < tiles; ++qt)
          steps += tile_steps(prm, offs[h + 1] - offs[h], q_pos0, n_queries, 256, qt, TCA_PART_ALL);
    many = steps >= 130 * tiles * Hs;
  }
  if (gather) return {variant == 3 || (variant != 1 && many) ? 8 : 4, 1};
  if (variant == 3 || (variant == 0 && many)) return {8, 1};
  if (variant == 2) return {4, 2};
  return {4, 1};
}

// The chunks of a call (plan_split), or 0.  Not for a part: the two parts may run side by side on one workspace, which has
// room for one call's chunks.
static int64_t choose_split(SplitPlan& sp, const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part,
                            WgShape sh, size_t ws_left) {
  const int Hq = prm->n_q_heads, GS = sel_group(prm);
  const int64_t n_qt = (n_queries + 127) / 128;
  if (sh.nw != 4 || sh.qb != 1 || part != TCA_PART_ALL || prefill_variant() != 0 || n_qt * Hq >= 2 * kSplitSlots) return 0;
  // when the plain launch would end
  double plain = 0.0;
  if (n_qt * Hq <= kSplitSlots) {
    plain = whole_steps(prm, offs, q_pos0, n_queries, part);
  } else if ((Hq & 7) == 0) {
    PrefillHeads ph;
    int64_t makespan = 0;
    plan_xcds(ph, prm, offs, q_pos0, n_queries, 128, part, 64, &makespan);
    plain = (double)makespan;
  } else {                                         // no plan for such head counts: what the longest takes alone, at least
    for (int h = 0; h < Hq; h += GS)
      plain = std::max(plain, 0.6 * (kFixedSteps + tile_steps(prm, offs[h / GS + 1] - offs[h / GS], q_pos0, n_queries, 128, n_qt - 1, part)));
  }
  return plan_split(sp, prm, offs, q_pos0, n_queries, ws_left, plain);
}

template <int D>
static void run_mfma(const tca_params* prm, const uint16_t* Q, int64_t q_pos0, int64_t n_queries,
                     const uint16_t* K, const uint16_t* V, int64_t kv_stride, const int32_t* idx,
                     const uint16_t* Kg, const uint16_t* Vg, const int64_t* offs, const int32_t* n_rows,
                     uint16_t* O, float* lse, void* ws, size_t ws_bytes, hipStream_t st, int part) {
  const int Hq = prm->n_q_heads, Hkv = prm->n_kv_heads, Hs = sel_heads(prm), w = prm->window;
  PrefillHeads ph;
  int32_t run = 0;
  for (int h = 0; h <= Hs; ++h) {
    ph.offs[h] = offs[h];
    ph.tile_off[h] = run;
    if (h < Hs) run += (int32_t)((offs[h + 1] - offs[h] + kBN - 1) / kBN);
  }
  MfmaWs mw = mfma_ws(ws, prm, n_queries, offs[Hs]);
  // cycle counters only when asked for (and not for a part: two parts may run side by side on one workspace)
  unsigned long long* clk = diag_prefill_clocks() && part == TCA_PART_ALL ? mw.clk : nullptr;
  if (clk) hipLaunchKernelGGL(clear_clocks_kernel, dim3(1), dim3(4), 0, st, clk);
  const bool gather = Kg == nullptr;               // no compacted copy of the kept rows

  // Shape of a workgroup.  Long calls: eight waves of 32 queries (256 queries, one workgroup per CU,
  // two waves per SIMD).  Calls with few query tiles: four waves of 32 queries
  // (128 queries, two workgroups per CU), which keeps more of the chip busy.  Four waves of 64
  // queries (one wave per SIMD, every LDS fragment feeds two MFMAs, half the LDS reads) stay
  // selectable through the diagnostics switch: measured 5-8 % slower on 128K tokens, because a
  // lone wave cannot issue its vector, LDS and scalar instructions fast enough beside the MFMAs.
  const WgShape sh = choose_shape(prm, offs, q_pos0, n_queries, gather, (((uintptr_t)V | (uintptr_t)Vg) & 15) == 0);
  SplitPlan sp;
  {
    const int64_t n_wg = choose_split(sp, prm, offs, q_pos0, n_queries, part, sh, ws_bytes > mw.need ? ws_bytes - mw.need : 0);
    if (n_wg) {
      sp.part = mw.part;
      auto launch_split = [&](auto gather_tag) {
        hipLaunchKernelGGL((prefill_mfma_kernel<D, 4, 1, decltype(gather_tag)::value, true>), dim3(8u * sp.run * (unsigned)((n_wg + 8 * sp.run - 1) / (8 * sp.run))),
                           dim3(256), 0, st, Q, q_pos0, n_queries, K, V, kv_stride, idx, Kg, Vg, n_rows,
                           0, 0, ph, Hq, Hq / Hkv, sel_group(prm), w, (float)logit_scale(prm), O, lse, clk, part, sp);
      };
      if (gather) launch_split(std::true_type{});
      else launch_split(std::false_type{});
      launch_merge_split(prm, sp, n_queries, O, lse, st);
      return;
    }
  }
  auto launch = [&](auto nw_tag, auto qb_tag, auto gather_tag) {
    constexpr int NW = decltype(nw_tag)::value, QB = decltype(qb_tag)::value;
    constexpr bool GATHER = decltype(gather_tag)::value;
    const int n_qt = (int)((n_queries + NW * QB * 32 - 1) / (NW * QB * 32));
    const unsigned n_wg = (Hq & 7) == 0 ? 8u * (unsigned)plan_xcds(ph, prm, offs, q_pos0, n_queries, NW * QB * 32, part, xcd_slots(sh))
                                        : (unsigned)n_qt * Hq;
    const uint16_t *v = V, *vg = Vg;
    const int64_t dt0 = (q_pos0 - w + 1 > 0 ? q_pos0 - w + 1 : 0) / kBN;         // the dense tiles any query's window meets
    const int d_tiles = (int)((q_pos0 + n_queries - 1) / kBN - dt0 + 1);
    if constexpr (uses_transposed_v(NW)) {
      const int region_tiles = part == TCA_PART_WINDOW ? 0 : run;
      const int tiles = region_tiles + (part == TCA_PART_GLOBAL ? 0 : d_tiles * Hkv);
      if (tiles > 0)
        hipLaunchKernelGGL((transpose_tiles_kernel<D>), dim3((unsigned)((tiles + 256 / D - 1) / (256 / D))), dim3(256), 0, st, Vg, V,
                           kv_stride, n_rows, GATHER ? idx : (const int32_t*)nullptr, Hs / Hkv, Hs, region_tiles, tiles, d_tiles,
                           dt0 * kBN, q_pos0 + n_queries, mw.Vgt, mw.Vt, ph);
      v = mw.Vt;
      vg = mw.Vgt;
    }
    hipLaunchKernelGGL((prefill_mfma_kernel<D, NW, QB, GATHER>), dim3(n_wg), dim3(NW * 64), 0, st, Q,
                       q_pos0, n_queries, K, v, kv_stride, idx, Kg, vg, n_rows, dt0, d_tiles, ph, Hq, Hq / Hkv,
                       sel_group(prm), w, (float)logit_scale(prm), O, lse, clk, part, NoSplit{});
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  if (gather) {
    if (sh.nw == 8) launch(I8{}, I1{}, std::true_type{});
    else launch(I4{}, I1{}, std::true_type{});
  } else if (sh.nw == 8) launch(I8{}, I1{}, std::false_type{});
  else if (sh.qb == 2) launch(I4{}, I2{}, std::false_type{});
  else launch(I4{}, I1{}, std::false_type{});
}

int64_t prefill_mfma_xcd_plan(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part,
                              bool gather, int32_t* start_out) {
  if ((prm->n_q_heads & 7) != 0) return -1;
  const WgShape sh = choose_shape(prm, offs, q_pos0, n_queries, gather, true);
  PrefillHeads ph;
  const int64_t longest = plan_xcds(ph, prm, offs, q_pos0, n_queries, sh.nw * sh.qb * 32, part, xcd_slots(sh));
  for (int x = 0; x <= 8; ++x) start_out[x] = ph.xcd_start[x];
  return 8 * longest;
}

int prefill_mfma_walk(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part, bool gather,
                      size_t ws_bytes, int32_t* heads_out, int64_t* chunks_out) {
  const WgShape sh = choose_shape(prm, offs, q_pos0, n_queries, gather, true);
  const size_t need = prefill_mfma_workspace_need(prm, n_queries, offs[sel_heads(prm)]);
  SplitPlan sp;
  const int64_t chunks = choose_split(sp, prm, offs, q_pos0, n_queries, part, sh, ws_bytes > need ? ws_bytes - need : 0);
  if (chunks_out) *chunks_out = chunks;
  if ((prm->n_q_heads & 7) != 0) return -1;
  PrefillHeads ph;
  plan_xcds(ph, prm, offs, q_pos0, n_queries, sh.nw * sh.qb * 32, part, xcd_slots(sh));
  for (int h = 0; heads_out && h < prm->n_q_heads; ++h) heads_out[h] = ph.order ? ph.perm[h] : h;
  return ph.order;
}

int launch_prefill_mfma(const tca_params* prm, const bf16_t* Q, int64_t q_pos0, int64_t n_queries,
                        const bf16_t* K, const bf16_t* V, int64_t kv_stride, const int32_t* idx,
                        const bf16_t* Kg, const bf16_t* Vg, const int64_t* offs, const int32_t* n_rows,
                        bf16_t* O, float* lse, void* ws, size_t ws_bytes, hipStream_t st, int part) {
  // the kernel addresses tiles with 32-bit byte offsets inside each buffer
  const int64_t row_bytes = (int64_t)prm->head_dim * 2;
  int64_t max_rows = q_pos0 + n_queries + prm->window + 2 * kBN;
  for (int h = 0; h < sel_heads(prm); ++h)
    if (offs[h + 1] - offs[h] + kBN > max_rows) max_rows = offs[h + 1] - offs[h] + kBN;
  if (max_rows * row_bytes > (int64_t)INT32_MAX)
    return fail(TCA_ERR_UNSUPPORTED, "tca_prefill (bf16): %lld rows of %lld bytes exceed 2 GiB per head buffer",
                (long long)max_rows, (long long)row_bytes);
  auto u = [](const bf16_t* p) { return reinterpret_cast<const uint16_t*>(p); };
  if (prm->head_dim == 128)
    run_mfma<128>(prm, u(Q), q_pos0, n_queries, u(K), u(V), kv_stride, idx, u(Kg), u(Vg), offs, n_rows,
                  reinterpret_cast<uint16_t*>(O), lse, ws, ws_bytes, st, part);
  else
    run_mfma<64>(prm, u(Q), q_pos0, n_queries, u(K), u(V), kv_stride, idx, u(Kg), u(Vg), offs, n_rows,
                 reinterpret_cast<uint16_t*>(O), lse, ws, ws_bytes, st, part);
  return TCA_OK;
}

}  // namespace tca
