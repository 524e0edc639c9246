// Layer integration in front of the path (an extension; the paper's method starts from Q, K, V):
// the projections Q = X W_Q, K = X W_K, V = X W_V of Sec. III for all heads in one launch, written
// straight into the layouts tca_select / tca_prefill (head-major) or tca_decode (token-major) read.
//
// bf16: a dense contraction, so it runs on the matrix cores.  qkv_mfma_kernel forms tiles of Y^T = W X^T
// with v_mfma_f32_32x32x16_bf16, 256 features x 256 tokens per workgroup for long calls (8 waves, two per SIMD,
// a wave owning 128 features x 64 tokens = 4 x 2 accumulator blocks, so that a k-step of 16 takes six
// fragment reads for eight MFMAs) down to 64 x 64 for short ones.  The hidden dimension is walked in stages of
// 64; the W and X slices of a stage go global -> LDS with the LDS modifier of the buffer loads (no staging
// registers), XOR-swizzled so that the 16-byte fragment reads are free of bank conflicts, two to six stages
// resident.  The one barrier of a stage sits in front of the stage's last k-step, whose fragments are in
// registers by then: after it no wave reads the stage any more, so the copies of a later stage start there, and
// the first fragments of the next stage are read under the last MFMAs.  Features are the rows of the MFMA
// result, so a lane ends up with four consecutive features of one token: one 8-byte store each.
// qkv_skinny_kernel takes the calls of a few rows, which are one pass over the weights.
//
// fp32 (qkv_f32_kernel): fp32 multiply-adds in the order of the hidden index (small cases and an independent check of
// the bf16 kernels' indexing).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tca_common.h"
#include "tca_device.h"

namespace tca {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;

constexpr int kPK = 64;                          // the hidden size must be a multiple of this

// Where the projected rows go.  Part 0 = Q, 1 = K, 2 = V; feature f belongs to head f / d of the
// concatenation (Hq query heads, Hkv key heads, Hkv value heads).  Element e of head h (counted
// inside its part) of token t lands at base[part] + h * head_stride[part] + t * token_stride[part] + e.
struct QkvOut {
  void* base[3];
  int64_t head_stride[3], token_stride[3];
  int first_head[4];                             // part p holds the heads [first_head[p], first_head[p+1])
};

// 16 bytes per lane, global -> LDS (lanes deposit at consecutive addresses from lds_dst on); lane_off: the
// lane's byte offset into the buffer, tile_off: a scalar byte offset on top
__device__ __forceinline__ void copy16_to_lds(__amdgpu_buffer_rsrc_t rsrc, int lane_off, int tile_off,
                                              unsigned char* lds_dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds_dst, 16, lane_off,
                                           tile_off, 0, 0);
}

__device__ __forceinline__ int part_of_head(const QkvOut& o, int hg) { return hg < o.first_head[1] ? 0 : hg < o.first_head[2] ? 1 : 2; }

// Stores the blocks of 32 features (from fblk on) x TB * 32 tokens (from t0 on) of a wave: the lane holds token
// column lrow of block tb; register 4 q4 + j is feature 8 q4 + 4 hh + j.
template <int TB>
__device__ __forceinline__ void store_block(const QkvOut& out, const uint16_t* __restrict__ bias, int64_t fblk, int n_feat,
                                            int d, int64_t t0, int64_t n_tok, int lrow, int hh, const f32x16_t (&acc)[TB]) {
  if (fblk >= n_feat) return;                                // n_feat is a multiple of d >= 64: whole blocks
  const int hg = (int)(fblk / d), e0 = (int)(fblk - (int64_t)hg * d);
  const int p = part_of_head(out, hg);
  uint16_t* const hbase = (uint16_t*)out.base[p] + (int64_t)(hg - out.first_head[p]) * out.head_stride[p] + e0;
  float bs[4][4];
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
    for (int j = 0; j < 4; ++j) bs[q4][j] = bias ? bf16_to_f32(bias[fblk + 8 * q4 + 4 * hh + j]) : 0.f;
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int64_t t = t0 + tb * 32 + lrow;
    if (t >= n_tok) continue;
    uint16_t* const row = hbase + t * out.token_stride[p];
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      bf16x4_t pk;
#pragma unroll
      for (int j = 0; j < 4; ++j) pk[j] = (__bf16)(acc[tb][4 * q4 + j] + bs[q4][j]);
      *reinterpret_cast<bf16x4_t*>(row + 8 * q4 + 4 * hh) = pk;
    }
  }
}

// A workgroup of NWF x NWT waves forms a tile of NWF * FBW * 32 features x NWT * TBW * 32 tokens, a wave FBW x TBW
// accumulator blocks of it; stages of 64 hidden elements, NST of them resident in LDS.
// Which shape takes which call: see tca_qkv_project.
template <int FBW, int TBW, int NWF, int NWT, int NST>
__global__ __launch_bounds__(NWF * NWT * 64) __attribute__((amdgpu_waves_per_eu(NWF * NWT / 4, NWF * NWT / 4)))
void qkv_mfma_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ X, const uint16_t* __restrict__ bias,
                     int n_feat, int64_t n_tok, int hidden, int d, QkvOut out, int n_ft, int n_tt) {
  constexpr int NW = NWF * NWT;
  constexpr int PF = NWF * FBW * 32, PT = NWT * TBW * 32;
  constexpr int BK = kPK, ROWB = BK * 2;         // a stage is one 128-byte line of every row
  constexpr int CPR = ROWB / 16;                 // 16-byte chunks per tile row
  constexpr int WB = PF * ROWB, XB = PT * ROWB, STAGEB = WB + XB;
  constexpr int NLW = WB / 1024 / NW, NLX = XB / 1024 / NW, NL = NLW + NLX;      // wave-loads per wave and stage
  static_assert(NST * STAGEB <= 160 * 1024 && NLW >= 1 && NLX >= 1, "shape");
  __shared__ __attribute__((aligned(16))) unsigned char lds[NST * STAGEB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroup ids go round-robin over the 8 XCDs.  The tiles are walked in groups of four token tiles, feature
  // tiles inside a group, and XCD x takes the x-th eighth of that sequence without holes: the 32 workgroups it
  // runs at a time are 8 feature tiles x 4 token tiles, which go through the hidden dimension side by side, so
  // that their L2 sees a W slice four times and an X slice eight times.  (Ids that return at once must not be
  // spread among the others: an XCD deals its ids to its CUs in order.)
  const int n_items = n_ft * n_tt, per_xcd = (n_items + 7) >> 3;
  const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (item >= n_items) return;
  const int grp = item / (4 * n_ft), in = item - grp * (4 * n_ft);
  const int gw = n_tt - grp * 4 < 4 ? n_tt - grp * 4 : 4;          // token tiles of this group
  const int ft = in / gw, ts = grp * 4 + (in - ft * gw);
  // Place ts of the token tiles' order: every eighth tile from 0 on, then from 1 on, ..: the XCDs then walk neighbouring
  // tiles side by side (335 us at 8192 rows, hidden 4096, 6144 features; 340 with an eighth of the rows to each)
  const int tq = n_tt >> 3, tr = n_tt & 7, cut = tr * (tq + 1);
  const int tt = ts < cut ? ts / (tq + 1) + 8 * (ts % (tq + 1)) : tr + (ts - cut) / tq + 8 * ((ts - cut) % tq);
  const int wf = wv % NWF, wt = wv / NWF;        // the wave's place inside the tile
  const int64_t f0 = (int64_t)ft * PF, t0 = (int64_t)tt * PT;
  const int rows_w = n_feat - f0 < PF ? (int)(n_feat - f0) : PF;
  const int rows_x = n_tok - t0 < PT ? (int)(n_tok - t0) : PT;

  // ---- copies.  Chunk c of tile row r sits at chunk position c ^ swz(r), where swz makes the 16 rows a
  // quarter-wave reads at one chunk column fall into distinct banks.  Rows past the end of W or X read
  // as zero (range check of the descriptor).
  auto swz_of = [](int r) { return (r >> 1) & 7; };
  constexpr int kRsrcFlags = 0x00020000;         // raw buffer, 32-bit data format
  const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void*)(W + f0 * hidden), 0, rows_w * hidden * 2, kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void*)(X + t0 * hidden), 0, rows_x * hidden * 2, kRsrcFlags);
  int low[NLW], lox[NLX];                        // this lane's byte offsets into the operands, per wave-load
  auto lane_offset = [&](int q) {                // 16-byte chunk of the LDS tile this lane fills in wave-load q
    const int cid = q * 64 + lane, r = cid / CPR, pch = cid % CPR;
    return r * hidden * 2 + ((pch ^ swz_of(r)) << 4);
  };
#pragma unroll
  for (int j = 0; j < NLW; ++j) low[j] = lane_offset(wv * NLW + j);
#pragma unroll
  for (int j = 0; j < NLX; ++j) lox[j] = lane_offset(wv * NLX + j);
  // copy i of this wave's share of stage kt into place sp, the operands taking turns
  constexpr int kBoth = NLW < NLX ? NLW : NLX;
  auto issue_one = [&](int kt, int sp, int i) {
    unsigned char* const dst = lds + sp * STAGEB;
    const bool is_w = i < 2 * kBoth ? (i & 1) == 0 : NLW > NLX;
    const int j = i < 2 * kBoth ? i >> 1 : i - kBoth;
    if (is_w) copy16_to_lds(rs_w, low[j < NLW ? j : 0], kt * ROWB, dst + (wv * NLW + j) * 1024);
    else copy16_to_lds(rs_x, lox[j < NLX ? j : 0], kt * ROWB, dst + WB + (wv * NLX + j) * 1024);
  };

  // ---- fragments: lane = (row lane & 31, k half lane >> 5) of a 32-row block
  constexpr int KS = BK / 16;                    // k-steps per stage
  const int lrow = lane & 31, hh = lane >> 5;
  int fo[KS];                                    // byte offset inside a block of 32 rows, per k-step of a stage
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) fo[kk] = lrow * ROWB + (((kk * 2 + hh) ^ swz_of(lrow)) << 4);
  const unsigned char* const wbase = lds + wf * (FBW * 32 * ROWB);
  const unsigned char* const xbase = lds + WB + wt * (TBW * 32 * ROWB);
  f32x16_t acc[FBW][TBW];
#pragma unroll
  for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[fb][tb][i] = 0.f;

  // Stage kt lives in place kt % NST.  The loop is cut at the barriers: a stretch starts behind the
  // barrier of stage kt - 1 with that stage's last k-step (its fragments are in registers), under
  // which the copies of stage kt + NST - 1 start, into the place stage kt - 1 has just left, and the
  // first fragments of stage kt arrive; then come the other k-steps of stage kt and its barrier.  There
  // is one copy of the stretch in the code (the place is a run-time offset; the first stretch
  // multiplies zeros for the stage that is not there, the last ones copy the last stage again instead
  // of stages that are not there), because every further copy of it costs registers the accumulators
  // need.  The order of a stretch's instructions is written out and fenced (sched_barrier): one MFMA,
  // behind it a fragment read of the next k-step in the order of need and, behind each of the stretch's first
  // ones, a copy.  Left to itself the compiler issues the copies in one burst and the
  // fragment reads in clumps (5 % slower, as is an order merely suggested through sched_group_barrier).
  // The barrier is the bare instruction behind a wait of our own: a __syncthreads() would wait for every
  // copy in flight, whatever NST is.
  static_assert(KS == 4 && NST >= 2, "the stretch below is four k-steps");
  const int nk = hidden / BK;
  constexpr int kAhead = (NST - 2) * NL;         // loads that may still be in flight when the next stage must be in
  static_assert(kAhead < 64, "vmcnt is six bits wide");
  // vmcnt(kAhead) (bits [3:0] and [15:14]); lgkmcnt(0): this wave's reads of the stage it leaves have returned
  constexpr int kWaitNext = 0x0070 | (kAhead & 15) | ((kAhead >> 4) << 14);
  bf16x8_t a0[FBW], b0[TBW], a1[FBW], b1[TBW];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
#pragma unroll
    for (int fb = 0; fb < FBW; ++fb) a1[fb][i] = (__bf16)0.f;
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb) b1[tb][i] = (__bf16)0.f;
  }
#pragma unroll
  for (int j = 0; j + 1 < NST; ++j)
#pragma unroll
    for (int i = 0; i < NL; ++i) issue_one(j < nk ? j : nk - 1, j, i);
  __builtin_amdgcn_s_waitcnt(kWaitNext);         // stage 0 is in
  __builtin_amdgcn_s_barrier();
  int s = 0;                                     // place of stage kt
  // fragment i of k-step kk of the stage in place sp, in the order the MFMAs need them: W block 0, the X
  // blocks, the other W blocks
  auto read_one = [&](int sp, int kk, int i, bf16x8_t (&a)[FBW], bf16x8_t (&b)[TBW]) {
    if (i == 0) a[0] = *reinterpret_cast<const bf16x8_t*>(wbase + sp * STAGEB + fo[kk]);
    else if (i <= TBW) b[i - 1] = *reinterpret_cast<const bf16x8_t*>(xbase + sp * STAGEB + (i - 1) * (32 * ROWB) + fo[kk]);
    else a[i - TBW] = *reinterpret_cast<const bf16x8_t*>(wbase + sp * STAGEB + (i - TBW) * (32 * ROWB) + fo[kk]);
  };
  // k-step number n of a stretch: the MFMAs of the current fragments (ca, cb); the reads of the fragments
  // (na, nb) of k-step kk of place sp; this k-step's share of the copies of stage ckt into place cs
  constexpr int NM = FBW * TBW, NR = FBW + TBW;
  auto kstep = [&](const bf16x8_t (&ca)[FBW], const bf16x8_t (&cb)[TBW], bf16x8_t (&na)[FBW], bf16x8_t (&nb)[TBW], int sp, int kk,
                   auto n_tag, int ckt, int cs) {
    constexpr int N = decltype(n_tag)::value;
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      const int fb = j / TBW, tb = j % TBW;
      acc[fb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ca[fb], cb[tb], acc[fb][tb], 0, 0, 0);
#pragma unroll
      for (int i = j; i < (j + 1 < NM ? j + 1 : NR); ++i)
        if (i < NR) read_one(sp, kk, i, na, nb);
      if (N * NM + j < NL) issue_one(ckt, cs, N * NM + j);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_assert(NL <= 4 * NM, "the copies of a stage fit its stretch");
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  for (int kt = 0; kt < nk; ++kt) {
    const int s_prev = s == 0 ? NST - 1 : s - 1;
    const int ckt = kt + NST - 1 < nk ? kt + NST - 1 : nk - 1;
    __builtin_amdgcn_sched_barrier(0);
    kstep(a1, b1, a0, b0, s, 0, I0{}, ckt, s_prev);          // the last k-step of stage kt - 1
    kstep(a0, b0, a1, b1, s, 1, I1{}, ckt, s_prev);
    kstep(a1, b1, a0, b0, s, 2, I2{}, ckt, s_prev);
    kstep(a0, b0, a1, b1, s, 3, I3{}, ckt, s_prev);
    __builtin_amdgcn_s_waitcnt(kWaitNext);       // this wave's share of stage kt + 1 has landed
    __builtin_amdgcn_s_barrier();                // everyone's has, and nobody reads stage kt any more
    s = s + 1 == NST ? 0 : s + 1;
  }
#pragma unroll
  for (int fb = 0; fb < FBW; ++fb)               // the last k-step of the last stage
#pragma unroll
    for (int tb = 0; tb < TBW; ++tb) acc[fb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[fb], b1[tb], acc[fb][tb], 0, 0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);            // no copy into this workgroup's LDS may outlive it
#pragma unroll
  for (int fb = 0; fb < FBW; ++fb)
    store_block<TBW>(out, bias, f0 + wf * (FBW * 32) + fb * 32, n_feat, d, t0 + wt * (TBW * 32), n_tok, lrow, hh, acc[fb]);
}

// ---- calls of few rows (a decoding batch): bound by one pass over the weights
//
// One workgroup of sixteen waves forms nf features (FB blocks of 16, the last of them not always full) x TB * 16
// tokens with v_mfma_f32_16x16x32_bf16.  The waves split the hidden dimension in units of 64 elements (one 128-byte
// line of a weight row each), interleaved, and load their fragments straight from global memory: nothing is reused
// inside a workgroup that would pay for a stage in LDS, and a wave has U units of loads in flight at once, which is
// what keeps HBM busy.  A lane's chunks of a unit are kb and kb + 4 (kb = lane / 16): the order of the hidden index
// inside a unit does not matter as long as W and X agree.  The waves' fp32 sums are added through LDS in
// wave order.
// Every workgroup reads the whole of X, and one CU takes in weights only so fast: the features are dealt out so that
// every CU has one workgroup (nf: see launch_skinny).  Sixteen waves with U units instead of eight with four or two
// make no difference up to 32 features a workgroup and 5 % at 40; eight units in flight, non-temporal loads of W
// (14.1 against 12.2 us at 16 rows) or another first unit per workgroup gain nothing.
template <int FB, int TB, int U>
__global__ __launch_bounds__(1024) void qkv_skinny_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ X,
                                                          const uint16_t* __restrict__ bias, int n_feat, int nf, int64_t n_tok,
                                                          int hidden, int d, QkvOut out) {
  typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
  constexpr int NW = 16;
  __shared__ __attribute__((aligned(16))) f32x4_t red[NW][FB * TB][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kb = lane >> 4;
  const int f0 = blockIdx.x * nf, mine = min(nf, n_feat - f0);       // multiples of 4
  const int64_t t0 = (int64_t)blockIdx.y * (TB * 16);
  const uint16_t* wp[FB];
  const uint16_t* xp[TB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) wp[fb] = W + (size_t)(f0 + min(fb * 16 + r, mine - 1)) * hidden + kb * 8;     // (as the tokens' below)
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int64_t t = t0 + tb * 16 + r;
    xp[tb] = X + (size_t)(t < n_tok ? t : n_tok - 1) * hidden + kb * 8;      // rows past the end repeat the last, never stored
  }
  f32x4_t acc[FB][TB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) acc[fb][tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nu = hidden >> 6;
  auto units = [&](int u0, auto n_tag) {           // units u0, u0 + NW, .. (N of them), all inside the hidden dimension
    constexpr int N = decltype(n_tag)::value;
    bf16x8_t w[N][2][FB], x[N][2][TB];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = (u0 + i * NW) * 64 + s * 32;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) w[i][s][fb] = *reinterpret_cast<const bf16x8_t*>(wp[fb] + k);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) x[i][s][tb] = *reinterpret_cast<const bf16x8_t*>(xp[tb] + k);
      }
    __builtin_amdgcn_sched_barrier(0);             // all of them requested before the first is used
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb)
            acc[fb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i][s][fb], x[i][s][tb], acc[fb][tb], 0, 0, 0);
  };
  int u = wv;
  for (; u + (U - 1) * NW < nu; u += U * NW) units(u, std::integral_constant<int, U>{});
  for (; u < nu; u += NW) units(u, std::integral_constant<int, 1>{});
#pragma unroll
  for (int fb = 0; fb < FB; ++fb)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) red[wv][fb * TB + tb][lane] = acc[fb][tb];
  __syncthreads();
  // lane (token r, kb) of a block holds the features 4 kb .. 4 kb + 3 of one token
  for (int g = tid; g < FB * TB * 64; g += NW * 64) {
    const int blk = g >> 6, ln = g & 63;
    f32x4_t s = red[0][blk][ln];
#pragma unroll
    for (int x = 1; x < NW; ++x) s += red[x][blk][ln];
    const int f = f0 + (blk / TB) * 16 + 4 * (ln >> 4);
    const int64_t t = t0 + (blk % TB) * 16 + (ln & 15);
    if (t >= n_tok || f - f0 >= mine) continue;
    const int hg = f / d, e0 = f - hg * d, p = part_of_head(out, hg);
    uint16_t* const row = (uint16_t*)out.base[p] + (int64_t)(hg - out.first_head[p]) * out.head_stride[p] + t * out.token_stride[p] + e0;
    bf16x4_t pk;
#pragma unroll
    for (int j = 0; j < 4; ++j) pk[j] = (__bf16)(s[j] + (bias ? bf16_to_f32(bias[f + j]) : 0.f));
    *reinterpret_cast<bf16x4_t*>(row) = pk;
  }
}

// fp32: a workgroup takes FT features x TT tokens, a thread RF x RT of them, each summed over the hidden index in
// order: fused multiply-adds onto one accumulator, the same bits whatever the tile.  The vector ALU and, for a few
// rows, the reads of the weights bound it: KC columns of both operands sit in LDS (rows padded by 16 bytes, so that
// the 16-byte reads of neighbouring features fall on different banks), the next KC are on their way into registers
// meanwhile.  Lanes run over the features, so that the tokens' reads are broadcasts and the stores are contiguous.
// ALIGNED: hidden % 4 == 0 and 16-byte operands.
// grid (ceil(n_feat / FT), ceil(n_tok / TT)); block 256.
template <int FT, int TT, int RF, int RT, int KC, bool ALIGNED>
__global__ __launch_bounds__(256) void qkv_f32_kernel(const float* __restrict__ W, const float* __restrict__ X,
                                                      const float* __restrict__ bias, int n_feat, int64_t n_tok, int hidden,
                                                      int d, QkvOut out) {
  constexpr int LF = FT / RF, LS = KC + 4, C4 = KC / 4, NL = (FT + TT) * C4 / 256;
  static_assert(LF * (TT / RT) == 256 && (FT + TT) * C4 % 256 == 0, "256 threads");
  __shared__ __align__(16) float lds[(FT + TT) * LS];           // FT rows of W, then TT rows of X
  const int tid = threadIdx.x, lf = tid % LF, lt = tid / LF;
  const int f0 = blockIdx.x * FT;
  const int64_t t0 = (int64_t)blockIdx.y * TT;

  const float* row[NL];                                         // rows past the end repeat the last one
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int r = (tid + i * 256) / C4;
    row[i] = r < FT ? W + (size_t)min(f0 + r, n_feat - 1) * hidden : X + (size_t)min(t0 + (r - FT), n_tok - 1) * hidden;
  }
  float4 next[NL];
  auto fetch = [&](int c0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int c = c0 + ((tid + i * 256) % C4) * 4;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if constexpr (ALIGNED) {
        if (c < hidden) v = *reinterpret_cast<const float4*>(row[i] + c);
      } else {
        if (c < hidden) v.x = row[i][c];
        if (c + 1 < hidden) v.y = row[i][c + 1];
        if (c + 2 < hidden) v.z = row[i][c + 2];
        if (c + 3 < hidden) v.w = row[i][c + 3];
      }
      next[i] = v;
    }
  };

  float acc[RF][RT];
#pragma unroll
  for (int a = 0; a < RF; ++a)
#pragma unroll
    for (int b = 0; b < RT; ++b) acc[a][b] = 0.f;

  fetch(0);
  for (int c0 = 0; c0 < hidden; c0 += KC) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NL; ++i)
      *reinterpret_cast<float4*>(lds + ((tid + i * 256) / C4) * LS + ((tid + i * 256) % C4) * 4) = next[i];
    __syncthreads();
    if (c0 + KC < hidden) fetch(c0 + KC);
    const int n = min(KC, hidden - c0);
    auto step4 = [&](int c) {
      float4 w[RF], x[RT];
#pragma unroll
      for (int a = 0; a < RF; ++a) w[a] = *reinterpret_cast<const float4*>(lds + (lf + a * LF) * LS + c);
#pragma unroll
      for (int b = 0; b < RT; ++b) x[b] = *reinterpret_cast<const float4*>(lds + (FT + lt * RT + b) * LS + c);
#pragma unroll
      for (int a = 0; a < RF; ++a)
#pragma unroll
        for (int b = 0; b < RT; ++b) {
          acc[a][b] = fmaf(x[b].x, w[a].x, acc[a][b]);
          acc[a][b] = fmaf(x[b].y, w[a].y, acc[a][b]);
          acc[a][b] = fmaf(x[b].z, w[a].z, acc[a][b]);
          acc[a][b] = fmaf(x[b].w, w[a].w, acc[a][b]);
        }
    };
    if (n == KC) {
#pragma unroll 8
      for (int c = 0; c < KC; c += 4) step4(c);
    } else {
      int c = 0;
      for (; c + 4 <= n; c += 4) step4(c);
      for (; c < n; ++c)                                        // no product with the padding: it would turn -0 into +0
#pragma unroll
        for (int a = 0; a < RF; ++a)
#pragma unroll
          for (int b = 0; b < RT; ++b)
            acc[a][b] = fmaf(lds[(FT + lt * RT + b) * LS + c], lds[(lf + a * LF) * LS + c], acc[a][b]);
    }
  }

#pragma unroll
  for (int a = 0; a < RF; ++a) {
    const int f = f0 + lf + a * LF;
    if (f >= n_feat) continue;
    const int hg = f / d, e = f - hg * d, p = part_of_head(out, hg);
    float* const o = (float*)out.base[p] + (int64_t)(hg - out.first_head[p]) * out.head_stride[p] + e;
    const float bf = bias ? bias[f] : 0.f;
#pragma unroll
    for (int b = 0; b < RT; ++b) {
      const int64_t t = t0 + lt * RT + b;
      if (t < n_tok) o[t * out.token_stride[p]] = bias ? acc[a][b] + bf : acc[a][b];
    }
  }
}

}  // namespace tca

using namespace tca;

namespace {
constexpr int kCUs = 256;

struct QkvCall {
  const uint16_t *W, *X, *bias;
  int n_feat;
  int64_t n_tok;
  int hidden, d;
  QkvOut out;
  hipStream_t st;
};

template <int FB, int TB>
void launch_skinny(const QkvCall& c, int nf) {
  constexpr int U = 4 / (FB * TB) > 1 ? 4 / (FB * TB) : 1;
  const dim3 grid((unsigned)((c.n_feat + nf - 1) / nf), (unsigned)((c.n_tok + 16 * TB - 1) / (16 * TB)));
  hipLaunchKernelGGL((qkv_skinny_kernel<FB, TB, U>), grid, dim3(1024), 0, c.st, c.W, c.X, c.bias, c.n_feat, nf, c.n_tok, c.hidden,
                     c.d, c.out);
}

template <int TB>
void launch_skinny(const QkvCall& c) {
  // Features per workgroup: as many as give each CU one (the same number of) workgroups, in fours (a store) and 16 at least.
  const int rounds = (c.n_feat + 64 * kCUs - 1) / (64 * kCUs), share = (c.n_feat + rounds * kCUs - 1) / (rounds * kCUs);
  const int nf = share <= 16 ? 16 : (share + 3) / 4 * 4;
  if (nf <= 16) launch_skinny<1, TB>(c, nf);
  else if (nf <= 32) launch_skinny<2, TB>(c, nf);
  else if (nf <= 48) launch_skinny<3, TB>(c, nf);
  else launch_skinny<4, TB>(c, nf);
}

template <int FBW, int TBW, int NWF, int NWT, int NST>
void launch_tiles(const QkvCall& c) {
  constexpr int PF = NWF * FBW * 32, PT = NWT * TBW * 32;
  const int n_ft = (c.n_feat + PF - 1) / PF, n_tt = (int)((c.n_tok + PT - 1) / PT);
  const unsigned n_wg = 8u * (unsigned)(((int64_t)n_ft * n_tt + 7) / 8);
  hipLaunchKernelGGL((qkv_mfma_kernel<FBW, TBW, NWF, NWT, NST>), dim3(n_wg), dim3(NWF * NWT * 64), 0, c.st, c.W, c.X, c.bias,
                     c.n_feat, c.n_tok, c.hidden, c.d, c.out, n_ft, n_tt);
}

struct F32Call {
  const float *W, *X, *bias;
  int n_feat;
  int64_t n_tok;
  int hidden, d;
  QkvOut out;
  hipStream_t st;
};

template <int FT, int TT, int RF, int RT, int KC>
void launch_f32(const F32Call& c) {
  const dim3 grid((unsigned)((c.n_feat + FT - 1) / FT), (unsigned)((c.n_tok + TT - 1) / TT));
  const bool aligned = c.hidden % 4 == 0 && !(((uintptr_t)c.W | (uintptr_t)c.X) & 15);
  auto* const kernel = aligned ? qkv_f32_kernel<FT, TT, RF, RT, KC, true> : qkv_f32_kernel<FT, TT, RF, RT, KC, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, c.st, c.W, c.X, c.bias, c.n_feat, c.n_tok, c.hidden, c.d, c.out);
}
}  // namespace

extern "C" int tca_qkv_project(const tca_params* prm, const void* X, int64_t n_tokens, int hidden, const void* W,
                               const void* bias, void* Q, int64_t q_token_stride, int64_t q_head_stride, void* K,
                               void* V, int64_t kv_token_stride, int64_t kv_head_stride, void* stream) {
  int rc = check_params(prm);
  if (rc) return rc;
  if (!X || !W || !Q || !K || !V || n_tokens < 0 || hidden < 1)
    return fail(TCA_ERR_INVALID, "tca_qkv_project: NULL pointer argument, n_tokens=%lld or hidden=%d", (long long)n_tokens,
                hidden);
  const int Hq = prm->n_q_heads, Hkv = prm->n_kv_heads, d = prm->head_dim;
  const int n_feat = (Hq + 2 * Hkv) * d;
  if (q_token_stride < d && n_tokens > 1) return fail(TCA_ERR_INVALID, "tca_qkv_project: q_token_stride=%lld", (long long)q_token_stride);
  if (kv_token_stride < d && n_tokens > 1) return fail(TCA_ERR_INVALID, "tca_qkv_project: kv_token_stride=%lld", (long long)kv_token_stride);
  if (q_head_stride < d || kv_head_stride < d)
    return fail(TCA_ERR_INVALID, "tca_qkv_project: head strides %lld, %lld", (long long)q_head_stride, (long long)kv_head_stride);
  if (n_tokens == 0) return TCA_OK;
  QkvOut out;
  out.base[0] = Q; out.base[1] = K; out.base[2] = V;
  out.head_stride[0] = q_head_stride; out.head_stride[1] = out.head_stride[2] = kv_head_stride;
  out.token_stride[0] = q_token_stride; out.token_stride[1] = out.token_stride[2] = kv_token_stride;
  out.first_head[0] = 0; out.first_head[1] = Hq; out.first_head[2] = Hq + Hkv; out.first_head[3] = Hq + 2 * Hkv;
  hipStream_t st = (hipStream_t)stream;
  if (prm->dtype == TCA_F32) {
    if (n_tokens > 65535) return fail(TCA_ERR_UNSUPPORTED, "tca_qkv_project (fp32): more than 65535 rows per call");
    // Fewer rows, smaller tiles: more workgroups and no work for missing rows; 64 x 64 once that gives every CU one.
    // us, one thread per output before -> now, hidden 4096 and 6144 features: 2 rows 493 -> 48, 16: 1275 -> 72,
    // 17: 1532 -> 97, 100: 10444 -> 156, 256: 23389 -> 292 (22 T multiply-adds a second, of about 36 that the vector
    // ALU has); hidden 1024, 384 features: 2 rows 117 -> 14, 256: 254 -> 27.
    const F32Call call{(const float*)W, (const float*)X, (const float*)bias, n_feat, n_tokens, hidden, d, out, st};
    if (n_tokens <= 8) launch_f32<32, 8, 1, 1, 128>(call);
    else if (n_tokens <= 16) launch_f32<32, 16, 1, 2, 64>(call);
    else if ((int64_t)((n_feat + 63) / 64) * ((n_tokens + 63) / 64) < kCUs) launch_f32<32, 32, 2, 2, 64>(call);
    else launch_f32<64, 64, 4, 4, 64>(call);
  } else {
    if (hidden % kPK) return fail(TCA_ERR_UNSUPPORTED, "tca_qkv_project (bf16): hidden=%d is not a multiple of %d", hidden, kPK);
    if ((int64_t)256 * hidden * 2 > INT32_MAX) return fail(TCA_ERR_UNSUPPORTED, "tca_qkv_project (bf16): hidden=%d", hidden);
    if ((q_token_stride | q_head_stride | kv_token_stride | kv_head_stride) & 3 || ((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V) & 7 ||
        ((uintptr_t)X | (uintptr_t)W) & 15)
      return fail(TCA_ERR_INVALID, "tca_qkv_project (bf16): strides must be multiples of 4 elements, outputs 8-byte and inputs 16-byte aligned");
    const QkvCall call{(const uint16_t*)W, (const uint16_t*)X, (const uint16_t*)bias, n_feat, n_tokens, hidden, d, out, st};
    // Up to 32 rows one pass over the weights is all there is to do.  Measured at 6144 features, hidden 4096 (50 MB of
    // weights), with 256 x 256 tiles / 32 features per workgroup / an equal share of 24 per CU: 1 row 196 / 13.8 / 10.5 us,
    // 16 rows 208 / 15.8 / 12.2, 30 rows 196 / 18.1 / 15.4; 10240 features, hidden 8192 (168 MB), 64 / 40 per workgroup:
    // 1 row 40.7 / 32.3, 16 rows 44.5 / 32.1, 30 rows 51.9 / 38.8.
    if (n_tokens <= 16) {
      launch_skinny<1>(call);
    } else if (n_tokens <= 32) {
      launch_skinny<2>(call);
    } else {
      // Tiles.  What a workgroup waits for is the passage of its stages from L2 into LDS, about 24 bytes per clock and
      // CU whatever the shape and however many stages are resident: a call takes (rounds of 256 workgroups) x
      // (features + tokens of the tile), and the 256 x 256 tile, where the matrix pipe takes as long, 1.35 times that.
      // The shape with the smallest product is taken (the larger tile if equal); us measured at 6144 features,
      // hidden 4096 (64x64 / 64x128 / 128x128 / 128x256 / 256x256), the choice in brackets:
      //   128 rows [23] 31 42 47 98;  256: 41 [31] 41 58 107;  413: 54 49 [36] 52 103;  1024: 119 84 80 [63] 106;
      //   1500: 129 110 102 104 [91];  4096: 338 272 221 [185] 199;  8192: 687 574 459 379 [342]
      // (256 x 256 alone, with ids that skipped CUs when the token tiles were not a multiple of 32, took 196 - 221
      // us up to 1500 rows, 230 us at 2048 and 295 at 4096).
      constexpr int kTiles[5][2] = {{256, 256}, {128, 256}, {128, 128}, {64, 128}, {64, 64}};      // features, tokens
      int best = -1;
      int64_t best_cost = 0;
      for (int i = 0; i < 5; ++i) {
        const int64_t items = (int64_t)((n_feat + kTiles[i][0] - 1) / kTiles[i][0]) * ((n_tokens + kTiles[i][1] - 1) / kTiles[i][1]);
        if (items > INT32_MAX - 8) continue;       // the grid, rounded up to a multiple of 8
        const int64_t cost = (items + kCUs - 1) / kCUs * (i == 0 ? 690 : kTiles[i][0] + kTiles[i][1]);
        if (best < 0 || cost < best_cost) { best = i; best_cost = cost; }
      }
      switch (best) {
        case 0: launch_tiles<4, 2, 2, 4, 2>(call); break;
        case 1: launch_tiles<2, 2, 2, 4, 3>(call); break;
        case 2: launch_tiles<2, 1, 2, 4, 4>(call); break;
        case 3: launch_tiles<1, 1, 2, 4, 4>(call); break;
        case 4: launch_tiles<1, 1, 2, 2, 6>(call); break;
        default: return fail(TCA_ERR_UNSUPPORTED, "tca_qkv_project: n_tokens=%lld", (long long)n_tokens);
      }
    }
  }
  TCA_HIP_CHECK(hipGetLastError());
  return TCA_OK;
}
