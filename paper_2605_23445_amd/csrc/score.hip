// Hierarchical block scoring (paper Sec. 5.2; Algorithm 1 step 2; Eq. 2 and Eq. 8).
//
//   pool_kernel   : Q_hat, K_hat = mean over the real rows of each sub-block, an HBM stream.  The fp32
//                   means (Q_hat already times 1/sqrt(d)) are scaled, four consecutive sub-blocks at a time,
//                   by the power of two that brings their largest magnitude to 2^11..2^12, and stored as two
//                   fp16 terms x = hi + lo, which together carry 22 bits of the value.
//   score_lse_kernel / score_fold_kernel : S_hat[u,v] = sum over the r x r sub-block pairs of
//                   softmax(Q_hat K_hat^T / sqrt(d)).  The sub-block attention matrix A_hat is never stored.
//                   One pass over the contraction: per (query sub-block, key block) the base-2 log of the
//                   summed exponentials of the block's key sub-blocks and per query sub-block the row
//                   log-sum-exp; a second, memory-bound kernel turns these into probabilities and folds the r
//                   query sub-blocks of a query block.  The logits run on the fp16 matrix cores as three
//                   partial products hi.hi + hi.lo + lo.hi with fp32 accumulation: every fp16 product is exact
//                   in fp32 and the dropped lo.lo term is below 2^-22 of the result, so the logits are as
//                   accurate as an fp32 contraction at several times its speed (the mask decision that
//                   follows stays an fp32 one); the scaling is undone, exactly, on the fp32 result.
//   fold_select_kernel : the second of the two with the selection of a row behind it (select_row.h).
//   score_small_kernel : all of it behind the pooling, for small problems.
#include <type_traits>

#include "score_small.h"
#include "select_row.h"

namespace dfs {

// ------------------------------------------------------------------------------------ pooling

// One wave per sub-block.  Lanes of a row sit side by side (16 bytes each); several rows are in
// flight per load; partial sums of the row groups are folded with cross-lane exchanges.
// Output: the hi and lo fp16 planes of the row times its group's scale (layouts above); the inverse scale of group s / 4 goes
// to q_down / k_down.
// blockIdx.z: 0 pools Q, 1 pools K, 2 only reorders V.  With an index (the permutation) Q, K (if k_src) and V come in source
// order and their rows are gathered; K (if k_out) and V are written out in the reordered layout on the way (pads as
// zeros, text rows too), so that a step that refreshes the mask reads and writes each of them once, in one launch.
// An HBM stream; a wave requests up to eight row groups (the positions first, then the rows) before it uses one,
// because on small problems a sub-block is a chain of dependent loads.  With V's reorder in a launch of its own and
// one row group at a time: 75 600 tokens x 40 heads, d = 128, 715 -> 643 us (6.0 TB/s); 17 550 x 48, d = 64, 105 -> 83
// us; 5 589 x 7, d = 128, 21.5 -> 11 us.
template <bool BF16, int D>
__global__ void __launch_bounds__(256) pool_kernel(const void* __restrict__ q_in, const void* __restrict__ k_in, const void* __restrict__ v_in,
                                                   uint16_t* __restrict__ q_hat, uint16_t* __restrict__ k_hat,
                                                   float* __restrict__ q_down, float* __restrict__ k_down,
                                                   const int32_t* __restrict__ index, void* __restrict__ k_out, void* __restrict__ v_out,
                                                   int64_t N_src, int64_t N_pad, int64_t N_v, int Bs, int M_s, float q_scale, bool tiled, bool k_src,
                                                   int32_t* __restrict__ zero, int n_zero) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
    for (int i = threadIdx.x; i < n_zero; i += 256) zero[i] = 0;
  constexpr int EPL = BF16 ? 8 : 4;           // elements per lane (16 bytes)
  constexpr int TPR = D / EPL;                // lanes per row
  constexpr int RPP = 64 / TPR;               // rows per pass
  constexpr int AHEAD = 32 / RPP < 8 ? 32 / RPP : 8;         // passes in flight
  const int lane = threadIdx.x & 63;
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  const bool pooled = s < M_s && blockIdx.z < 2;             // this wave has a sub-block to pool
  void* out = blockIdx.z == 0 ? nullptr : blockIdx.z == 1 ? k_out : v_out;
  const bool copied = out != nullptr && int64_t(s) * Bs < N_pad;
  const bool gather = index != nullptr && (blockIdx.z != 1 || k_src);
  const int head = blockIdx.y;
  const void* src = blockIdx.z == 0 ? q_in : blockIdx.z == 1 ? k_in : v_in;
  uint16_t* dst = blockIdx.z == 0 ? q_hat : k_hat;
  const int c = lane % TPR, rg = lane / TPR;
  const int64_t row0 = int64_t(s) * Bs;
  int64_t left = N_v - row0;
  const int cnt = left <= 0 ? 0 : (left < Bs ? int(left) : Bs);
  float acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
  const u32x4* base = reinterpret_cast<const u32x4*>(src) + (gather ? int64_t(head) * N_src * TPR : (int64_t(head) * N_pad + row0) * TPR) + c;
  u32x4* copy = reinterpret_cast<u32x4*>(out) + (int64_t(head) * N_pad + row0) * TPR + c;
  const int rows = copied ? Bs : pooled ? cnt : 0;           // a copy covers the pad rows of the sub-block as well
  for (int i0 = rg; i0 - rg < rows; i0 += RPP * AHEAD) {
    int32_t from[AHEAD];
    u32x4 val[AHEAD];
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
      const int i = i0 + p * RPP;
      from[p] = i >= rows ? -1 : gather ? index[row0 + i] : i;
    }
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
      if (gather && from[p] >= N_src) from[p] = -1;
      val[p] = u32x4{0u, 0u, 0u, 0u};
      if (from[p] >= 0) val[p] = __builtin_nontemporal_load(base + int64_t(from[p]) * TPR);
    }
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
      const int i = i0 + p * RPP;
      if (copied && i < rows) __builtin_nontemporal_store(val[p], copy + int64_t(i) * TPR);
      if (from[p] < 0 || i >= cnt) continue;
      if (BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] += __uint_as_float(val[p][e] << 16);
          acc[2 * e + 1] += __uint_as_float(val[p][e] & 0xFFFF0000u);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __uint_as_float(val[p][e]);
      }
    }
  }
  if (blockIdx.z == 2) return;                               // the whole work-group
#pragma unroll
  for (int off = TPR; off < 64; off <<= 1) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
  }
  // every lane now holds the column sums of its 16 bytes of the row; the row's largest magnitude, then the group's
  const float inv = pooled && cnt > 0 ? (blockIdx.z == 0 ? q_scale : 1.0f) / float(cnt) : 0.f;
  float mx = 0.f;
#pragma unroll
  for (int e = 0; e < EPL; ++e) {
    acc[e] *= inv;
    mx = fmaxf(mx, fabsf(acc[e]));
  }
#pragma unroll
  for (int off = 1; off < TPR; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  __shared__ float s_max[4];
  if (lane == 0) s_max[threadIdx.x >> 6] = mx;
  __syncthreads();                             // reached by all four waves: none has left the kernel
  if (!pooled) return;                         // copied only, or beyond the last sub-block
  float up, down;
  group_scale(fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3])), up, down);
  if (threadIdx.x == 0) (blockIdx.z == 0 ? q_down : k_down)[int64_t(head) * ((M_s + 3) / 4) + blockIdx.x] = down;
  if (rg == 0) {
    const int in_tile = tile_rows(M_s, s / 32);
    uint16_t* o = dst + int64_t(head) * M_s * (2 * D) +
                  (tiled ? tile_at<D>(s / 32) + chunk_at<D>(0, c * EPL / 8, in_tile, s % 32) + c * EPL % 8 : int64_t(s) * (2 * D) + c * EPL);
    uint16_t hi[EPL], lo[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) split2(acc[e] * up, hi[e], lo[e]);
    typedef unsigned int pairs __attribute__((ext_vector_type(EPL / 2)));
    pairs h2, l2;
#pragma unroll
    for (int e = 0; e < EPL; e += 2) {
      h2[e / 2] = uint32_t(hi[e]) | (uint32_t(hi[e + 1]) << 16);
      l2[e / 2] = uint32_t(lo[e]) | (uint32_t(lo[e + 1]) << 16);
    }
    *reinterpret_cast<pairs*>(o) = h2;
    *reinterpret_cast<pairs*>(o + (tiled ? chunk_at<D>(1, 0, in_tile, 0) : D)) = l2;
  }
}

// Pooling of bf16 tensors that nothing is written out of on the way: one wave per scale group of four sub-blocks, so that what follows the sums
// (row groups folded, magnitude, scale, split) is done once for four, each row of sixteen lanes with a sub-block of its own, and without a way
// through LDS; the same sums in the same order as above.  An HBM stream that was bound by the issue of some 240 instructions per
// sub-block beside its loads (counted from the source), now some 130.  See pool_reads_groups for the rule and what it measured.
template <int D>
__global__ void __launch_bounds__(256) pool_read_kernel(const uint16_t* __restrict__ q_in, const uint16_t* __restrict__ k_in, uint16_t* __restrict__ q_hat,
                                                        uint16_t* __restrict__ k_hat, float* __restrict__ q_down, float* __restrict__ k_down,
                                                        const int32_t* __restrict__ index, int64_t N_src, int64_t N_pad, int64_t N_v, int Bs, int M_s,
                                                        float q_scale, bool tiled, bool k_src, int32_t* __restrict__ zero, int n_zero) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
    for (int i = threadIdx.x; i < n_zero; i += 256) zero[i] = 0;
  constexpr int TPR = D / 8, RPP = 64 / TPR, AHEAD = 4, CR = RPP * AHEAD;        // lanes per row, rows per pass, passes in flight of each sub-block
  constexpr int NP = 4 * CR / 64;                            // positions a lane looks up for them
  const int lane = threadIdx.x & 63, g = blockIdx.x * 4 + (threadIdx.x >> 6), G4 = (M_s + 3) / 4;
  if (g >= G4) return;
  const int c = lane % TPR, rg = lane / TPR, head = blockIdx.y;
  const bool keys = blockIdx.z == 1, gather = index != nullptr && (!keys || k_src);
  const int64_t limit = gather ? N_src : N_pad, row0 = int64_t(4 * g) * Bs;
  const u32x4* base = reinterpret_cast<const u32x4*>(keys ? k_in : q_in) + int64_t(head) * limit * TPR + c;
  float acc[4][8];
#pragma unroll
  for (int sb = 0; sb < 4; ++sb)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[sb][e] = 0.f;
  for (int i0 = 0; i0 < Bs; i0 += CR) {
    int pos[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int x = m * 64 + lane, i = i0 + x % CR;
      const int64_t row = row0 + x / CR * Bs + i;
      pos[m] = i >= Bs || row >= N_v ? -1 : gather ? index[row] : int(row);
      if (pos[m] >= limit) pos[m] = -1;
    }
    u32x4 val[4][AHEAD];
#pragma unroll
    for (int sb = 0; sb < 4; ++sb)
#pragma unroll
      for (int p = 0; p < AHEAD; ++p) {
        const int x = sb * CR + p * RPP, from = __shfl(pos[x / 64], x % 64 + rg, 64);
        val[sb][p] = u32x4{0u, 0u, 0u, 0u};
        if (from >= 0) val[sb][p] = __builtin_nontemporal_load(base + int64_t(from) * TPR);
      }
#pragma unroll
    for (int sb = 0; sb < 4; ++sb)
#pragma unroll
      for (int p = 0; p < AHEAD; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) {                        // zeros change no sum that starts from zero
          acc[sb][2 * e] += __uint_as_float(val[sb][p][e] << 16);
          acc[sb][2 * e + 1] += __uint_as_float(val[sb][p][e] & 0xFFFF0000u);
        }
  }
  const int sb = lane >> 4, s = 4 * g + sb;                  // this lane's sub-block from here on
  const int64_t left = N_v - int64_t(s) * Bs;
  const float cnt = left <= 0 ? 0.f : float(left < Bs ? int(left) : Bs), by = left <= 0 ? 0.f : (keys ? 1.0f : q_scale) / cnt;
  float own[8], mx = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (RPP == 8) {                                          // two row groups in sixteen lanes
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x][e] += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(acc[x][e]), 0x128, 0xF, 0xF, true));
    }
    own[e] = sum_32(sum_16(acc[0][e], acc[1][e]), sum_16(acc[2][e], acc[3][e])) * by;
    mx = fmaxf(mx, fabsf(own[e]));
  }
  float up, down;
  group_scale(max_32(max_16(max_of_16(mx))), up, down);
  if (lane == 0) (keys ? k_down : q_down)[int64_t(head) * G4 + g] = down;
  if (s >= M_s || (lane & 15) >= TPR) return;
  const int in_tile = tile_rows(M_s, s / 32);
  uint16_t* o = (keys ? k_hat : q_hat) + int64_t(head) * M_s * (2 * D) +
                (tiled ? tile_at<D>(s / 32) + chunk_at<D>(0, c, in_tile, s % 32) : int64_t(s) * (2 * D) + c * 8);
  uint16_t hi[8], lo[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) split2(own[e] * up, hi[e], lo[e]);
  u32x4 h4, l4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h4[e] = uint32_t(hi[2 * e]) | (uint32_t(hi[2 * e + 1]) << 16);
    l4[e] = uint32_t(lo[2 * e]) | (uint32_t(lo[2 * e + 1]) << 16);
  }
  *reinterpret_cast<u32x4*>(o) = h4;
  *reinterpret_cast<u32x4*>(o + (tiled ? chunk_at<D>(1, 0, in_tile, 0) : D)) = l4;
}

// ------------------------------------------------------------------------------------ scoring

// T is stored with its rows padded to whole query groups (128 sub-blocks) and its row count to whole key tiles,
// so that the contraction kernel stores without a bounds check: [heads][t_rows][t_cols] fp32.
__host__ __device__ inline int t_cols(int M_s) { return (M_s + 127) / 128 * 128; }
__host__ __device__ inline int t_rows(int M_s, int R) { return (M_s + 31) / 32 * (32 / R); }

__device__ __forceinline__ float vmax3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Pass 1 (the contraction, once).  A work-group owns 128 query sub-blocks (32 per wave) and one of KSPLIT
// ranges of key tiles (32 key sub-blocks each).  The logits are computed transposed, keys along the rows of
// the matrix instruction's result, so that a lane holds, for ONE query sub-block (its column), runs of four
// consecutive key sub-blocks: the R key sub-blocks of a key block fold inside the lane (R = 8: plus one
// exchange between the two lane halves).  Per (query sub-block i, key block v) it stores
//   T[v][i] = log2 sum over the key sub-blocks j of v of 2^logit(i, j)          (logits already in base 2)
// which needs no row reference, and per query sub-block the log-sum-exp over its key range.  Pass 2 turns
// T into probabilities and folds the R query sub-blocks of a query block.
template <int D, int R>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
score_lse_kernel(const uint16_t* __restrict__ q_hat, const uint16_t* __restrict__ k_hat, const float* __restrict__ q_down,
                 const float* __restrict__ k_down, float* __restrict__ tt, float* __restrict__ lse, int M_s, int n_live, int tiles_per_split, int ksplit,
                 int wgs_per_head, int total_wgs, int wgs_per_xcd) {
  constexpr int RS = 2 * D;                   // elements of a centroid row (hi, lo planes)
  constexpr int RSP = RS + 8;                 // LDS row stride: 16 bytes of skew keep the row-per-lane reads conflict-free
  constexpr int KS = D / 16;                  // product steps of 16 features
  constexpr int CPT = 32 * RS / 8 / 256;      // 16-byte chunks of a key tile per thread (6 at d=128)
  constexpr int G = R < 4 ? R : 4;            // key sub-blocks of one key block that sit in consecutive registers
  __shared__ __attribute__((aligned(16))) uint16_t s_k[2][32 * RSP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, half = lane >> 5;
  // Work-group ids are dealt round-robin to the 8 XCDs, each with an L2 of its own.  Every XCD takes a contiguous
  // eighth of the (head, query group, key range) list, so that the work-groups resident on an XCD belong to one or
  // two heads and that head's key centroids (re-read by every one of them) stay in its L2.
  const int logical = (blockIdx.x % 8) * wgs_per_xcd + blockIdx.x / 8;
  if (logical >= total_wgs) return;           // the whole work-group: no barrier has been reached yet
  const int head = logical / wgs_per_head, in_head = logical % wgs_per_head;
  const int split = in_head % ksplit;
  const int i0 = (in_head / ksplit) * 128 + wave * 32;      // first query sub-block of this wave
  const uint16_t* qh = q_hat + int64_t(head) * M_s * RS;
  const uint16_t* kh = k_hat + int64_t(head) * M_s * RS;

  // Query centroids as the B operand: lane (n, half) holds row i0 + n, features 16 kk + 8 half .. + 7, two planes.
  const int G4 = (M_s + 3) / 4;               // scale groups (four consecutive sub-blocks) per head
  f16x8 bq[2][KS];
  float q_dn = 1.0f;                          // inverse scale of this lane's query row
  {
    const int row = i0 + n;
    if (row < M_s) q_dn = q_down[int64_t(head) * G4 + row / 4];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (row < M_s) v = *reinterpret_cast<const u32x4*>(qh + int64_t(row) * RS + p * D + 16 * kk + 8 * half);
        bq[p][kk] = __builtin_bit_cast(f16x8, v);
      }
  }
  const int n_tiles = (n_live + 31) / 32;     // key sub-blocks at or beyond n_live are empty
  const int t_begin = split * tiles_per_split;
  const int t_end = t_begin + tiles_per_split < n_tiles ? t_begin + tiles_per_split : n_tiles;

  // key tile t (32 centroid rows, contiguous in memory) -> registers -> LDS
  u32x4 kreg[CPT];
  auto fetch = [&](int t) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      // rows at or beyond M_s re-read the last row instead (no branch): they are at or beyond n_live and masked later
      const int c = tid + i * 256;
      const int row = t * 32 + c / (RS / 8);
      const int from = row < M_s ? row : M_s - 1;
      kreg[i] = *reinterpret_cast<const u32x4*>(kh + int64_t(from) * RS + (c % (RS / 8)) * 8);
    }
  };
  auto commit = [&](int buf) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + i * 256;
      *reinterpret_cast<u32x4*>(&s_k[buf][(c / (RS / 8)) * RSP + (c % (RS / 8)) * 8]) = kreg[i];
    }
  };
  float m_row = LSE_START, z_row = 0.f;       // this lane's share of the row log-sum-exp of query sub-block i0 + n
  const int q_row = i0 + n;
  const int TC = t_cols(M_s);
  float* tt_h = tt + int64_t(head) * t_rows(M_s, R) * TC;
  const int t_lane = (R == 8 ? 0 : half) * (R == 1 ? 4 : R == 2 ? 2 : 1) * TC + q_row;   // this lane's share of a T index
  // inverse scales for the four row groups of tile t that this lane's registers cover, times the query row's
  auto load_dn = [&](int t, float (&dn)[4]) {
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {            // scale group of key rows 32 t + 8 gq + 4 half .. + 3
      const int grp = 8 * t + 2 * gq + half;
      dn[gq] = k_down[int64_t(head) * G4 + (grp < G4 ? grp : G4 - 1)] * q_dn;     // beyond the last group: masked rows
    }
  };

  // One pipeline stage, written out in issue order: the matrix instructions of tile t and, in their shadow, the
  // epilogue of the tile before, cut into 24 slices.  (Two waves of a SIMD that each run their matrix phase and
  // then their vector phase fall into step, and the two kinds of work then add up instead of overlapping.)
  //   matrix part: transposed logits of the 32 x 32 tile, a[i] = <k_hat[row 8 (i/4) + 4 half + i%4 of the tile],
  //     q_hat[i0 + n]>, as hi.hi + hi.lo + lo.hi products (lo.lo is below 2^-22 of the result) with fp32
  //     accumulation, dealt to two accumulators c0, c1 in turn so that no matrix instruction waits for the one
  //     before it; the operands of two product steps are requested from LDS one pair ahead; tile t + 1 goes from
  //     its staging registers to LDS early in the stage, and only then the loads of tile t + 2 are issued, so
  //     they have a whole stage to land.
  //   epilogue of tile tp from its accumulators p0, p1: logits = (p0 + p1) x inverse scales (registers 4 g .. 4 g + 3
  //     of a lane are four consecutive key rows, one scale group); one reference for the whole tile, the running
  //     row maximum including this tile (finite from the start, so no difference is ever inf - inf; masked logits
  //     give 2^-inf = 0; R == 8: a key block is split over the two lane halves, which therefore share the
  //     reference); then per key block the log of its summed exponentials.
  constexpr int NS = 3 * KS;                  // matrix instructions of a tile
  auto stage = [&](auto do_mm, auto do_ep, int t, int buf, f32x16& c0, f32x16& c1, float (&dn_next)[4], const f32x16& p0,
                   const f32x16& p1, const float (&dn_prev)[4], int tp) {
    constexpr bool MM = decltype(do_mm)::value, EP = decltype(do_ep)::value;
    const uint16_t* krow = &s_k[buf][n * RSP + 8 * half];
    f16x8 fr[2][4];
    auto load_pair = [&](int p) {
      fr[p & 1][0] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(krow + 32 * p));
      fr[p & 1][1] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(krow + D + 32 * p));
      fr[p & 1][2] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(krow + 32 * p + 16));
      fr[p & 1][3] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(krow + D + 32 * p + 16));
    };
    float dp[4], c[16];
    float mt = 0.f, m_new = 0.f, zt = 0.f;
    if (EP) {
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) dp[gq] = dn_prev[gq];      // dn_next may be the same array
    }
    if (MM) {
      load_pair(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) { c0[i] = 0.f; c1[i] = 0.f; }
    }
    auto slice = [&](int sl) {
      if (sl < 8) {
#pragma unroll
        for (int i = 2 * sl; i < 2 * sl + 2; ++i) c[i] = (p0[i] + p1[i]) * dp[i / 4];
      } else if (sl == 8) {
        if (__builtin_expect(tp * 32 + 32 > n_live, 0)) {   // ragged end: key sub-blocks without rows count for nothing
          asm volatile("");                   // keeps this a branch: as selects it would run on every tile
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (tp * 32 + 8 * (i / 4) + 4 * half + (i % 4) >= n_live) c[i] = -INFINITY;
        }
        mt = vmax3(c[0], c[1], c[2]);
      } else if (sl < 12) {
        const int i = 3 + 4 * (sl - 9);
        mt = vmax3(mt, c[i], c[i + 1]);
        mt = vmax3(mt, c[i + 2], c[i + 3]);
      } else if (sl == 12) {
        mt = fmaxf(mt, c[15]);
        if (R == 8) {
          float lo, hi;
          both_halves(mt, lo, hi);
          mt = fmaxf(lo, hi);
        }
        m_new = fmaxf(m_row, mt);
        z_row *= __builtin_amdgcn_exp2f(m_row - m_new);
        m_row = m_new;
      } else {
        if (sl < 21) {
#pragma unroll
          for (int i = 2 * (sl - 13); i < 2 * (sl - 13) + 2; ++i) {
            const float e = __builtin_amdgcn_exp2f(c[i] - m_new);
            if (G == 1) zt += e; else c[i] = e;
          }
        }
        if (sl >= 20) {
          // fold the key sub-blocks of each key block: groups of G consecutive registers
          constexpr int NG = 16 / G;
#pragma unroll
          for (int gi = (sl - 20) * NG / 4; gi < (sl - 19) * NG / 4; ++gi) {
            float tv;
            if (G == 1) {
              tv = c[gi];
            } else {
              float sg = 0.f;
#pragma unroll
              for (int e = 0; e < G; ++e) sg += c[gi * G + e];
              zt += sg;                        // this lane's own share of the row sum
              if (R == 8) {
                float lo, hi;
                both_halves(sg, lo, hi);
                sg = lo + hi;
              }
              // a block whose sum vanishes against the row maximum (below 2^-126 of it) scores nothing: log2(0) = -inf
              tv = m_new + __builtin_amdgcn_logf(sg);
            }
            // key sub-block of the group's first register: 8 (first / 4) + 4 half + first % 4
            // key block = (32 tp + 8 (first / 4) + first % 4) / R + the lane half's share, which is in t_lane; the
            // uniform part goes into a scalar base.  No bounds check: T is padded, and at R = 8 both lane halves
            // store the same value to the same place.
            const int first = gi * G;
            const int v_uniform = (tp * 32 + 8 * (first / 4) + (first % 4)) / R;
            (tt_h + int64_t(v_uniform) * TC)[t_lane] = tv;
          }
          if (sl == 23) z_row += zt;
        }
      }
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      if (MM) {
        const int p = m / 6, j = m % 6, kk = 2 * p;
        if (j == 0 && p + 1 < KS / 2) load_pair(p + 1);
        const f16x8(&f)[4] = fr[p & 1];
        if (j == 0) c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[0], bq[0][kk], c0, 0, 0, 0);          // hi.hi
        if (j == 1) c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[0], bq[1][kk], c1, 0, 0, 0);          // hi.lo
        if (j == 2) c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[1], bq[0][kk], c0, 0, 0, 0);          // lo.hi
        if (j == 3) c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[2], bq[0][kk + 1], c1, 0, 0, 0);
        if (j == 4) c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[2], bq[1][kk + 1], c0, 0, 0, 0);
        if (j == 5) c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[3], bq[0][kk + 1], c1, 0, 0, 0);
        if (m == 2 && t + 1 < t_end) commit(buf ^ 1);      // the other buffer was last read before the previous barrier
        if (m == 4 && t + 2 < t_end) fetch(t + 2);
        if (m == NS / 2 && t + 1 < t_end) load_dn(t + 1, dn_next);   // the epilogue is done with dn_prev by now
      }
      if (EP) {
#pragma unroll
        for (int sl = m * 24 / NS; sl < (m + 1) * 24 / NS; ++sl) slice(sl);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (MM) __syncthreads();                  // tile t has been read by every wave; tile t + 1 is in LDS
  };

  if (t_begin < t_end) {
    using yes = std::true_type;
    using no = std::false_type;
    // tiles alternate between two sets of accumulators and inverse scales (the second set is handed, unused, to the
    // first stage, which has no epilogue)
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 xa0 = zero16, xa1 = zero16, ya0 = zero16, ya1 = zero16;
    float dx[4] = {1.f, 1.f, 1.f, 1.f}, dy[4] = {1.f, 1.f, 1.f, 1.f};
    load_dn(t_begin, dx);
    fetch(t_begin);
    commit(0);
    if (t_begin + 1 < t_end) fetch(t_begin + 1);
    __syncthreads();
    int t = t_begin;
    stage(yes{}, no{}, t, 0, xa0, xa1, dy, ya0, ya1, dy, t);
    ++t;
    for (; t + 1 < t_end; t += 2) {
      stage(yes{}, yes{}, t, 1, ya0, ya1, dx, xa0, xa1, dx, t - 1);
      stage(yes{}, yes{}, t + 1, 0, xa0, xa1, dy, ya0, ya1, dy, t);
    }
    if (t < t_end) {
      stage(yes{}, yes{}, t, 1, ya0, ya1, dx, xa0, xa1, dx, t - 1);
      stage(no{}, yes{}, t, 0, xa0, xa1, dx, ya0, ya1, dy, t);
    } else {
      stage(no{}, yes{}, t, 0, ya0, ya1, dy, xa0, xa1, dx, t - 1);
    }
  }
  // the two lane halves of a column hold different key blocks of the same query sub-block
  {
    const float m2 = __shfl_xor(m_row, 32, 64), z2 = __shfl_xor(z_row, 32, 64);
    lse_merge(m_row, z_row, m2, z2);
  }
  if (half == 0 && q_row < M_s)
    lse[(int64_t(head) * ksplit + split) * M_s + q_row] = z_row > 0.f ? m_row + __builtin_amdgcn_logf(z_row) : -INFINITY;
}

// Pass 2: S_hat[u][v] = sum over the R query sub-blocks i of u of 2^(T[v][i] - lse(i)), lse(i) merged over the
// key ranges.  A work-group handles 32 query blocks x 32 key blocks; T is read along i (contiguous), the
// scores are written along v (contiguous), the transposition goes through LDS.
template <int R>
__global__ void __launch_bounds__(256) score_fold_kernel(const float* __restrict__ tt, const float* __restrict__ lse,
                                                         float* __restrict__ score, int M_s, int M_v, int n_live, int ksplit) {
  __shared__ float s_t[32][33];
  const int head = blockIdx.z, u0 = blockIdx.x * 32, v0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;          // 32 x 8
  const int TC = t_cols(M_s);
  const float* tt_h = tt + int64_t(head) * t_rows(M_s, R) * TC;
  const float* lse_h = lse + int64_t(head) * ksplit * M_s;
  // row log-sum-exp of the R sub-blocks of query block u0 + tx
  float l[R];
#pragma unroll
  for (int a = 0; a < R; ++a) {
    const int i = (u0 + tx) * R + a;
    float m = LSE_START, z = 0.f;
    if (u0 + tx < M_v && i < n_live) {
      for (int sp = 0; sp < ksplit; ++sp) lse_add(m, z, lse_h[int64_t(sp) * M_s + i]);
    }
    l[a] = z > 0.f ? m + __builtin_amdgcn_logf(z) : INFINITY;       // +inf: an empty query sub-block scores nothing
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = v0 + ty + 8 * k;
    float acc = 0.f;
    if (v < M_v && u0 + tx < M_v) {
      const float* row = tt_h + int64_t(v) * TC + int64_t(u0 + tx) * R;
#pragma unroll
      for (int a = 0; a < R; ++a) acc += __builtin_amdgcn_exp2f(row[a] - l[a]);
    }
    s_t[ty + 8 * k][tx] = acc;                                       // [v][u]
  }
  __syncthreads();
  float* out = score + int64_t(head) * M_v * M_v;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int u = u0 + ty + 8 * k, v = v0 + tx;
    if (u < M_v && v < M_v) out[int64_t(u) * M_v + v] = s_t[tx][ty + 8 * k];
  }
}

// Pass 2 and the selection in one, for callers that want the lists only: eight query blocks of a head per work-group.  The
// scores of their rows (the same sums as above, in the same order) go to LDS as ordered keys, then each wave selects one
// row.  Eight rows because at R = 4 their query sub-blocks are one 128-byte line of a row of T.  The scores never go to
// memory and one launch goes: 75 600 tokens x 40 heads 134 -> 71 us, 17 550 x 48 19 -> 14, 2 565 x 12 and its gap 10 + 2 -> 7.
constexpr int FS_ROWS = 8, FS_T = 64 * FS_ROWS;
__host__ __device__ inline int fs_stride(int M_v) { return (M_v + 63) / 64 * 64 + 8; }   // lanes (block, row) hit every bank once
template <int R>
__global__ void __launch_bounds__(FS_T) fold_select_kernel(const float* __restrict__ tt, const float* __restrict__ lse, int M_s, int M_v,
                                                           int M_x, int n_live, int ksplit, int k_fixed, int k_cap, double mass,
                                                           uint8_t* __restrict__ mask, int32_t* __restrict__ kv_idx,
                                                           int32_t* __restrict__ kv_cnt, int K_max, int32_t* __restrict__ k_head) {
  extern __shared__ unsigned long long lds64[];
  uint32_t* hists = reinterpret_cast<uint32_t*>(lds64);                  // 256 words per wave, then the keys
  uint32_t* keys = hists + FS_ROWS * 256;
  const int stride = fs_stride(M_v);
  const int head = blockIdx.y, u0 = blockIdx.x * FS_ROWS;
  const int TC = t_cols(M_s);
  const int r = threadIdx.x % FS_ROWS, u = u0 + r;
  if (u < M_v) {
    const float* tt_h = tt + int64_t(head) * t_rows(M_s, R) * TC + int64_t(u) * R;
    const float* lse_h = lse + int64_t(head) * ksplit * M_s;
    float l[R];
#pragma unroll
    for (int a = 0; a < R; ++a) {
      const int i = u * R + a;
      float m = LSE_START, z = 0.f;
      if (i < n_live)
        for (int sp = 0; sp < ksplit; ++sp) lse_add(m, z, lse_h[int64_t(sp) * M_s + i]);
      l[a] = z > 0.f ? m + __builtin_amdgcn_logf(z) : INFINITY;
    }
    typedef float trow __attribute__((ext_vector_type(R < 4 ? R : 4)));   // R T-values side by side, 4 R bytes aligned
    constexpr int W = R < 4 ? R : 4;
#pragma unroll 4
    for (int v = threadIdx.x / FS_ROWS; v < M_v; v += FS_T / FS_ROWS) {
      float acc = 0.f;
#pragma unroll
      for (int w = 0; w < R / W; ++w) {
        const trow t = reinterpret_cast<const trow*>(tt_h + int64_t(v) * TC)[w];
#pragma unroll
        for (int e = 0; e < W; ++e) acc += __builtin_amdgcn_exp2f(t[e] - l[w * W + e]);
      }
      keys[r * stride + v] = order_key(acc);
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, uw = u0 + wave, M = M_v + M_x;
  if (uw >= M) return;
  const int64_t out = int64_t(head) * M + uw;
  uint8_t* mrow = mask ? mask + out * M : nullptr;
  if (uw >= M_v) {
    select_text_row(M, mrow, kv_cnt + out);
    return;
  }
  const uint32_t* row = keys + wave * stride;
  uint32_t* hist = hists + wave * 256;
  int k = k_fixed;
  if (mass > 0.0) {                                                      // every row its own count, clamped
    const int ku = mass_count_row(row, reinterpret_cast<unsigned long long*>(hist), M_v, mass);
    k = ku < k_fixed ? k_fixed : (ku > k_cap ? k_cap : ku);
  } else if (k_head && uw == 0 && (threadIdx.x & 63) == 0) {
    k_head[head] = k;
  }
  select_row<1 << 30, ss_columns(R, 128)>(row, hist, M_v, M_x, k, mrow, kv_idx + out * K_max, kv_cnt + out);     // shorter rows are score_small_kernel's
}
static size_t fs_lds(int M_v) { return size_t(FS_ROWS) * (256 + fs_stride(M_v)) * sizeof(uint32_t); }

// Scoring of small problems in one kernel: a work-group owns 32 query sub-blocks (32 / R query blocks) of a head, its eight
// waves take key tiles in turn, straight from memory, and T and the row sums never leave LDS.  The same sums as the two kernels
// above, except that a row's keys are summed by eight waves and its reference and sum stay apart; so one kernel serves the
// calls that want scores (`score`) and those that want lists (`kv_idx`), and both decide alike.  What bounds it is latency: a
// tile's rows, its product chain, three barriers, the selection; it saves a launch and the way of T through memory.  256 fp32
// tokens x 2 heads 18.4 -> 16.6 us a refresh, 2 565 + 77 tokens x 12 heads, blocks of 64, 39.1 -> 35.5 (both sides in turn).
template <int D, int R>
__global__ void __launch_bounds__(SS_T) score_small_kernel(const uint16_t* __restrict__ q_hat, const uint16_t* __restrict__ k_hat,
                                                           const float* __restrict__ q_down, const float* __restrict__ k_down,
                                                           float* __restrict__ score, int M_s, int M_v, int M_x, int n_live, int k_fixed,
                                                           int k_cap, double mass, uint8_t* __restrict__ mask, int32_t* __restrict__ kv_idx,
                                                           int32_t* __restrict__ kv_cnt, int K_max, int32_t* __restrict__ k_head) {
  constexpr int RS = 2 * D, ROWS = 32 / R;
  extern __shared__ unsigned long long lds64[];
  uint32_t* hists = reinterpret_cast<uint32_t*>(lds64);                  // 256 words per wave
  float* s_t = reinterpret_cast<float*>(hists + SS_WAVES * 256);         // T [M_v][SS_STRIDE], then keys in the first of R
  __shared__ float s_m[SS_WAVES][32], s_z[SS_WAVES][32], s_ref[32], s_inv[32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int head = blockIdx.y, u0 = blockIdx.x * ROWS, i0 = blockIdx.x * 32, M = M_v + M_x;
  if (u0 < M_v) {
    const uint16_t* qh = q_hat + int64_t(head) * M_s * RS;
    const uint16_t* kh = k_hat + int64_t(head) * M_s * RS;
    const int G4 = (M_s + 3) / 4;
    small_scores<D, R>(MemoryOperands<D>{qh, kh, q_down + int64_t(head) * G4, k_down + int64_t(head) * G4, M_s, i0}, s_t, s_m, s_z, s_ref, s_inv, M_v, n_live, i0);
    for (int x = tid; x < ROWS * M_v; x += SS_T) {
      const int r = x / M_v, v = x % M_v;
      float* t = s_t + v * SS_STRIDE + r * R;
      const float acc = small_score<R>(t, s_ref + r * R, s_inv + r * R);
      if (score) {
        if (u0 + r < M_v) score[(int64_t(head) * M_v + u0 + r) * M_v + v] = acc;
      } else {
        *reinterpret_cast<uint32_t*>(t) = order_key(acc);
      }
    }
    __syncthreads();
  }
  if (score) return;
  for (int r = wave; r < ROWS && u0 + r < M; r += SS_WAVES) {
    const int u = u0 + r;
    const int64_t out = int64_t(head) * M + u;
    uint8_t* mrow = mask ? mask + out * M : nullptr;
    if (u >= M_v) {
      select_text_row(M, mrow, kv_cnt + out);
      continue;
    }
    const StridedKeys row = {reinterpret_cast<const uint32_t*>(s_t) + r * R, SS_STRIDE};
    uint32_t* hist = hists + wave * 256;
    int k = k_fixed;
    if (mass > 0.0) {                                      // every row its own count, clamped
      const int ku = mass_count_row(row, reinterpret_cast<unsigned long long*>(hist), M_v, mass);
      k = ku < k_fixed ? k_fixed : (ku > k_cap ? k_cap : ku);
    } else if (k_head && u == 0 && lane == 0) {
      k_head[head] = k;
    }
    select_row<ss_columns(R, D)>(row, hist, M_v, M_x, k, mrow, kv_idx + out * K_max, kv_cnt + out);
  }
}
static size_t ss_lds(int M_v) { return (size_t(SS_WAVES) * 256 + size_t(M_v) * SS_STRIDE) * sizeof(uint32_t); }
// Where the one kernel is the faster of the two ways: a wave selects 4 / R .. 1 rows one after the other, and every 32 query
// sub-blocks read all key tiles.  Time of the two kernels over that of the one, whole refresh calls in bf16 on one card:
//   R = 8, d = 64: 16 blocks x 8 heads 1.30, 48 x 40 1.07, 200 x 8 1.04, 200 x 40 1.03, 313 x 1 1.09, 313 x 8 0.98;
//          d = 128: 16 x 8 1.23, 88 x 40 0.99, 200 x 8 1.02, 200 x 40 1.00, 313 x 8 0.97
//   R = 4, d = 64: 24 x 8 1.13, 138 x 48 1.00, 200 x 8 1.03, 313 x 1 1.08, 313 x 40 1.00; d = 128: 24 x 8 1.10, 138 x 40 1.00, 313 x 8 1.01, 313 x 40 1.00
//   R = 2, d = 64: 8 x 8 1.12, 48 x 8 1.03, 72 x 8 1.01, 138 x 1 0.96; d = 128: 24 x 8 1.04, 48 x 8 1.00, 72 x 8 0.99
//   R = 1: 8 x 8 1.04, 16 x 8 0.99 (d = 64) and 1.02 (128), 24 x 8 0.95 and 0.97, 138 x 1 0.78
bool score_small(const dfs_geom* g, const dfs_sizes& s) { return s.M_v <= ss_columns(s.r, g->d); }   // at 320, R = 4, 52 KB of the 64 KB of LDS

// Workspace: Q_hat, K_hat (two fp16 planes each, followed by the inverse scales of their row groups),
// T [heads][t_rows][t_cols] fp32 (padded, see t_cols), row log-sum-exp [heads][KSPLIT_MAX][M_s] fp32.
constexpr int KSPLIT_MAX = 4;
static size_t ws_planes_bytes(const dfs_geom* g, const dfs_sizes& s) { return align256(size_t(g->heads) * s.M_s * 2 * g->d * sizeof(uint16_t)); }
static size_t ws_hat_bytes(const dfs_geom* g, const dfs_sizes& s) {
  return ws_planes_bytes(g, s) + align256(size_t(g->heads) * ((s.M_s + 3) / 4) * sizeof(float));
}
static size_t ws_tt_bytes(const dfs_geom* g, const dfs_sizes& s) {
  return align256(size_t(g->heads) * t_rows(s.M_s, s.r) * t_cols(s.M_s) * sizeof(float));
}
static size_t ws_lse_bytes(const dfs_geom* g, const dfs_sizes& s) { return align256(size_t(g->heads) * KSPLIT_MAX * s.M_s * sizeof(float)); }
size_t ws_block_score(const dfs_geom* g, const dfs_sizes& s) {
  return 2 * ws_hat_bytes(g, s) + ws_tt_bytes(g, s) + ws_lse_bytes(g, s);
}

// Key ranges per query group: the split that wastes the least of the last round of work-groups
// (512 work-groups of 4 waves are resident on the chip at two waves per SIMD).
static int choose_ksplit(int64_t groups_times_heads, int n_tiles) {
  int best = 1;
  double best_cost = 1e300;
  for (int k = 1; k <= KSPLIT_MAX; ++k) {
    const int per = (n_tiles + k - 1) / k;
    const int64_t wgs = groups_times_heads * k;
    const int64_t rounds = (wgs + 511) / 512;
    const double cost = double(rounds) * (per + 2);       // +2: prologue / epilogue of a work-group, in tile units
    if (cost < best_cost - 1e-9) { best_cost = cost; best = k; }
  }
  return best;
}

template <int D, int R>
static void launch_score(const dfs_geom* g, const dfs_sizes& s, const uint16_t* q_hat, const uint16_t* k_hat, const float* q_down,
                         const float* k_down, float* tt, float* lse, float* score, const SelectPlan* sel, int n_live, hipStream_t st) {
  if (score_small(g, s)) {
    const int rows = 32 / R, n_rows = sel ? s.M : s.M_v;
    score_small_kernel<D, R><<<dim3(unsigned((n_rows + rows - 1) / rows), unsigned(g->heads)), SS_T, ss_lds(s.M_v), st>>>(
        q_hat, k_hat, q_down, k_down, sel ? nullptr : score, s.M_s, s.M_v, s.M_x, n_live, sel ? sel->k_fixed : 0, sel ? sel->k_cap : 0,
        sel ? sel->mass : 0.0, sel ? sel->mask : nullptr, sel ? sel->kv_idx : nullptr, sel ? sel->kv_cnt : nullptr, sel ? sel->K_max : 0,
        sel ? sel->k_head : nullptr);
    return;
  }
  const int groups = (s.M_s + 127) / 128, n_tiles = (n_live + 31) / 32;
  const int ksplit = choose_ksplit(int64_t(groups) * g->heads, n_tiles);
  const int per = (n_tiles + ksplit - 1) / ksplit;
  const int wgs_per_head = groups * ksplit;
  const int64_t total = int64_t(wgs_per_head) * g->heads;
  const int per_xcd = int((total + 7) / 8);
  score_lse_kernel<D, R><<<dim3(unsigned(per_xcd * 8)), 256, 0, st>>>(q_hat, k_hat, q_down, k_down, tt, lse, s.M_s, n_live, per, ksplit,
                                                                      wgs_per_head, int(total), per_xcd);
  if (sel) {
    fold_select_kernel<R><<<dim3(unsigned((s.M + FS_ROWS - 1) / FS_ROWS), unsigned(g->heads)), FS_T, fs_lds(s.M_v), st>>>(
        tt, lse, s.M_s, s.M_v, s.M_x, n_live, ksplit, sel->k_fixed, sel->k_cap, sel->mass, sel->mask, sel->kv_idx, sel->kv_cnt, sel->K_max, sel->k_head);
    return;
  }
  const unsigned tb = unsigned((s.M_v + 31) / 32);
  score_fold_kernel<R><<<dim3(tb, tb, unsigned(g->heads)), 256, 0, st>>>(tt, lse, score, s.M_s, s.M_v, n_live, ksplit);
}

bool can_select_in_fold(const dfs_sizes& s, int mode) { return mode != DFS_SELECT_MASS_HEAD && fs_lds(s.M_v) <= 65536; }

// Where a wave pools four sub-blocks: rows that it can have in flight together, and enough groups to fill the chip with as long waves
// all the same.  Measured (us, one sub-block a wave -> four): pooling under the profiler, 17 550 tokens x 48 heads, d = 64, sub-blocks of 32, 42.6 -> 35.4,
// 2 565 x 12, of 16, 5.5 -> 5.1, 75 600 x 40, d = 128, of 32, 272 -> 272 (HBM); refresh steps: 38 400 x 5, d = 64, of 32, 138.8 -> 134.5, 7 200 x 6, d = 128, of
// 8, 58.0 -> 55.6, 1 024 x 8, d = 64, of 16 (128 groups), 16.1 -> 16.6, 3 072 x 8, d = 128, of 64, 27.6 -> 31.2.
static bool pool_reads_groups(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* k_out) {
  return dtype == DFS_BF16 && !k_out && g->Bs <= 32 && int64_t(g->heads) * ((s.M_s + 3) / 4) >= 384;
}

int run_block_score(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* q_perm, const void* k_perm, float* score,
                    void* ws, const int32_t* index, bool k_src, void* k_out, const void* v, void* v_out, int32_t* zero, int n_zero, const SelectPlan* sel,
                    hipStream_t st) {
  if (g->heads > 65535) return fail(DFS_ESHAPE, "heads=%d exceeds 65535", g->heads);
  if ((s.M_v + 31) / 32 > 65535) return fail(DFS_ESHAPE, "M_v=%d is too large for the scoring grid", s.M_v);
  char* base = static_cast<char*>(ws);
  uint16_t* q_hat = reinterpret_cast<uint16_t*>(base);
  uint16_t* k_hat = reinterpret_cast<uint16_t*>(base + ws_hat_bytes(g, s));
  float* q_down = reinterpret_cast<float*>(base + ws_planes_bytes(g, s));
  float* k_down = reinterpret_cast<float*>(base + ws_hat_bytes(g, s) + ws_planes_bytes(g, s));
  float* tt = reinterpret_cast<float*>(base + 2 * ws_hat_bytes(g, s));
  float* lse = reinterpret_cast<float*>(base + 2 * ws_hat_bytes(g, s) + ws_tt_bytes(g, s));
  const int64_t pool_subs = k_out ? s.N_pad / g->Bs : s.M_s;   // with k_out (and v_out) the text blocks are copied as well
  dim3 pg(unsigned((pool_subs + 3) / 4), unsigned(g->heads), v_out ? 3 : 2);
  const bool bf = dtype == DFS_BF16;
  // 1/sqrt(d) of Eq. 2 and the change to base 2 go into Q_hat, so that the logits come out of the contraction in base 2
  const float scale = 1.4426950408889634f / sqrtf(float(g->d));
#define POOL(BF, DD) pool_kernel<BF, DD><<<pg, 256, 0, st>>>(q_perm, k_perm, v, q_hat, k_hat, q_down, k_down, index, k_out, v_out, s.N, s.N_pad, s.N_v, g->Bs, s.M_s, scale, score_small(g, s), k_src, zero, n_zero)
#define POOL_READ(DD) pool_read_kernel<DD><<<dim3(unsigned(((s.M_s + 3) / 4 + 3) / 4), unsigned(g->heads), 2), 256, 0, st>>>(static_cast<const uint16_t*>(q_perm), static_cast<const uint16_t*>(k_perm), q_hat, k_hat, q_down, k_down, index, s.N, s.N_pad, s.N_v, g->Bs, s.M_s, scale, score_small(g, s), k_src, zero, n_zero)
  if (pool_reads_groups(g, s, dtype, k_out)) { if (g->d == 64) POOL_READ(64); else POOL_READ(128); }
  else if (g->d == 64) { if (bf) POOL(true, 64); else POOL(false, 64); }
  else                 { if (bf) POOL(true, 128); else POOL(false, 128); }
#undef POOL_READ
#undef POOL
  const int n_live = int((s.N_v + g->Bs - 1) / g->Bs);
#define SCORE(DD, RR) launch_score<DD, RR>(g, s, q_hat, k_hat, q_down, k_down, tt, lse, score, sel, n_live, st)
#define SCORE_R(DD)                                                                 \
  switch (s.r) {                                                                    \
    case 1: SCORE(DD, 1); break;                                                    \
    case 2: SCORE(DD, 2); break;                                                    \
    case 4: SCORE(DD, 4); break;                                                    \
    case 8: SCORE(DD, 8); break;                                                    \
    default: return fail(DFS_ESHAPE, "B/Bs=%d is not 1, 2, 4 or 8", s.r);           \
  }
  if (g->d == 64) { SCORE_R(64) } else { SCORE_R(128) }
#undef SCORE_R
#undef SCORE
  return launch_status("dfs_block_score");
}

}  // namespace dfs

using namespace dfs;

extern "C" int dfs_block_score(const dfs_geom* g, int dtype, const void* q_perm, const void* k_perm, float* score, void* ws,
                               size_t ws_bytes, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (dtype != DFS_F32 && dtype != DFS_BF16) return fail(DFS_EDTYPE, "dtype %d is not DFS_F32 or DFS_BF16", dtype);
  if (!q_perm || !k_perm || !score) return fail(DFS_EINVAL, "dfs_block_score: NULL argument");
  if (misaligned(16, {q_perm, k_perm}) || misaligned(4, {score})) return fail(DFS_EINVAL, "dfs_block_score: tensors must be 16-byte aligned, the score array 4-byte aligned");
  const size_t need = ws_block_score(g, s);
  if (!ws || (uintptr_t(ws) & 255) || ws_bytes < need)
    return fail(DFS_EWORKSPACE, "dfs_block_score: workspace of %zu bytes needed (256-byte aligned), got %zu", need, ws_bytes);
  return run_block_score(g, s, dtype, q_perm, k_perm, score, ws, nullptr, false, nullptr, nullptr, nullptr, nullptr, 0, nullptr, as_stream(stream));
}

extern "C" int dfs_block_score_src(const dfs_geom* g, int dtype, const void* q, const int32_t* perm_pad, const void* k_perm,
                                   float* score, void* ws, size_t ws_bytes, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (dtype != DFS_BF16) return fail(DFS_EDTYPE, "dfs_block_score_src: bf16 tensors only");
  if (!q || !perm_pad || !k_perm || !score) return fail(DFS_EINVAL, "dfs_block_score_src: NULL argument");
  if (misaligned(16, {q, k_perm}) || misaligned(4, {perm_pad, score}))
    return fail(DFS_EINVAL, "dfs_block_score_src: tensors must be 16-byte aligned, index and score arrays 4-byte aligned");
  const size_t need = ws_block_score(g, s);
  if (!ws || (uintptr_t(ws) & 255) || ws_bytes < need)
    return fail(DFS_EWORKSPACE, "dfs_block_score_src: workspace of %zu bytes needed (256-byte aligned), got %zu", need, ws_bytes);
  return run_block_score(g, s, dtype, q, k_perm, score, ws, perm_pad, false, nullptr, nullptr, nullptr, nullptr, 0, nullptr, as_stream(stream));
}

extern "C" int dfs_block_score_fused(const dfs_geom* g, int dtype, const void* q, const void* k, const int32_t* perm_pad,
                                     void* k_perm, float* score, void* ws, size_t ws_bytes, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (dtype != DFS_BF16) return fail(DFS_EDTYPE, "dfs_block_score_fused: bf16 tensors only");
  if (!q || !k || !perm_pad || !k_perm || !score) return fail(DFS_EINVAL, "dfs_block_score_fused: NULL argument");
  if (misaligned(16, {q, k, k_perm}) || misaligned(4, {perm_pad, score}))
    return fail(DFS_EINVAL, "dfs_block_score_fused: tensors must be 16-byte aligned, index and score arrays 4-byte aligned");
  if (k == k_perm) return fail(DFS_EINVAL, "dfs_block_score_fused: k_perm must not alias k");
  const size_t need = ws_block_score(g, s);
  if (!ws || (uintptr_t(ws) & 255) || ws_bytes < need)
    return fail(DFS_EWORKSPACE, "dfs_block_score_fused: workspace of %zu bytes needed (256-byte aligned), got %zu", need, ws_bytes);
  return run_block_score(g, s, dtype, q, k, score, ws, perm_pad, true, k_perm, nullptr, nullptr, nullptr, 0, nullptr, as_stream(stream));
}
