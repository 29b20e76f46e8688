// Scoring of small problems (device code shared by the kernel behind the pooling and the one that pools, scores, selects and attends):
// layout and scaling of the centroids, and what a work-group of eight waves does for 32 query sub-blocks.
#pragma once
#include <math.h>

#include "common.h"

namespace dfs {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// x (already scaled so that its group's largest magnitude is in [2^11, 2^12)) -> (hi, lo) with hi = fp16(x),
// lo = fp16(x - hi).  The subtraction is exact and |x - hi| <= 2^-11 |x|, so x = hi + lo to within 2^-22 |x| as long
// as lo is a normal fp16 number, which it is for |x| >= 2^-3: an element more than 2^14 times smaller than the
// largest of its group is kept to 2^-25 absolute instead, i.e. to 2^-36 of that largest one.
__device__ __forceinline__ void split2(float x, uint16_t& hi, uint16_t& lo) {
  const _Float16 h = (_Float16)x;
  const _Float16 l = (_Float16)(x - (float)h);
  hi = __builtin_bit_cast(uint16_t, h);
  lo = __builtin_bit_cast(uint16_t, l);
}
// Rows are scaled in groups of four consecutive sub-blocks (the four waves of a pooling work-group) by a power of
// two that brings the group's largest magnitude into [2^11, 2^12); `down` is the inverse.  Powers of two: exact.
constexpr int SHIFT_MAX = 126;                 // keeps both factors finite and normal for groups of vanishing magnitude
                                               // (the largest finite fp32 needs a shift of -116)
__device__ __forceinline__ void group_scale(float gmax, float& up, float& down) {
  up = 1.0f; down = 1.0f;
  if (gmax > 0.f && gmax < INFINITY) {
    int ex;
    (void)frexpf(gmax, &ex);                   // gmax = m 2^ex, m in [0.5, 1)
    int sh = 12 - ex;
    sh = sh > SHIFT_MAX ? SHIFT_MAX : (sh < -SHIFT_MAX ? -SHIFT_MAX : sh);
    up = ldexpf(1.0f, sh);
    down = ldexpf(1.0f, -sh);
  }
}

// Layouts of Q_hat and K_hat.  For the two-kernel contraction, row after row, [2][D] fp16 (hi, lo planes).  For the one-kernel
// form (`tiled`), per head, tiles of 32 sub-blocks (the last one with what is left, `rows`), a tile chunk by chunk as
// the matrix instructions' operands want it, [2 D / 8][rows][8] fp16: chunks 0 .. D / 8 - 1 are features 8 c .. 8 c + 7 of the hi
// plane, the others of the lo plane.  The lanes of an operand load, one row each, then read a kilobyte
// in one piece; with whole rows behind one another they read 16 bytes of 32 rows: 2 565 tokens x 12 heads, d = 64, blocks of 64,
// 36.5 -> 35.5 us a refresh.  It costs the pooling, which writes rows of a tile in pieces of 64 bytes, 4 % where it is an HBM stream
// (75 600 tokens x 40 heads 399 -> 418 us for Q and K), and the two-kernel contraction, which goes through LDS, would gain 2 %
// (184 -> 181).
__host__ __device__ __forceinline__ int tile_rows(int M_s, int t) { return M_s - 32 * t < 32 ? M_s - 32 * t : 32; }
template <int D> __device__ __forceinline__ int64_t tile_at(int t) { return int64_t(t) * (32 * 2 * D); }      // elements
template <int D> __device__ __forceinline__ int chunk_at(int p, int c, int rows, int n) { return ((p * (D / 8) + c) * rows + n) * 8; }

constexpr float LSE_START = -1.0e30f;          // finite stand-in for "nothing seen yet" (keeps differences finite)

// The value of the other lane half (lane ^ 32) beside this lane's own, through the vector unit (a shuffle through
// LDS would make the wave wait for every LDS read in flight).  Returns {lower half's value, upper half's value}.
__device__ __forceinline__ void both_halves(float x, float& lo, float& hi) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(sw[0]);
  hi = __uint_as_float(sw[1]);
}

// x' and y' hold the lower and the upper lanes' (of 32, of 64) values of a pair: x' + y' is x summed over the pair in its lower lanes and y
// in its upper ones.
__device__ __forceinline__ float sum_16(float x, float y) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float sum_32(float x, float y) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float max_16(float x) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float max_32(float x) {
  float lo, hi;
  both_halves(x, lo, hi);
  return fmaxf(lo, hi);
}
template <int CTRL> __device__ __forceinline__ float dpp_max(float x) {
  return fmaxf(x, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), CTRL, 0xF, 0xF, true)));
}
__device__ __forceinline__ float max_of_16(float x) {        // over each row of sixteen lanes
  x = dpp_max<0xB1>(x);                                       // lanes 1 0 3 2
  x = dpp_max<0x4E>(x);                                       // lanes 2 3 0 1
  x = dpp_max<0x141>(x);                                      // eight, mirrored
  return dpp_max<0x140>(x);                                   // sixteen, mirrored
}

// Running base-2 log-sum-exp (reference m, sum z of 2^(x - m)): add one term, merge two partial sums.
__device__ __forceinline__ void lse_add(float& m, float& z, float x) {
  const float mn = fmaxf(m, x);
  z = z * __builtin_amdgcn_exp2f(m - mn) + __builtin_amdgcn_exp2f(x - mn);
  m = mn;
}
__device__ __forceinline__ void lse_merge(float& m, float& z, float m2, float z2) {
  const float mn = fmaxf(m, m2);
  z = z * __builtin_amdgcn_exp2f(m - mn) + z2 * __builtin_amdgcn_exp2f(m2 - mn);
  m = mn;
}

// Centroids in memory, in operand order: chunk c (eight features of plane p) of a row.
template <int D> struct MemoryOperands {
  const uint16_t *qh, *kh;
  const float *q_down, *k_down;
  int M_s, i0;
  __device__ __forceinline__ f16x8 q(int p, int c, int n) const {        // rows beyond the last repeat it; nothing reads their results
    const int from = i0 + n < M_s ? n : M_s - 1 - i0;
    return __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(qh + tile_at<D>(i0 / 32) + chunk_at<D>(p, c, tile_rows(M_s, i0 / 32), from)));
  }
  __device__ __forceinline__ float q_inverse(int n) const { return q_down[(i0 + n < M_s ? i0 + n : M_s - 1) / 4]; }
  __device__ __forceinline__ f16x8 k(int t, int p, int c, int n) const {                 // beyond the last: masked by the caller
    const int rows = tile_rows(M_s, t);
    return __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(kh + tile_at<D>(t) + (n < rows ? n : rows - 1) * 8 + chunk_at<D>(p, c, rows, 0)));
  }
  __device__ __forceinline__ float k_inverse(int grp) const {
    const int G4 = (M_s + 3) / 4;
    return k_down[grp < G4 ? grp : G4 - 1];
  }
};

// Key blocks up to which one kernel scores a head behind the pooling, see score_small.
__host__ __device__ constexpr int ss_columns(int r, int d) { return r == 8 ? 256 : r == 4 ? 320 : r == 2 ? 4096 / d : 12; }

// T of the query sub-blocks i0 .. i0 + 31 of a head, [M_v][SS_STRIDE] in LDS, and their references and inverse sums: the waves take key
// tiles in turn.  Ends behind a barrier.
constexpr int SS_T = 512, SS_WAVES = SS_T / 64, SS_STRIDE = 33;
template <int D, int R, class Operands>
__device__ __forceinline__ void small_scores(const Operands& x, float* s_t, float (*s_m)[32], float (*s_z)[32], float* s_ref, float* s_inv, int M_v,
                                             int n_live, int i0) {
  constexpr int KS = D / 16;
  constexpr int G = R < 4 ? R : 4, NG = 16 / G;            // as in score_lse_kernel
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, half = lane >> 5;
  const float q_dn = x.q_inverse(n);
  f16x8 bq[2][KS];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) bq[p][kk] = x.q(p, 2 * kk + half, n);
  float m_row = LSE_START, z_row = 0.f;
  // At d = 64 a tile's operands are requested as soon as the matrix instructions have taken those of the tile before, in front of its
  // exponentials; at d = 128 the registers that this takes would leave a CU one work-group instead of two.  Rows of R <= 2 are at most a
  // tile for each wave: without room for a next one R = 1 takes 88 registers instead of 139, two work-groups a CU instead of one (us a launch, 12
  // blocks x 1 024 heads 20.8 -> 14.7, x 512 10.4 -> 7.7, x 200 5.9 -> 6.1; with no operand ahead of its use 17.5, 9.1 and 7.5).
  constexpr bool AHEAD = D == 64, ONE = AHEAD && ss_columns(R, D) * R <= 32 * SS_WAVES;
  f16x8 ak[2][KS];
  float k_dn[4];
  auto ask = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) ak[p][kk] = x.k(t, p, 2 * kk + half, n);
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) k_dn[gq] = x.k_inverse(8 * t + 2 * gq + half);
  };
  if (AHEAD && wave * 32 < n_live) ask(wave);
  if (ONE) __builtin_amdgcn_sched_barrier(0);          // all of them, not in turn with the products
  for (int t = wave; t * 32 < n_live; t += SS_WAVES) {
    if (!AHEAD) ask(t);
    float dn[4];
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) dn[gq] = k_dn[gq] * q_dn;
    f32x16 c0, c1;
#pragma unroll
    for (int i = 0; i < 16; ++i) { c0[i] = 0.f; c1[i] = 0.f; }
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {                    // hi.hi, hi.lo, lo.hi, dealt to the accumulators as there
      f32x16& a = kk % 2 ? c1 : c0;
      f32x16& b = kk % 2 ? c0 : c1;
      a = __builtin_amdgcn_mfma_f32_32x32x16_f16(ak[0][kk], bq[0][kk], a, 0, 0, 0);
      b = __builtin_amdgcn_mfma_f32_32x32x16_f16(ak[0][kk], bq[1][kk], b, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_32x32x16_f16(ak[1][kk], bq[0][kk], a, 0, 0, 0);
    }
    if (AHEAD && !ONE) {
      if ((t + SS_WAVES) * 32 < n_live) ask(t + SS_WAVES);
      __builtin_amdgcn_sched_barrier(0);
    }
    float c[16], mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      c[i] = (c0[i] + c1[i]) * dn[i / 4];
      if (t * 32 + 8 * (i / 4) + 4 * half + (i % 4) >= n_live) c[i] = -INFINITY;
      mt = fmaxf(mt, c[i]);
    }
    if (R == 8) {                                        // a key block is split over the lane halves: one reference
      float lo, hi;
      both_halves(mt, lo, hi);
      mt = fmaxf(lo, hi);
    }
    const float m_new = fmaxf(m_row, mt);
    z_row *= __builtin_amdgcn_exp2f(m_row - m_new);
    m_row = m_new;
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      float sg = 0.f;
#pragma unroll
      for (int e = 0; e < G; ++e) sg += __builtin_amdgcn_exp2f(c[gi * G + e] - m_new);
      z_row += sg;
      if (R == 8) {
        float lo, hi;
        both_halves(sg, lo, hi);
        sg = lo + hi;
      }
      const int first = gi * G, v = (t * 32 + 8 * (first / 4) + (R == 8 ? 0 : 4 * half) + first % 4) / R;
      if (v < M_v) s_t[v * SS_STRIDE + n] = m_new + __builtin_amdgcn_logf(sg);  // R == 8: both halves store the same
    }
    if (ONE) break;
  }
  const float m2 = __shfl_xor(m_row, 32, 64), z2 = __shfl_xor(z_row, 32, 64);
  lse_merge(m_row, z_row, m2, z2);
  if (half == 0) {
    s_m[wave][n] = m_row;
    s_z[wave][n] = z_row;
  }
  __syncthreads();
  if (tid < 32) {
    float m = s_m[0][tid], z = s_z[0][tid];
#pragma unroll
    for (int w = 1; w < SS_WAVES; ++w) {
      if (w * 32 >= n_live) break;                         // a wave without tiles: nothing to add
      lse_merge(m, z, s_m[w][tid], s_z[w][tid]);
    }
    // Reference and sum stay apart: their log-sum-exp in one number, of magnitude log2(M_s) and more, would be rounded by up
    // to 2^-21 there (error of the scores, 2-norm: 2.8e-7 at 688 sub-blocks, the two kernels with their key ranges 1.6e-7).
    const bool any = i0 + tid < n_live && z > 0.f;                                         // an empty query sub-block scores nothing
    s_ref[tid] = any ? m : INFINITY;
    s_inv[tid] = any ? 1.f / z : 0.f;
  }
  __syncthreads();
}

// The score of a query block from T, its references and inverse sums at its first query sub-block.
template <int R>
__device__ __forceinline__ float small_score(const float* t, const float* ref, const float* inv) {
  float acc = 0.f;
#pragma unroll
  for (int a = 0; a < R; ++a) acc = fmaf(__builtin_amdgcn_exp2f(t[a] - ref[a]), inv[a], acc);
  return acc;
}

}  // namespace dfs
