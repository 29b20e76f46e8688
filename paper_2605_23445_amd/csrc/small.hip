// A refresh step of a small fp32 problem in one kernel: pooling, scoring, selection and attention (paper Algorithm 1, steps 2 and 3).
// Three kernels behind one another, each four to nine microseconds, are mostly launches and chains of dependent loads, and most of the
// chip stands idle in all of them.  A work-group therefore does everything that its 32 query rows need: it pools the keys of its head and
// its own query block, scores and selects that block's row, and attends.  What it repeats of other work-groups' work (the pooled
// keys, once per work-group; the row, once per 32 query rows of a block) costs less than the two launches as long as a head is small; see
// forward_small_fits.  The same sums in the same order as the kernels of their own, so the same lists and the same output, bit for bit.
// 256 tokens x 2 heads, d = 64: 16.4 -> 12.4 us.
#include "attn_f32.h"
#include "score_small.h"
#include "select_row.h"

namespace dfs {

// The most of a head: video tokens times d (256 KB of keys), sub-blocks, rows in the order, blocks; of a sub-block: tokens times d.
constexpr int FS_NUMEL = 65536, FS_SUBS = 64, FS_ROWS_MAX = 2048, FS_BLOCKS = FS_ROWS_MAX / 64, FS_SUB = 8192;

template <int D> struct SmallRoom {                   // LDS
  static constexpr int V_BLOCKS = FS_NUMEL / D / 64;
  union {
    struct {
      __attribute__((aligned(16))) uint16_t k[FS_SUBS * 2 * D], q[8 * 2 * D];                // centroids in operand order; of at most 8 query sub-blocks
      float k_inv[FS_SUBS / 4], q_inv[2];
      float t[V_BLOCKS * SS_STRIDE], m[SS_WAVES][32], z[SS_WAVES][32], ref[32], inv[32];
      __attribute__((aligned(8))) uint32_t hist[256];
    } score;
    AttnF32Room<D, true> attn;
  };
  int32_t pos[FS_ROWS_MAX];                            // source row of every row of the order, -1 for none
  int32_t list[FS_BLOCKS], cnt;
};

// One wave: the centroids of groups first, first + step, ... < groups, four sub-blocks each, as pool_kernel forms them, the same sums in the same
// order.  A group's rows are requested while the group before is finished.  rows_of(g): the tensor's head and the factor; put(g, sb, c, up, hi, lo):
// features 4 c .. 4 c + 3 of sub-block sb of the group, and inverse(g, x).
template <int D, class Rows, class Sub, class Put, class Inverse>
__device__ __forceinline__ void pool_groups(int first, int step, int groups, const int32_t* pos, int N_v, int Bs, Rows rows_of, Sub sub_of, Put put,
                                            Inverse inverse) {
  constexpr int TPR = D / 4, RPP = 64 / TPR, AHEAD = 4, OWN = 4 / RPP;   // lanes per row, rows per pass, passes in flight of each sub-block, sub-blocks a lane ends with
  const int lane = threadIdx.x & 63, c = lane % TPR, rg = lane / TPR;
  f32x4 val[4][AHEAD];
  auto ask = [&](int g, int i0) {
    float factor;
    const float* x = rows_of(g, factor);
    const int s0 = sub_of(g);
    int from[4][AHEAD];
#pragma unroll
    for (int sb = 0; sb < 4; ++sb)
#pragma unroll
      for (int p = 0; p < AHEAD; ++p) {
        const int i = i0 + rg + p * RPP, row = (s0 + sb) * Bs + i;
        from[sb][p] = i < Bs && row < N_v ? pos[row] : -1;
      }
#pragma unroll
    for (int sb = 0; sb < 4; ++sb)
#pragma unroll
      for (int p = 0; p < AHEAD; ++p) {
        val[sb][p] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (from[sb][p] >= 0) val[sb][p] = *reinterpret_cast<const f32x4*>(x + int64_t(from[sb][p]) * D + 4 * c);
      }
  };
  if (first < groups) ask(first, 0);
  for (int g = first; g < groups; g += step) {
    float acc[4][4];
#pragma unroll
    for (int sb = 0; sb < 4; ++sb)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[sb][e] = 0.f;
    for (int i0 = 0; i0 < Bs; i0 += RPP * AHEAD) {
#pragma unroll
      for (int sb = 0; sb < 4; ++sb)
#pragma unroll
        for (int p = 0; p < AHEAD; ++p)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[sb][e] += val[sb][p][e];       // zeros change no sum that starts from zero
      if (i0 + RPP * AHEAD < Bs) ask(g, i0 + RPP * AHEAD);
      else if (g + step < groups) ask(g + step, 0);
    }
    // sums over the row groups: lanes of row group rg end with sub-block rg (d = 64), or rg and 2 + rg (d = 128)
    float own[OWN][4], mx[OWN], factor;
    rows_of(g, factor);
#pragma unroll
    for (int w = 0; w < OWN; ++w) {
      const int sb = w * RPP + rg, left = N_v - (sub_of(g) + sb) * Bs, cnt = left < Bs ? left : Bs;
      const float by = cnt > 0 ? factor / float(cnt) : 0.f;
      mx[w] = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        own[w][e] = RPP == 4 ? sum_32(sum_16(acc[0][e], acc[1][e]), sum_16(acc[2][e], acc[3][e])) : sum_32(acc[2 * w][e], acc[2 * w + 1][e]);
        own[w][e] *= by;
        mx[w] = fmaxf(mx[w], fabsf(own[w][e]));
      }
      mx[w] = max_of_16(mx[w]);
    }
    float up, down;
    group_scale(max_32(max_16(OWN == 1 ? mx[0] : fmaxf(mx[0], mx[OWN - 1]))), up, down);
    if (lane == 0) inverse(g, down);
#pragma unroll
    for (int w = 0; w < OWN; ++w) {
      uint16_t hi[4], lo[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) split2(own[w][e] * up, hi[e], lo[e]);
      typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
      put(g, w * RPP + rg, c, u32x2{uint32_t(hi[0]) | (uint32_t(hi[1]) << 16), uint32_t(hi[2]) | (uint32_t(hi[3]) << 16)},
          u32x2{uint32_t(lo[0]) | (uint32_t(lo[1]) << 16), uint32_t(lo[2]) | (uint32_t(lo[3]) << 16)});
    }
  }
}

// Centroids in LDS; the query sub-blocks are rows 0 .. 7 of a tile of eight.
template <int D> struct RoomOperands {
  const uint16_t *qh, *kh;
  const float *q_inv, *k_inv;
  int M_s;
  __device__ __forceinline__ f16x8 q(int p, int c, int n) const {        // rows beyond the eighth repeat it; nothing reads their results
    return __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(qh + chunk_at<D>(p, c, 8, n < 8 ? n : 7)));
  }
  __device__ __forceinline__ float q_inverse(int n) const { return q_inv[n < 4 ? 0 : 1]; }
  __device__ __forceinline__ f16x8 k(int t, int p, int c, int n) const {
    const int rows = tile_rows(M_s, t);
    return __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(kh + tile_at<D>(t) + chunk_at<D>(p, c, rows, n < rows ? n : rows - 1)));
  }
  __device__ __forceinline__ float k_inverse(int grp) const {
    const int G4 = (M_s + 3) / 4;
    return k_inv[grp < G4 ? grp : G4 - 1];
  }
};

template <int D, int R>
__global__ void __launch_bounds__(SS_T) forward_small_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                             const int32_t* __restrict__ row_index, float* __restrict__ o, int N, int N_v, int n_text,
                                                             int M_v, int M, int B, int n_live, float q_scale, int k_fixed, int k_cap, double mass,
                                                             uint8_t* __restrict__ mask, int32_t* __restrict__ kv_idx,
                                                             int32_t* __restrict__ kv_cnt, int K_max, int32_t* __restrict__ k_head, float scale) {
  __shared__ SmallRoom<D> room;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int parts = B / 32, head = blockIdx.y, u = M - 1 - int(blockIdx.x) / parts, part = int(blockIdx.x) % parts;
  const int64_t out = int64_t(head) * M + u;
  uint8_t* mrow = mask && part == 0 ? mask + out * M : nullptr;
  for (int i = tid; i < M * B; i += SS_T) {
    const int at = row_index[i];
    room.pos[i] = at < N ? at : -1;
  }
  __syncthreads();
  QueryRow<D> query;                                          // requested here, used at the end
  query.load(q, N, head, room.pos[u * B + part * 32 + (lane & 31)]);
  if (u < M_v) {
    auto& x = room.score;
    const int Bs = B / R, M_s = M_v * R, i0 = u * R & ~3, q_groups = (R + 3) / 4, k_groups = (M_s + 3) / 4;
    const float *qh = q + int64_t(head) * N * D, *kh = k + int64_t(head) * N * D;
    pool_groups<D>(
        wave, SS_WAVES, q_groups + k_groups, room.pos, N_v, Bs,
        [&](int g, float& factor) {
          factor = g < q_groups ? q_scale : 1.0f;
          return g < q_groups ? qh : kh;
        },
        [&](int g) { return g < q_groups ? i0 + 4 * g : 4 * (g - q_groups); },
        [&](int g, int sb, int c, auto hi, auto lo) {
          const int s = 4 * (g - q_groups) + sb, rows = g < q_groups ? 8 : tile_rows(M_s, s / 32);
          if (g >= q_groups && s >= M_s) return;
          uint16_t* at = g < q_groups ? x.q + chunk_at<D>(0, c / 2, 8, 4 * g + sb) : x.k + tile_at<D>(s / 32) + chunk_at<D>(0, c / 2, rows, s % 32);
          at += c % 2 * 4;
          *reinterpret_cast<decltype(hi)*>(at) = hi;
          *reinterpret_cast<decltype(lo)*>(at + chunk_at<D>(1, 0, rows, 0)) = lo;
        },
        [&](int g, float inverse) { (g < q_groups ? x.q_inv + g : x.k_inv + g - q_groups)[0] = inverse; });
    __syncthreads();
    small_scores<D, R>(RoomOperands<D>{x.q, x.k, x.q_inv, x.k_inv, M_s}, x.t, x.m, x.z, x.ref, x.inv, M_v, n_live, i0);
    if (wave == 0) {
      const int first = u * R - i0;
      if (lane < M_v) {
        float* t = x.t + lane * SS_STRIDE + first;
        const float score = small_score<R>(t, x.ref + first, x.inv + first);
        *reinterpret_cast<uint32_t*>(t) = order_key(score);
      }
      wave_sync();
      const StridedKeys row = {reinterpret_cast<const uint32_t*>(x.t) + first, SS_STRIDE};
      int n = k_fixed;
      if (mass > 0.0) {                                      // every row its own count, clamped
        const int ku = mass_count_row(row, reinterpret_cast<unsigned long long*>(x.hist), M_v, mass);
        n = ku < k_fixed ? k_fixed : (ku > k_cap ? k_cap : ku);
      } else if (k_head && u == 0 && part == 0 && lane == 0) {
        k_head[head] = n;
      }
      select_row<16>(row, x.hist, M_v, M - M_v, n, mrow, room.list, &room.cnt);
    }
  } else if (wave == 0) {
    select_text_row(M, mrow, &room.cnt);
  }
  __syncthreads();
  const int cnt = __builtin_amdgcn_readfirstlane(room.cnt);
  if (part == 0) {
    if (tid == 0) kv_cnt[out] = cnt;
    if (u < M_v && tid < cnt) kv_idx[out * K_max + tid] = room.list[tid];
  }
  attn_f32_rows<D, true>(room.attn, query, k, v, [&](int i) { return __builtin_amdgcn_readfirstlane(room.list[i]); }, cnt, K_max, o, nullptr, N, [&](int64_t at) { return room.pos[at]; }, N,
                         int64_t(M) * B, N_v, n_text, M_v, M, B, scale, head, u, part);
}

// Small enough that what every work-group repeats costs less than the launches do, in one round of work-groups.  Measured (us, three kernels
// -> one, half the blocks kept; in brackets a first pass over new inputs, waited for, medians of 180): d = 64, 256 tokens x 2 heads 16.4 -> 12.4 (32.5 ->
// 27.7), x 8 18.0 -> 12.6 (34 -> 28.5), 512 + 40 x 1 26.5 -> 18.9 (42 -> 34), 512 x 8 with 64 sub-blocks 21.1 -> 19.4 (38 -> 34), 1 024 x 1 25.2 -> 24.8 (40.7 ->
// 40.1), x 4, blocks of 128, 26.9 -> 26.6 (43.4 -> 42.3), x 1 with 128 sub-blocks 22.6 -> 24.6; d = 128, 256 x 8 25.2 -> 22.5 (41.2 -> 38.3), 512 x 8
// 31.1 -> 30.7 (48 -> 48), x 1 29.2 -> 28.9 (44.0 -> 45.8).  Sub-blocks of 128 rows at d = 128, a wave's serial way through 64 KB, lose: 128 x 1 34.8 -> 36.2, 256 x 4
// 36.0 -> 37.1, 512 x 1 44.3 -> 45.5 (of 64 rows 35.4 -> 34.5, of 128 at d = 64 27.7 -> 24.8).  The output must not lie over the queries either, whose neighbours' rows a work-group
// pools where a block has fewer than four sub-blocks.
bool forward_small_fits(const dfs_geom* g, const dfs_sizes& s, int dtype, int mode, const void* q, const void* k, const void* v, const void* o) {
  return dtype == DFS_F32 && mode != DFS_SELECT_MASS_HEAD && s.N_v * g->d <= FS_NUMEL && s.M_s <= FS_SUBS && s.N_pad <= FS_ROWS_MAX && g->Bs * g->d <= FS_SUB && score_small(g, s) &&
         int64_t(g->heads) * s.M * (g->B / 32) <= 256 && apart(g, s, dtype, q, o) && apart(g, s, dtype, k, o) && apart(g, s, dtype, v, o);
}

int run_forward_small(const dfs_geom* g, const dfs_sizes& s, const void* q, const void* k, const void* v, const int32_t* perm_pad, const SelectPlan& sel,
                      float scale, void* o, hipStream_t st) {
  const int n_live = int((s.N_v + g->Bs - 1) / g->Bs);
  const float q_scale = 1.4426950408889634f / sqrtf(float(g->d));        // as run_block_score has it
  const dim3 grid(unsigned(s.M * (g->B / 32)), unsigned(g->heads));
#define SMALL(DD, RR)                                                                                                                          \
  forward_small_kernel<DD, RR><<<grid, SS_T, 0, st>>>(static_cast<const float*>(q), static_cast<const float*>(k), static_cast<const float*>(v), perm_pad, \
                                                      static_cast<float*>(o), int(s.N), int(s.N_v), g->n_text, s.M_v, s.M, g->B, n_live, q_scale,          \
                                                      sel.k_fixed, sel.k_cap, sel.mass, sel.mask, sel.kv_idx, sel.kv_cnt, sel.K_max, sel.k_head, scale)
#define SMALL_R(DD)                       \
  switch (s.r) {                          \
    case 1: SMALL(DD, 1); break;          \
    case 2: SMALL(DD, 2); break;          \
    case 4: SMALL(DD, 4); break;          \
    default: SMALL(DD, 8); break;         \
  }
  if (g->d == 64) { SMALL_R(64) } else { SMALL_R(128) }
#undef SMALL_R
#undef SMALL
  return launch_status("dfs_forward");
}

}  // namespace dfs
