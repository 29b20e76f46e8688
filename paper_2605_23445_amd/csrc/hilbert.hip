// Token permutation by 3D Hilbert index (paper Sec. 5.1; Algorithm 1 step 1) and by the other
// traversal orders of the ablation in Sec. 6.3.
//
// No keys are sorted or counted.  A token's rank among the cells of the grid has a closed form under every
// order: walking down the levels of the curve, the cells that come before it are those of the sibling octants the
// curve visits earlier, and an octant clipped by the grid holds the product of its three clipped extents.  So one
// kernel without scratch memory gives perm, inverse and block sizes.  75 600 tokens take 3.4 us a launch among
// others in a graph, of which the launch itself is half, and 3.6 us a call from Python, whose host side is then the longer
// one; the six kernels before (keys marked in a bitmap over the enclosing cube, its prefix sum in three launches, keys turned
// into ranks) took 26 us with the gaps between them.  Run once per geometry.
#include "common.h"

namespace dfs {

// Rank of cell x among the cells of the grid [0, dim[0]) x ... in ascending order of their Hilbert index: the Butz
// curve in Skilling's transpose form on the enclosing cube of 2^b cells per axis, axis 0 the high bit of a digit.
// At level j the bits of the cell are read through the axis order and reflections that the levels above left
// behind (a set bit reflects axis 0 below this level, a clear one exchanges axis 0 with that axis); their parity,
// running over the axes and the levels, is the next bit of the index, and a set one means that the whole half of the
// sub-cube with that bit clear comes before the cell.
// A wave is alone on its SIMD here (75 600 tokens are 1 182 waves) and issues a vector instruction every eight cycles or so, so
// what bounds the kernel is their number, some fifty a level: an axis keeps its coordinate and the reflected one in one word, which is
// exchanged in one piece, and the extent of the present sub-cube inside the grid, which is halved with it; volumes are at most
// 2^23, their factors at most 2^18, so the products are 24-bit ones, at four times the rate.  With the extents worked out anew from
// the grid, reflections apart and 32-bit products and divisions a launch among others in a graph took 4.11 us, now 3.39 (75 600
// tokens; 64 tokens 1.96 and 1.76).
template <int N>
__device__ __forceinline__ uint32_t hilbert_rank(const uint32_t (&x)[N], const uint32_t (&dim)[N], int b) {
  constexpr int REFLECTED = 16;                      // first bit of the reflected coordinate
  uint32_t w[N], ext[N];
#pragma unroll
  for (int a = 0; a < N; ++a) {
    w[a] = x[a] | x[a] << REFLECTED;
    ext[a] = dim[a];
  }
  uint32_t digit = 0, rank = 0;                      // digit: bit of the index, running over the axes and levels
  for (int j = b - 1; j >= 0; --j) {
    const uint32_t side = 1u << j;
    bool bit[N];
    uint32_t mine[N], before[N];                     // extents of the half with this cell, and of the other if that comes first
#pragma unroll
    for (int a = 0; a < N; ++a) {
      bit[a] = (w[a] >> (REFLECTED + j)) & 1u;
      digit ^= bit[a];
      const uint32_t lower = ext[a] < side ? ext[a] : side;
      mine[a] = (w[a] >> j) & 1u ? ext[a] - lower : lower;
      before[a] = digit ? ext[a] - mine[a] : 0u;
    }
    uint32_t same = 1;                               // cells that agree with this one on the axes before
#pragma unroll
    for (int a = 0; a < N; ++a) {
      uint32_t v = same;
#pragma unroll
      for (int c = a + 1; c < N; ++c) v = __umul24(v, ext[c]);
      rank += __umul24(before[a], v);
      same = __umul24(same, mine[a]);
    }
#pragma unroll
    for (int a = 0; a < N; ++a) ext[a] = mine[a];
#pragma unroll
    for (int a = 0; a < N; ++a) {
      if (bit[a]) {
        w[0] ^= 0xFFFFu << REFLECTED;
      } else {
        uint32_t tmp = w[0]; w[0] = w[a]; w[a] = tmp;
        tmp = ext[0]; ext[0] = ext[a]; ext[a] = tmp;
      }
    }
  }
  return rank;
}

// Division of n < 2^23 (65 536 blocks, see check_geom) by d <= 512, by the high half of a product with ceil(2^32 / d): it exceeds
// 2^32 n / d by less than 2^23 x 512 / d, so that the floor is right.  0 stands for d = 1.
static uint32_t reciprocal(int d) { return d == 1 ? 0u : uint32_t((0x100000000ull + d - 1) / d); }
__device__ __forceinline__ uint32_t quotient(uint32_t n, uint32_t recip) { return recip ? __umulhi(n, recip) : n; }

// Rank of video token n under a traversal order:
//   hilbert3d  3D Hilbert index of (t,h,w) in the enclosing cube (Sec. 5.1)
//   raster     n itself (per-frame row-major, the model's own order)
//   hilbert2d  frame index, then the 2D Hilbert index of (h,w) (ablation of Sec. 6.3)
//   block3d    4x4x4 cubes in raster order of the cubes, raster inside a cube (ablation of Sec. 6.3)
__device__ __forceinline__ uint32_t token_rank(uint32_t n, int order, uint32_t T, uint32_t H, uint32_t W, uint32_t by_H, uint32_t by_W, int b, int b2) {
  const uint32_t th = quotient(n, by_W), w = n - __umul24(th, W);
  const uint32_t t = quotient(th, by_H), h = th - __umul24(t, H);
  switch (order) {
    case DFS_ORDER_RASTER: return n;
    case DFS_ORDER_HILBERT2D: {
      uint32_t x[2] = {h, w}, dim[2] = {H, W};
      return t * H * W + hilbert_rank<2>(x, dim, b2);
    }
    case DFS_ORDER_BLOCK3D: {
      const uint32_t t0 = t & ~3u, h0 = h & ~3u, w0 = w & ~3u;                   // the cube's corner and clipped extents
      const uint32_t nt = T - t0 < 4 ? T - t0 : 4, nh = H - h0 < 4 ? H - h0 : 4, nw = W - w0 < 4 ? W - w0 : 4;
      return (t0 * H + nt * h0) * W + nt * nh * w0 + ((t - t0) * nh + (h - h0)) * nw + (w - w0);
    }
    default: {
      uint32_t x[3] = {t, h, w}, dim[3] = {T, H, W};
      return hilbert_rank<3>(x, dim, b);
    }
  }
}

// Every video token writes itself at its rank; text tokens and pads are filled in beside them.
__global__ void __launch_bounds__(256) token_order_kernel(uint32_t N_v, int n_text, int order, int T, int H, int W, uint32_t by_H, uint32_t by_W, int b,
                                                          int b2, int B, int M_v, int64_t N_pad, int32_t* __restrict__ perm_pad,
                                                          int32_t* __restrict__ inv, int32_t* __restrict__ blk_valid) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < N_v) {
    const uint32_t rank = token_rank(i, order, uint32_t(T), uint32_t(H), uint32_t(W), by_H, by_W, b, b2);
    perm_pad[rank] = int32_t(i);
    inv[i] = int32_t(rank);
  }
  if (i < N_pad) {
    const uint32_t text_base = uint32_t(M_v) * uint32_t(B);
    if (i >= N_v && i < text_base) perm_pad[i] = -1;
    if (i >= text_base) {
      const int j = int(i - text_base);
      if (j < n_text) { perm_pad[i] = int32_t(N_v) + j; inv[int64_t(N_v) + j] = int32_t(i); }
      else perm_pad[i] = -1;
    }
    if (i % uint32_t(B) == 0) {
      const int64_t blk = i / uint32_t(B);
      int64_t real = blk < M_v ? int64_t(N_v) - blk * B : int64_t(n_text) - (blk - M_v) * B;
      blk_valid[blk] = int32_t(real > B ? B : (real < 0 ? 0 : real));
    }
  }
}

static inline int bits_for(int extent) {
  int b = 1;
  while ((1 << b) < extent) ++b;
  return b;
}

// The ranks need no scratch memory.  The size asked of callers is that of two bitmaps over the largest key space of
// an order and their chunk counts, which is what the interface has always asked for: a caller's buffer and what is
// refused stay the same.
// Number of key values an order can produce for a geometry (every token's key is below it).
static size_t key_space(const dfs_geom* g, const dfs_sizes& s, int order) {
  switch (order) {
    case DFS_ORDER_RASTER: return size_t(s.N_v);
    case DFS_ORDER_HILBERT2D: return size_t(g->T) << (2 * bits_for(g->H > g->W ? g->H : g->W));
    case DFS_ORDER_BLOCK3D: return size_t((g->T + 3) / 4) * ((g->H + 3) / 4) * ((g->W + 3) / 4) * 64;
    default: return size_t(1) << (3 * s.bits);
  }
}
static size_t ws_for_cells(size_t cells) {
  const size_t nw = (cells + 31) / 32, chunks = (nw + 255) / 256;
  return align256(nw * 4) * 2 + align256(chunks * 4);
}

size_t ws_hilbert(const dfs_geom* g, const dfs_sizes& s) {   // enough for every order
  size_t need = 0;
  for (int order = 0; order < 4; ++order) {
    const size_t w = ws_for_cells(key_space(g, s, order));
    need = w > need ? w : need;
  }
  return need;
}

static int run_token_order(const dfs_geom* g, const dfs_sizes& s, int order, int32_t* perm_pad, int32_t* inv, int32_t* blk_valid,
                           hipStream_t st) {
  const int b2 = bits_for(g->H > g->W ? g->H : g->W);
  token_order_kernel<<<dim3(unsigned((s.N_pad + 255) / 256)), 256, 0, st>>>(uint32_t(s.N_v), g->n_text, order, g->T, g->H, g->W, reciprocal(g->H),
                                                                          reciprocal(g->W), s.bits, b2, g->B, s.M_v, s.N_pad, perm_pad, inv, blk_valid);
  return launch_status("dfs_token_order");
}

}  // namespace dfs

using namespace dfs;

extern "C" int dfs_token_order(const dfs_geom* g, int order, int32_t* perm_pad, int32_t* inv, int32_t* blk_valid, void* ws,
                               size_t ws_bytes, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (order < DFS_ORDER_HILBERT3D || order > DFS_ORDER_BLOCK3D) return fail(DFS_EINVAL, "dfs_token_order: unknown order %d", order);
  if (!perm_pad || !inv || !blk_valid) return fail(DFS_EINVAL, "dfs_token_order: NULL output");
  const size_t need = ws_hilbert(g, s);
  if (!ws || (uintptr_t(ws) & 255) || ws_bytes < need)
    return fail(DFS_EWORKSPACE, "dfs_token_order: workspace of %zu bytes needed (256-byte aligned), got %zu", need, ws_bytes);
  return run_token_order(g, s, order, perm_pad, inv, blk_valid, as_stream(stream));
}

extern "C" int dfs_hilbert_perm(const dfs_geom* g, int32_t* perm_pad, int32_t* inv, int32_t* blk_valid, void* ws, size_t ws_bytes,
                                void* stream) {
  return dfs_token_order(g, DFS_ORDER_HILBERT3D, perm_pad, inv, blk_valid, ws, ws_bytes, stream);
}
