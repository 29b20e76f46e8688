// Token permutation by 3D Hilbert index (paper Sec. 5.1; Algorithm 1 step 1) and by the other
// traversal orders of the ablation in Sec. 6.3.
//
// No keys are sorted or counted.  A token's rank among the cells of the grid has a closed form under every
// order: walking down the levels of the curve, the cells that come before it are those of the sibling octants the
// curve visits earlier, and an octant clipped by the grid holds the product of its three clipped extents.  So one
// kernel without scratch memory gives perm, inverse and block sizes.  75 600 tokens take 5.8 us, of which the launch
// is half; the six kernels before (keys marked in a bitmap over the enclosing cube, its prefix sum in three launches,
// keys turned into ranks) took 26 us with the gaps between them, the call as a whole now 6.2.  Run once per geometry.
#include "common.h"

namespace dfs {

// Rank of cell x among the cells of the grid [0, dim[0]) x ... in ascending order of their Hilbert index: the Butz
// curve in Skilling's transpose form on the enclosing cube of 2^b cells per axis, axis 0 the high bit of a digit.
// At level j the bits of the cell are read through the axis order and reflections that the levels above left
// behind (a set bit reflects axis 0 below this level, a clear one exchanges axis 0 with that axis); their running
// parities, all inverted where `fix` says so, are the digit of the index, and a set digit bit means that the whole
// half of the sub-cube with that bit clear comes before the cell.
template <int N>
__device__ __forceinline__ uint32_t hilbert_rank(uint32_t (&x)[N], uint32_t (&dim)[N], int b) {
  uint32_t flip[N] = {};
  uint32_t fix = 0, rank = 0;
  for (int j = b - 1; j >= 0; --j) {
    const uint32_t side = 1u << j;
    uint32_t bit[N], mine[N], other[N];             // extents inside the grid of the half with this cell and of its sibling
#pragma unroll
    for (int a = 0; a < N; ++a) {
      const uint32_t raw = (x[a] >> j) & 1u;
      const uint32_t room = dim[a] - ((x[a] >> j) >> 1 << (j + 1));             // > 0: the cell itself is inside
      const uint32_t lower = room < side ? room : side, rest = room - lower;
      const uint32_t upper = rest < side ? rest : side;
      mine[a] = raw ? upper : lower;
      other[a] = raw ? lower : upper;
      bit[a] = raw ^ flip[a];
    }
    uint32_t parity = 0, same = 1;                   // same: cells that agree with this one on the axes before
#pragma unroll
    for (int a = 0; a < N; ++a) {
      parity ^= bit[a];
      uint32_t before = same * other[a];
#pragma unroll
      for (int c = a + 1; c < N; ++c) before *= mine[c] + other[c];
      rank += (parity ^ fix) ? before : 0u;
      same *= mine[a];
    }
    fix ^= parity;
#pragma unroll
    for (int a = 0; a < N; ++a) {
      if (bit[a]) {
        flip[0] ^= 1u;
      } else {
        uint32_t tmp = x[0]; x[0] = x[a]; x[a] = tmp;
        tmp = dim[0]; dim[0] = dim[a]; dim[a] = tmp;
        tmp = flip[0]; flip[0] = flip[a]; flip[a] = tmp;
      }
    }
  }
  return rank;
}

// Rank of video token n (< 2^23, see check_geom) under a traversal order:
//   hilbert3d  3D Hilbert index of (t,h,w) in the enclosing cube (Sec. 5.1)
//   raster     n itself (per-frame row-major, the model's own order)
//   hilbert2d  frame index, then the 2D Hilbert index of (h,w) (ablation of Sec. 6.3)
//   block3d    4x4x4 cubes in raster order of the cubes, raster inside a cube (ablation of Sec. 6.3)
__device__ __forceinline__ uint32_t token_rank(uint32_t n, int order, uint32_t T, uint32_t H, uint32_t W, int b, int b2) {
  const uint32_t w = n % W, th = n / W;
  const uint32_t t = th / H, h = th % H;
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
__global__ void __launch_bounds__(256) token_order_kernel(uint32_t N_v, int n_text, int order, int T, int H, int W, int b, int b2, int B,
                                                          int M_v, int64_t N_pad, int32_t* __restrict__ perm_pad,
                                                          int32_t* __restrict__ inv, int32_t* __restrict__ blk_valid) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < N_v) {
    const uint32_t rank = token_rank(i, order, uint32_t(T), uint32_t(H), uint32_t(W), b, b2);
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
  token_order_kernel<<<dim3(unsigned((s.N_pad + 255) / 256)), 256, 0, st>>>(uint32_t(s.N_v), g->n_text, order, g->T, g->H, g->W, s.bits, b2,
                                                                          g->B, s.M_v, s.N_pad, perm_pad, inv, blk_valid);
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
