// Block-mask selection (paper Eq. 9) and the cumulative-mass keep count.
//
// One wave owns one (head, query block) row of scores.  Scores are mapped to 32-bit keys whose
// unsigned order is the float order; the k-th largest key is found a byte at a time from the top (four
// histogram passes over the row in LDS), ties at the threshold are resolved towards the lower
// column index, and the kept columns are written in ascending order with ballot prefix sums.
// Everything is integer work on the bit patterns, so the result is exactly the total order
// "higher score first, equal scores by lower index".
#include <math.h>

#include <mutex>

#include "select_row.h"

namespace dfs {

// Scratch of dfs_select_mask_static: the per-row and per-head keep counts of the mass modes live here instead
// of in a caller-supplied workspace.  One copy per GPU, held until the process ends.  Host code never uses the
// symbol's name as an address: the device address is resolved once per device (static_scratch below).
constexpr size_t STATIC_SCRATCH_BYTES = size_t(1) << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

// k_row[head, u] = fewest top-ranked columns whose fixed-point scores reach ceil(mass * row total).
__global__ void __launch_bounds__(64) mass_count_kernel(const float* __restrict__ score, int M_v, double mass,
                                                        int32_t* __restrict__ k_row) {
  extern __shared__ unsigned long long lds[];
  uint32_t* keys = reinterpret_cast<uint32_t*>(lds + 64);
  const int lane = threadIdx.x;
  const float* row = score + (int64_t(blockIdx.y) * M_v + blockIdx.x) * M_v;
  for (int j = lane; j < M_v; j += 64) keys[j] = order_key(row[j]);
  wave_sync();
  const int k = mass_count_row(keys, lds, M_v, mass);
  if (lane == 0) k_row[int64_t(blockIdx.y) * M_v + blockIdx.x] = k;
}

// k_head[h] = clamp(max(ceil(mean_u k_row[h,u]), k_floor), 1, k_cap)
__global__ void __launch_bounds__(256) head_count_kernel(const int32_t* __restrict__ k_row, int M_v, int k_floor, int k_cap,
                                                         int32_t* __restrict__ k_used, int32_t* __restrict__ k_head_out) {
  __shared__ unsigned long long part[4];
  unsigned long long s = 0;
  for (int u = threadIdx.x; u < M_v; u += 256) s += uint32_t(k_row[int64_t(blockIdx.x) * M_v + u]);
  s = wave_sum_u64(s);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long tot = part[0] + part[1] + part[2] + part[3];
    int k = int((tot + M_v - 1) / M_v);
    if (k < k_floor) k = k_floor;
    if (k > k_cap) k = k_cap;
    if (k < 1) k = 1;
    k_used[blockIdx.x] = k;
    if (k_head_out) k_head_out[blockIdx.x] = k;
  }
}

// Top-k of one row.  k is `k_fixed`, or k_per_head[head], or clamp(k_per_row[head, u], k_fixed, k_cap).
__global__ void __launch_bounds__(64) select_kernel(const float* __restrict__ score, int M_v, int M_x, int k_fixed,
                                                    const int32_t* __restrict__ k_per_head, const int32_t* __restrict__ k_per_row,
                                                    int k_cap, uint8_t* __restrict__ mask,
                                                    int32_t* __restrict__ kv_idx, int32_t* __restrict__ kv_cnt, int K_max,
                                                    int32_t* __restrict__ k_head_out) {
  extern __shared__ uint32_t keys[];
  const int lane = threadIdx.x;
  const int head = blockIdx.y, u = blockIdx.x;
  const int M = M_v + M_x;
  const int64_t out = int64_t(head) * M + u;
  uint8_t* mrow = mask ? mask + out * M : nullptr;
  if (u >= M_v) {
    select_text_row(M, mrow, kv_cnt + out);
    return;
  }
  int k = k_per_head ? k_per_head[head] : k_fixed;
  if (k_per_row) {
    const int ku = k_per_row[int64_t(head) * M_v + u];
    k = ku < k_fixed ? k_fixed : (ku > k_cap ? k_cap : ku);
  }
  if (k_head_out && !k_per_head && !k_per_row && u == 0 && lane == 0) k_head_out[head] = k;
  const float* row = score + (int64_t(head) * M_v + u) * M_v;
  for (int j = lane; j < M_v; j += 64) keys[j] = order_key(row[j]);
  wave_sync();
  select_row(keys, keys + M_v, M_v, M_x, k, mrow, kv_idx + out * K_max, kv_cnt + out);
}

size_t ws_select_mask(const dfs_geom* g, const dfs_sizes& s) {
  return align256(size_t(g->heads) * s.M_v * sizeof(int32_t)) + align256(size_t(g->heads) * sizeof(int32_t));
}

int check_select(const dfs_geom* g, const dfs_sizes& s, int mode, double sparsity, double mass, int32_t K_max) {
  if (mode != DFS_SELECT_TOPK && mode != DFS_SELECT_MASS_HEAD && mode != DFS_SELECT_MASS_ROW)
    return fail(DFS_EINVAL, "dfs_select_mask: unknown mode %d", mode);
  if (!(sparsity >= 0.0 && sparsity <= 1.0)) return fail(DFS_EINVAL, "dfs_select_mask: sparsity %g is outside [0,1]", sparsity);
  if (g->heads > 65535) return fail(DFS_ESHAPE, "heads=%d exceeds 65535", g->heads);
  if (s.M_v > 16128) return fail(DFS_ESHAPE, "dfs_select_mask: M_v=%d exceeds 16128 (one score row and a histogram must fit in 64 KB of LDS)", s.M_v);
  const int k_base = dfs_keep_count(sparsity, s.M_v);
  if (K_max < k_base + s.M_x)
    return fail(DFS_ESHAPE, "dfs_select_mask: K_max=%d is below the %d kept blocks per row", K_max, k_base + s.M_x);
  if (mode != DFS_SELECT_TOPK && !(mass > 0.0 && mass <= 1.0)) return fail(DFS_EINVAL, "dfs_select_mask: mass %g is outside (0,1]", mass);
  return DFS_OK;
}

int run_select_mask(const dfs_geom* g, const dfs_sizes& s, const float* score, int mode, double sparsity, double mass,
                    uint8_t* mask, int32_t* kv_idx, int32_t* kv_cnt, int32_t K_max, int32_t* k_head, void* ws,
                    hipStream_t st) {
  const int rc = check_select(g, s, mode, sparsity, mass, K_max);
  if (rc) return rc;
  const int k_base = dfs_keep_count(sparsity, s.M_v);
  const size_t lds = size_t(s.M_v) * sizeof(uint32_t) + 64 * sizeof(uint64_t);       // one key per column and the mass bins
  const size_t lds_sel = size_t(s.M_v) * sizeof(uint32_t) + 256 * sizeof(uint32_t);  // ... or the byte histogram
  dim3 rows(unsigned(s.M), unsigned(g->heads));
  if (mode == DFS_SELECT_TOPK) {
    select_kernel<<<rows, 64, lds_sel, st>>>(score, s.M_v, s.M_x, k_base, nullptr, nullptr, 0, mask, kv_idx, kv_cnt, K_max, k_head);
  } else {
    int32_t* k_row = static_cast<int32_t*>(ws);
    int32_t* k_used = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + align256(size_t(g->heads) * s.M_v * sizeof(int32_t)));
    int k_cap = K_max - s.M_x;
    if (k_cap > s.M_v) k_cap = s.M_v;
    mass_count_kernel<<<dim3(unsigned(s.M_v), unsigned(g->heads)), 64, lds, st>>>(score, s.M_v, mass, k_row);
    if (mode == DFS_SELECT_MASS_HEAD) {
      head_count_kernel<<<dim3(unsigned(g->heads)), 256, 0, st>>>(k_row, s.M_v, k_base, k_cap, k_used, k_head);
      select_kernel<<<rows, 64, lds_sel, st>>>(score, s.M_v, s.M_x, 0, k_used, nullptr, 0, mask, kv_idx, kv_cnt, K_max, nullptr);
    } else {
      select_kernel<<<rows, 64, lds_sel, st>>>(score, s.M_v, s.M_x, k_base, nullptr, k_row, k_cap, mask, kv_idx, kv_cnt, K_max, nullptr);
    }
  }
  return launch_status("dfs_select_mask");
}

// Device address of `scratch` on the current device, resolved on the first call per device and kept.
static int static_scratch(void** out) {
  constexpr int MAX_DEV = 64;
  static std::mutex mu;
  static void* addr[MAX_DEV] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(DFS_EHIP, "dfs_select_mask_static: hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= MAX_DEV) return fail(DFS_EHIP, "dfs_select_mask_static: device ordinal %d is outside [0,%d)", dev, MAX_DEV);
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(DFS_EHIP, "dfs_select_mask_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
    addr[dev] = p;
  }
  *out = addr[dev];
  return DFS_OK;
}

}  // namespace dfs

using namespace dfs;

extern "C" int dfs_select_mask_static(const dfs_geom* g, const float* score, int mode, double sparsity, double mass, uint8_t* mask,
                                      int32_t* kv_idx, int32_t* kv_cnt, int32_t K_max, int32_t* k_head, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (!score || !kv_idx || !kv_cnt) return fail(DFS_EINVAL, "dfs_select_mask_static: NULL argument");
  if (misaligned(4, {score, kv_idx, kv_cnt, k_head})) return fail(DFS_EINVAL, "dfs_select_mask_static: score, list and count arrays must be 4-byte aligned");
  const size_t need = ws_select_mask(g, s);
  if (need > STATIC_SCRATCH_BYTES)
    return fail(DFS_EWORKSPACE, "dfs_select_mask_static: heads x M_v = %d x %d needs %zu bytes of scratch, the built-in buffer holds %zu; "
                                "use dfs_select_mask with a workspace", g->heads, s.M_v, need, STATIC_SCRATCH_BYTES);
  void* ws = nullptr;
  if ((rc = static_scratch(&ws))) return rc;
  return run_select_mask(g, s, score, mode, sparsity, mass, mask, kv_idx, kv_cnt, K_max, k_head, ws, as_stream(stream));
}

extern "C" int dfs_select_mask(const dfs_geom* g, const float* score, int mode, double sparsity, double mass, uint8_t* mask,
                               int32_t* kv_idx, int32_t* kv_cnt, int32_t K_max, int32_t* k_head, void* ws, size_t ws_bytes,
                               void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (!score || !kv_idx || !kv_cnt) return fail(DFS_EINVAL, "dfs_select_mask: NULL argument");
  if (misaligned(4, {score, kv_idx, kv_cnt, k_head})) return fail(DFS_EINVAL, "dfs_select_mask: score, list and count arrays must be 4-byte aligned");
  const size_t need = ws_select_mask(g, s);
  if ((mode == DFS_SELECT_MASS_HEAD || mode == DFS_SELECT_MASS_ROW) && (!ws || (uintptr_t(ws) & 255) || ws_bytes < need))
    return fail(DFS_EWORKSPACE, "dfs_select_mask: workspace of %zu bytes needed (256-byte aligned), got %zu", need, ws_bytes);
  return run_select_mask(g, s, score, mode, sparsity, mass, mask, kv_idx, kv_cnt, K_max, k_head, ws, as_stream(stream));
}
