// Internal helpers shared by the HIP translation units of libdfsattn (not part of the ABI).
#pragma once
#include <initializer_list>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/dfsattn.h"

namespace dfs {

constexpr int MAX_BLOCKS = 65536;                   // of a sequence (check_geom): at most 2^23 rows

// Records `msg` as the calling thread's last error and returns `code`.
int fail(int code, const char* fmt, ...);
// Validates a geometry (sets the error on failure) and fills the derived sizes.
int check_geom(const dfs_geom* g, dfs_sizes* s);
// Turns the error state left by a kernel launch into a status code.
int launch_status(const char* what);

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
// Tensor rows move 16 bytes at a time, so every Q/K/V/O tensor must start on a 16-byte boundary
// (index, count and fp32 arrays on a 4-byte boundary).  True if any of the pointers does not.
inline bool misaligned(size_t a, std::initializer_list<const void*> ps) {
  for (const void* p : ps)
    if (reinterpret_cast<uintptr_t>(p) & (a - 1)) return true;
  return false;
}
inline int elem_size(int dtype) { return dtype == DFS_BF16 ? 2 : 4; }

// Stage entry points without argument checks, used by dfs_forward after it has validated once.
// x2, x2_perm (may be NULL): a second tensor, reordered in the same launch.  n_zero words at `zero` are cleared.
int run_permute(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* x, const int32_t* perm_pad,
                void* x_perm, const void* x2, void* x2_perm, int32_t* zero, int n_zero, hipStream_t st);
// What the selection of a row needs when the scoring does it on the way: the keep count, or with mass > 0 its bounds.
struct SelectPlan {
  int k_fixed, k_cap;
  double mass;
  uint8_t* mask;
  int32_t *kv_idx, *kv_cnt;
  int32_t K_max;
  int32_t* k_head;
};
// index (may be NULL): the permutation; Q is then read in source order and gathered while pooling, and so is K with k_src.
// With k_out (which needs k_src) K is written out reordered on the way, and so is V with v_out (which needs k_out).  n_zero words at
// `zero` are cleared on the way.  With sel the block lists are written instead of the scores (`score` may be NULL then).
int run_block_score(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* q_perm, const void* k_perm,
                    float* score, void* ws, const int32_t* index, bool k_src, void* k_out, const void* v, void* v_out, int32_t* zero,
                    int n_zero, const SelectPlan* sel, hipStream_t st);
// Whether one kernel scores a problem of this size behind the pooling.
bool score_small(const dfs_geom* g, const dfs_sizes& s);
// A refresh step of a small fp32 problem in one kernel, and whether a call is one.
bool forward_small_fits(const dfs_geom* g, const dfs_sizes& s, int dtype, int mode, const void* q, const void* k, const void* v, const void* o);
int run_forward_small(const dfs_geom* g, const dfs_sizes& s, const void* q, const void* k, const void* v, const int32_t* perm_pad, const SelectPlan& sel,
                      float scale, void* o, hipStream_t st);
// Whether the scoring can select on the way: the rule needs one row's scores only and eight rows fit in 64 KB of LDS.
bool can_select_in_fold(const dfs_sizes& s, int mode);
int check_select(const dfs_geom* g, const dfs_sizes& s, int mode, double sparsity, double mass, int32_t K_max);
int run_select_mask(const dfs_geom* g, const dfs_sizes& s, const float* score, int mode, double sparsity,
                    double mass, uint8_t* mask, int32_t* kv_idx, int32_t* kv_cnt, int32_t K_max,
                    int32_t* k_head, void* ws, hipStream_t st);
// row_index (may be NULL): Q and O in source order, and K and V as well with kv_src.  scratch (may be NULL): room to split text rows
// over work-groups; its first split_tickets() words are zero when the kernel starts, already (zeroed) or by a launch of its own.
int run_sparse_attn(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* q, const void* k, const void* v,
                    const int32_t* kv_idx, const int32_t* kv_cnt, int32_t K_max, float scale, void* o, float* lse,
                    const int32_t* row_index, bool kv_src, bool maybe_dense, bool zeroed, void* scratch, size_t scratch_bytes, hipStream_t st);
// Whether two tensors in source order have no byte in common.
bool apart(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* a, const void* b);
// Whether dfs_forward hands the attention K and V in source order (kv_src above) instead of reordering them.
bool attn_reads_source(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* k, const void* v, const void* o);
// One per text block, and with 512 query blocks and more one for each that the last round of work-groups may share (at most 127
// per XCD).
inline size_t split_tickets(const dfs_geom* g, const dfs_sizes& s) {
  return size_t(g->heads) * s.M_x + (int64_t(g->heads) * s.M >= 512 ? 8 * 128 : 0);
}
int run_unperm(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* o_perm, const int32_t* inv, void* o,
               hipStream_t st);
size_t ws_block_score(const dfs_geom* g, const dfs_sizes& s);
size_t ws_select_mask(const dfs_geom* g, const dfs_sizes& s);
size_t ws_hilbert(const dfs_geom* g, const dfs_sizes& s);

// bf16 <-> fp32 on raw bits (round to nearest even on the way down)
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(uint32_t(b) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}

}  // namespace dfs
