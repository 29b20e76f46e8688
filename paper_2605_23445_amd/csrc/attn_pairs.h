// Which query blocks attn_pairs_kernel takes, in which order, and which it leaves to the kernel behind it (rules alone, for host and device).
#pragma once

namespace dfs {

// A pair is two neighbouring video blocks of a head (the last one may be alone) or two text blocks.  Slots of an XCD: the text pairs of
// all heads in turn with the other XCDs, then its eighth of the video pairs of head 0, of head 1, ...  Its PAIR_WGS work-groups take a
// slot each per round; what lies behind the last full round is left over: fewer than PAIR_WGS pairs an XCD, and no text (an eighth of the
// video pairs of a head is a round and more, see pair_rounds).
// The eighths are not those of the kernel behind, which cuts a head's blocks: cut in the same way, an odd eighth has a pair of one block in every
// head and XCD, whose idle half costs the clock (600 blocks x 40 heads, all kept, 94.9 -> 98.3 ms, 929 + 2 x 24 137.5 -> 140.0).
// A head has (M - M_v + 1) / 2 text pairs; with that in a function of its own the compiler laid the registers of the pairs' loop out in another way (four heads
// of 591 blocks with log-sum-exp, all kept, 8.45 -> 8.69 ms).
constexpr int PAIR_WGS = 32;
__host__ __device__ __forceinline__ int pair_text_slots(int M_v, int M, int n_heads) { return (n_heads * ((M - M_v + 1) / 2) + 7) / 8; }
__host__ __device__ __forceinline__ int pair_chunk(int M_v) { return ((M_v + 1) / 2 + 7) / 8; }                        // video pairs of a head and XCD
__host__ __device__ __forceinline__ int pair_slots(int M_v, int M, int n_heads) { return pair_text_slots(M_v, M, n_heads) + n_heads * pair_chunk(M_v); }

// First block of the pair in a slot, -1 for none.
__host__ __device__ __forceinline__ int pair_at(int xcd, int slot, int M_v, int M, int n_heads, int& head) {
  const int XP = (M - M_v + 1) / 2, C = pair_chunk(M_v), text_slots = pair_text_slots(M_v, M, n_heads);
  if (slot < text_slots) {
    const int id = slot * 8 + xcd;
    head = XP > 0 ? id / XP : 0;
    return head < n_heads && XP > 0 ? M_v + 2 * (id % XP) : -1;
  }
  const int s2 = slot - text_slots, u = 2 * (xcd * C + s2 % C);
  head = s2 / C;
  return head < n_heads && u < M_v ? u : -1;
}
// First block of the pair that holds block u, and that pair's slot.
__host__ __device__ __forceinline__ int pair_of(int u, int M_v) { return u < M_v ? u & ~1 : M_v + ((u - M_v) & ~1); }
__host__ __device__ __forceinline__ int pair_slot(int head, int u, int M_v, int M, int n_heads) {
  const int C = pair_chunk(M_v);
  return u < M_v ? pair_text_slots(M_v, M, n_heads) + head * C + u / 2 % C : (head * ((M - M_v + 1) / 2) + (u - M_v) / 2) / 8;
}

}  // namespace dfs
