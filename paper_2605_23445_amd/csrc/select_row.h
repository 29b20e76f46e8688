// One wave's selection over one row of block scores held as ordered keys in LDS (device code shared by the kernels that
// read the scores from memory and the one that forms them).
#pragma once
#include "common.h"

namespace dfs {

constexpr int MASS_FRAC_BITS = 24;

__device__ __forceinline__ uint32_t order_key(float s) {
  uint32_t b = __float_as_uint(s);
  if (b == 0x80000000u) b = 0u;                     // -0 ranks with +0
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t key) {             // the score of a key (+0 for -0)
  return __uint_as_float((key & 0x80000000u) ? key & 0x7FFFFFFFu : ~key);
}

__device__ __forceinline__ unsigned long long mass_fixed(float s) {
  const double c = fmin(fmax(double(s), 0.0), 4096.0);   // NaN clamps to 0
  return static_cast<unsigned long long>(c * double(1 << MASS_FRAC_BITS));
}

__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long v, int from) {
  const uint32_t lo = __shfl(uint32_t(v), from, 64), hi = __shfl(uint32_t(v >> 32), from, 64);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += shfl_u64(v, (threadIdx.x & 63) ^ off);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Orders a wave's LDS accesses among its own lanes.  The LDS serves a wave in order, so the compiler is all that has to
// be held back; no other wave touches the row.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

struct StridedKeys {                                 // a row whose keys lie `stride` words apart
  const uint32_t* first;
  int stride;
  __device__ __forceinline__ uint32_t operator[](int j) const { return first[j * stride]; }
};

// Fewest top-ranked columns whose fixed-point scores reach ceil(mass * row total).  The column at which the sum from
// the top reaches the target is found six bits of its key at a time: a 64-bin histogram of the masses of the keys that
// match the bits fixed so far, one bin per lane, and a scan over the lanes.  Integers throughout, so the result does
// not depend on any order.  (One bit per pass, each with a sum over the row: 355 us at 75 600 tokens x 40 heads and
// reading the scores again; this form 101.)
// (keys: a pointer, or whatever else gives the key of column j as keys[j].)
template <class Keys>
__device__ __forceinline__ int mass_count_row(Keys keys, unsigned long long* bins /*[64]*/, int M_v, double mass) {
  const int lane = threadIdx.x & 63;
  unsigned long long tot = 0;
  for (int j = lane; j < M_v; j += 64) tot += mass_fixed(key_score(keys[j]));
  tot = wave_sum_u64(tot);
  const unsigned long long target = static_cast<unsigned long long>(ceil(mass * double(tot)));
  if (target == 0) return 1;
  uint32_t T = 0, fixed = 0;
  unsigned long long above = 0;                     // mass of the keys above those that match T on `fixed`
  for (int shift = 26; shift >= -4; shift -= 6) {
    const int down = shift < 0 ? 0 : shift;         // the last pass takes the two bits left
    const uint32_t field = shift < 0 ? 3u : 63u;
    bins[lane] = 0ull;
    wave_sync();
    for (int j = lane; j < M_v; j += 64) {
      const uint32_t key = keys[j];
      const unsigned long long q = (key & fixed) == T ? mass_fixed(key_score(key)) : 0ull;
      if (q) atomicAdd(&bins[(key >> down) & field], q);
    }
    wave_sync();
    const unsigned long long mine = bins[63 - lane];                   // lane order is descending key order
    unsigned long long incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned long long up = shfl_u64(incl, lane - off < 0 ? lane : lane - off);
      if (lane >= off) incl += up;
    }
    const unsigned long long reached = __ballot(above + incl >= target);           // never empty: the sum reaches the target
    const int sel = __ffsll(reached) - 1;
    above += shfl_u64(incl - mine, sel);
    T |= uint32_t(63 - sel) << down;
    fixed |= field << down;
    wave_sync();                                                       // the bins are cleared next
  }
  uint32_t n_above = 0;
  for (int j = lane; j < M_v; j += 64) n_above += keys[j] > T ? 1u : 0u;
  n_above = wave_sum_u32(n_above);
  const unsigned long long at = mass_fixed(key_score(T)), need = target - above;   // both > 0 by choice of T
  return int(n_above + (need + at - 1) / at);
}

// The row in registers, NK keys a lane: the k-th largest key a bit at a time from the top, the count of the keys that reach it from ballots and scalar
// additions.  Then its kept columns in ascending order, ties at the threshold the lowest first.
template <int NK, class Keys>
__device__ __forceinline__ void select_in_registers(Keys keys, int M_v, int k, uint8_t* mrow, int32_t* idx) {
  const int lane = threadIdx.x & 63;
  uint32_t key[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) key[i] = 64 * i + lane < M_v ? keys[64 * i + lane] : 0u;     // zeros reach no threshold that is tried
  uint32_t T = 0;
  constexpr int BITS = NK <= 3 ? 2 : 1;                // two at a time where the chain from count to count is longer than the counting
  for (int shift = 32 - BITS; shift >= 0; shift -= BITS) {
    uint32_t digit = 0;                              // the counts fall from digit to digit
#pragma unroll
    for (uint32_t x = 1; x < 1u << BITS; ++x) {
      int reached = 0;
#pragma unroll
      for (int i = 0; i < NK; ++i) reached += __popcll(__ballot(key[i] >= (T | x << shift)));
      digit += reached >= k ? 1 : 0;
    }
    T |= digit << shift;
  }
  int above = 0;
#pragma unroll
  for (int i = 0; i < NK; ++i) above += __popcll(__ballot(64 * i + lane < M_v && key[i] > T));
  const unsigned long long below_me = (1ull << lane) - 1ull;
  int ties_left = k - above, written = 0;
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const int j = 64 * i + lane;
    const bool is_tie = j < M_v && key[i] == T;
    const unsigned long long ties = __ballot(is_tie);
    const bool keep = j < M_v && (key[i] > T || (is_tie && __popcll(ties & below_me) < ties_left));
    const unsigned long long kept = __ballot(keep);
    if (keep) idx[written + __popcll(kept & below_me)] = j;
    if (mrow && j < M_v) mrow[j] = keep ? 1 : 0;
    ties_left -= __popcll(ties) < ties_left ? __popcll(ties) : ties_left;
    written += __popcll(kept);
  }
}

// Top-k of a row: kept columns in ascending order into idx, the text blocks behind them, the mask row if there is one.
// Rows of up to 640 columns are selected in registers.  In longer ones the k-th largest key is found a byte at a time from the top: a 256-bin
// histogram of the next byte of the keys that still match the bytes fixed so far, then the bin in which the count from the top
// reaches what is still wanted; counts are integers, so it is the same key.
// With the histogram for rows of more than 64 columns and a rank of every column below (us a launch, under the profiler): 41 columns x 12 heads with
// the scoring 7.6 -> 6.2, 138 x 48 35.0 -> 31.2 (d = 64, with the operands ahead), 591 x 40 with the fold 78 -> 72.
// Where the lines lie (histogram -> registers, with the fold, x 24 heads): seven keys a lane 330 columns 22.1 -> 20.6, 360 28.8 -> 25.5, 448 36.3
// -> 31.9 (ten: 24.4, 29.4, 35.8, so up to 360 slower than the histogram); ten 470 41.3 -> 39.3, 576 41.9 -> 37.6, 640 48.3 -> 42.6.  Fifteen would lose
// again at 704 (x 40 heads 106 -> 108, x 8 31 -> 33) and win at 929 (97 -> 89 in 18 ms).
// MOST: rows have no more columns than that, LEAST: they have more (the ways for longer and shorter ones are left out).
template <int MOST = 1 << 30, int LEAST = 0, class Keys>
__device__ __forceinline__ void select_row(Keys keys, uint32_t* hist /*[256]*/, int M_v, int M_x, int k, uint8_t* mrow,
                                           int32_t* idx, int32_t* cnt) {
  const int lane = threadIdx.x & 63;
  for (int j = lane; j < M_x; j += 64) {             // text key blocks are always kept
    idx[k + j] = M_v + j;
    if (mrow) mrow[M_v + j] = 1;
  }
  if (lane == 0) *cnt = k + M_x;
  if (LEAST < 16 && (MOST <= 16 || M_v <= 16)) {                   // ranked outright, each lane counting the columns ahead of its own
    const uint32_t key = lane < M_v ? keys[lane] : 0u;
    int ahead = 0;
    for (int i0 = 0; i0 < M_v; i0 += 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e;
        const uint32_t other = keys[i < M_v ? i : M_v - 1];
        ahead += i < M_v && (other > key || (other == key && i < lane)) ? 1 : 0;
      }
    }
    const bool keep = lane < M_v && ahead < k;
    const unsigned long long kept = __ballot(keep);
    if (keep) idx[__popcll(kept & ((1ull << lane) - 1ull))] = lane;
    if (mrow && lane < M_v) mrow[lane] = keep ? 1 : 0;
    return;
  }
  if (LEAST < 64 && (MOST <= 64 || M_v <= 64)) return select_in_registers<1>(keys, M_v, k, mrow, idx);
  if (LEAST < 192 && M_v <= 192) return select_in_registers<3>(keys, M_v, k, mrow, idx);
  if (LEAST < 320 && (MOST <= 320 || M_v <= 320)) return select_in_registers<5>(keys, M_v, k, mrow, idx);
  if (M_v <= 448) return select_in_registers<7>(keys, M_v, k, mrow, idx);
  if (M_v <= 640) return select_in_registers<10>(keys, M_v, k, mrow, idx);
  uint32_t T = 0, fixed = 0, want = uint32_t(k);      // want: rank of the key looked for among the keys matching T on `fixed`
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int b = lane; b < 256; b += 64) hist[b] = 0u;
    wave_sync();
    for (int j = lane; j < M_v; j += 64) {
      const uint32_t key = keys[j];
      if ((key & fixed) == T) atomicAdd(&hist[(key >> shift) & 255u], 1u);
    }
    wave_sync();
    // lane l owns bins 255 - 4 l .. 252 - 4 l, so that lane order is descending key order
    uint32_t c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = hist[255 - 4 * lane - i];
    const uint32_t mine = c[0] + c[1] + c[2] + c[3];
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
    const unsigned long long reached = __ballot(incl >= want);     // never empty: at least `want` keys match
    const int sel = __ffsll(reached) - 1;
    uint32_t left = want - (incl - mine), digit = 0u;              // meaningful in lane `sel` only
#pragma unroll
    for (int i = 3; i >= 0; --i) {                                 // the first bin (from the top) whose running count reaches `left`
      const uint32_t before = (i > 0 ? c[0] : 0u) + (i > 1 ? c[1] : 0u) + (i > 2 ? c[2] : 0u);
      if (before < left && left <= before + c[i]) digit = uint32_t(255 - 4 * lane - i) | ((left - before) << 8);
    }
    digit = __shfl(digit, sel, 64);
    T |= (digit & 255u) << shift;
    want = digit >> 8;
    fixed |= 255u << shift;
    wave_sync();                                                   // the histogram is cleared next
  }
  const uint32_t ties_wanted = want;                               // lowest-index columns equal to T; the k - want keys above T are all kept
  uint32_t ties_seen = 0, written = 0;
  const unsigned long long below_me = (1ull << lane) - 1ull;
  for (int j0 = 0; j0 < M_v; j0 += 64) {
    const int j = j0 + lane;
    const uint32_t key = j < M_v ? keys[j] : 0u;
    const bool is_tie = j < M_v && key == T;
    const unsigned long long tie_ballot = __ballot(is_tie);
    const uint32_t tie_rank = ties_seen + __popcll(tie_ballot & below_me);
    const bool keep = j < M_v && (key > T || (is_tie && tie_rank < ties_wanted));
    const unsigned long long keep_ballot = __ballot(keep);
    if (keep) idx[written + __popcll(keep_ballot & below_me)] = j;
    if (mrow && j < M_v) mrow[j] = keep ? 1 : 0;
    ties_seen += __popcll(tie_ballot);
    written += __popcll(keep_ballot);
  }
}

// A text query block: keeps every key block.
__device__ __forceinline__ void select_text_row(int M, uint8_t* mrow, int32_t* cnt) {
  const int lane = threadIdx.x & 63;
  if (mrow)
    for (int j = lane; j < M; j += 64) mrow[j] = 1;
  if (lane == 0) *cnt = M;
}

}  // namespace dfs
