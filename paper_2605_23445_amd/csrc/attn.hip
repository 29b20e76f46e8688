// Block-sparse attention forward over the reordered sequence (paper Algorithm 1 step 3: Eq. 1
// restricted to the kept block pairs, softmax normalised over the kept keys).
//
// bf16 kernel (the hot one).  A work-group owns one query block of one head; each of its waves
// owns 32 query rows.  Key/value blocks named by kv_idx stream through LDS in tiles of 64 rows.
// Per tile a wave forms S^T = K Q^T on the matrix cores (32x32x16 bf16), so that every lane holds
// logits of ONE query row: the softmax reference and normaliser are per-lane scalars.  The probabilities, still in
// registers, are already laid out as the B operand of O^T += V^T P^T; the V^T operand comes out of
// LDS through the transposing LDS read, so V is stored row-major like K and never transposed in
// memory.
#include <float.h>
#include <math.h>
#include <type_traits>

#include "attn_f32.h"
#include "attn_pairs.h"

namespace dfs {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define LDS_PTR(T) __attribute__((address_space(3))) T*

constexpr int KN = 64;   // key rows per LDS tile

// XOR swizzles of the 16-byte chunks inside a tile row.  Tiles are stored without padding (the
// direct-to-LDS load writes 64 consecutive chunks per wave instruction); the swizzle, applied on the
// global side of the load and again on every LDS read, spreads the rows a wave reads at once over
// all banks.  K is read one row per lane (16 B each), V four rows x 64 B per half-wave pass.
template <int CH> __device__ __forceinline__ int swz_k(int row) { return (row / (16 / CH)) % CH; }
template <int CH> __device__ __forceinline__ int swz_v(int row) { return 4 * ((row / (16 / CH)) % (CH / 4)); }

constexpr int swz_period(int step, int mod) {    // smallest P with (P * step) % mod == 0
  int p = 1;
  while ((p * step) % mod != 0) ++p;
  return p;
}

// XLSE: the caller wants the log-sum-exp.  The normaliser of O sums the probabilities as rounded to bf16
// (see the row sums below), which is right for O but leaves ln(sum) off by up to bf16's unit roundoff 2^-8; with
// XLSE a second running sum of the unrounded fp32 probabilities is kept for the log-sum-exp alone.
//
// Waves per SIMD: two at d = 128 (about 250 registers each).  At d = 64 the kernel needs about 160 registers, so
// three waves fit (measured 36 -> 43 % of the matrix cycles, +8 % throughput on the 17 550- and 75 600-token
// shapes); the variants that would have to spill for that (64-row blocks, log-sum-exp output) stay at two.
//
// Text rows keep every block and are many times longer than the others; where too few of the others follow to hide
// them, SPLIT work-groups share one text block, each with a run of its list.  They leave their unnormalised sums in
// `part`; the one that takes the last ticket merges them, in list order, so the result does not depend on who is last.
// The query blocks of the last round of work-groups are shared in the same way where they would leave slots idle (tail_split),
// by an instance of its own (TAIL): the work behind it costs every work-group some 0.3 us on its way to the list.
// (Only calls without log-sum-exp are given a `part`.)
//
// KS: where the query blocks are too few to give every SIMD its two waves, KS groups of waves share one query block, each
// with a KS-th of its tiles, tile buffers of its own and a softmax of its own; they merge through LDS at the end.  A lone
// wave per SIMD reaches three fifths of the matrix rate, two together three quarters; see key_split below for the rule.
//
// SLIM (d = 128, 64 query rows): at 16 KB a tile, two buffers each for K and V leave room for two work-groups of two waves, one
// wave per SIMD.  With one buffer each, whose halves take turns, four work-groups fit; a half is then requested a stage
// ahead instead of a tile.  See `slim` below for the rule.
//
// SRC: keys and values come in source order, like the queries, and their tiles are gathered through row_index, so that nothing is
// reordered in front of the kernel.  The rows of a block are 64 times 128 or 256 contiguous bytes either way; what it costs
// is the lookup of positions and their way to the lanes.  See attn_reads_source below for the rule.
template <int D, int BM, bool XLSE, int KS>
constexpr int attn_waves() { return D == 64 && BM == 128 && !XLSE && KS == 1 ? 3 : 2; }
// Whether the pair's rows are dense.  Text rows always are; they go with the head's first video rows, so that they run beside what
// takes as long.
__device__ __forceinline__ bool pair_dense(const int32_t* __restrict__ kv_cnt, int head, int u, int M_v, int M) {
  const int32_t* cnt = kv_cnt + int64_t(head) * M;
  const int end = u < M_v ? M_v : M, v1 = M_v > 1 ? 1 : 0;
  return cnt[u] >= M && cnt[u + 1 < end ? u + 1 : u] >= M && (u < M_v || (cnt[0] >= M && cnt[v1] >= M));
}
// Whether a dense row is in such a pair in front of slot `end`.
__device__ __forceinline__ bool in_pairs(const int32_t* __restrict__ kv_cnt, int head, int u, int M_v, int M, int n_heads, int end) {
  return pair_slot(head, u, M_v, M, n_heads) < end && pair_dense(kv_cnt, head, pair_of(u, M_v), M_v, M);
}

// What a work-group does: the query block u of `head` (BM = 256: blocks u and u + 1, which keep every key block), or with TAIL and
// for text rows the share `split` of it; xcd and slot name it among the tail's.
template <int D, int BM, bool XLSE, int KS, bool SLIM, bool TAIL, bool SRC, bool REST>
__device__ __forceinline__ void
attn_rows(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
          const int32_t* __restrict__ kv_idx, const int32_t* __restrict__ kv_cnt, int K_max, uint16_t* __restrict__ o,
          float* __restrict__ lse, const int32_t* __restrict__ row_index, int64_t N_src, int64_t N_pad, int64_t N_v, int n_text,
          int M_v, int M, int total_wg, float scale, unsigned long long* __restrict__ clock_probe, float* __restrict__ part,
          int32_t* __restrict__ tickets, int text_splits, int split_blocks, int tail_from, int tail_rows, int pairs_end, int head, int u, int split,
          int splits, int xcd, int slot, bool tail) {
  constexpr int NW = BM / 32;                      // waves per group: one per 32 query rows
  constexpr int CH = D / 8;                        // 16-byte chunks per row
  constexpr int TILE = KN * D;                     // elements per tile
  constexpr int LPW = KN * CH / (64 * NW);         // load instructions per wave and tile
  constexpr int RJ = NW * 64 / CH;                 // tile rows between two load instructions of a wave
  constexpr int BK = BM > 128 ? 128 : BM;          // rows of a block
  constexpr int STEPS = BK / KN;                   // tiles per key block
  constexpr int NF = D / 8;                        // operand fragments per stage: D/16 of V^T, D/16 of K
  constexpr int ESL = NF - 1;                      // matrix instructions the sixteen exponentials of a half tile are spread over
  constexpr float HEADROOM = 4.f, SUM_LIMIT = 2.25f;                      // see "A row's reference" below
  // Two K and two V tile buffers per group (tile t lives in the pair of parity t & 1), at fixed byte offsets.
  static_assert(!SLIM || KS == 1, "the merge of wave groups wants all four buffers");
  static_assert(!TAIL || (KS == 1 && !XLSE), "see run_sparse_attn");
  static_assert(!SRC || !XLSE, "see run_sparse_attn");
  constexpr bool PAIR = BM > 128, END_WAVE = XLSE || (D == 128 && BM == 128);
  static_assert(!PAIR || (KS == 1 && !SLIM && !TAIL), "see attn_pairs_kernel");
  __shared__ __attribute__((aligned(16))) uint16_t tiles[KS * (SLIM ? 2 : 4) * TILE];
  constexpr int K0 = 0, K1 = SLIM ? 0 : 2 * TILE, V0 = SLIM ? 2 * TILE : 4 * TILE, V1 = SLIM ? 2 * TILE : 6 * TILE;

  // diagnostic: shader-clock cycles and constant-rate (100 MHz) ticks this work-group lives for
  const unsigned long long probe_c0 = clock_probe ? clock64() : 0, probe_w0 = clock_probe ? wall_clock64() : 0;
  auto probe_end = [&]() {
    if (clock_probe && threadIdx.x == 0) {
      atomicAdd(&clock_probe[0], clock64() - probe_c0);
      atomicAdd(&clock_probe[1], wall_clock64() - probe_w0);
      atomicAdd(&clock_probe[2], 1ull);
    }
  };

  int tid = threadIdx.x;
  if (PAIR) asm volatile("" : "+v"(tid));             // see attn_pairs_kernel
  const int lane = tid & 63;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / (64 * NW)), wave = (tid >> 6) - grp * NW;
  const int n = lane & 31, h = lane >> 5;
  const int cnt_in = PAIR ? M : kv_cnt[int64_t(head) * M + u];
  const bool dense = PAIR || cnt_in >= M;
  if (REST && dense && in_pairs(kv_cnt, head, u, M_v, M, total_wg / M, pairs_end)) return;       // another work-group's
  const bool shared_row = !XLSE && splits > 1;
  int cnt = dense ? M : (cnt_in < 0 ? 0 : (cnt_in > K_max ? K_max : cnt_in));
  const int run = tail ? (cnt + splits - 1) / splits : split_blocks;
  const int blk_first = shared_row ? split * run : 0;                     // this work-group's run of the list
  if (shared_row) cnt = cnt - blk_first < 0 ? 0 : cnt - blk_first < run ? cnt - blk_first : run;
  const int32_t* idx = kv_idx + (int64_t(head) * M + u) * K_max + blk_first;
  const int64_t head_off = int64_t(head) * (SRC ? N_src : N_pad) * D;
  const uint16_t* kh = k + head_off;
  const uint16_t* vh = v + head_off;
  const int64_t q_row0 = int64_t(u) * BK + wave * 32 + n;
  // PAIR: this wave's block, and whether there is one (the last video or text block may be alone)
  const int u_wave = PAIR ? u + wave / (BK / 32) : u;
  const bool owned = !PAIR || u_wave < (u < M_v ? M_v : M);

  // Where this lane's query rows live.  With row_index (the permutation) Q is read from, and O written to,
  // the tensors in source order, which spares the reorder passes of Q and O; -1 marks a pad row.
  int64_t io_row = !owned ? -1 : row_index ? int64_t(row_index[q_row0]) : q_row0;
  if (row_index && io_row >= N_src) io_row = -1;
  const int64_t io_off = int64_t(head) * (row_index ? N_src : N_pad) * D;

  // Q rows as the B operand of S^T = K Q^T: lane (n, h) holds Q[row][16 kk + 8 h .. + 7]
  bf16x8 qf[D / 16];
  {
    const u32x4* qp = reinterpret_cast<const u32x4*>(q + io_off + (io_row < 0 ? 0 : io_row) * D);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, io_row < 0 ? u32x4{0u, 0u, 0u, 0u} : qp[2 * kk + h]);
  }

  f32x16 oacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
  // reference in the base-2 exponent's units (logit x c2), row sum, row sum of the unrounded probabilities (XLSE only)
  float m_run = 0.f, l_run = 0.f, x_run = 0.f;
  // Row sums of the probabilities as rounded to bf16 (numerator and denominator then use exactly the same weights, so
  // a dominant key leaves no systematic rounding bias), on the matrix cores: a 16x16x32 product takes the same B operand
  // registers as the 32x32x16 one, but reads lanes 16 g + n as keys 8 g .. 8 g + 7 of column n.  With ones where the
  // parity of the key group equals that of the result row's group, every lane's result is the sum over both lane
  // halves of its own query row.  Every half tile is summed from zero and added to the row's sum on the vector unit: a matrix
  // instruction that accumulates the row's sum rounds each weight against it, and a long row of small weights behind large
  // ones loses 3e-4 to 5e-4 of the sum (131 072 keys; this form below 1.2e-4); as one 2:4 sparse product of half the
  // matrix cycles it was up to 2 % faster (75 600 tokens dense 95.8 -> 95.0 ms, 118 800 x 24 heads 18.0 -> 17.6, 17 550 x 48,
  // d = 64 674 -> 668 us).
  const uint32_t one_pair = (((lane >> 4) ^ (lane >> 2)) & 1) == 0 ? 0x3F803F80u : 0u;
  const bf16x8 row_ones = __builtin_bit_cast(bf16x8, u32x4{one_pair, one_pair, one_pair, one_pair});
  const float c2 = scale * 1.4426950408889634f;     // softmax in base 2

  // Tile loads, global memory straight into LDS: instruction j of this wave fills the 64 consecutive
  // 16-byte chunks (j NW + wave) 64 + lane of the tile buffer; the chunk swizzle is applied on the
  // global side.  The swizzle repeats every PK (PV) instructions, so that few per-lane offsets serve all.
  constexpr int PK = swz_period(RJ / (16 / CH) > 0 ? RJ / (16 / CH) : 1, CH);
  constexpr int PV = swz_period(RJ / (16 / CH) > 0 ? RJ / (16 / CH) : 1, CH / 4);
  static_assert(RJ % (16 / CH) == 0 && LPW % PK == 0 && LPW % PV == 0, "tile load pattern");
  // This group's tiles are t_first .. t_first + n_tiles - 1 of the list's, whole key blocks (whose first row is real: the
  // softmax starts from it).  `rounds`: as many as any group has.
  const int rounds = (cnt + KS - 1) / KS * STEPS, t_first = grp * rounds;
  const int own_tiles = cnt * STEPS - t_first, n_tiles = KS == 1 || own_tiles > rounds ? rounds : own_tiles < 0 ? 0 : own_tiles;
  auto tile_block = [&](int tile) {
    tile += t_first;
    int blk = dense ? blk_first + tile / STEPS : idx[tile / STEPS];
    return unsigned(blk) < unsigned(M) ? blk : 0;     // a corrupt list must not read out of bounds
  };
  auto lane_off = [&](int j, bool is_v) {             // byte offset inside the tile of the chunk this lane fetches
    const int p = (j * NW + wave) * 64 + lane;
    const int row = p / CH, pc = p % CH;
    return uint32_t(2 * ((SRC ? 0 : row * D) + ((pc ^ (is_v ? swz_v<CH>(row) : swz_k<CH>(row))) * 8)));
  };
  uint32_t k_off[PK], v_off[PV];
#pragma unroll
  for (int j = 0; j < PK; ++j) k_off[j] = lane_off(j, false);
#pragma unroll
  for (int j = 0; j < PV; ++j) v_off[j] = lane_off(j, true);
  // The load is issued from an asm statement so that it stays outside the compiler's wait-count
  // bookkeeping: the compiler cannot tell that reads of one tile buffer are independent of loads in
  // flight into another and would wait for every outstanding load before each LDS read.  The waits
  // that are needed are the explicit vmcnt(0) + barrier pairs in the loop below.  (Loads retire in
  // order, so the compiler's own counts for its few other memory operations stay conservative.)
  // LDS address of this wave's first chunk in the first buffer, as a scalar, once (taken from a vector register
  // inside the loop it costs a vector-to-scalar hand-over per tile)
  const uint32_t lds_tiles = uint32_t(reinterpret_cast<uintptr_t>((LDS_PTR(void))(tiles))) + uint32_t(grp * 8 * TILE);
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_tiles + uint32_t(wave * 1024));
  auto tile_src = [&](const uint16_t* base, int tile, int blk) {
    return reinterpret_cast<uint64_t>(base + (int64_t(blk) * BK + (tile % STEPS) * KN) * D);
  };
  auto issue_one = [&](uint64_t src, int buf, bool is_v, int j) {
    const int P = is_v ? PV : PK;
    const uint32_t voff = is_v ? v_off[j % PV] : k_off[j % PK];
    const uint64_t sj = src + uint64_t(j / P) * (P * RJ) * D * 2;
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(sj)), hi = __builtin_amdgcn_readfirstlane(uint32_t(sj >> 32));
    const uint64_t sbase = (uint64_t(hi) << 32) | lo;
    const uint32_t lds = lds_wave + uint32_t(buf + j * NW * 1024);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(sbase) : "memory", "m0");
  };
  auto issue = [&](const uint16_t* base, int buf, bool is_v, int tile, int blk) {
    const uint64_t src = tile_src(base, tile, blk);
#pragma unroll
    for (int j = 0; j < LPW; ++j) issue_one(src, buf, is_v, j);
  };

  // SRC: tiles are gathered from the tensors in source order.  The lanes of a row of load j need that row's position; of four loads,
  // the lanes of a quad look up one each and exchange them inside the quad, on the way of an addition that is needed anyway, so that a
  // tile costs LQ lookups instead of LPW (75 600 tokens dense, d = 128, 1 % of the call; 60 of 591 blocks 1.5 %).  The
  // requests go through a buffer descriptor of the head, whose bounds turn positions that are none (pads, -1; a damaged order) into
  // zeros: their offsets, 2^32 - 2 D and more, lie behind any head.  With a mask of the lanes in its
  // place the calls took 2 to 5 % longer.
  constexpr int LQ = (LPW + 3) / 4;
  const int lane_row = 4 * ((lane % (LPW < 4 ? LPW : 4) * NW * 64 + wave * 64 + lane) / CH);             // bytes of row_index
  auto descriptor = [&](const uint16_t* base) {
    const uint64_t at = reinterpret_cast<uint64_t>(base);
    return u32x4{uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(at))), uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(at >> 32))) & 0xFFFFu,
                 uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(N_src * (2 * D)))), 0x00020000u};
  };
  const u32x4 k_desc = descriptor(kh), v_desc = descriptor(vh);
  struct Rows { uint32_t at[LQ]; };
  auto index_desc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(row_index), 0, int(N_pad * 4), 0x00020000);
  auto look_up = [&](int step, int blk) {            // positions of tile `step` of block blk
    Rows r;
#pragma unroll
    for (int i = 0; i < LQ; ++i) r.at[i] = __builtin_amdgcn_raw_buffer_load_b32(index_desc, lane_row + i * 16 * RJ, (blk * BK + step * KN) * 4, 0);
    return r;
  };
  // The list entry of a tile further ahead, by a vector load: the wait at the tile's barrier covers it, while a scalar one is waited for
  // on the spot, together with the operand reads in flight (d = 128, 17 550 tokens x 24 heads 565 -> 543 us).
  auto list_desc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(idx), 0, dense ? 0 : cnt * 4, 0x00020000);
  auto ask_block = [&](int tile) { return __builtin_amdgcn_raw_buffer_load_b32(list_desc, 0, (t_first + (tile < n_tiles ? tile : n_tiles - 1)) / STEPS * 4, 0); };
  auto told_block = [&](int tile, uint32_t entry) {
    const uint32_t blk = dense ? uint32_t(blk_first + (t_first + (tile < n_tiles ? tile : n_tiles - 1)) / STEPS) : uint32_t(__builtin_amdgcn_readfirstlane(entry));
    return blk < uint32_t(M) ? int(blk) : 0;
  };
  auto offsets = [&](const Rows& r) {                // byte offsets of the rows inside the head
    constexpr uint32_t OUT = 0xFFFFFFFFu / uint32_t(2 * D);
    static_assert(int64_t(MAX_BLOCKS) * BK <= OUT, "no row of a head lies at the offset of a position that is none, or behind 32 bits");
    Rows o;
#pragma unroll
    for (int i = 0; i < LQ; ++i) o.at[i] = (r.at[i] < OUT ? r.at[i] : OUT) * uint32_t(2 * D);
    return o;
  };
  auto gather_one = [&](const Rows& off, int buf, bool is_v, int j) {
    const int x = int(off.at[j / 4]);
    const int y = j % 4 == 0 ? __builtin_amdgcn_mov_dpp(x, 0x00, 0xF, 0xF, true) : j % 4 == 1 ? __builtin_amdgcn_mov_dpp(x, 0x55, 0xF, 0xF, true)
                : j % 4 == 2 ? __builtin_amdgcn_mov_dpp(x, 0xAA, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(x, 0xFF, 0xF, 0xF, true);
    const uint32_t voff = uint32_t(y) + (is_v ? v_off[j % PV] : k_off[j % PK]);
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 ::"s"(lds_wave), "v"(voff), "s"(is_v ? v_desc : k_desc), "i"(buf + j * NW * 1024) : "memory", "m0", "scc");
  };
  auto gather = [&](const Rows& off, int buf, bool is_v) {
#pragma unroll
    for (int j = 0; j < LPW; ++j) gather_one(off, buf, is_v, j);
  };

  // LDS byte addresses of this lane's operand reads in the first buffer, loop invariant: one per K fragment and one per
  // value column group, everything else (buffer, half tile, key rows) is in the instruction's offset.  The empty asm keeps
  // the compiler from working each out anew per buffer, which took thirty registers more, spilled some and redid eight of
  // them per tile: 4 heads of 75 600 tokens with log-sum-exp, dense and sparse, 13.5 -> 12.2 ms; d = 64, 17 550 tokens x 48
  // heads, 667 -> 658 us.
  const int k_sw = swz_k<CH>(n);                                    // rows 32 t + n: swizzle depends on n only
  const int v_r = (lane & 15) >> 2;                                 // row inside the 4-row group
  const int v_row = 4 * h + v_r;
  const int v_sw = swz_v<CH>(v_r);                                  // rows 16 s + 4 h + v_r (+8): same swizzle
  const int v_c = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);        // chunk inside the 32-column group
  const int v_b = (lane & 1) * 4;                                   // 8-byte half of the chunk
  uint32_t k_addr[D / 16], v_addr[D / 32];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    k_addr[kk] = lds_tiles + uint32_t(2 * (n * D + ((2 * kk + h) ^ k_sw) * 8));
    asm volatile("" : "+v"(k_addr[kk]));
  }
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) {
    v_addr[dt] = lds_tiles + uint32_t(2 * (v_row * D + v_b + ((4 * dt + v_c) ^ v_sw) * 8));
    asm volatile("" : "+v"(v_addr[dt]));
  }

  // The loop works on half tiles (32 key rows).  Logits of a half tile:
  // sx[i] = logit(key row 32 half + 8 (i/4) + 4 h + i%4, query row n of the wave).
  auto k_frag = [&](int kbuf, int half, int kk) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<LDS_PTR(const u32x4)>(k_addr[kk] + uint32_t(kbuf + half * 64 * D)));
  };
  // One product piece of O^T += V^T P^T for a half tile: piece j = (D/32) s2 + dt.  Product step s2
  // covers key rows 16 s2 + {4h..4h+3} and 16 s2 + 8 + {4h..4h+3}, which is what registers 8 s2 .. 8 s2 + 7
  // of the logit tile hold; the transposing LDS read hands each lane four consecutive key rows of one
  // value column.
  auto v_frag = [&](int vbuf, int half, int j) {
    const int s2 = j / (D / 32), dt = j % (D / 32);
    const uint32_t p0 = v_addr[dt] + uint32_t(vbuf + half * 64 * D + s2 * 32 * D);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_PTR(s16x4)>(p0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_PTR(s16x4)>(p0 + 16 * D));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto logits = [&](int kbuf, int half, f32x16& sx) {
#pragma unroll
    for (int i = 0; i < 16; ++i) sx[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) sx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(kbuf, half, kk), qf[kk], sx, 0, 0, 0);
  };
  // pad keys of a ragged block never count.  Only two blocks can be ragged, the last video block and the last text
  // block; their ids and real-row counts are worked out once, so that the check per half tile is two scalar compares
  // on a block id that is already at hand (measured: the 64-bit arithmetic of the general form, twice per tile, cost
  // 2 % of the kernel).
  const int real_v_last = block_real_rows(M_v - 1, BK, M_v, N_v, n_text);
  const int real_x_last = M > M_v ? block_real_rows(M - 1, BK, M_v, N_v, n_text) : BK;
  const int ragged_v = real_v_last < BK ? M_v - 1 : -1, ragged_x = real_x_last < BK ? M - 1 : -1;
  auto mask_pads = [&](int blk, int tile, int half, f32x16& sx) {
    if (__builtin_expect(blk == ragged_v || blk == ragged_x, 0)) {
      asm volatile("");                               // keeps this a branch: turned into selects it would run on every half tile
      const int real = blk == ragged_v ? real_v_last : real_x_last;
      const int base = (tile % STEPS) * KN + 32 * half;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (base + 8 * (i / 4) + 4 * h + (i % 4) >= real) sx[i] = -INFINITY;
    }
  };

  // One pipeline stage, written out in issue order.  Fragments alternate between K of the next half tile (logit chain
  // into `sn`) and V^T of the previous half tile (products O^T += V^T P^T with its probabilities `pp`).  In the shadow
  // of the matrix instructions the vector units turn the logits `sx` of the current half tile into probabilities `pc`,
  // which are summed at the end.  Scheduling fences and empty asm statements keep the compiler from separating the matrix
  // and vector work again.
  //
  // A row's reference m_run is a maximum of its logits times 2^HEADROOM: to start with that of its first half tile and of
  // its own 32 keys, where many rows have their largest logit; later that of a half tile whose weights sum to more than
  // SUM_LIMIT.  32 weights of 2^-HEADROOM sum to 2, so a row moves when one weight has grown by 2^5.2 or many have by less,
  // and raises its reference by at least an eighth.  The sums come from the matrix cores, so that watching them costs two
  // vector instructions per half tile, an addition and a comparison (a running maximum and its factor: some fifteen), and
  // `settle` does the half tile again when a row moves: about 1 % of the half tiles of a wave at 75 600 tokens, 2 % at
  // 17 550, 5 % in rows of 13 blocks of 64.
  // Weights are then below SUM_LIMIT whatever comes, and exact in bf16 where they are largest, which is what the reference
  // is followed for: with that of the first half tile kept, the outputs' error against 64 bits was 1.86e-3 of the result
  // instead of 1.77e-3 (75 600 tokens, 60 of 591 blocks), 2.29e-3 instead of 2.17e-3 (17 550 tokens, dense, d = 64,
  // logits of standard deviation 2).  What it costs against keeping it, on one card: d = 64, 17 550 tokens x 48 heads 654 ->
  // 674 us; d = 128, 75 600 tokens, 40 heads, 60 of 591 blocks 10.99 -> 11.16 ms, 8 heads dense 19.56 -> 19.66; against a
  // running maximum it wins 743 -> 674, 11.92 -> 11.16, 21.09 -> 19.66.
  auto half_max = [&](const f32x16& x) __attribute__((always_inline)) {      // row maximum of a half tile, in both lane halves
    float mx = x[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  auto pack = [&](float a, float b) __attribute__((always_inline)) {
    const bf16x2 pk = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, pk);
  };
  auto half_sum = [&](const u32x4& p, f32x4 sum) __attribute__((always_inline)) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(row_ones, __builtin_bit_cast(bf16x8, p), sum, 0, 0, 0);
  };
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  // Adds a half tile's sums (`sum` of the rounded weights pc, xsum of the unrounded) to the row's.  If a row of the wave has
  // outgrown its reference, the rows that have grown at all move first (logits sx).  The comparison is one that a NaN does not
  // pass: where rows n and 16 + n both reach infinite weights, each sum holds the other's infinity times a zero.
  auto settle = [&](const f32x16& sx, u32x4 (&pc)[2], f32x4 sum, float xsum) __attribute__((always_inline)) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(sum[0] <= SUM_LIMIT)) != 0, 0)) {
      const float mx = fmaf(half_max(sx), c2, HEADROOM);
      const float m_new = mx > m_run ? mx : m_run;   // not fmaxf: a NaN leaves the reference where it is
      float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      // The accumulators are scaled in place, so that they keep one home across the branch.  The compiler does not see what
      // these statements read, so the waits for the matrix instructions in flight (at most 19 states) and for the
      // exponential (one) are written out, in a statement that they depend on.
      asm volatile("s_nop 15\n\ts_nop 3" : "+v"(alpha));
      m_run = m_new;
      l_run *= alpha;
      if (XLSE) x_run *= alpha;
      asm volatile("" : "+v"(l_run), "+v"(x_run));    // not fused with the additions below: the same bits in every instance
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          float y = oacc[dt][i];
          asm volatile("v_mul_f32 %0, %1, %0" : "+v"(y) : "v"(alpha));
          oacc[dt][i] = y;
        }
      xsum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float a = __builtin_amdgcn_exp2f(fmaf(sx[i], c2, -m_run)), b = __builtin_amdgcn_exp2f(fmaf(sx[i + 1], c2, -m_run));
        pc[i / 8][(i % 8) / 2] = pack(a, b);
        if (XLSE) xsum += a + b;
      }
      sum = half_sum(pc[1], half_sum(pc[0], zero4));
      asm volatile("" : "+v"(sum));                   // one home as well
    }
    l_run += sum[0];
    if (XLSE) x_run += xsum;
  };
  auto stage = [&](auto do_pv, auto do_s, int vbuf, int pv_half, const u32x4 (&pp)[2], int kbuf,
                   int s_half, f32x16& sn, const f32x16& sx, u32x4 (&pc)[2], f32x4& sum, float& xsum, auto mem) __attribute__((always_inline)) {
    constexpr bool DO_PV = decltype(do_pv)::value, DO_S = decltype(do_s)::value;
    bf16x8 frag[NF];
    auto load = [&](int f) {
      if (f % 2 == 1) {
        if (DO_PV) frag[f] = v_frag(vbuf, pv_half, f / 2);
      } else if (DO_S) {
        frag[f] = k_frag(kbuf, s_half, f / 2);
      }
    };
    float pe[16];
    xsum = 0.f;
    if (DO_S) {
#pragma unroll
      for (int i = 0; i < 16; ++i) sn[i] = 0.f;
    }
    constexpr int AHEAD = 3;                          // fragments requested ahead of their matrix instruction
#pragma unroll
    for (int f = 0; f < AHEAD; ++f) load(f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      if (f + AHEAD < NF) load(f + AHEAD);
      mem(f);
      if (f % 2 == 1) {
        if (DO_PV) {
          const int j = f / 2, s2 = j / (D / 32), dt = j % (D / 32);
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[f], __builtin_bit_cast(bf16x8, pp[s2]), oacc[dt], 0, 0, 0);
        }
      } else if (DO_S) {
        sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[f], qf[f / 2], sn, 0, 0, 0);
      }
      if (f < ESL) {
#pragma unroll
        for (int i = f * 16 / ESL; i < (f + 1) * 16 / ESL; ++i) {
          pe[i] = __builtin_amdgcn_exp2f(fmaf(sx[i], c2, -m_run));
          asm volatile("" : "+v"(pe[i]));
        }
      }
      if (f > 0 && f <= ESL) {                        // pairs completed in the slot before: their exponentials have retired
#pragma unroll
        for (int i = (f - 1) * 16 / ESL; i < f * 16 / ESL; ++i)
          if (i % 2 == 1) {
            pc[i / 8][(i % 8) / 2] = pack(pe[i - 1], pe[i]);
            if (XLSE) xsum += pe[i - 1] + pe[i];
          }
      }
      if (f == NF - 1) {
#pragma unroll
        for (int i = (ESL - 1) * 16 / ESL; i < 16; ++i) asm volatile("" : "+v"(pc[i / 8][(i % 8) / 2]));
      }
      if (f == NF - 2) sum = half_sum(pc[0], zero4);
      if (f == NF - 1) sum = half_sum(pc[1], sum);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using yes = std::true_type;
  using no = std::false_type;

  // Software pipeline over half tiles.  K(t+2) and V(t+1) are requested once per tile, right after the
  // barrier in the middle of tile t, into the buffers K(t) and V(t-1) have just left; they are first
  // read a full tile later.
  f32x16 s0, s1;
  u32x4 p0[2], p1[2];                              // probabilities as bf16 pairs: B operands of the products
  // Key blocks of tiles t and t + 1; the list is looked up where tile t + 2 starts another block.  (With a lookup for every tile, K and V
  // reordered, blocks of 128: d = 64, 17 550 tokens x 48 heads, 21 of 138 blocks, 627 -> 621 us; d = 128, 75 600 x 40, 60 of 591, 11 331 -> 11 298,
  // x 8 dense 20 105 -> 19 994, x 4 dense with log-sum-exp 10 981 -> 10 892.)
  int b_cur = 0, b_nxt = 0;
  // SRC: block of tile t + 2, list entry of tile t + 3, positions of the rows of K(t + 2), offsets of those of V(t + 1); SLIM: all a
  // tile less.  Positions are looked up a tile before the tile is requested and two before it is read.
  int b_far = 0;
  uint32_t entry = 0;
  Rows k_rows, v_rows;
  auto tile_step = [&](auto parity, auto first, auto last, int t) __attribute__((always_inline)) {
    constexpr bool ODD = decltype(parity)::value, FIRST = decltype(first)::value, LAST = decltype(last)::value;
    constexpr int k_cur = ODD ? K1 : K0;             // K(t); K(t+2) goes here
    constexpr int k_nxt = ODD ? K0 : K1;             // K(t+1)
    constexpr int v_cur = ODD ? V1 : V0;             // V(t)
    constexpr int v_nxt = ODD ? V0 : V1;             // V(t-1); V(t+1) goes here
    // SLIM: every stage requests a half of V(t) and a half of K(t+1), in its first slots, into the halves that the stage before
    // has left; they are read in the next stage.
    Rows next;
    const int b_told = SRC && SLIM ? told_block(t + 2, entry) : 0;
    if (SRC && SLIM) k_rows = offsets(k_rows);
    auto request = [&](int half) {
      const uint64_t k_src = tile_src(kh, t + 1, b_nxt), v_src = tile_src(vh, t, b_cur);
      return [&, half, k_src, v_src](int f) {
        if (!SLIM || f >= NF / 2) return;
        if (SRC && f == 0 && half == 0 && !LAST) {
          next = look_up(0, b_told);
          entry = ask_block(t + 3);
        }
#pragma unroll
        for (int j = f * 2 * LPW / NF; j < (f + 1) * 2 * LPW / NF; ++j) {
          if (LAST && j >= LPW / 2) return;
          if (SRC) {
            gather_one(j < LPW / 2 ? v_rows : k_rows, j < LPW / 2 ? V0 : K0, j < LPW / 2, half * LPW / 2 + j % (LPW / 2));
            continue;
          }
          issue_one(j < LPW / 2 ? v_src : k_src, j < LPW / 2 ? V0 : K0, j < LPW / 2, half * LPW / 2 + j % (LPW / 2));
        }
      };
    };
    // first half: products of (t-1, 1), logits of (t, 1), probabilities of (t, 0)
    f32x4 sum;
    float xsum;
    stage(std::integral_constant<bool, !FIRST>{}, yes{}, v_nxt, 1, p1, k_cur, 1, s1, s0, p0, sum, xsum, request(0));
    mask_pads(b_cur, t, 1, s1);
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): this wave's parts of K(t+1) and V(t) landed
    __syncthreads();                                 // all parts landed; every wave is past the first half of tile t
    settle(s0, p0, sum, xsum);
    // Second half: products of (t, 0), logits of (t+1, 0), probabilities of (t, 1); between its matrix instructions the
    // loads of K(t+2) and V(t+1) (in one run behind the barrier they kept the matrix cores waiting for some fifty
    // instructions: +2.0 % on lists that hit in L2, +2.5 % on scattered ones, +4.7 % dense at d = 128).  Behind the
    // last tile K(t+2) is that tile once more, into a buffer that nothing reads.
    const int b_new = SRC && SLIM ? b_told : SRC ? b_far : STEPS == 2 && ODD ? b_nxt : tile_block(t + 2 < n_tiles ? t + 2 : n_tiles - 1);
    const uint64_t k_src = tile_src(kh, t + 2, b_new), v_src = tile_src(vh, t + 1, b_nxt);
    if constexpr (SLIM) {
      stage(yes{}, std::integral_constant<bool, !LAST>{}, V0, 0, p0, K0, 0, s0, s1, p1, sum, xsum, request(1));
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      if (SRC) {
        v_rows = k_rows;
        if (!LAST) k_rows = next;
      }
    } else if constexpr (SRC) {
      const int b_pos = STEPS == 2 && !ODD ? b_far : told_block(t + 3, entry);
      k_rows = offsets(k_rows);
      stage(yes{}, std::integral_constant<bool, !LAST>{}, v_cur, 0, p0, k_nxt, 0, s0, s1, p1, sum, xsum, [&](int f) {
        if (LAST) return;
        if (f == 0) {
          next = look_up(STEPS == 2 && !ODD, b_pos);
          if (STEPS == 1 || !ODD) entry = ask_block(t + 4);
        }
#pragma unroll
        for (int j = f * 2 * LPW / NF; j < (f + 1) * 2 * LPW / NF; ++j) {
          if (j < LPW) gather_one(v_rows, v_nxt, true, j);
          else gather_one(k_rows, k_cur, false, j - LPW);
        }
      });
      v_rows = k_rows;
      if (!LAST) k_rows = next;
      b_far = b_pos;
    } else {
      stage(yes{}, std::integral_constant<bool, !LAST>{}, v_cur, 0, p0, k_nxt, 0, s0, s1, p1, sum, xsum, [&](int f) {
        if (LAST) return;
#pragma unroll
        for (int j = f * 2 * LPW / NF; j < (f + 1) * 2 * LPW / NF; ++j)
          issue_one(j < LPW ? v_src : k_src, j < LPW ? v_nxt : k_cur, j < LPW, j % LPW);
      });
    }
    settle(s1, p1, sum, xsum);
    if (!LAST) mask_pads(b_nxt, t + 1, 0, s0);
    b_cur = b_nxt;
    b_nxt = b_new;
  };
  auto products = [&](int vbuf, int half, const u32x4 (&pp)[2]) __attribute__((always_inline)) {    // O^T += V^T P^T
#pragma unroll
    for (int j = 0; j < 2 * (D / 32); ++j) {
      const bf16x8 pj = __builtin_bit_cast(bf16x8, pp[j / (D / 32)]);
      oacc[j % (D / 32)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(vbuf, half, j), pj, oacc[j % (D / 32)], 0, 0, 0);
    }
  };
  if (n_tiles > 0) {
    // The keys of this wave's own rows, for the reference to start from if their block is among this group's.  The list is
    // requested in front of the tiles: behind them the wave waited for tiles and list before it asked for the keys (44
    // blocks x 4 heads, 9 kept, 27.8 -> 27.2 us a reuse step).
    const int own_first = t_first / STEPS, own_blks = n_tiles / STEPS;
    const int listed = !dense && lane < own_blks ? idx[own_first + lane] : -1;
    b_cur = tile_block(0);
    b_nxt = n_tiles > 1 ? tile_block(1) : b_cur;
    if constexpr (SRC) {
      Rows rows_0 = look_up(0, b_cur);
      k_rows = look_up(STEPS - 1, b_nxt);            // behind a lone tile its block once more, into a buffer that nothing reads
      if (SLIM) {
        entry = ask_block(2);
        v_rows = offsets(rows_0);
        gather(v_rows, K0, false);
      } else {
        v_rows = k_rows;
        b_far = tile_block(n_tiles > 2 ? 2 : n_tiles - 1);
        k_rows = look_up(0, b_far);
        if (STEPS == 1) entry = ask_block(3);
        rows_0 = offsets(rows_0);
        gather(rows_0, K0, false);
        gather(rows_0, V0, true);
        v_rows = offsets(v_rows);
        gather(v_rows, K1, false);
      }
    } else {
      issue(kh, K0, false, 0, b_cur);
      if (!SLIM) issue(vh, V0, true, 0, b_cur);
    }
    bf16x8 own_k[D / 16];
    {
      const u32x4* kp = reinterpret_cast<const u32x4*>(kh + (SRC ? io_row < 0 ? 0 : io_row : owned ? q_row0 : 0) * D);
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) own_k[kk] = __builtin_bit_cast(bf16x8, SRC && io_row < 0 ? u32x4{0u, 0u, 0u, 0u} : kp[2 * kk + h]);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (!SRC && !SLIM && n_tiles > 1) issue(kh, K1, false, 1, b_nxt);
    logits(K0, 0, s0);
    if (SLIM) __syncthreads();                       // the first half of K(0) has been read
    mask_pads(b_cur, 0, 0, s0);
    m_run = half_max(s0);
    bool own = dense ? u_wave - blk_first >= own_first && u_wave - blk_first < own_first + own_blks : listed == u;
    if (!dense)
      for (int i = 64 + lane; i < own_blks; i += 64) own |= idx[own_first + i] == u;
    if (__builtin_amdgcn_ballot_w64(own) != 0) {     // as logits and mask_pads, with the keys from registers
#pragma unroll
      for (int i = 0; i < 16; ++i) s1[i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(own_k[kk], qf[kk], s1, 0, 0, 0);
      if (u_wave == ragged_v || u_wave == ragged_x) {
        const int real = u_wave == ragged_v ? real_v_last : real_x_last;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (wave % (BK / 32) * 32 + 8 * (i / 4) + 4 * h + (i % 4) >= real) s1[i] = -INFINITY;
      }
      m_run = fmaxf(m_run, half_max(s1));
    }
    m_run = fmaxf(fmaf(m_run, c2, HEADROOM), -FLT_MAX);              // finite: logits of -inf have weight 0, not NaN
    if (n_tiles == 1) {
      tile_step(no{}, yes{}, yes{}, 0);
    } else {
      tile_step(no{}, yes{}, no{}, 0);
      int t = 1;
      for (; t + 2 < n_tiles; t += 2) {              // middle tiles in pairs: buffer parities are compile-time
        tile_step(yes{}, no{}, no{}, t);
        tile_step(no{}, no{}, no{}, t + 1);
      }
      if (t + 1 < n_tiles) { tile_step(yes{}, no{}, no{}, t); ++t; }
      if (t & 1) tile_step(yes{}, no{}, yes{}, t);
      else tile_step(no{}, no{}, yes{}, t);
    }
    products((n_tiles - 1) & 1 ? V1 : V0, 1, p1);  // drain: the last half tile
  }
  // The groups share their barriers, one in front of the first tile and one per tile: a group with fewer tiles meets the
  // others at those it has not come to.  (It walked its last tile again with weights of zero instead, which turned
  // infinite values there into NaN.)
  if (KS > 1)
    for (int t = n_tiles > 0 ? n_tiles : -1; t < rounds; ++t) __syncthreads();

  if constexpr (KS > 1) {
    // Merge.  A group's accumulators go where its tiles were (one buffer holds one wave's), its reference and sums beside
    // them; the first group brings all to the largest reference and adds.  A group without tiles (reference -inf) adds zeros.
    __shared__ float s_part[KS][NW][3][64];
    auto acc_buf = [&](int g) {
      return reinterpret_cast<float*>(tiles + (g * 4 + wave) * TILE) + lane;
    };
    static_assert(TILE * 2 == (D / 32) * 16 * 64 * 4, "one tile buffer holds the accumulators of one wave");
    if (rounds == 0) {
      if (grp > 0) {
        if constexpr (END_WAVE) __builtin_amdgcn_endpgm();
        return;
      }
    } else {
      if (n_tiles == 0) m_run = -INFINITY;
      __syncthreads();                               // every wave is done with the tiles
      if (grp > 0) {
        float* part = acc_buf(grp);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i) part[(dt * 16 + i) * 64] = oacc[dt][i];
        s_part[grp][wave][0][lane] = m_run;
        s_part[grp][wave][1][lane] = l_run;
        s_part[grp][wave][2][lane] = x_run;
      }
      __syncthreads();
      // With END_WAVE the end of the wave itself: as a return, a way to the end of the kernel, it kept the accumulators of the first group in scratch
      // (187 registers spilled with log-sum-exp, d = 128, blocks of 128, instead of 15; recall's calls on one head of 44 blocks 174 us instead of 153).
      // Where none are spilled the return is the faster one (us a reuse step of 2 048 tokens: x 8 heads, d = 128, blocks of 64, 16.23 -> 15.97, x 3 20.65
      // -> 20.42, x 8, d = 64, 9.20 -> 9.12).
      if (grp > 0) {
        if constexpr (END_WAVE) __builtin_amdgcn_endpgm();
        return;
      }
      float m_all = m_run;
#pragma unroll
      for (int g = 1; g < KS; ++g) m_all = fmaxf(m_all, s_part[g][wave][0][lane]);
      const float own = __builtin_amdgcn_exp2f(m_run - m_all);
      m_run = m_all;
      l_run *= own;
      x_run *= own;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dt][i] *= own;
#pragma unroll
      for (int g = 1; g < KS; ++g) {
        const float share = __builtin_amdgcn_exp2f(s_part[g][wave][0][lane] - m_all);
        const float* part = acc_buf(g);
        l_run = fmaf(share, s_part[g][wave][1][lane], l_run);
        x_run = fmaf(share, s_part[g][wave][2][lane], x_run);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[dt][i] = fmaf(share, part[(dt * 16 + i) * 64], oacc[dt][i]);
      }
    }
  }

  if constexpr (!XLSE) {
    if (shared_row) {
      // Stores and loads at the chip's scope go past the L2, which belongs to one XCD: a release and an acquire around
      // the ticket instead would write the whole L2 back and drop it (2 565 + 77 tokens x 12 heads 43 -> 55 us).  The order
      // that they would give is here: no store is in flight when its wave arrives at the barrier in front of the ticket,
      // and no load is issued before the ticket has come back.
      auto put = [](float* p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      auto get = [](const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      constexpr int REGS = D / 2 + 2;                // of a lane: accumulators, reference, row sum
      // tickets and partial rows: those of the text rows, then those of the tail
      const int M_x = M - M_v, text_rows = total_wg / M * M_x, tail_row = xcd * tail_rows + slot - tail_from;
      const int row = tail ? text_rows + tail_row : head * M_x + (u - M_v);
      const int64_t first = tail ? int64_t(text_splits > 1 ? text_rows : 0) * text_splits + int64_t(tail_row) * splits : int64_t(row) * splits;
      float* rows = part + (first * NW + wave) * REGS * 64 + lane;
      float* mine = rows + int64_t(split) * NW * REGS * 64;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) put(mine + (dt * 16 + i) * 64, oacc[dt][i]);
      put(mine + (REGS - 2) * 64, n_tiles == 0 ? -INFINITY : m_run);
      put(mine + (REGS - 1) * 64, l_run);
      __shared__ int s_ticket;
      __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wave's sums have reached memory
      __syncthreads();                               // and every wave's, before the ticket is taken
      if (tid == 0) s_ticket = __hip_atomic_fetch_add(&tickets[row], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      if (s_ticket != splits - 1) {
        probe_end();
        return;
      }
      float m_all = -INFINITY;
      for (int sp = 0; sp < splits; ++sp) m_all = fmaxf(m_all, get(rows + (int64_t(sp) * NW * REGS + REGS - 2) * 64));
      const float ref = m_all == -INFINITY ? 0.f : m_all;
      l_run = 0.f;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
      for (int sp = 0; sp < splits; ++sp) {
        const float* p = rows + int64_t(sp) * NW * REGS * 64;
        const float share = __builtin_amdgcn_exp2f(get(p + (REGS - 2) * 64) - ref);
        l_run = fmaf(share, get(p + (REGS - 1) * 64), l_run);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[dt][i] = fmaf(share, get(p + (dt * 16 + i) * 64), oacc[dt][i]);
      }
    }
  }

  probe_end();
  // epilogue: normalise, round to bf16, store.  Lane (n, h) holds O[row][32 dt + 8 j + 4 h + 0..3].
  const float inv = l_run > 0.f ? 1.0f / l_run : 0.f;
  if (io_row >= 0) {
    uint16_t* orow = o + io_off + io_row * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (__bf16)(oacc[dt][4 * j + e] * inv);
        *reinterpret_cast<u32x2*>(orow + 32 * dt + 8 * j + 4 * h) = __builtin_bit_cast(u32x2, w);
      }
  }
  if (XLSE) {
    const float x_tot = x_run + __shfl_xor(x_run, 32, 64);
    if (lse && h == 0 && owned)
      lse[int64_t(head) * N_pad + q_row0] = x_tot > 0.f ? (m_run + __builtin_amdgcn_logf(x_tot)) * 0.6931471805599453f : -INFINITY;
  }
}

// REST: behind attn_pairs_kernel.  Dense pairs in front of slot pairs_end are left out, which it has done or, behind its `pair_rounds`, the work-groups
// from slot left_from on do: left_rows / 2 pairs an XCD, whose blocks left_splits work-groups share each.
template <int D, int BM, bool XLSE, int KS, bool SLIM, bool TAIL, bool SRC, bool REST>
__device__ __forceinline__ void
attn_work_group(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                const int32_t* __restrict__ kv_idx, const int32_t* __restrict__ kv_cnt, int K_max, uint16_t* __restrict__ o,
                float* __restrict__ lse, const int32_t* __restrict__ row_index, int64_t N_src, int64_t N_pad, int64_t N_v, int n_text,
                int M_v, int M, int total_wg, int wg_per_xcd, int mapping, float scale, unsigned long long* __restrict__ clock_probe,
                float* __restrict__ part, int32_t* __restrict__ tickets, int text_splits, int split_blocks, int tail_from, int tail_rows,
                int tail_splits, int pair_rounds, int pairs_end, int left_from, int left_rows, int left_splits) {
  // Work-group to (head, query block).  Ids are dealt round-robin to the 8 XCDs, so id % 8 names the XCD
  // and id / 8 the order inside it.
  //   mapping 2 (long sequences): every XCD takes its own eighth of the query blocks of head 0, then of
  //     head 1, ...  All XCDs are on the same head at the same time, so the key/value working set of the
  //     chip is one or two heads and stays in the memory-side cache, while the blocks that meet in one
  //     L2 are neighbours on the curve, which share key blocks.  The dense text blocks of all heads, the
  //     longest work-groups, come first.
  //   mapping 1 (an eighth of a head would not fill an XCD): each XCD walks whole heads of its own,
  //     query blocks last-first so that the text blocks of a head start first.
  //   mapping 3: mapping 1 with the text blocks, split, of all heads in front as in mapping 2.
  // Behind slot tail_from, where the query blocks left would not fill the XCD once more, tail_splits work-groups share each.
  int head, u, split = 0, splits = 1, slot = blockIdx.x / 8;
  const int xcd = blockIdx.x % 8;
  const bool left = REST && TAIL && slot >= left_from;
  bool tail = TAIL && slot >= tail_from;
  if (tail && !left) {
    splits = tail_splits;
    split = (slot - tail_from) / tail_rows;
    slot -= split * tail_rows;
  }
  if (left) {
    const int row = (slot - left_from) % left_rows;
    splits = left_splits;
    split = (slot - left_from) / left_rows;
    u = pair_at(xcd, pair_rounds * PAIR_WGS + row / 2, M_v, M, total_wg / M, head);
    if (u < 0 || !pair_dense(kv_cnt, head, u, M_v, M)) return;
    u += row & 1;
    if (u >= M_v) return;
    // their tickets and partial rows lie behind the tail's
    tickets += 8 * tail_rows;
    part += int64_t(8 * tail_rows * tail_splits) * (BM * (D + 4));
    tail = true;
    tail_from = 0;
    tail_rows = left_rows;
    slot = row;
    pairs_end = 0;
  } else if (mapping >= 2) {
    const int M_x = M - M_v, n_heads = total_wg / M;
    const int text_wgs = n_heads * M_x * text_splits, text_slots = (text_wgs + 7) / 8;
    if (slot < text_slots) {
      const int id = slot * 8 + xcd;
      if (id >= text_wgs) return;
      u = M_v + id % M_x;
      split = id / M_x % text_splits;
      splits = text_splits;
      head = id / M_x / text_splits;
    } else if (mapping == 2) {
      const int C = (M_v + 7) / 8, s2 = slot - text_slots;
      head = s2 / C;
      u = xcd * C + s2 % C;
      if (head >= n_heads || u >= M_v) return;
    } else {
      const int logical = xcd * wg_per_xcd + slot - text_slots;
      if (slot - text_slots >= wg_per_xcd || logical >= n_heads * M_v) return;
      head = logical / M_v;
      u = M_v - 1 - logical % M_v;
    }
  } else {
    const int logical = xcd * wg_per_xcd + slot;
    if (slot >= wg_per_xcd || logical >= total_wg) return;
    head = logical / M;
    u = M - 1 - logical % M;
  }
  attn_rows<D, BM, XLSE, KS, SLIM, TAIL, SRC, REST>(q, k, v, kv_idx, kv_cnt, K_max, o, lse, row_index, N_src, N_pad, N_v, n_text, M_v, M, total_wg,
                                                    scale, clock_probe, part, tickets, text_splits, split_blocks, tail_from, tail_rows, pairs_end,
                                                    head, u, split, splits, xcd, slot, tail);
}

template <int D, int BM, bool XLSE, int KS, bool SLIM, bool TAIL, bool SRC>
__global__ void __launch_bounds__(BM * 2 * KS)
__attribute__((amdgpu_waves_per_eu(attn_waves<D, BM, XLSE, KS>(), attn_waves<D, BM, XLSE, KS>())))
attn_bf16_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                 const int32_t* __restrict__ kv_idx, const int32_t* __restrict__ kv_cnt, int K_max, uint16_t* __restrict__ o,
                 float* __restrict__ lse, const int32_t* __restrict__ row_index, int64_t N_src, int64_t N_pad, int64_t N_v, int n_text,
                 int M_v, int M, int total_wg, int wg_per_xcd, int mapping, float scale, unsigned long long* __restrict__ clock_probe,
                 float* __restrict__ part, int32_t* __restrict__ tickets, int text_splits, int split_blocks, int tail_from, int tail_rows,
                 int tail_splits) {
  attn_work_group<D, BM, XLSE, KS, SLIM, TAIL, SRC, false>(q, k, v, kv_idx, kv_cnt, K_max, o, lse, row_index, N_src, N_pad, N_v, n_text, M_v, M, total_wg,
                                                          wg_per_xcd, mapping, scale, clock_probe, part, tickets, text_splits, split_blocks, tail_from,
                                                          tail_rows, tail_splits, 0, 0, 0, 0, 0);
}

// The same behind attn_pairs_kernel (its look at the pairs costs a work-group 0.3 us on its way to the list).
template <int D, int BM, bool XLSE, bool TAIL, bool SRC>
__global__ void __launch_bounds__(BM * 2) __attribute__((amdgpu_waves_per_eu(2, 2)))
attn_rest_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                 const int32_t* __restrict__ kv_idx, const int32_t* __restrict__ kv_cnt, int K_max, uint16_t* __restrict__ o,
                 float* __restrict__ lse, const int32_t* __restrict__ row_index, int64_t N_src, int64_t N_pad, int64_t N_v, int n_text,
                 int M_v, int M, int total_wg, int wg_per_xcd, int mapping, float scale, unsigned long long* __restrict__ clock_probe,
                 float* __restrict__ part, int32_t* __restrict__ tickets, int text_splits, int split_blocks, int tail_from, int tail_rows,
                 int tail_splits, int pair_rounds, int pairs_end, int left_from, int left_rows, int left_splits) {
  attn_work_group<D, BM, XLSE, 1, false, TAIL, SRC, true>(q, k, v, kv_idx, kv_cnt, K_max, o, lse, row_index, N_src, N_pad, N_v, n_text, M_v, M, total_wg,
                                                         wg_per_xcd, mapping, scale, clock_probe, part, tickets, text_splits, split_blocks, tail_from,
                                                         tail_rows, tail_splits, pair_rounds, pairs_end, left_from, left_rows, left_splits);
}

// Dense rows (the first quarter of a sampling run's steps): two neighbouring query blocks of 128 rows that keep every key block, in one
// work-group of eight waves, so that a tile is brought into LDS once for both.  What bounds them is the clock that the chip grants, and
// it pays for every byte on its way: half the tile loads are 4.5 % (75 600 tokens x 40 heads 102.4 -> 97.7 ms, 1.15 -> 1.20 PFLOP/s on one
// card), the same bits.  The kernel looks the counts up and leaves if no pair is dense; its work-groups, one per CU, walk
// their slots in step.  The blocks behind the last full round, pairs that are not dense and single blocks are the other kernel's, in a
// launch behind this one.
template <int D, bool XLSE, bool SRC>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
attn_pairs_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                  const int32_t* __restrict__ kv_cnt, uint16_t* __restrict__ o, float* __restrict__ lse, const int32_t* __restrict__ row_index,
                  int64_t N_src, int64_t N_pad, int64_t N_v, int n_text, int M_v, int M, int n_heads, float scale,
                  unsigned long long* __restrict__ clock_probe, int rounds) {
  const int xcd = blockIdx.x % 8, first = blockIdx.x / 8, lane = threadIdx.x & 63;
  for (int r0 = 0; r0 < rounds; r0 += 64) {
    int head, u = -1;
    if (r0 + lane < rounds) {
      u = pair_at(xcd, (r0 + lane) * PAIR_WGS + first, M_v, M, n_heads, head);
      if (u >= 0 && !pair_dense(kv_cnt, head, u, M_v, M)) u = -1;
    }
    unsigned long long todo = __builtin_amdgcn_ballot_w64(u >= 0);         // the same in every wave
    while (todo != 0) {
      const int r = r0 + __builtin_ctzll(todo);
      todo &= todo - 1;
      u = pair_at(xcd, r * PAIR_WGS + first, M_v, M, n_heads, head);
      // What a pair needs is worked out anew for each: kept from pair to pair, forty registers of it would be spilled.
      asm volatile("" : "+s"(q), "+s"(k), "+s"(v), "+s"(o), "+s"(lse), "+s"(row_index), "+s"(N_src), "+s"(N_pad), "+s"(N_v), "+s"(n_text), "+s"(scale),
                   "+s"(head), "+s"(u));
      attn_rows<D, 256, XLSE, 1, false, false, SRC, false>(q, k, v, nullptr, kv_cnt, 0, o, lse, row_index, N_src, N_pad, N_v, n_text, M_v, M, n_heads * M, scale,
                                                    clock_probe, nullptr, nullptr, 1, M, 0, 1, 0, head, u, 0, 1, xcd, 0, false);
      __syncthreads();                               // every wave is done with the tiles
    }
  }
}

// Attention of fp32 tensors (attn_f32.h).
template <int D, bool SRC>
__global__ void __launch_bounds__(64 * AF_WAVES) attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                                 const int32_t* __restrict__ kv_idx, const int32_t* __restrict__ kv_cnt, int K_max,
                                                                 float* __restrict__ o, float* __restrict__ lse, const int32_t* __restrict__ row_index,
                                                                 int64_t N_src, int64_t N_pad, int64_t N_v, int n_text, int M_v, int M, int B,
                                                                 float scale) {
  __shared__ AttnF32Room<D, SRC || D == 128> room;
  const int parts = B / 32, head = blockIdx.y, u = M - 1 - int(blockIdx.x) / parts;      // the dense text rows start first
  const int64_t row = int64_t(head) * M + u;
  const int part = int(blockIdx.x) % parts, cnt = kv_cnt[row];
  const int64_t q_row = int64_t(u) * B + part * 32 + (threadIdx.x & 31), head_rows = row_index ? N_src : N_pad;
  QueryRow<D> query;
  query.load(q, head_rows, head, row_index ? int64_t(row_index[q_row]) : q_row);       // see the bf16 kernel
  attn_f32_rows<D, SRC>(
      room, query, k, v, [&](int i) { return kv_idx[row * K_max + i]; }, cnt, K_max, o, lse, head_rows, [&](int64_t at) { return row_index[at]; }, N_src,
      N_pad, N_v, n_text, M_v, M, B, scale, head, u, part);
}

// The tickets of shared rows, for calls with no kernel in front that clears them on its way (1.4 us at the least under the profiler, 5.5
// on average; a memset may not be recorded into a graph).
__global__ void __launch_bounds__(256) clear_tickets_kernel(int32_t* __restrict__ tickets, int n) {
  for (int i = threadIdx.x; i < n; i += 256) tickets[i] = 0;
}

static unsigned long long* g_clock_probe = nullptr;   // set by dfs_attn_clock_probe (diagnostic)

// Groups of waves that share a query block (kernel's KS): two where the work-groups leave SIMDs with less than one wave
// each.  A second wave per SIMD raises the matrix rate by a fifth, the merge costs some 4 us, so short lists of the one
// shape whose lone waves do well (d = 128, 128 rows) stay whole.  Measured (us a reuse step, one group -> two), 128 rows:
// d = 128, 44 blocks x 1 head 28.0 -> 29.2 with 9 kept, 83.6 -> 73.0 with all kept, 176 work-groups 92.8 -> 83.0, 264
// 140 -> 165; d = 64, 88 work-groups 22.5 -> 21.9, 264 31.5 -> 39.5.  64 rows (two waves per group): d = 64, 164
// work-groups 18.3 -> 16.9, 492 25.1 -> 23.3, 656 26.9 -> 30.7; d = 128, 246 29.4 -> 28.6, 328 31.0 -> 43.1.
// The host knows a list's room, K_max, not its length, and the two differ: a dense call whose lists have room for 9 blocks
// stays on one group (83.7 and 92.9 us above instead of 73.0 and 83.0), a list of 9 with room for all 44 takes two.
static int key_split(int d, int B, int64_t work_groups, int K_max) {
  if (B == 64 && d == 64) return work_groups <= 512 ? 2 : 1;
  if (B == 128 && d == 128 && K_max <= 16) return 1;
  return work_groups <= 256 ? 2 : 1;
}

// One tile buffer instead of two where the work-groups are more than two per CU (kernel's SLIM, d = 128, 64 rows).  Measured (two
// buffers over one, whole calls): 528 work-groups x 14 of 88 blocks 48.3 -> 41.3 us, 1 056 76.5 -> 72.4, 6 600 x 42 of 275 765 ->
// 711, dense 4 013 -> 3 630, 704 dense with log-sum-exp 182 -> 147; 328 work-groups x 14 of 82 30.5 -> 35.8, 352 dense 97 -> 136.  Not
// for sequences that all XCDs walk together (mapping 2), whose lists come from beyond L2: 2 364 work-groups x 178 of 1 182 blocks
// 1 049 -> 1 052, 14 184 8 104 -> 8 412.
static bool slim(int64_t work_groups, int ks, int mapping) { return ks == 1 && work_groups > 512 && mapping != 2; }

// Whether all XCDs walk one head together (kernel's mapping 2), an eighth of its video blocks each: once that fills the XCD's 64
// work-group slots (measured +3..6 % on the 75 600- and 118 800-token shapes, -4 % on the 17 550-token one, which stays on mapping 1).
static int xcd_blocks(const dfs_sizes& s) { return (s.M_v + 7) / 8; }
static bool walked_together(const dfs_sizes& s) { return xcd_blocks(s) >= 64; }

// Text rows in pieces of `blocks` key blocks, as long as a video row, or of five eighths of that: the merge of a text row, some 4 us, comes behind the
// last video row where all work-groups start at once.  For that all of them must, in the form that they had (key_split, slim): in blocks of 128 no more of them on
// a CU than before (query blocks: 512 at the most); in blocks of 64 up to the chip's 1 024 slots and at most 64 more than before, and a piece must lose a block and more
// for each that a row gains, which the merge reads; at d = 64, where a block is half the work, up to 768 and three blocks.
// Measured (us a reuse step, long -> short): 2 624 + 30 x 4, 20 kept, d = 64, blocks of 64, 17.6 -> 15.5,
// 2 624 + 77 x 8, 21 kept, d = 128 38.6 -> 32.1, 5 248 + 259 x 2, 16 kept, blocks of 128, d = 64 29.1 -> 25.0, d = 128 43.6 -> 36.3; not so, blocks of 64, d = 64:
// 960 + 259 x 20, 10 -> 8 blocks a piece, 500 -> 600 work-groups, 17.4 -> 21.1 (another form), 1 344 + 300 x 15, 11 -> 8, 540 -> 615, 20.5 -> 21.6, 2 624 + 259 x 12, 12 -> 8,
// 732 -> 852, 22.7 -> 25.0, 4 480 + 30 x 2, 12 -> 8, six -> nine pieces, 16.8 -> 17.3; blocks of 128, d = 128: 3 712 + 200 x 7, 15 -> 9, 245 -> 259, 45.2 -> 50.4.  592
// shapes in all: the 489 taken 0.98 to 1.21 times as fast, 1.073 in the mean; the others would be 0.82 to 1.11 times, 0.978.
static int shorter_pieces(const dfs_geom* g, const dfs_sizes& s, int K_max, int blocks) {
  const int shorter = blocks * 5 / 8 < 8 ? 8 : blocks * 5 / 8, pieces = (s.M + blocks - 1) / blocks, more = (s.M + shorter - 1) / shorter;
  const auto groups = [&](int n) { return int64_t(g->heads) * (s.M_v + int64_t(s.M_x) * n); };
  const auto form = [&](int n) {
    const int ks = key_split(g->d, g->B, groups(n), K_max);
    return 2 * ks + (g->d == 128 && g->B == 64 && slim(groups(n), ks, walked_together(s) ? 2 : 3) ? 1 : 0);
  };
  const int64_t few = groups(pieces), many = groups(more);
  if (form(pieces) != form(more)) return blocks;
  if (g->B == 128) return int64_t(g->heads) * s.M <= 512 && (few + 255) / 256 == (many + 255) / 256 ? shorter : blocks;
  if (many - few > 64 || many > (g->d == 64 ? 768 : 1024)) return blocks;
  return blocks - shorter >= (g->d == 64 ? 3 : 1) * (more - pieces) ? shorter : blocks;
}

// Work-groups per text block, and the key blocks each takes: about as many as a video row keeps (an eighth of all where
// K_max does not tell), at least eight, or fewer (shorter_pieces).  One where the video rows' work, in rounds of the chip's work-group slots, hides
// the text rows, which start first.  Measured (us a reuse step, whole -> split), 17 550 video + 77 text tokens, 21 of 138
// blocks kept: d = 64 x 2 heads 194 -> 58, x 12 331 -> 199, x 40 679 -> 618; d = 128 x 2 264 -> 88, x 12 519 -> 348, x 40
// 1 187 -> 1 142 (work of 1.7 text rows: whole by the rule, which is drawn for lists of the room they are given);
// 75 600 + 256 tokens x 8 heads 2 435 -> 2 436 (work of 0.96: whole).  A dense call with room for 22 blocks is taken for a
// short one and split: 1 209 -> 1 213 (d = 128, 8 heads).  Below 16 blocks there is nothing to win.
struct TextSplit { int splits, blocks; };
static TextSplit text_split(const dfs_geom* g, const dfs_sizes& s, int K_max, size_t scratch_bytes) {
  const TextSplit whole = {1, s.M};
  if (s.M_x == 0 || s.M < 16 || scratch_bytes == 0) return whole;
  const int64_t slots = g->B == 128 ? 512 : 1024, kept = K_max < s.M ? K_max : s.M;
  const int64_t likely = kept == s.M ? kept / 3 : kept;                  // adaptive lists are given room for all
  if (int64_t(g->heads) * s.M_v * likely * 5 >= 4 * slots * s.M) return whole;
  int blocks = int(2 * kept <= s.M ? kept : s.M / 8);
  if (blocks < 8) blocks = 8;
  if (2 * kept <= s.M) blocks = shorter_pieces(g, s, K_max, blocks);
  const size_t row = size_t(g->B) * (g->d + 4) * sizeof(float) * s.M_x * g->heads;         // one split of every text block
  const int64_t room = int64_t((scratch_bytes - align256(split_tickets(g, s) * sizeof(int32_t))) / row);
  if ((s.M + blocks - 1) / blocks > room) {
    if (room < 2) return whole;
    blocks = int((s.M + room - 1) / room);
  }
  return {(s.M + blocks - 1) / blocks, blocks};
}

// The last round of work-groups: `rows` query blocks of an XCD from slot `from` on, shared by `splits` work-groups each where a
// whole one would leave slots idle: a third of them and less at d = 128 with blocks of 128 (a lone wave per SIMD does most of
// what two do), half and less elsewhere, pieces of four key blocks and more.  Within eight rounds: beyond, the last one is short
// against the rest; two for the form with one buffer, whose work-groups end less evenly.  Measured (us, whole -> shared, kept of
// blocks x heads): d = 128, 44 of 107 x 5 (1.05 rounds) 253 -> 207, 60 of 342 x 6 (4.02) 1 006 -> 942, 107 of 228 x 3 (1.34, two
// pieces: whole by the rule) 573 -> 582; d = 64, 47 of 102 x 8 (1.06) 211 -> 181, 39 of 148 x 21 (4.06) 559 -> 542, blocks of 64, 63 of
// 492 x 3 (1.45) 142 -> 133; d = 128, blocks of 64, 130 of 279 x 4 (1.09) 391 -> 332, 28 of 159 x 27 (4.20: whole by the rule) 353 -> 368.
struct TailSplit { int from, rows, splits; };
static TailSplit tail_split(const dfs_geom* g, const dfs_sizes& s, int32_t K_max, int order, int text_slots, const TextSplit& ts, bool one_buffer,
                            size_t scratch_bytes) {
  const TailSplit none = {0, 1, 1};
  const int slots = 32 * (g->B == 128 ? (g->d == 64 ? 3 : 2) : g->d == 64 || one_buffer ? 4 : 2);     // resident work-groups of an XCD
  const int full = order / slots * slots, rows = order - full;
  if (scratch_bytes == 0 || int64_t(g->heads) * s.M < 512 || full == 0 || rows == 0 || full < text_slots) return none;
  if (full > (one_buffer ? 2 : 8) * slots) return none;
  const int64_t kept = K_max < s.M ? K_max : s.M, likely = kept == s.M ? kept / 3 : kept;     // as in text_split
  int splits = slots / rows;
  if (splits > 4) splits = 4;
  const int pieces = int(likely / (full == slots ? 4 : 6));
  if (splits > pieces) splits = pieces;
  if (splits < (g->d == 128 && g->B == 128 ? 3 : 2)) return none;
  const int64_t parts = 8 * int64_t(rows) * splits + (ts.splits > 1 ? int64_t(g->heads) * s.M_x * ts.splits : 0);
  const size_t have = scratch_bytes - align256(split_tickets(g, s) * sizeof(int32_t));
  if (size_t(parts) * g->B * (g->d + 4) * sizeof(float) > have) return none;
  return {full, rows, splits};
}

// Whether dfs_forward's attention gathers keys and values itself (kernel's SRC) instead of having them reordered in front.  It saves
// the reorder's way through memory, and on a reuse step its launch; it costs a tile's loads some ten instructions, 0.3 % of a long dense
// call.  Measured (us a call, reordered -> gathered; medians of three runs each, in turn on one card, whose spread is 0.1 to 1 %),
// reuse steps: d = 64, 512 tokens x 8 heads 11.9 -> 8.7, 2 565 + 77 x 12, blocks of 64, 30.0 -> 22.6, 17 550 x 48, 21 of 138 blocks,
// 689 -> 631; d = 128, 5 632 x 24, 9 of 44 blocks, 131 -> 99, 17 550 x 24, 21 of 138, 634 -> 573, 75 600 x 40, 60 of 591, 11 874 ->
// 11 319; refresh steps, whose pooling reorders on its way: 2 565 + 77 x 12 36.8 -> 35.5, 17 550 x 48, d = 64, 730 -> 692, 75 600 x 40
// 12 258 -> 11 982, 118 800 + 256 x 24, 93 of 929, 18 023 -> 17 850; dense: 17 550 x 12, d = 64, 988 -> 987, 75 600 x 40 98.8 ->
// 99.1 ms.  Not for sequences that all XCDs walk together at d = 64 or in blocks of 64, where the reorder is a smaller part: 75 600 tokens, dense, d = 64
// x 8 11 307 -> 11 476, d = 128, blocks of 64, x 2 6 633 -> 7 203, 119 of 1 182 blocks x 10 3 746 -> 3 854; d = 64 would win 2 to 3 %
// on short lists (48 of 591 blocks x 10 1 305 -> 1 267, 119 of 1 182 of 64 x 10 1 859 -> 1 824).  The host does not know whether a
// call is dense, so the line lies where dense calls break even.
// Not where the output lies over the keys or values either: they are then reordered before the first row is written.
bool attn_reads_source(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* k, const void* v, const void* o) {
  if (dtype == DFS_BF16 && walked_together(s) && !(g->d == 128 && g->B == 128)) return false;
  // fp32 tensors (on reuse steps, see dfs_forward): calls of 2^31 operations and less with every block kept, whose reorder is a launch more than it
  // is work.  (us) 256 tokens x 2 heads, d = 64, 11.0 -> 8.9; 1 024 x 3, d = 64 17.5 -> 14.2, d = 128 29.8 -> 24.7; 1 920 x 1, d = 64, dense 46.5 ->
  // 45.7; larger ones lose, the rows of a run lying apart: 1 920 + 30 x 6, d = 128, 127 -> 131, 3 968 x 8 236 -> 252.
  // One head dense at d = 128, a lone wave per SIMD at the most, loses all the same (768 tokens 39.0 -> 40.4, 2 048 87.7 -> 91.6) where its masked steps win (768, 2
  // of 12 blocks, 18.0 -> 14.8, half 26.5 -> 25.3, 2 048, half, 52.5 -> 51.5): the host does not know which they are.
  if (dtype == DFS_F32 && 4 * int64_t(g->heads) * g->d * double(s.N_pad) * double(s.N_pad) > 2147483648.0) return false;
  return apart(g, s, dtype, k, o) && apart(g, s, dtype, v, o);
}

// Rounds of attn_pairs_kernel, full ones; what is left is the other kernel's, whose work-groups are half as long.  The kernel is launched
// where lists may be dense, the host does not know, and costs a call whose lists are not 4.5 us (10 heads of 138 blocks, 7 kept, 100 -> 102.6
// us): so from 2 048 query blocks on, four rounds of work-groups.  Measured (ms, blocks one by one -> in pairs; all 591 kept): 3 heads 7.78 ->
// 7.56, 4 10.57 -> 10.15, 8 20.7 -> 19.9, 40 102.4 -> 97.7; 929 + 2 text blocks x 4 25.8 -> 25.25; with log-sum-exp, 4 heads of 591, recall's
// two calls and what is around them 12.26 -> 11.92; 60 of 591 kept x 40 11.05 -> 11.11, two runs of one side as far apart.  Not for
// sequences that an XCD takes whole (mapping 1): the blocks left over are then one XCD's (138 blocks x 24 heads, all kept, 3.33 -> 5.29).  At d
// = 64 eight waves would leave the CU two per SIMD instead of three (138 blocks x 48 heads, all kept, 3.74 -> 4.07).
static int pair_rounds(const dfs_geom* g, const dfs_sizes& s) {
  if (g->d != 128 || g->B != 128 || !walked_together(s) || int64_t(g->heads) * s.M < 2048) return 0;
  return pair_slots(s.M_v, s.M, g->heads) / PAIR_WGS;
}

// The dense pairs behind the last full round: their blocks, `rows` an XCD, shared by `splits` work-groups each where there is room (dfs_forward) and
// up to 32 are left, so that a whole one each would leave half of the XCD's slots and more idle for as long as a dense row takes.  Two
// pieces are worth their merge here, other than in tail_split, which shares masked rows behind pairs as elsewhere.  Measured (ms, whole
// -> shared; all kept): 591 blocks x 40 heads (16 rows left an XCD) 94.4 -> 93.6, x 8 19.28 -> 18.76, 520 x 5 (10) 9.58 -> 9.01; in two pieces
// 591 x 16 (32) 37.97 -> 37.15, 600 x 40 (32) 96.4 -> 96.0, 929 + 2 x 24 (22) 139.3 -> 138.9.  Masked calls that find nothing to share: 520 x 5, 52 kept,
// 1.020 -> 1.022, 929 + 2 x 24, 93 kept, 17.1 -> 17.1, two runs of one side as far apart.
struct PairsLeft { int rows, splits; };
static PairsLeft pairs_left(const dfs_geom* g, const dfs_sizes& s, int pairs, const TailSplit& tail, const TextSplit& ts, size_t scratch_bytes) {
  const int rows = 2 * (pair_slots(s.M_v, s.M, g->heads) - pairs * PAIR_WGS);
  if (scratch_bytes == 0 || rows == 0 || rows > 32) return {0, 1};
  const int splits = 64 / rows < 4 ? 64 / rows : 4;
  const int64_t parts = 8 * (int64_t(rows) * splits + int64_t(tail.rows) * tail.splits) + (ts.splits > 1 ? int64_t(g->heads) * s.M_x * ts.splits : 0);
  if (size_t(parts) * g->B * (g->d + 4) * sizeof(float) > scratch_bytes - align256(split_tickets(g, s) * sizeof(int32_t))) return {0, 1};
  return {rows, splits};
}

int run_sparse_attn(const dfs_geom* g, const dfs_sizes& s, int dtype, const void* q, const void* k, const void* v,
                    const int32_t* kv_idx, const int32_t* kv_cnt, int32_t K_max, float scale, void* o, float* lse,
                    const int32_t* row_index, bool kv_src, bool maybe_dense, bool zeroed, void* scratch, size_t scratch_bytes, hipStream_t st) {
  if (K_max < 1) return fail(DFS_ESHAPE, "dfs_sparse_attn_fwd: K_max=%d must be positive", K_max);
  if (dtype == DFS_BF16) {
    const int64_t total = int64_t(g->heads) * s.M;
    if (total > (int64_t(1) << 30)) return fail(DFS_ESHAPE, "dfs_sparse_attn_fwd: heads*M too large");
    const int chunk = xcd_blocks(s);
    const TextSplit ts = lse ? TextSplit{1, s.M} : text_split(g, s, K_max, scratch_bytes);
    const int mapping = walked_together(s) ? 2 : ts.splits > 1 ? 3 : 1;
    const int text_slots = (g->heads * s.M_x * ts.splits + 7) / 8, video_slots = int((int64_t(g->heads) * s.M_v + 7) / 8);
    const int per_xcd = mapping == 2 ? g->heads * chunk : mapping == 3 ? video_slots : int((total + 7) / 8);
    int32_t* tickets = static_cast<int32_t*>(scratch);
    float* part = reinterpret_cast<float*>(static_cast<char*>(scratch) + align256(split_tickets(g, s) * sizeof(int32_t)));
    const int64_t work_groups = total + int64_t(g->heads) * s.M_x * (ts.splits - 1);
    const int ks = key_split(g->d, g->B, work_groups, K_max);
    const bool one_buffer = g->d == 128 && g->B == 64 && slim(work_groups, ks, mapping);
    const int order = mapping >= 2 ? text_slots + per_xcd : per_xcd;     // slots of an XCD
    const int pairs = maybe_dense ? pair_rounds(g, s) : 0;
    TailSplit tail = lse || ks > 1 ? TailSplit{0, 1, 1} : tail_split(g, s, K_max, order, mapping >= 2 ? text_slots : 0, ts, one_buffer, scratch_bytes);
    const PairsLeft left = lse || pairs == 0 ? PairsLeft{0, 1} : pairs_left(g, s, pairs, tail, ts, scratch_bytes);
    if (left.rows > 0 && tail.splits == 1) tail = {order, 0, 1};         // nothing but what the pairs leave is shared
    if (!zeroed && (ts.splits > 1 || tail.splits > 1 || left.splits > 1)) clear_tickets_kernel<<<1, 256, 0, st>>>(tickets, int(split_tickets(g, s)));
    if (pairs > 0) {
#define ATTN_PAIRS(XX, SRC)                                                                                                            \
  attn_pairs_kernel<128, XX, SRC><<<8 * PAIR_WGS, 512, 0, st>>>(static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),            \
                                                                static_cast<const uint16_t*>(v), kv_cnt, static_cast<uint16_t*>(o), lse, row_index, \
                                                                s.N, s.N_pad, s.N_v, g->n_text, s.M_v, s.M, g->heads, scale, g_clock_probe, pairs)
      if (kv_src) ATTN_PAIRS(false, true);
      else if (lse) ATTN_PAIRS(true, false);
      else ATTN_PAIRS(false, false);
#undef ATTN_PAIRS
    }
    const int walked = order + tail.rows * (tail.splits - 1);
    dim3 grid(unsigned(8 * (walked + left.rows * left.splits)));
#define ATTN_X(DD, BB, XX, KS, SLIM, TAIL, SRC)                                                                                            \
  attn_bf16_kernel<DD, BB, XX, KS, SLIM, TAIL, SRC><<<grid, BB * 2 * KS, 0, st>>>(static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k), \
                                                        static_cast<const uint16_t*>(v), kv_idx, kv_cnt, K_max,                 \
                                                        static_cast<uint16_t*>(o), lse, row_index, s.N, s.N_pad, s.N_v,         \
                                                        g->n_text, s.M_v, s.M, int(total), per_xcd, mapping, scale, g_clock_probe, \
                                                        part, tickets, ts.splits, ts.blocks, tail.from, tail.rows, tail.splits)
#define ATTN_REST(XX, TAIL, SRC)                                                                                                           \
  attn_rest_kernel<128, 128, XX, TAIL, SRC><<<grid, 256, 0, st>>>(static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),               \
                                                                  static_cast<const uint16_t*>(v), kv_idx, kv_cnt, K_max,                         \
                                                                  static_cast<uint16_t*>(o), lse, row_index, s.N, s.N_pad, s.N_v,                 \
                                                                  g->n_text, s.M_v, s.M, int(total), per_xcd, mapping, scale, g_clock_probe,      \
                                                                  part, tickets, ts.splits, ts.blocks, tail.from, tail.rows, tail.splits, pairs,     \
                                                                  left.rows > 0 ? pair_slots(s.M_v, s.M, g->heads) : pairs * PAIR_WGS, walked, left.rows, left.splits)
#define ATTN_LSE(DD, BB, KS, SLIM) do { if (lse) ATTN_X(DD, BB, true, KS, SLIM, false, false); else ATTN_X(DD, BB, false, KS, SLIM, false, false); } while (0)
#define ATTN_WHOLE(DD, BB, KS, SLIM) do { if (kv_src) ATTN_X(DD, BB, false, KS, SLIM, false, true); else ATTN_LSE(DD, BB, KS, SLIM); } while (0)
#define ATTN_TAIL(DD, BB, SLIM) do { if (kv_src) ATTN_X(DD, BB, false, 1, SLIM, true, true); else ATTN_X(DD, BB, false, 1, SLIM, true, false); } while (0)
#define ATTN_1(DD, BB, SLIM) do { if (tail.splits > 1) ATTN_TAIL(DD, BB, SLIM); else ATTN_WHOLE(DD, BB, 1, SLIM); } while (0)
#define ATTN_KS(DD, BB) do { if (ks == 2) ATTN_WHOLE(DD, BB, 2, false); else ATTN_1(DD, BB, false); } while (0)
    if (pairs > 0) {
      if (lse) ATTN_REST(true, false, false);
      else if (tail.splits > 1 || left.splits > 1) { if (kv_src) ATTN_REST(false, true, true); else ATTN_REST(false, true, false); }
      else if (kv_src) ATTN_REST(false, false, true);
      else ATTN_REST(false, false, false);
    }
    else if (g->d == 64) { if (g->B == 64) ATTN_KS(64, 64); else ATTN_KS(64, 128); }
    else if (g->B == 128) ATTN_KS(128, 128);
    else if (one_buffer) ATTN_1(128, 64, true);
    else if (tail.splits > 1) ATTN_X(128, 64, false, 1, false, true, false);      // only sequences that all XCDs walk together: none is gathered
    else if (ks == 2) ATTN_WHOLE(128, 64, 2, false);
    else ATTN_WHOLE(128, 64, 1, false);
#undef ATTN_KS
#undef ATTN_1
#undef ATTN_TAIL
#undef ATTN_WHOLE
#undef ATTN_LSE
#undef ATTN_REST
#undef ATTN_X
  } else {
    if (g->heads > 65535) return fail(DFS_ESHAPE, "heads=%d exceeds 65535", g->heads);
    dim3 grid(unsigned(s.M * (g->B / 32)), unsigned(g->heads));
#define ATTN_F32(DD, SRC)                                                                                                       \
  attn_f32_kernel<DD, SRC><<<grid, 512, 0, st>>>(static_cast<const float*>(q), static_cast<const float*>(k),                         \
                                            static_cast<const float*>(v), kv_idx, kv_cnt, K_max, static_cast<float*>(o), lse,   \
                                            row_index, s.N, s.N_pad, s.N_v, g->n_text, s.M_v, s.M, g->B, scale)
    if (g->d == 64) { if (kv_src) ATTN_F32(64, true); else ATTN_F32(64, false); }
    else            { if (kv_src) ATTN_F32(128, true); else ATTN_F32(128, false); }
#undef ATTN_F32
  }
  return launch_status("dfs_sparse_attn_fwd");
}

}  // namespace dfs

using namespace dfs;

extern "C" int dfs_attn_clock_probe(uint64_t* counters) {
  if (misaligned(8, {counters})) return fail(DFS_EINVAL, "dfs_attn_clock_probe: counters must be 8-byte aligned");
  g_clock_probe = reinterpret_cast<unsigned long long*>(counters);
  return DFS_OK;
}

extern "C" int dfs_sparse_attn_fwd(const dfs_geom* g, int dtype, const void* q_perm, const void* k_perm, const void* v_perm,
                                   const int32_t* kv_idx, const int32_t* kv_cnt, int32_t K_max, float scale, void* o_perm,
                                   float* lse, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (dtype != DFS_F32 && dtype != DFS_BF16) return fail(DFS_EDTYPE, "dtype %d is not DFS_F32 or DFS_BF16", dtype);
  if (!q_perm || !k_perm || !v_perm || !kv_idx || !kv_cnt || !o_perm) return fail(DFS_EINVAL, "dfs_sparse_attn_fwd: NULL argument");
  if (misaligned(16, {q_perm, k_perm, v_perm, o_perm}) || misaligned(4, {kv_idx, kv_cnt, lse}))
    return fail(DFS_EINVAL, "dfs_sparse_attn_fwd: tensors must be 16-byte aligned, index and fp32 arrays 4-byte aligned");
  if (!(scale > 0.f)) return fail(DFS_EINVAL, "dfs_sparse_attn_fwd: scale must be positive");
  return run_sparse_attn(g, s, dtype, q_perm, k_perm, v_perm, kv_idx, kv_cnt, K_max, scale, o_perm, lse, nullptr, false, true, false, nullptr, 0, as_stream(stream));
}

extern "C" int dfs_sparse_attn_fwd_src(const dfs_geom* g, int dtype, const void* q, const int32_t* perm_pad, const void* k_perm,
                                       const void* v_perm, const int32_t* kv_idx, const int32_t* kv_cnt, int32_t K_max, float scale,
                                       void* o, float* lse, void* stream) {
  dfs_sizes s;
  int rc = check_geom(g, &s);
  if (rc) return rc;
  if (dtype != DFS_BF16) return fail(DFS_EDTYPE, "dfs_sparse_attn_fwd_src: bf16 tensors only");
  if (!q || !perm_pad || !k_perm || !v_perm || !kv_idx || !kv_cnt || !o) return fail(DFS_EINVAL, "dfs_sparse_attn_fwd_src: NULL argument");
  if (misaligned(16, {q, k_perm, v_perm, o}) || misaligned(4, {perm_pad, kv_idx, kv_cnt, lse}))
    return fail(DFS_EINVAL, "dfs_sparse_attn_fwd_src: tensors must be 16-byte aligned, index and fp32 arrays 4-byte aligned");
  if (!(scale > 0.f)) return fail(DFS_EINVAL, "dfs_sparse_attn_fwd_src: scale must be positive");
  return run_sparse_attn(g, s, dtype, q, k_perm, v_perm, kv_idx, kv_cnt, K_max, scale, o, lse, perm_pad, false, true, false, nullptr, 0, as_stream(stream));
}
