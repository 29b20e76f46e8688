// Attention of fp32 tensors: what a work-group does for 32 query rows (device code shared by the kernel of its own and the one that scores
// and selects in front of it).
#pragma once
#include <math.h>

#include "common.h"

namespace dfs {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int block_real_rows(int blk, int B, int M_v, int64_t N_v, int n_text) {
  int64_t real = blk < M_v ? N_v - int64_t(blk) * B : int64_t(n_text) - int64_t(blk - M_v) * B;
  return real >= B ? B : (real <= 0 ? 0 : int(real));
}

// A work-group owns 32 query rows of one (head, query block); its eight waves split the kept keys, 32 at a
// time in turn, each with a softmax of its own, and merge through LDS at the end, because calls on fp32 tensors are
// small (a few thousand tokens) and have few query rows to fill the chip with, so what bounds them is one row's serial
// walk through its keys.  Both products run on the fp32 matrix instruction (32x32x2: full fp32, the chip's fastest fp32
// rate), transposed as in the bf16 kernel, with operands straight from memory: no key is shared between waves.  The
// order of the summed features and of the output features is free, so lanes load 16 bytes of a key row (features
// 8 c + 4 h ..) and D / 32 consecutive value features each.
// Measured against one thread per query row with operands from LDS (which at d = 128 spilled its rows): 256 tokens x
// 2 heads, d = 64, 2 of 4 blocks 89 -> 9 us; 3 600 tokens + 30 text rows x 6 heads, d = 128, 9 of 29 blocks 6 670 ->
// 268 us (16 and 330 without the requests ahead of their use); error against 64 bits a half to a ninth of that kernel's
// (3.2e-7 instead of 2.1e-6 at d = 128), since a row's sums are now eight shorter ones.
// SRC: keys and values in source order, as in the bf16 kernel.  A lane looks up the position of one key of a run, a run ahead; for the values
// the positions go to the lanes that want them through scalars (through LDS, each a wait, the kernel took up to 2 % longer).
constexpr int AF_WAVES = 8;
// Room in LDS.  The waves' outputs are added ((0 + 4) + (2 + 6)) + ((1 + 5) + (3 + 7)) either way: at once, an eighth by every wave, behind one
// barrier; or, with half the room, wave onto wave in three steps, where the waves that are done leave early and the next work-group starts
// beside the rest.  At once is the faster way for short lists (256 tokens x 2 heads, a reuse step 9.2 -> 8.9 us) and at d = 128, where no second
// work-group fits (3 968 tokens x 8 heads, 10 of 31 blocks, 235.9 -> 231.9 us); d = 64 there 130.7 -> 134.2, dense 336 -> 345.
template <int D, bool AT_ONCE_> struct AttnF32Room {
  static constexpr bool AT_ONCE = AT_ONCE_;
  float m[AF_WAVES][32], l[AF_WAVES][32];
  float o[AT_ONCE ? AF_WAVES : AF_WAVES / 2][D / 32 * 16 * 64];
};
// A lane's query row, lane (n, h): features 8 c + 4 h .. + 3 of row n.  `at`: where it lives, -1 for a pad row (which reads row 0; it is not
// written); of a tensor of head_rows rows a head.
template <int D> struct QueryRow {
  int64_t at;
  f32x4 x[D / 8];
  __device__ __forceinline__ void load(const float* __restrict__ q, int64_t head_rows, int head, int64_t row) {
    const int h = (threadIdx.x >> 5) & 1;
    at = row < head_rows ? row : -1;
#pragma unroll
    for (int c = 0; c < D / 8; ++c) x[c] = *reinterpret_cast<const f32x4*>(q + (int64_t(head) * head_rows + (at < 0 ? 0 : at)) * D + 8 * c + 4 * h);
  }
};
// Rows 32 part .. of query block u, whose own (`query`) live in a tensor of head_rows rows a head, as the output's do; idx(i): its list, of cnt_in
// blocks; position(row): with SRC, where a row of the order lives.
template <int D, bool SRC, class Room, class List, class Position>
__device__ __forceinline__ void attn_f32_rows(Room& room, const QueryRow<D>& query, const float* __restrict__ k, const float* __restrict__ v,
                                              List idx, int cnt_in, int K_max, float* __restrict__ o, float* __restrict__ lse, int64_t head_rows,
                                              Position position, int64_t N_src, int64_t N_pad, int64_t N_v, int n_text, int M_v, int M, int B,
                                              float scale, int head, int u, int part) {
  constexpr int NW = AF_WAVES, DT = D / 32;
  typedef float vrow __attribute__((ext_vector_type(DT)));
  auto &s_m = room.m, &s_l = room.l;
  auto& s_o = room.o;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int log_parts = B == 128 ? 2 : 1, parts = 1 << log_parts;        // per block: groups of 32 query rows, runs of 32 keys
  const bool dense = cnt_in >= M;
  const int cnt = dense ? M : (cnt_in < 0 ? 0 : (cnt_in > K_max ? K_max : cnt_in));
  const float* kh = k + int64_t(head) * (SRC ? N_src : N_pad) * D;
  const float* vh = v + int64_t(head) * (SRC ? N_src : N_pad) * D;
  f32x4 qf[D / 8];
#pragma unroll
  for (int c = 0; c < D / 8; ++c) qf[c] = query.x[c];
  // Softmax in base 2.  The factor is positive, so that masked logits (-inf) stay what they are and a row's maximum is the
  // largest exponent; the sign of a scale that is not goes to Q (0 as well: every logit is 0 then).
  float c2 = scale * 1.4426950408889634f;
  if (!(scale > 0.f)) {
    const float sign = scale < 0.f ? -1.f : scale;
    c2 = scale < 0.f ? -c2 : 1.f;
#pragma unroll
    for (int c = 0; c < D / 8; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) qf[c][e] *= sign;
  }
  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;              // reference in the exponent's units, this lane half's share of the sum
  // This wave's next run of keys, skipping what lies wholly behind the real rows of a ragged block.
  const int runs = cnt << log_parts;
  int64_t row = 0;                                   // first key row of the run, the real ones among its 32
  int real = 1;
  auto next_run = [&](int j) {
    for (; j < runs; j += NW) {
      int blk = dense ? j >> log_parts : idx(j >> log_parts);
      blk = unsigned(blk) < unsigned(M) ? blk : 0;   // a corrupt list must not read out of bounds
      const int r0 = j % parts * 32;
      const int left = block_real_rows(blk, B, M_v, N_v, n_text) - r0;
      if (left <= 0) continue;
      row = int64_t(blk) * B + r0;
      real = left < 32 ? left : 32;
      break;
    }
    return j;
  };
  // pad rows are never read: their keys and values repeat the last real one and are masked
  f32x4 kf[D / 8];
  vrow vf[16];
  auto load_k = [&](const float* base, uint32_t off, int c) { kf[c] = *reinterpret_cast<const f32x4*>(base + off + 8 * c); };
  // SRC: rows come through buffer descriptors of the head, whose bounds make zeros of positions that are none (a damaged order); a
  // select of its own behind the load waits for it there (3 968 tokens x 8 heads dense, d = 128, 605 -> 721 us).
  auto k_desc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kh), 0, int(N_src * (4 * D)), 0x00020000);
  auto v_desc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vh), 0, int(N_src * (4 * D)), 0x00020000);
  auto gather_k = [&](uint32_t off, int c) { kf[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(k_desc, off + 16 * h, 32 * c, 0)); };
  auto gather_v = [&](uint32_t off, int i) {
    if constexpr (DT == 2) vf[i] = __builtin_bit_cast(vrow, __builtin_amdgcn_raw_buffer_load_b64(v_desc, off + 4 * DT * n, 0, 0));
    else vf[i] = __builtin_bit_cast(vrow, __builtin_amdgcn_raw_buffer_load_b128(v_desc, off + 4 * DT * n, 0, 0));
  };
  // byte offset of a position
  auto offset_of = [&](uint32_t at) { return (at < uint32_t(N_src) ? at : 0x80000000u / (4 * D)) * uint32_t(4 * D); };
  auto look_up = [&]() { return offset_of(uint32_t(position(row + n))); };         // of key n of the run at hand (row: whole runs)
  uint32_t pos = 0;
  int j = next_run(wave);
  // The keys of a run are requested during the value products of the run before; without SRC at d = 64 at its own start, where the two waves of a
  // SIMD cover for one another and loads between the products cost more (3 968 tokens x 8 heads, dense, 336 -> 345 us).
  constexpr bool AHEAD = SRC || D == 128;
  if (SRC && j < runs) pos = look_up();
  if (AHEAD && j < runs) {
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      if (SRC) gather_k(pos, c);
      else load_k(kh + row * D, uint32_t(n < real ? n : real - 1) * D + 4 * h, c);
    }
  }
  while (j < runs) {
    const float* vb = vh + row * D;
    const int here = real;
    const uint32_t at = pos;
    if (SRC) {
      j = next_run(j + NW);
      pos = look_up();                               // behind the last run: that run's once more
    }
    if (!AHEAD) {
#pragma unroll
      for (int c = 0; c < D / 8; ++c) load_k(kh + row * D, uint32_t(n < real ? n : real - 1) * D + 4 * h, c);
    }
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    // the values are requested while the logits are formed, the keys of the next run during the value products
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c][e], qf[c][e], s, 0, 0, 0);
#pragma unroll
      for (int i = c * 128 / D; i < (c + 1) * 128 / D; ++i) {
        const int key = 8 * (i / 4) + 4 * h + i % 4;
        if (SRC) {
          const uint32_t at0 = __builtin_amdgcn_readlane(at, 8 * (i / 4) + i % 4), at1 = __builtin_amdgcn_readlane(at, 8 * (i / 4) + i % 4 + 4);
          gather_v(h == 0 ? at0 : at1, i);
        } else {
          vf[i] = *reinterpret_cast<const vrow*>(vb + (uint32_t(key < here ? key : here - 1) * D + DT * n));
        }
      }
    }
    if (!SRC) j = next_run(j + NW);
    // s[i]: key 8 (i / 4) + 4 h + i % 4 of the run against query row n
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (8 * (i / 4) + 4 * h + i % 4 >= here) s[i] = -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    const float m_new = fmaxf(m_run, fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * c2);
    const float ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - ref);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c2, -ref));
      l_run += s[i];
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
    const float* kb = kh + row * D;                  // behind the last run: that run once more
    const uint32_t k_off = uint32_t(n < real ? n : real - 1) * D + 4 * h;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bool pad = 8 * (i / 4) + 4 * h + i % 4 >= here;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(pad ? 0.f : vf[i][dt], s[i], oacc[dt], 0, 0, 0);
#pragma unroll
      for (int c = i * D / 128; c < (i + 1) * D / 128; ++c) {
        if (SRC) gather_k(pos, c);
        else if (AHEAD) load_k(kb, k_off, c);
      }
    }
  }
  // merge: a common reference, then the sums, wave onto wave in a tree
  const auto lw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
  s_m[wave][n] = m_run;
  s_l[wave][n] = __uint_as_float(lw[0]) + __uint_as_float(lw[1]);
  __syncthreads();
  float m_all = s_m[0][n], l_all = 0.f;
#pragma unroll
  for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, s_m[w][n]);
  const float ref = m_all == -INFINITY ? 0.f : m_all;
#pragma unroll
  for (int w = 0; w < NW; ++w) l_all += s_l[w][n] * __builtin_amdgcn_exp2f(s_m[w][n] - ref);
  const float share = __builtin_amdgcn_exp2f(m_run - ref);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] *= share;
  // no keys: a zero row; keys whose weights all vanish (logits of -inf only): undefined, NaN as 0 / 0
  const float inv = l_all > 0.f ? 1.0f / l_all : cnt > 0 ? NAN : 0.f;
  float* orow = o + (int64_t(head) * head_rows + query.at) * D + DT * 4 * h;
  auto put = [&](int i, const vrow& w) { *reinterpret_cast<vrow*>(orow + DT * (8 * (i / 4) + i % 4)) = w; };
  if constexpr (Room::AT_ONCE) {
    if (wave < runs) {                               // the others had no run: nothing to add
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) s_o[wave][(dt * 16 + i) * 64 + lane] = oacc[dt][i];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int i = 2 * wave + e;
      vrow w;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        float p[NW];
#pragma unroll
        for (int x = 0; x < NW; ++x) p[x] = x < runs ? s_o[x][(dt * 16 + i) * 64 + lane] : 0.f;
#pragma unroll
        for (int half = NW / 2; half >= 1; half /= 2)
#pragma unroll
          for (int x = 0; x < half; ++x) p[x] += p[x + half];
        w[dt] = p[0] * inv;
      }
      if (query.at >= 0) put(i, w);
    }
  } else {
#pragma unroll
    for (int half = NW / 2; half >= 1; half /= 2) {
      if (runs <= half) continue;                    // the upper waves had no run: nothing to add
      if (wave >= half && wave < 2 * half) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i) s_o[wave - half][(dt * 16 + i) * 64 + lane] = oacc[dt][i];
      }
      __syncthreads();
      if (wave < half) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[dt][i] += s_o[wave][(dt * 16 + i) * 64 + lane];
      }
      __syncthreads();
    }
    if (wave != 0) return;
    if (query.at >= 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        vrow w;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) w[dt] = oacc[dt][i] * inv;
        put(i, w);
      }
    }
  }
  if (lse && wave == 0 && h == 0)
    lse[int64_t(head) * N_pad + int64_t(u) * B + part * 32 + n] = l_all > 0.f ? (ref + __builtin_amdgcn_logf(l_all)) * 0.6931471805599453f : -INFINITY;
}

}  // namespace dfs
