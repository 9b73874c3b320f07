// Importance scores of the prompt tokens (the H2O accumulated attention at
// the end of prefill, Section 3.1 / Section 4.1): every prompt query i
// attends causally to keys 0..i, and token j's score is the sum of its
// softmax probabilities over all queries i >= j and over the query heads
// that share its KV head,
//   score[b, h, j] = sum_{g in group(h)} sum_{i >= j} softmax_i(q_i . k / sqrt(d))_j.
// The logits are a dense contraction (Q K^T per head), so both passes run
// on the matrix cores (v_mfma_f32_32x32x16_f16, fp16 operands as given, fp32
// accumulation):
//   pass 1  a wave holds 64 queries of one query head and streams the causal
//           keys past them: running maximum (raised lazily) and normaliser of
//           every query, in log2 units;
//   pass 2  a wave holds 64 keys of one KV head and streams the queries of
//           every head of the group past them: the logits again, turned into
//           probabilities with the pass-1 statistics and summed per key.
// In both the streamed rows pass through LDS, shared by the block's four
// waves, and the C tile has keys along its rows and queries along its columns,
// so a lane holds one query per tile: its statistics are two scalars, and a
// logit costs one FMA, one exp2 and one add (pass 1) or FMA (pass 2).
// Tiles entirely below the causal diagonal (nearly all) skip the mask.
// Short prompts have a kernel of their own for each pass (short_pass).
// Bound: the matrix cores and the VALU together, at the clock the chip holds
// under both (about 2 GHz): per 32 x 32 tile 256 cycles of MFMA beside some 300
// of FMA, exp2 and add.  Streaming through LDS instead of by every wave from
// L2, one VALU instruction less per logit and no wait inside the loop:
// 16 x 32/8 heads x 16384 tokens 77.9 -> 36.8 ms (0.96 PFLOP/s on the matrix
// cores, a large fp16 library product reaches 1.31), 8 x 32 x 4096 3.51 ->
// 1.38 ms, 1 x 40 x 1531 224 -> 56 us.  Three waves per SIMD with 32-row
// tiles, priorities around the MFMAs and register staging measured even.
// Lane l of a wave: operand row l % 32, channels [16 i + 8 (l / 32), + 8) of
// MFMA i (the same split on both sides, so eight MFMAs cover 128 channels);
// result register r is tile row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
#include <algorithm>

#include "mikv_internal.h"

namespace mikv {

namespace {

constexpr int kThreads = 256;
constexpr int kWaveRows = 64;          // stationary rows per wave (two 32-row tiles)
constexpr int kRowWords = kHeadDim / 8;  // 16-byte words per fp16 row
constexpr float kLog2e = 1.4426950408889634f;
// Raise a query's running maximum when a lane's 16 terms of a tile sum past
// this.
constexpr float kRaise = 1024.0f;

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));

__device__ inline h8_t as_h8(u4_t v) { return __builtin_bit_cast(h8_t, v); }

// Rows of an LDS tile: 16-byte word c of row r sits at word c ^ (r % 16), so
// that the 16 lanes that one LDS cycle serves touch every bank once, both
// when a row is written and when 16 rows are read at the same word.
__device__ inline int lds_word(int row, int c) { return row * kRowWords + (c ^ (row & 15)); }

// The streamed tile of TR rows goes from memory straight to LDS (each wave
// instruction moves 1 KiB: four rows, lane l the word that belongs at word
// l % 16 of row l / 16), through a descriptor that ends with the last row:
// rows past it arrive as zeros.  The whole offset is in the vector operand: the
// scalar one is no part of the bounds check.  REPEAT: past the prompt the last
// row again instead (pass 2, whose sums take every query of the tile: such a
// query's logit is infinite or NaN only where the last query's is, and its
// statistics make it a probability of 0, where zeros would make NaN of an
// infinite key; pass 1 masks the keys past its queries, where the clamp would
// cost 0.3 %).
template <int TR, bool REPEAT>
__device__ inline void stage(u4_t *lds, const uint16_t *rows, int row0, int T) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = 4 * wave + (lane >> 4), last = min(TR, T - row0) - 1;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t *>(rows + (int64_t)row0 * kHeadDim), (short)0, (last + 1) * kHeadDim * 2, 0x00020000);
  const uint32_t word = 16u * (uint32_t)((lane & 15) ^ row);
#pragma unroll
  for (int u = 0; u < TR / 16; ++u) {
    const int r = REPEAT ? min(row + 16 * u, last) : row + 16 * u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(lds + (16 * u + 4 * wave) * kRowWords),
                                             16, (uint32_t)r * (kHeadDim * 2) + word, 0, 0, 0);
  }
}

__device__ inline void load_stationary(const uint16_t *base, int row0, int T, u4_t op[2][8]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const uint16_t *r = base + (int64_t)min(row0 + 32 * b + (lane & 31), T - 1) * kHeadDim + 8 * (lane >> 5);
#pragma unroll
    for (int i = 0; i < 8; ++i) op[b][i] = *reinterpret_cast<const u4_t *>(r + 16 * i);
  }
}

// Byte offset of the lane's word 0 of row 0 of a tile; its word i of row r
// (r a multiple of 32) is at (offset ^ 32 i) + 256 r.
__device__ inline uint32_t tile_offset() {
  const int lane = threadIdx.x & 63;
  return 16u * (uint32_t)lds_word(lane & 31, lane >> 5);
}
__device__ inline u4_t read_word(const u4_t *lds, uint32_t off, int row0, int i) {
  return *reinterpret_cast<const u4_t *>(reinterpret_cast<const char *>(lds) + (off ^ (32u * i)) + 256 * row0);
}
__device__ inline void read_tile(const u4_t *lds, uint32_t off, int row0, u4_t op[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) op[i] = read_word(lds, off, row0, i);
}

__device__ inline void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

__device__ inline f16_t splat(float v) {
  f16_t d;
#pragma unroll
  for (int r = 0; r < 16; ++r) d[r] = v;
  return d;
}

// 32 x 32 logits: rows `key` tile, columns `query` tile.
__device__ inline f16_t logits(const u4_t key[8], const u4_t query[8]) {
  f16_t d = splat(0.0f);
#pragma unroll
  for (int i = 0; i < 8; ++i) d = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_h8(key[i]), as_h8(query[i]), d, 0, 0, 0);
  return d;
}

// One pipeline step: the logits `next` = key x query on the matrix cores and,
// between their eight MFMAs (32 cycles each), the exponentials of the previous
// tile `cur` on the VALU: per MFMA two FMAs, two exp2 and two uses, which fill
// those 32 cycles.  use(r, p) takes the term p of tile register r.  With LOAD
// the words of the LDS tile at row0 are read into `ahead` on the way.
template <bool LOAD, class Use>
__device__ inline void step(f16_t &next, const u4_t (&key)[8], const u4_t (&query)[8], const f16_t &cur, float s2scale,
                            float m, u4_t (&ahead)[8], const u4_t *lds, uint32_t off, int row0, Use use) {
  f16_t d = splat(0.0f);
  float x0 = fmaf(cur[0], s2scale, -m), x1 = fmaf(cur[1], s2scale, -m), e0 = 0.0f, e1 = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    d = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_h8(key[i]), as_h8(query[i]), d, 0, 0, 0);
    if constexpr (LOAD) ahead[i] = read_word(lds, off, row0, i);
    const float p0 = __builtin_amdgcn_exp2f(x0), p1 = __builtin_amdgcn_exp2f(x1);
    if (i < 7) {
      x0 = fmaf(cur[2 * i + 2], s2scale, -m);
      x1 = fmaf(cur[2 * i + 3], s2scale, -m);
    }
    if (i > 0) {
      use(2 * i - 2, e0);
      use(2 * i - 1, e1);
    }
    e0 = p0;
    e1 = p1;
    __builtin_amdgcn_sched_barrier(0);
  }
  use(14, e0);
  use(15, e1);
  next = d;
}

__device__ inline int tile_row(int r) { return 8 * (r >> 2) + 4 * ((threadIdx.x & 63) >> 5) + (r & 3); }

__device__ inline float exp_sum(const f16_t &d, float s2scale, float m) {
  float t[2] = {0.0f, 0.0f};
#pragma unroll
  for (int r = 0; r < 16; ++r) t[r & 1] += __builtin_amdgcn_exp2f(fmaf(d[r], s2scale, -m));
  return t[0] + t[1];
}

// Block -> (unit, index) with index 0 the longest.  A unit's blocks stream the
// same head's rows.  Workgroups go to the eight XCDs in turn: a unit keeps to
// one XCD, and `run` of its blocks, about equally long, follow each other there,
// so that its L2 serves most of their rows; over the runs the longest go first
// for every unit, so that the grid ends on its shortest blocks.  False: no work
// (the last group's units count as eight, the last run's blocks as `run`).
__device__ inline bool block_unit(int units, int per_unit, int run, int &unit, int &idx) {
  const int groups = (units + 7) / 8, e = blockIdx.x >> 3;
  const int r = e / (groups * run), rem = e % (groups * run);
  unit = 8 * (rem / run) + (blockIdx.x & 7);
  idx = r * run + rem % run;
  return unit < units && idx < per_unit;
}

// Rows per streamed tile with WS waves on the same stationary rows, and the
// 32-row subtiles each wave takes of it.
template <int WS>
constexpr int tile_rows() { return WS == 4 ? 128 : 64; }
template <int WS>
constexpr int subtiles() { return tile_rows<WS>() / 32 / WS; }

// Pass 1: (max, 1 / normaliser) of every query, log2 units.  WS waves of the
// block take the same 64 queries and share out the 32-key subtiles.
template <int WS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void prefill_rowstats_kernel(const uint16_t *q, const uint16_t *k, int q_heads, int kv_heads, int units, int nblk,
                             int run, int T, float s2scale, float2 *stats) {
  constexpr int TR = tile_rows<WS>(), SUBS = subtiles<WS>(), kCols = kWaveRows * 4 / WS;
  __shared__ u4_t s_rows[2][TR * kRowWords];
  __shared__ float2 s_ml[WS > 1 ? 4 : 1][kWaveRows];
  const int lane = threadIdx.x & 63, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform for the compiler too
  const int wc = wave / WS, ws = wave % WS;
  const int G = q_heads / kv_heads;
  int hk, idx;
  if (!block_unit(units, nblk * G, run, hk, idx)) return;
  const int qh = hk * G + idx % G;                       // = b * q_heads + head
  const int i_base = (nblk - 1 - idx / G) * kCols;       // longest first
  const int i_wave = i_base + kWaveRows * wc;
  const uint16_t *qb = q + (int64_t)qh * T * kHeadDim, *kb = k + (int64_t)hk * T * kHeadDim;
  stage<TR, false>(s_rows[0], kb, 0, T);
  u4_t bq[2][8];
  load_stationary(qb, i_wave, T, bq);
  const uint32_t off = tile_offset();
  const int sub0 = ws * SUBS;  // the wave's subtiles of each tile
  // Each lane keeps the maximum and the sum of its own half of a query's
  // keys.  The maximum is raised only where a tile's terms sum past kRaise
  // (or to infinity: it starts at -inf), so that the common tile needs no
  // maximum at all.
  float m[2] = {-__builtin_huge_valf(), -__builtin_huge_valf()}, l[2] = {0.0f, 0.0f};
  auto add = [&](const f16_t &d, int cb, float ts) {
    if (__ballot(!(ts <= kRaise))) {
      if (!(ts <= kRaise)) {
        float mx = d[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, d[r]);
        const float mn = fmaxf(m[cb], mx * s2scale);
        // without a finite logit so far the sum is 0, or NaN (which the maximum
        // passes over)
        const float ref = mn == -__builtin_huge_valf() ? 0.0f : mn;
        l[cb] *= m[cb] == -__builtin_huge_valf() ? 0.0f : __builtin_amdgcn_exp2f(m[cb] - ref);
        m[cb] = mn;
        ts = exp_sum(d, s2scale, ref);
      }
    }
    l[cb] += ts;
  };
  const int n_tiles = (min(T, i_base + kCols) + TR - 1) / TR, n_full = i_base / TR;
  wait_loads();
  __syncthreads();
  // tiles wholly below the diagonal for every wave of the block
  f16_t d0, d1 = splat(-__builtin_huge_valf());  // the first step's previous tile adds nothing
  for (int t = 0; t < n_full; ++t) {
    const u4_t *rows = s_rows[t & 1];
    u4_t a[SUBS][8];
    read_tile(rows, off, 32 * sub0, a[0]);
#pragma unroll
    for (int s = 0; s < SUBS; ++s) {
      float ts[2] = {0.0f, 0.0f};
      auto use = [&](int r, float p) { ts[r & 1] += p; };
      if constexpr (SUBS == 2) {
        if (s == 0)
          step<true>(d0, a[s], bq[0], d1, s2scale, m[1], a[1], rows, off, 32 * (sub0 + 1), use);
        else
          step<false>(d0, a[s], bq[0], d1, s2scale, m[1], a[0], rows, off, 0, use);
      } else {
        step<false>(d0, a[s], bq[0], d1, s2scale, m[1], a[0], rows, off, 0, use);
      }
      add(d1, 1, ts[0] + ts[1]);
      // after the tile's last LDS read: the compiler holds LDS reads back for
      // loads to LDS that are under way
      if (s == 0) stage<TR, false>(s_rows[(t + 1) & 1], kb, min(t + 1, n_tiles - 1) * TR, T);
      ts[0] = ts[1] = 0.0f;
      step<false>(d1, a[s], bq[1], d0, s2scale, m[0], a[0], rows, off, 0, use);
      add(d0, 0, ts[0] + ts[1]);
    }
    wait_loads();
    __syncthreads();
  }
  add(d1, 1, exp_sum(d1, s2scale, m[1]));
  // the tiles on the diagonal
  for (int t = n_full; t < n_tiles; ++t) {
    const u4_t *rows = s_rows[t & 1];
#pragma unroll
    for (int s = 0; s < SUBS; ++s) {
      const int j0 = t * TR + 32 * (sub0 + s);
      if (j0 >= i_wave + kWaveRows) continue;  // above the diagonal (wave-uniform)
      u4_t a[8];
      read_tile(rows, off, 32 * (sub0 + s), a);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        f16_t d = logits(a, bq[cb]);
        const int i = i_wave + 32 * cb + n;
#pragma unroll
        for (int r = 0; r < 16; ++r) d[r] = j0 + tile_row(r) <= i ? d[r] : -__builtin_huge_valf();
        add(d, cb, exp_sum(d, s2scale, m[cb]));
      }
    }
    stage<TR, false>(s_rows[(t + 1) & 1], kb, min(t + 1, n_tiles - 1) * TR, T);
    wait_loads();
    __syncthreads();
  }
  // merge the two lanes of a query, then the WS waves
  auto merge = [](float &ma, float &la, float mb, float lb) {
    const float M = fmaxf(ma, mb);
    // (a side without a finite logit has the sum 0, or NaN)
    la = (ma == -__builtin_huge_valf() ? la : la * __builtin_amdgcn_exp2f(ma - M)) +
         (mb == -__builtin_huge_valf() ? lb : lb * __builtin_amdgcn_exp2f(mb - M));
    ma = M;
  };
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) merge(m[cb], l[cb], __shfl_xor(m[cb], 32, 64), __shfl_xor(l[cb], 32, 64));
  if constexpr (WS > 1) {
    if (lane < 32) {
      s_ml[wave][n] = make_float2(m[0], l[0]);
      s_ml[wave][32 + n] = make_float2(m[1], l[1]);
    }
    __syncthreads();
    if (ws != 0) return;
#pragma unroll
    for (int o = 1; o < WS; ++o)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const float2 v = s_ml[wave + o][32 * cb + n];
        merge(m[cb], l[cb], v.x, v.y);
      }
  }
  if (lane < 32) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      const int qi = i_wave + 32 * cb + n;
      if (qi < T) stats[(int64_t)qh * T + qi] = make_float2(m[cb], 1.0f / l[cb]);
    }
  }
}

// Pass 2: sums of the probabilities per key, over the causal queries of
// every query head of the KV head's group.  WS waves of the block take the
// same 64 keys and share out the 32-query subtiles.
template <int WS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void prefill_colsum_kernel(const uint16_t *q, const uint16_t *k, int q_heads, int kv_heads, int units, int nblk, int run,
                           int T, float s2scale, const float2 *stats, float *scores) {
  constexpr int TR = tile_rows<WS>(), SUBS = subtiles<WS>(), kKeys = kWaveRows * 4 / WS;
  __shared__ u4_t s_rows[2][TR * kRowWords];
  __shared__ float2 s_stat[2][TR];
  __shared__ float s_sum[4][kWaveRows];
  const int lane = threadIdx.x & 63, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wc = wave / WS, ws = wave % WS;
  const int G = q_heads / kv_heads;
  int hk, idx;
  if (!block_unit(units, nblk, run, hk, idx)) return;
  const int j_base = idx * kKeys, j_wave = j_base + kWaveRows * wc;  // longest first
  const uint16_t *qb = q + (int64_t)hk * G * T * kHeadDim, *kb = k + (int64_t)hk * T * kHeadDim;
  const float2 *stb = stats + (int64_t)hk * G * T;
  // of each query head: the tiles [t_first, t_full) on the diagonal, then
  // those wholly below it for every wave of the block
  const int t_first = j_base / TR, t_end = (T + TR - 1) / TR, t_full = min(t_end, (j_base + kKeys - 1 + TR - 1) / TR);
  float2 ml = make_float2(0.0f, 0.0f);
  auto load = [&](int buf, int g, int t) {
    stage<TR, true>(s_rows[buf], qb + (int64_t)g * T * kHeadDim, t * TR, T);
    if (threadIdx.x < TR) {
      const int i = min(t * TR + (int)threadIdx.x, T - 1);
      ml = stb[(int64_t)g * T + i];
      // a query past the prompt adds exp2(-inf) * 0
      if (t * TR + (int)threadIdx.x >= T) ml = make_float2(__builtin_huge_valf(), 0.0f);
    }
  };
  int buf = 0;
  auto load_next = [&](int g, int t) {  // the tile after (g, t); after the last, any
    const bool wrap = t + 1 == t_end;
    load(buf ^ 1, wrap ? min(g + 1, G - 1) : g, wrap ? t_first : t + 1);
  };
  auto flip = [&]() {
    buf ^= 1;
    if (threadIdx.x < TR) s_stat[buf][threadIdx.x] = ml;
    wait_loads();
    __syncthreads();
  };
  load(0, 0, t_first);
  u4_t ak[2][8];
  load_stationary(kb, j_wave, T, ak);
  const uint32_t off = tile_offset();
  const int sub0 = ws * SUBS;
  f16_t cs[2] = {splat(0.0f), splat(0.0f)};
  if (threadIdx.x < TR) s_stat[0][threadIdx.x] = ml;
  wait_loads();
  __syncthreads();
  for (int g = 0; g < G; ++g) {
    for (int t = t_first; t < t_full; ++t) {
      const u4_t *rows = s_rows[buf];
#pragma unroll
      for (int s = 0; s < SUBS; ++s) {
        const int i0 = t * TR + 32 * (sub0 + s);
        if (i0 + 31 < j_wave) continue;  // above the diagonal (wave-uniform)
        u4_t b[8];
        read_tile(rows, off, 32 * (sub0 + s), b);
        const float2 qs = s_stat[buf][32 * (sub0 + s) + n];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          const f16_t d = logits(ak[cb], b);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f(fmaf(d[r], s2scale, -qs.x)) * qs.y;
            cs[cb][r] += j_wave + 32 * cb + tile_row(r) <= i0 + n ? p : 0.0f;
          }
        }
      }
      load_next(g, t);
      flip();
    }
    f16_t d0, d1 = splat(0.0f);  // the first step's previous tile adds exp2(-inf) * 0
    float2 qp = make_float2(__builtin_huge_valf(), 0.0f);
    for (int t = t_full; t < t_end; ++t) {
      const u4_t *rows = s_rows[buf];
      u4_t b[SUBS][8];
      read_tile(rows, off, 32 * sub0, b[0]);
      float2 qst[SUBS];
#pragma unroll
      for (int s = 0; s < SUBS; ++s) qst[s] = s_stat[buf][32 * (sub0 + s) + n];
#pragma unroll
      for (int s = 0; s < SUBS; ++s) {
        const float2 qs = qst[s];
        float inv = qp.y;
        auto use1 = [&](int r, float p) { cs[1][r] = fmaf(p, inv, cs[1][r]); };
        if constexpr (SUBS == 2) {
          if (s == 0)
            step<true>(d0, ak[0], b[s], d1, s2scale, qp.x, b[1], rows, off, 32 * (sub0 + 1), use1);
          else
            step<false>(d0, ak[0], b[s], d1, s2scale, qp.x, b[0], rows, off, 0, use1);
        } else {
          step<false>(d0, ak[0], b[s], d1, s2scale, qp.x, b[0], rows, off, 0, use1);
        }
        if (s == 0) load_next(g, t);  // after the tile's last LDS read (see pass 1)
        auto use0 = [&](int r, float p) { cs[0][r] = fmaf(p, qs.y, cs[0][r]); };
        step<false>(d1, ak[1], b[s], d0, s2scale, qs.x, b[0], rows, off, 0, use0);
        qp = qs;
      }
      flip();
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) cs[1][r] = fmaf(__builtin_amdgcn_exp2f(fmaf(d1[r], s2scale, -qp.x)), qp.y, cs[1][r]);
  }
  // over the tile's 32 query columns, then over the WS waves
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float v = cs[cb][r];
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (n == 0) s_sum[wave][32 * cb + tile_row(r)] = v;
    }
  __syncthreads();
  if (ws != 0) return;
  float v = s_sum[wave][lane];
#pragma unroll
  for (int o = 1; o < WS; ++o) v += s_sum[wave + o][lane];
  const int kj = j_wave + lane;
  if (kj < T) scores[(int64_t)hk * T + kj] = v;
}

// The passes of short prompts: one wave per 64 stationary rows, the streamed
// rows straight from memory, 16 at a time, through v_mfma_f32_16x16x32_f16.
// Bound: latency (a wave's chain is at most a few tiles); so 64-thread blocks without
// LDS, many to a CU, instead of two blocks of four waves that fill a 128-row
// tile first (short_pass has both sides' times).  Lane 16 a + n: operand row n
// of a tile, channels [32 c + 8 a, + 8) of MFMA c; result registers r are
// rows (queries) 4 a + r, column (key) n.
constexpr int kShortTiles = 4;  // 16-row tiles per wave (64 rows)
constexpr int kGridHeads = 65535;  // heads along the grid's y (its limit), the rest along z; a head's blocks follow each other
constexpr float kLazy = 8.0f;   // raise a query's running maximum only past this (log2 units)

typedef float f4_t __attribute__((ext_vector_type(4)));

// Operands of row `row` of a [T, 128] fp16 matrix (zero past T).
__device__ inline void load_rows16(const uint16_t *base, int row, int T, int a, u4_t op[4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c)
    op[c] = row < T ? *reinterpret_cast<const u4_t *>(base + (int64_t)row * kHeadDim + 32 * c + 8 * a) : u4_t{0, 0, 0, 0};
}

__device__ inline f4_t logits16(const u4_t query[4], const u4_t key[4]) {
  f4_t d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int c = 0; c < 4; ++c) d = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(query[c]), as_h8(key[c]), d, 0, 0, 0);
  return d;
}

// Reductions over the 16 lanes of one logit row.
__device__ inline float max16(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));
  v = fmaxf(v, dpp_mov<0x4E>(v));
  v = fmaxf(v, dpp_mov<0x141>(v));
  return fmaxf(v, dpp_mov<0x140>(v));
}
__device__ inline float sum16(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  return v + dpp_mov<0x140>(v);
}

// Pass 1, block = 64 queries of one query head.
__global__ __launch_bounds__(64) void short_rowstats_kernel(const uint16_t *q, const uint16_t *k, int q_heads,
                                                            int kv_heads, int heads, int T, float s2scale, float2 *stats) {
  const int lane = threadIdx.x, n = lane & 15, a = lane >> 4;
  const int qh = blockIdx.z * kGridHeads + blockIdx.y, i_base = blockIdx.x * 16 * kShortTiles;
  if (qh >= heads) return;
  const int hk = qh / (q_heads / kv_heads);
  const uint16_t *qb = q + (int64_t)qh * T * kHeadDim, *kb = k + (int64_t)hk * T * kHeadDim;
  u4_t aq[kShortTiles][4];
#pragma unroll
  for (int rb = 0; rb < kShortTiles; ++rb) load_rows16(qb, i_base + 16 * rb + n, T, a, aq[rb]);
  // The maximum is the same in the 16 lanes of a row and raised only when a
  // logit exceeds it by more than kLazy, decided for the whole wave with one
  // ballot; each lane sums its own terms.
  float m[kShortTiles][4], l[kShortTiles][4];
#pragma unroll
  for (int rb = 0; rb < kShortTiles; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      m[rb][r] = -__builtin_huge_valf();
      l[rb][r] = 0.0f;
    }
  const int j_end = min(T, i_base + 16 * kShortTiles);  // keys past the last query are masked
  for (int j0 = 0; j0 < j_end; j0 += 16) {
    u4_t bk[4];
    load_rows16(kb, j0 + n, T, a, bk);
    const int kj = j0 + n;
#pragma unroll
    for (int rb = 0; rb < kShortTiles; ++rb) {
      if (j0 > i_base + 16 * rb + 15) continue;  // above the diagonal (wave-uniform)
      const f4_t d = logits16(aq[rb], bk);
      // a tile below the diagonal and inside the prompt needs no mask
      const bool full = j0 + 15 <= i_base + 16 * rb && i_base + 16 * rb + 15 < T;  // wave-uniform
      float s[4];
      bool raise = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qi = i_base + 16 * rb + 4 * a + r;
        s[r] = full || (kj <= qi && qi < T) ? d[r] * s2scale : -__builtin_huge_valf();
        raise = raise || s[r] > m[rb][r] + kLazy;
      }
      if (__ballot(raise)) {  // wave-uniform
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float mn = fmaxf(m[rb][r], max16(s[r]));
          if (mn != m[rb][r]) {  // row-uniform; mn is finite here
            l[rb][r] *= m[rb][r] == -__builtin_huge_valf() ? 0.0f : __builtin_amdgcn_exp2f(m[rb][r] - mn);
            m[rb][r] = mn;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) l[rb][r] += s[r] == -__builtin_huge_valf() ? 0.0f : __builtin_amdgcn_exp2f(s[r] - m[rb][r]);
    }
  }
#pragma unroll
  for (int rb = 0; rb < kShortTiles; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float sum = sum16(l[rb][r]);
      const int qi = i_base + 16 * rb + 4 * a + r;
      if (n == 0 && qi < T) stats[(int64_t)qh * T + qi] = make_float2(m[rb][r], 1.0f / sum);
    }
}

// Pass 2, block = 64 keys of one KV head.
__global__ __launch_bounds__(64) void short_colsum_kernel(const uint16_t *q, const uint16_t *k, int q_heads, int kv_heads,
                                                          int heads, int T, float s2scale, const float2 *stats,
                                                          float *scores) {
  const int lane = threadIdx.x, n = lane & 15, a = lane >> 4;
  const int hk = blockIdx.z * kGridHeads + blockIdx.y, j_base = blockIdx.x * 16 * kShortTiles;
  if (hk >= heads) return;
  const int G = q_heads / kv_heads;
  const uint16_t *kb = k + (int64_t)hk * T * kHeadDim;
  u4_t bk[kShortTiles][4];
#pragma unroll
  for (int cb = 0; cb < kShortTiles; ++cb) load_rows16(kb, j_base + 16 * cb + n, T, a, bk[cb]);
  float cs[kShortTiles];
#pragma unroll
  for (int cb = 0; cb < kShortTiles; ++cb) cs[cb] = 0.0f;
  for (int g = 0; g < G; ++g) {
    const int qh = hk * G + g;  // = b * q_heads + head
    const uint16_t *qb = q + (int64_t)qh * T * kHeadDim;
    const float2 *st = stats + (int64_t)qh * T;
    for (int i0 = j_base; i0 < T; i0 += 16) {
      u4_t aq[4];
      load_rows16(qb, i0 + n, T, a, aq);
      float2 ml[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qi = i0 + 4 * a + r;
        ml[r] = qi < T ? st[qi] : make_float2(0.0f, 0.0f);
      }
#pragma unroll
      for (int cb = 0; cb < kShortTiles; ++cb) {
        if (j_base + 16 * cb > i0 + 15) continue;  // above the diagonal (wave-uniform)
        const f4_t d = logits16(aq, bk[cb]);
        const int kj = j_base + 16 * cb + n;
        const bool full = j_base + 16 * cb + 15 <= i0 && i0 + 15 < T;  // no mask (wave-uniform)
        if (full) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            cs[cb] = fmaf(__builtin_amdgcn_exp2f(fmaf(d[r], s2scale, -ml[r].x)), ml[r].y, cs[cb]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int qi = i0 + 4 * a + r;
            const bool valid = kj <= qi && qi < T;
            const float p = __builtin_amdgcn_exp2f(fmaf(d[r], s2scale, -ml[r].x)) * ml[r].y;
            cs[cb] += valid ? p : 0.0f;
          }
        }
      }
    }
  }
#pragma unroll
  for (int cb = 0; cb < kShortTiles; ++cb) {
    float v = cs[cb] + __shfl_xor(cs[cb], 16, 64);
    v += __shfl_xor(v, 32, 64);
    const int kj = j_base + 16 * cb + n;
    if (a == 0 && kj < T) scores[(int64_t)hk * T + kj] = v;
  }
}

// Launch of one pass: WS (0: a short prompt's kernel), the blocks of a head and
// the length of a run.
struct Grid {
  int ws, nblk, run;
  dim3 blocks;
};

// Whether a pass (its stationary rows in `heads` heads, G the query heads it
// streams per block in pass 2, 0 in pass 1) takes the short kernel.  Per block of
// 64 rows that one does about half the work per time once the tiles are
// full, but its blocks take neither LDS nor a whole 128-row tile, and some
// eight times as many fit the chip.  Pass 1 (few rows to stream): a handful of
// tokens, up to 112 as the heads fill the chip several times, and up to 192 where
// blocks of 128 and 256 rows would be mostly padding.  Pass 2, which ends
// in a reduction over 32 columns and four waves, up to 192 tokens in all over
// the streamed heads or with many heads, and just past 256 likewise.  Measured
// (both passes, us, the long kernels -> this): 1 x 4/4 heads x 1 token 14.5 ->
// 7.0, 1 x 32/8 x 33 20.3 -> 15, 32 x 40 x 64 48 -> 20, 512 x 32 x 100 688 -> 398,
// 512 x 32 x 300 2273 -> 1540, 1 x 64/8 x 100 26.8 against 50.8.
bool short_pass(int heads, int G, int T) {
  if (G == 0) return T <= std::min(112, 16 + heads / 16) || (heads >= 2048 && T > 128 && T <= std::min(192, 128 + heads / 64));
  return T <= (heads >= 1024 ? 192 : 32 + 160 / G) || (heads >= (G == 1 ? 512 : 1024) && T > 256 && T <= 320 + 64 / G);
}

// `heads` heads of T stationary rows in `units` units of the same streamed
// rows.  WS = 1 streams each row past 256 stationary ones, WS = 2 and 4 past 128
// and 64, in two and four times as many blocks of a half and a quarter of the
// work: better only while the grid leaves CUs idle (two blocks fit a CU, so
// 512 fill the chip; pass 2 in one round of equal blocks, T <= 256, stays with
// WS = 1: 512 x 4/4 x 160 93 against 100 us) or where 256 rows are mostly
// padding.  Measured (us for both passes, WS = 1 / 2 / 4, by the
// blocks of WS = 1): 4096 blocks 1511 / 1557 / 1954, 1024: 347 / 365 / 440,
// 256: 701 / 648 / 695, 240: 77 / 57 / 66, 64: 36 / 27 / 22.
// Runs of 32 read less from beyond L2 than runs of 4 (4096 blocks: 1380
// against 1481 us, 32768: 35.2 against 36.7 ms), but leave a longer tail,
// which decides while the grid is only a few rounds (1024 blocks: 410 against
// 336 us).
Grid plan_pass(int heads, int units, int G, int T) {
  Grid g;
  if (short_pass(heads, G, T)) {
    g.ws = 0;
    g.run = 1;
    g.nblk = (T + 16 * kShortTiles - 1) / (16 * kShortTiles);
    g.blocks = dim3(g.nblk, std::min(heads, kGridHeads), (heads + kGridHeads - 1) / kGridHeads);
    return g;
  }
  const int64_t n1 = (int64_t)heads * ((T + 255) / 256);
  g.ws = n1 >= (G && T <= 256 ? 512 : 768) ? 1 : n1 >= 192 ? 2 : 4;
  const bool half_empty = T % 256 != 0 && T % 256 <= 128;  // of the last 256 rows
  if (T <= 64)
    g.ws = 4;
  else if (g.ws == 1 && half_empty && T < (G ? 320 : 512))
    g.ws = 2;
  const int cols = kWaveRows * 4 / g.ws;
  g.nblk = (T + cols - 1) / cols;
  const int per_unit = g.nblk * (heads / units);
  g.run = n1 >= 4096 ? 32 : 4;
  if (g.run > per_unit) g.run = per_unit;
  g.blocks = dim3(8 * ((units + 7) / 8) * ((per_unit + g.run - 1) / g.run * g.run));
  return g;
}

}  // namespace

}  // namespace mikv

using namespace mikv;

extern "C" size_t mikv_prefill_importance_workspace_size(int32_t batch, int32_t q_heads, int32_t tokens) {
  if (batch < 1 || q_heads < 1 || tokens < 1) return 0;
  return (size_t)((int64_t)batch * q_heads * tokens * 8);
}

extern "C" int mikv_prefill_importance(const uint16_t *q_prefill, const uint16_t *k_prefill, int32_t batch,
                                       int32_t q_heads, int32_t kv_heads, int32_t tokens, int32_t head_dim,
                                       float scale, float *scores, void *ws, size_t ws_bytes, void *stream) {
  if (!q_prefill || !k_prefill || !scores)
    return set_error(MIKV_ERR_INVALID_ARG, "mikv_prefill_importance: NULL pointer");
  if (batch < 1 || q_heads < 1 || kv_heads < 1 || tokens < 1 || q_heads % kv_heads != 0)
    return set_error(MIKV_ERR_INVALID_ARG, "mikv_prefill_importance: bad sizes");
  const int G = q_heads / kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8)
    return set_error(MIKV_ERR_UNSUPPORTED, "mikv_prefill_importance: query heads per KV head must be 1, 2, 4 or 8");
  if (head_dim != kHeadDim) return set_error(MIKV_ERR_UNSUPPORTED, "mikv_prefill_importance: head_dim must be 128");
  if (!(scale > 0.0f)) return set_error(MIKV_ERR_INVALID_ARG, "mikv_prefill_importance: scale must be > 0");
  if (((uintptr_t)q_prefill | (uintptr_t)k_prefill) % 16 != 0)
    return set_error(MIKV_ERR_INVALID_ARG, "mikv_prefill_importance: q_prefill and k_prefill must be 16-byte aligned");
  if (!ws || ws_bytes < mikv_prefill_importance_workspace_size(batch, q_heads, tokens))
    return set_error(MIKV_ERR_CAPACITY, "mikv_prefill_importance: workspace too small");
  const float s2scale = scale * kLog2e;
  hipStream_t st = (hipStream_t)stream;
  float2 *stats = (float2 *)ws;
  const int units = batch * kv_heads;
  const Grid g1 = plan_pass(batch * q_heads, units, 0, tokens), g2 = plan_pass(units, units, G, tokens);
  if (g1.ws == 0) {
    hipLaunchKernelGGL(short_rowstats_kernel, g1.blocks, dim3(64), 0, st, q_prefill, k_prefill, q_heads, kv_heads,
                       batch * q_heads, tokens, s2scale, stats);
  } else {
    auto rowstats = g1.ws == 1 ? prefill_rowstats_kernel<1> : g1.ws == 2 ? prefill_rowstats_kernel<2> : prefill_rowstats_kernel<4>;
    hipLaunchKernelGGL(rowstats, g1.blocks, dim3(kThreads), 0, st, q_prefill, k_prefill, q_heads, kv_heads, units, g1.nblk,
                       g1.run, tokens, s2scale, stats);
  }
  if (g2.ws == 0) {
    hipLaunchKernelGGL(short_colsum_kernel, g2.blocks, dim3(64), 0, st, q_prefill, k_prefill, q_heads, kv_heads, units,
                       tokens, s2scale, (const float2 *)stats, scores);
  } else {
    auto colsum = g2.ws == 1 ? prefill_colsum_kernel<1> : g2.ws == 2 ? prefill_colsum_kernel<2> : prefill_colsum_kernel<4>;
    hipLaunchKernelGGL(colsum, g2.blocks, dim3(kThreads), 0, st, q_prefill, k_prefill, q_heads, kv_heads, units, g2.nblk,
                       g2.run, tokens, s2scale, (const float2 *)stats, scores);
  }
  return check_launch("mikv_prefill_importance");
}
