// Saliency scoring on the matrix cores for bf16, head_dim 128, 32 query rows (Sec. 3.3 second
// equation, aggregated over the block's queries and the query heads of a KV group as in Alg. 1).
//
// The softmax-normalised score needs each query row's max and sum over ALL candidates before any
// column can be reduced, so it takes two streaming passes over K (the logits are recomputed; they
// are cheap next to the K read):
//   pass 1 (row_stats): logits^T = K_tile Q_h^T, lane = query row, online (max, sum) per row;
//   pass 2 (col_reduce): logits = Q_h K_tile^T, lane = candidate key, p = exp2(s - max)/sum summed
//                        over the 32 rows (in registers) and over the G query heads of the group.
// A workgroup serves one (batch, KV head) and a contiguous range of candidate tiles, so K is read from HBM once per
// pass however large G is.  Its waves take tiles round-robin into wave-private LDS tiles (no barrier in the loop), the Q
// fragments of all G heads in LDS; or, in pass 2 of grouped-query heads as a launch of its own, one head each while there is little work per CU.
// Probabilities stay fp32 end to end: the retained set must match a float64 reference except for
// scores within 1e-4 relative of the k-th value.
#include <type_traits>

#include "mfma_tile.h"

namespace sdllm {

struct CandTiles {
  const char* k0; const char* k1;   // first row of the prefix / suffix candidates of this (b, g)
  uint32_t stride;                  // bytes per key row
  int n0, n1, tiles0;
};

__device__ __forceinline__ CandTiles cand_tiles(const ScoreParams& p, int b, int g) {
  CandTiles ct;
  ct.stride = (uint32_t)(p.k_sr * 2);
  const char* base = (const char*)p.k + 2 * (b * p.k_sb + g * p.k_sh);
  ct.k0 = base;
  ct.k1 = base + (size_t)(p.block_off + p.block_len) * ct.stride;
  ct.n0 = min(p.n_cand, p.block_off);
  ct.n1 = p.n_cand - ct.n0;
  ct.tiles0 = (ct.n0 + kTileKeys - 1) / kTileKeys;
  return ct;
}

// tile -> (first row pointer, valid rows, candidate index of its first row)
__device__ __forceinline__ const char* tile_rows(const CandTiles& ct, int tile, int& rows, int& cand0) {
  if (tile < ct.tiles0) {
    cand0 = tile * kTileKeys;
    rows = min(kTileKeys, ct.n0 - cand0);
    return ct.k0 + (size_t)cand0 * ct.stride;
  }
  const int first = (tile - ct.tiles0) * kTileKeys;
  cand0 = ct.n0 + first;
  rows = min(kTileKeys, ct.n1 - first);
  return ct.k1 + (size_t)first * ct.stride;
}

// Q rows of all G heads of the group -> LDS, padded like a K tile so both are read the same way.
// Row `row` of head h; with two blocks of query rows per head (q_shift 1) h counts blocks.  Rows past the end are copies of the last one:
// they weigh nothing (row_statistics).
__device__ __forceinline__ const char* query_row(const ScoreParams& p, int b, int h, int row) {
  return (const char*)p.q + 2 * (b * p.q_sb + (int64_t)(h >> p.q_shift) * p.q_sh + (int64_t)min((h & p.q_shift) * 32 + row, p.nq - 1) * p.q_sr);
}

template <int G>
__device__ __forceinline__ void stage_queries(const ScoreParams& p, int b, int g, uint8_t* lds_q) {
  for (int i = threadIdx.x; i < G * 32 * 16; i += blockDim.x) {
    const int chunk = i & 15, row = (i >> 4) & 31, hh = i >> 9;
    const char* src = query_row(p, b, g * G + hh, row) + chunk * 16;
    *reinterpret_cast<u32x4*>(lds_q + hh * kTileBytes + tile_off(row, chunk)) = *reinterpret_cast<const u32x4*>(src);
  }
}

// The column reduction over this workgroup's tiles (pass 2): lds_q holds the group's Q rows, lds_ml the
// final (max, 1/sum) of every (head, row).
template <int G, bool BACKWARDS>
__device__ __forceinline__ void score_columns(const ScoreParams& p, int b, int g, int bg, int part, const uint8_t* lds_q,
                                              uint8_t* lds_k, const float2* lds_ml, int wave, int nw, int lane, int half,
                                              int col) {
  const CandTiles ct = cand_tiles(p, b, g);
  const int ntiles = ct.tiles0 + (ct.n1 + kTileKeys - 1) / kTileKeys;
  const int t_begin = part * p.tiles_per_part;
  const int t_end = min(ntiles, t_begin + p.tiles_per_part);
  const float inv_count = p.inv_count;
  float* score_row = p.score + (size_t)bg * p.score_stride;

  u32x4 kreg[8];
  int rows = 0, cand0 = 0;
  // BACKWARDS (the sweep that follows the statistics pass inside one launch): last tile first, because
  // the rows that pass read last are the ones this XCD's L2 may still hold
  const int n_mine = t_end - t_begin;
  auto tile_at = [&](int i) { return BACKWARDS ? t_end - 1 - i : t_begin + i; };   // i-th tile of this workgroup's walk
  int i_t = wave;
  if (i_t < n_mine) {
    const char* src = tile_rows(ct, tile_at(i_t), rows, cand0);
    load_rows(src, rows, ct.stride, lane, kreg);
  }
  for (; i_t < n_mine; i_t += nw) {
    store_rows(lds_k, lane, kreg);
    wave_lds_sync();
    const int rows_now = rows, cand_now = cand0;
    if (i_t + nw < n_mine) {
      const char* src = tile_rows(ct, tile_at(i_t + nw), rows, cand0);
      load_rows(src, rows, ct.stride, lane, kreg);
    }
    bf16x8 kf[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) kf[kk] = *reinterpret_cast<const bf16x8*>(lds_k + tile_off(col, kk * 2 + half));
    float total = 0.f;
    if (G > 1 && p.softmax) {
      // Software pipeline over the heads: while the vector ALU turns head hh's logits into
      // probabilities, the matrix core works on head hh+1 and the LDS returns the Q fragments of
      // head hh+2.  A wave issues in order, so the three streams are interleaved in program order
      // (one MFMA, its share of LDS reads and of ALU work, eight times per head); a modest gain,
      // 20.5 -> 19.4 us with seven heads per group at batch 8.
      bf16x8 qf[2][8];
      f32x16 sn[2];
      auto q_frag = [&](int hh, int kk) {
        return *reinterpret_cast<const bf16x8*>(lds_q + hh * kTileBytes + tile_off(col, kk * 2 + half));
      };
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) qf[0][kk] = q_frag(0, kk);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) qf[1][kk] = q_frag(1, kk);
#pragma unroll
      for (int i = 0; i < 16; ++i) sn[0][i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) sn[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[0][kk], kf[kk], sn[0], 0, 0, 0);
      // row statistics of register i of head hh: query row 8*(i/4) + 4*half + i%4 (this lane's key is `col`)
      auto row_ml = [&](int hh, int i) { return lds_ml[hh * 32 + (i >> 2) * 8 + half * 4 + (i & 3)]; };
      float2 ml[2] = {row_ml(0, 0), row_ml(0, 1)};
#pragma unroll
      for (int hh = 0; hh < G; ++hh) {
        const int cur = hh & 1, nxt = cur ^ 1;
        if (hh + 1 < G) {
#pragma unroll
          for (int i = 0; i < 16; ++i) sn[nxt][i] = 0.f;
        }
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          if (hh + 1 < G) sn[nxt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[nxt][kk], kf[kk], sn[nxt], 0, 0, 0);
          if (hh + 2 < G) qf[cur][kk] = q_frag(hh + 2, kk);
          // the statistics are requested one group ahead of their use
          float2 ml_next[2] = {ml[0], ml[1]};
          if (kk < 7) { ml_next[0] = row_ml(hh, 2 * kk + 2); ml_next[1] = row_ml(hh, 2 * kk + 3); }
          else if (hh + 1 < G) { ml_next[0] = row_ml(hh + 1, 0); ml_next[1] = row_ml(hh + 1, 1); }
          total += __builtin_amdgcn_exp2f(sn[cur][2 * kk] * p.scale_log2 - ml[0].x) * ml[0].y;
          total += __builtin_amdgcn_exp2f(sn[cur][2 * kk + 1] * p.scale_log2 - ml[1].x) * ml[1].y;
          ml[0] = ml_next[0]; ml[1] = ml_next[1];
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);   // 3 LDS reads
          __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);   // 6 vector ALU
        }
      }
    } else {
#pragma unroll
      for (int hh = 0; hh < G; ++hh) {
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          const bf16x8 qf = *reinterpret_cast<const bf16x8*>(lds_q + hh * kTileBytes + tile_off(col, kk * 2 + half));
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[kk], s, 0, 0, 0);   // rows = queries, columns = keys
        }
        // register i is query row 8*(i/4) + 4*half + i%4, this lane's key is `col`
        float part_sum = 0.f;
        if (p.softmax) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float2 ml = lds_ml[hh * 32 + (i >> 2) * 8 + half * 4 + (i & 3)];
            part_sum += __builtin_amdgcn_exp2f(s[i] * p.scale_log2 - ml.x) * ml.y;
          }
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) part_sum += s[i];
          part_sum *= p.scale;
        }
        total += part_sum;
      }
    }
    total += __shfl_xor(total, 32);
    if (half == 0 && col < rows_now) score_row[cand_now + col] = total * inv_count;
    wave_lds_sync();
  }
}

// ------------------------------------------------------------------ pass 1: row statistics
template <int G>
__global__ __launch_bounds__(512) void score_stats_mfma_kernel(const ScoreParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int part = blockIdx.x;
  const int bg = blockIdx.y;
  const int b = p.by_hkv.quotient(bg), g = bg - b * p.hkv;

  uint8_t* lds_q = smem;
  uint8_t* lds_k = smem + G * kTileBytes + wave * kTileBytes;
  float2* lds_ml = reinterpret_cast<float2*>(smem + (G + nw) * kTileBytes);
  stage_queries<G>(p, b, g, lds_q);
  __syncthreads();

  const CandTiles ct = cand_tiles(p, b, g);
  const int ntiles = ct.tiles0 + (ct.n1 + kTileKeys - 1) / kTileKeys;
  const int t_begin = part * p.tiles_per_part;
  const int t_end = min(ntiles, t_begin + p.tiles_per_part);

  float m_run[G], l_run[G];
#pragma unroll
  for (int hh = 0; hh < G; ++hh) { m_run[hh] = -INFINITY; l_run[hh] = 0.f; }

  u32x4 kreg[8];
  int rows = 0, cand0 = 0;
  int t = t_begin + wave;
  if (t < t_end) {
    const char* src = tile_rows(ct, t, rows, cand0);
    load_rows<false>(src, rows, ct.stride, lane, kreg);   // plain: the column pass reads these rows again
  }
  for (; t < t_end; t += nw) {
    store_rows(lds_k, lane, kreg);
    wave_lds_sync();
    const int rows_now = rows;
    const int tn = t + nw;
    if (tn < t_end) {
      const char* src = tile_rows(ct, tn, rows, cand0);
      load_rows<false>(src, rows, ct.stride, lane, kreg);   // plain: the column pass reads these rows again
    }
    bf16x8 kf[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) kf[kk] = *reinterpret_cast<const bf16x8*>(lds_k + tile_off(col, kk * 2 + half));
#pragma unroll
    for (int hh = 0; hh < G; ++hh) {
      f32x16 s;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const bf16x8 qf = *reinterpret_cast<const bf16x8*>(lds_q + hh * kTileBytes + tile_off(col, kk * 2 + half));
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf, s, 0, 0, 0);   // rows = keys, columns = queries
      }
      // each half-lane keeps the (max, sum) of the keys it has seen itself (the two halves of a row
      // are merged once, after the loop); the max is taken on the raw logits and the scale folded
      // into the exponent's multiply-add
      if (rows_now < kTileKeys) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if ((i >> 2) * 8 + half * 4 + (i & 3) >= rows_now) s[i] = -INFINITY;
      }
      float m_loc = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) m_loc = fmaxf(m_loc, s[i]);
      if (m_loc != -INFINITY) {   // a ragged tile can leave a half-lane without any key
        const float m_new = fmaxf(m_run[hh], m_loc * p.scale_log2);
        float l_loc = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) l_loc += __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], p.scale_log2, -m_new));
        l_run[hh] = l_run[hh] * __builtin_amdgcn_exp2f(m_run[hh] - m_new) + l_loc;
        m_run[hh] = m_new;
      }
    }
    wave_lds_sync();
  }

  // merge the waves: every wave parks (max, sum) per head and row in its own tile region
  float* mine = reinterpret_cast<float*>(lds_k);
#pragma unroll
  for (int hh = 0; hh < G; ++hh) {
    const float m_other = __shfl_xor(m_run[hh], 32), l_other = __shfl_xor(l_run[hh], 32);
    const float m_row = fmaxf(m_run[hh], m_other);
    float l_tot = 0.f;
    if (m_run[hh] != -INFINITY) l_tot += l_run[hh] * __builtin_amdgcn_exp2f(m_run[hh] - m_row);
    if (m_other != -INFINITY) l_tot += l_other * __builtin_amdgcn_exp2f(m_other - m_row);
    if (lane < 32) { mine[hh * 64 + lane] = m_row; mine[hh * 64 + 32 + lane] = l_tot; }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < G * 32; i += blockDim.x) {
    const int hh = i >> 5, row = i & 31;
    float m_tot = -INFINITY;
    for (int w = 0; w < nw; ++w)
      m_tot = fmaxf(m_tot, reinterpret_cast<const float*>(smem + (G + w) * kTileBytes)[hh * 64 + row]);
    float l_tot = 0.f;
    for (int w = 0; w < nw; ++w) {
      const float* o = reinterpret_cast<const float*>(smem + (G + w) * kTileBytes);
      const float m_w = o[hh * 64 + row];
      if (m_w != -INFINITY) l_tot += o[hh * 64 + 32 + row] * __builtin_amdgcn_exp2f(m_w - m_tot);
    }
    const size_t head = (size_t)b * p.hq + g * G + hh;
    float* dst = p.part_ml + (head * p.n_part + part) * 64;
    dst[row] = m_tot;
    dst[32 + row] = l_tot;
    if (p.cols_follow) lds_ml[i] = make_float2(m_tot, 1.f / l_tot);
  }
  // One workgroup per row: its statistics are final, and the column pass follows in the same launch
  // (no second launch with its fill and drain, and the walk back starts on rows still in L2).
  if (p.cols_follow) {
    __syncthreads();
    score_columns<G, true>(p, b, g, bg, part, lds_q, lds_k, lds_ml, wave, nw, lane, half, col);
  }
}

// ------------------------------------------------------------------ pass 2: column reduction
// (max, 1 / sum) of one row of a head from the partials of pass 1, in one sweep (there can be dozens per row and every load is
// a trip to L2: UNROLL pairs are requested together, then folded in).
template <int UNROLL>
__device__ __forceinline__ float2 row_statistics(const ScoreParams& p, size_t head, int row) {
  const float* src = p.part_ml + head * p.n_stat_part * 64 + row;
  float m_tot = -INFINITY, l_tot = 0.f;
#pragma unroll UNROLL
  for (int s = 0; s < p.n_stat_part; ++s) {
    const float m_s = src[s * 64];
    const float l_s = src[s * 64 + 32];
    const float m_new = fmaxf(m_tot, m_s);
    if (m_new != -INFINITY)
      l_tot = l_tot * __builtin_amdgcn_exp2f(m_tot - m_new) + l_s * __builtin_amdgcn_exp2f(m_s - m_new);
    m_tot = m_new;
  }
  return make_float2(m_tot, (int)(head & p.q_shift) * 32 + row < p.nq ? 1.f / l_tot : 0.f);
}

// One query head per KV head, and grouped-query heads with much work per CU (heads_pay): a wave per tile, which walks the heads.
template <int G>
__global__ __launch_bounds__(512) void score_cols_mfma_kernel(const ScoreParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int part = blockIdx.x;
  const int bg = blockIdx.y;
  const int b = p.by_hkv.quotient(bg), g = bg - b * p.hkv;

  uint8_t* lds_q = smem;
  uint8_t* lds_k = smem + G * kTileBytes + wave * kTileBytes;
  // per (head, row): max (log2 domain) and 1/sum of the whole row, from the partials of pass 1
  float2* lds_ml = reinterpret_cast<float2*>(smem + (G + nw) * kTileBytes);
  stage_queries<G>(p, b, g, lds_q);
  if (p.softmax)
    for (int i = threadIdx.x; i < G * 32; i += blockDim.x) lds_ml[i] = row_statistics<16>(p, (size_t)b * p.hq + g * G + (i >> 5), i & 31);
  __syncthreads();

  score_columns<G, false>(p, b, g, bg, part, lds_q, lds_k, lds_ml, wave, nw, lane, half, col);
}

template <int N>
__device__ __forceinline__ void wait_requests() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// The statistics of the rows that the registers of a lane's products belong to, 8*(i/4) + 4*half + i%4, from 32 pairs in LDS.
__device__ __forceinline__ void rows_of_registers(const float2* ml, int half, float (&row_m)[16], float (&row_il)[16]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float2 x = ml[(i >> 2) * 8 + half * 4 + (i & 3)];
    row_m[i] = x.x;
    row_il[i] = x.y;
  }
}

// ------------------------------------------------------------------ pass 2 for grouped-query heads: one wave per query head
// With the statistics there already (the dense attention of the same step left them) or not needed, a wave takes one of the
// G heads and keeps its 32 query rows and their statistics in registers; a tile of keys is fetched once for its G waves, into a
// ring in LDS, and the heads' sums of a tile meet in LDS.  One more wave does the fetching and the writing of the scores, so that
// the others, which meet at a barrier per tile, have nothing else between two barriers.
// Against a wave per tile that walks the heads: a third of the LDS reads (a tile's keys once per head instead of the head's
// queries and statistics once per tile: 0.5 us per tile and head on eight waves), and one round trip at the start instead of
// four, as queries, statistics and the first tiles are requested together.  Kernel, 28/4 heads: 4320 candidates 11.0 -> 5.2 us,
// 33 248 18.5 -> 13.7; whole cache-update step, 3 x 28/4 x 1200 positions 31.3 -> 26.2, 8 x 28/4 x 4600 80.3 -> 76.5, 4 x 32/8 x
// 1500 35.0 -> 32.8, 2 x 16/2 x 3000 33.3 -> 26.2.  Where it does not pay: heads_pay.
constexpr int heads_streams(int g) { return g <= 4 ? 2 : 1; }       // tiles worked on side by side
constexpr int heads_ring(int g) { return g <= 4 ? 4 : 6; }          // tiles of a stream in LDS
constexpr int heads_waves(int g) { return g * heads_streams(g); }   // and the one that fetches and writes
constexpr int heads_ring_bytes(int g) { return heads_streams(g) * heads_ring(g) * kRingK; }
constexpr int heads_lds_bytes(int g) { return heads_ring_bytes(g) + heads_waves(g) * (32 * 8 + 2 * 64 * 4 + kRingK); }

template <int G>
__global__ __launch_bounds__((heads_waves(G) + 1) * kWave) void score_cols_heads_kernel(const ScoreParams p, const int tiles_per_wg) {
  constexpr int T = heads_streams(G), R = heads_ring(G), W = heads_waves(G);
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, col = lane & 31;
  const int bg = blockIdx.y, b = p.by_hkv.quotient(bg), g = bg - b * p.hkv;

  const CandTiles ct = cand_tiles(p, b, g);
  const int ntiles = ct.tiles0 + (ct.n1 + kTileKeys - 1) / kTileKeys;
  const int t0 = blockIdx.x * tiles_per_wg, t1 = min(ntiles, t0 + tiles_per_wg);   // not empty: launch_heads
  const int nsteps = (t1 - t0 + T - 1) / T;                                        // step j: tiles t0 + T j + stream

  float2* ml = reinterpret_cast<float2*>(smem + heads_ring_bytes(G));               // [W][32] (max, 1 / sum) of a head's rows
  float* sums = reinterpret_cast<float*>(smem + heads_ring_bytes(G) + W * 32 * 8);   // [2][W][64] a tile's sums, per head and lane

  if (wave == W) {
    const uint32_t ring_at = lds_address(smem), k_chunk = fetch_k_chunk(lane);
    auto fetch = [&](int j) {
#pragma unroll
      for (int st = 0; st < T; ++st) {
        int rows, cand0;
        // past the end the last tile again, which is not written
        const char* base = in_scalars(tile_rows(ct, min(t0 + T * j + st, t1 - 1), rows, cand0));
#pragma unroll
        for (int c = 0; c < 8; ++c)
          fetch_to_lds(ring_at + (uint32_t)((st * R + j % R) * kRingK + c * kKGroup), base,
                       (uint32_t)min(c + 8 * (lane >> 4), rows - 1) * ct.stride + k_chunk);
      }
    };
    float* score_row = p.score + (size_t)bg * p.score_stride;
    const float inv_count = p.inv_count;
    auto write = [&](int j) {   // the scores of step j: a half-lane per stream
      const int tile = t0 + T * j + half;
      int rows, cand0;
      tile_rows(ct, min(tile, t1 - 1), rows, cand0);
      if (half >= T || tile >= t1 || col >= rows) return;
      const float* part = sums + ((j & 1) * W + half * G) * 64 + col;
      float total = 0.f;
#pragma unroll
      for (int k = 0; k < G; ++k) total += part[k * 64] + part[k * 64 + 32];
      score_row[cand0 + col] = total * inv_count;
    };
    for (int j = 0; j < R - 1; ++j)
      if (j < nsteps) fetch(j);
    in_issue_order();
    wait_requests<0>();
    bare_barrier();                        // tiles 0 .. R-2 are there
    for (int j = 0; j < nsteps; ++j) {
      bare_barrier();                      // tile j is in the others' registers, the sums of step j-1 are written
      if (j + R - 1 < nsteps) fetch(j + R - 1);
      in_issue_order();
      if (j > 0) write(j - 1);
      in_issue_order();
      // tile j+2, which is read behind the next barrier, has landed; behind it are at most R - 3 tiles and a few scores
      if (j + R - 1 < nsteps) wait_requests<(R - 3) * 8 * T>();
      else wait_requests<0>();
    }
    bare_barrier();
    write(nsteps - 1);
    return;
  }

  const int hh = wave % G, stream = wave / G, h = g * G + hh;
  // the head's query rows, whole rows at a time through LDS of the wave's own
  uint8_t* lds_q = smem + heads_ring_bytes(G) + W * (32 * 8 + 2 * 64 * 4) + wave * kRingK;
#pragma unroll
  for (int c = 0; c < 8; ++c)
    fetch_to_lds(lds_address(lds_q) + (uint32_t)(c * kKGroup),
                 query_row(p, b, h, c + 8 * (lane >> 4)) + fetch_k_chunk(lane));
  float row_m[16], row_il[16];
  if (p.softmax) {
    const float2 x = row_statistics<8>(p, (size_t)b * p.hq + h, col);
    if (half == 0) ml[wave * 32 + col] = x;
    wave_lds_sync();
    rows_of_registers(ml + wave * 32, half, row_m, row_il);
  }

  wait_requests<0>();
  wave_lds_sync();
  bf16x8 qf[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) qf[i] = shared_k_frag(shared_k_at(lds_q, half, col), i);

  // Step j: products of tile j, whose operands are in registers, requests for those of tile j + 1, then tile j's weights.
  const uint8_t* k_at = shared_k_at(smem + stream * R * kRingK, half, col);
  float* my_sum = sums + wave * 64 + lane;
  bf16x8 kf[8];
  bare_barrier();
#pragma unroll
  for (int i = 0; i < 8; ++i) kf[i] = shared_k_frag(k_at, i);
  int slot = kRingK;                       // of tile j + 1
  for (int j = 0; j < nsteps; ++j) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bare_barrier();
    f32x16 sc;
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[i], kf[i], sc, 0, 0, 0);   // rows = queries, columns = keys
#pragma unroll
    for (int i = 0; i < 8; ++i) kf[i] = shared_k_frag(k_at + slot, i);   // behind the last step: read, not used
    slot = slot + kRingK == R * kRingK ? 0 : slot + kRingK;
    __builtin_amdgcn_sched_barrier(0);
    float total = 0.f;
    if (p.softmax) {
#pragma unroll
      for (int i = 0; i < 16; ++i) total += __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i], p.scale_log2, -row_m[i])) * row_il[i];
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) total += sc[i];
      total *= p.scale;
    }
    my_sum[(j & 1) * W * 64] = total;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  bare_barrier();
}

static int candidate_tiles(const ScoreParams& p) {
  const int n0 = p.n_cand < p.block_off ? p.n_cand : p.block_off, n1 = p.n_cand - n0;
  return (n0 + kTileKeys - 1) / kTileKeys + (n1 + kTileKeys - 1) / kTileKeys;
}

// Which of the two kernels runs the column pass of grouped-query heads.  A wave per head starts sooner and reads LDS less per tile, but
// fills a CU with one workgroup of G or 2 G waves; from some number of tiles per CU on, eight waves that walk the heads, or two
// such workgroups, take less.  The line lies there, in rows ((batch, KV head) pairs) x tiles, by how many waves there are.
// us, walking / wave per head:
// * whole cache-update step, whose other kernels leave less of either one's code in the instruction cache: 2 heads, 16 rows x 93
//   tiles 29.9 / 27.0, 192 x 46 67.0 / 68.4, 256 x 187 244.7 / 260.8; 7 heads, 32 x 46 35.6 / 32.8, 192 x 93 179.5 / 183.1; with few
//   rows at any length, 7 heads, 2 x 1190 77.1 / 68.6; raw logits, 3 heads, 68 x 14 24.9 / 22.5;
// * on its own, raw logits, with the selection: 2 heads, 8 x 46 9.4 / 8.3, 32 x 24 8.9 / 9.2, 192 x 187 67.3 / 86.0; 4 heads,
//   8 x 46 10.1 / 9.0, 91 x 13 10.9 / 11.9, 96 x 93 23.3 / 25.4; 5 heads, 16 x 24 9.8 / 9.0, 192 x 24 17.6 / 20.7; 7 heads, 16 x 93
//   15.4 / 14.3, 96 x 93 29.9 / 33.0;
// * softmax with statistics from a launch of this file, which leaves the keys where they are read again soonest: 2 heads, 8 x 71
//   18.6 / 16.7, 48 x 12 13.9 / 14.5; 5 heads, 70 x 13 20.6 / 21.8; 7 heads, 8 x 94 26.8 / 22.7.  That leaves up to 256 partials a
//   row too, which a wave per head folds by itself: 1 x 1814 with 7 heads 53.3 / 56.9, 1 x 1948 with 2 43.9 / 48.0.  With 7 heads
//   and 45 to 64 rows of 24 to 50 tiles a wave per head takes 2 to 7 % less again.
// Beyond 256 rows the kernel that walks the heads has one workgroup per row, of ever fewer waves, of which from six heads on
// the queries' LDS lets a CU hold one: 7 heads, 512 rows x 24 tiles, raw logits 51.3 / 41.8.
static bool heads_pay(const ScoreParams& p, int tiles) {
  const int rows = p.batch * p.hkv, g = p.group;
  const int64_t work = (int64_t)rows * tiles;
  if (p.in_step) {
    static constexpr int kMost[9] = {0, 0, 3000, 4000, 6000, 3500, 6000, 5000, 4000};   // by heads per group
    if (rows > kNumCUs) return g >= 6 || (g >= 4 && tiles <= 9) || (g == 4 && p.softmax);
    return work <= kMost[g] || rows <= 8;
  }
  if (!p.softmax) {
    const int most = g <= 3 ? 600 : g <= 5 ? 1000 : 3000;
    if (rows > kNumCUs) return g >= 6 && (rows >= 400 || work <= most);
    if (rows > kNumCUs / 3) return tiles <= (g <= 5 ? 4 : 12);   // one or two workgroups per row
    return work <= most || (g >= 6 && rows <= 4);
  }
  if (p.n_stat_part > (g <= 3 ? 16 : g <= 5 ? 48 : 64)) return false;
  if (rows > (g == 4 ? 40 : g >= 6 ? 36 : 22)) return g >= 6 && rows <= 64 && tiles >= 24 && work <= 4000;
  return work <= (g == 5 ? 2500 : 5000) || (rows <= 12 && (g == 4 || g >= 6));
}

template <int G>
static hipError_t launch_heads(const ScoreParams& p, int tiles, hipStream_t s) {
  static LdsOptIn lds;
  const auto kernel = score_cols_heads_kernel<G>;
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), heads_lds_bytes(G));
  if (e != hipSuccess) return e;
  const int rows = p.batch * p.hkv;
  int parts = kNumCUs / rows;              // a workgroup per CU (two: the whole step 0 to 10 % slower below 32 rows, level above)
  if (parts < 1) parts = 1;
  const int per_wg = (tiles + parts - 1) / parts;
  parts = (tiles + per_wg - 1) / per_wg;   // none empty
  return launch(kernel, dim3(parts, rows), dim3((heads_waves(G) + 1) * kWave), heads_lds_bytes(G), s, p, per_wg);
}

static size_t score_lds_bytes(int group, int waves) { return (size_t)(group + waves) * kTileBytes + (size_t)group * 32 * 8; }

template <int G>
static hipError_t launch_g(const ScoreParams& p, hipStream_t s) {
  const size_t lds = score_lds_bytes(G, p.waves);
  const int max_lds = (int)score_lds_bytes(G, kMaxWavesPerWg);
  const dim3 grid(p.n_part, p.batch * p.hkv), block(p.waves * kWave);
  if (p.softmax && !p.skip_stats) {
    static LdsOptIn lds_stats;
    const hipError_t e = lds_stats.ensure(reinterpret_cast<const void*>(score_stats_mfma_kernel<G>), max_lds);
    if (e != hipSuccess) return e;
    ScoreParams q = p;
    q.cols_follow = p.n_part == 1;   // statistics final inside the workgroup: one launch does both passes
    const hipError_t launched = launch(score_stats_mfma_kernel<G>, grid, block, lds, s, q);
    if (launched != hipSuccess || q.cols_follow) return launched;
  }
  if constexpr (G > 1) {
    const int tiles = candidate_tiles(p);
    if (heads_pay(p, tiles)) return launch_heads<G>(p, tiles, s);
  }
  static LdsOptIn lds_cols;
  const hipError_t e = lds_cols.ensure(reinterpret_cast<const void*>(score_cols_mfma_kernel<G>), max_lds);
  if (e != hipSuccess) return e;
  return launch(score_cols_mfma_kernel<G>, grid, block, lds, s, p);
}

bool score_mfma_supports_group(int group) { return group >= 1 && group <= 8; }

hipError_t launch_score_mfma_bf16(const ScoreParams& p, hipStream_t s) {
  if (p.n_cand <= 0) return hipSuccess;
  switch (p.group) {
    case 1: return launch_g<1>(p, s);
    case 2: return launch_g<2>(p, s);
    case 3: return launch_g<3>(p, s);
    case 4: return launch_g<4>(p, s);
    case 5: return launch_g<5>(p, s);
    case 6: return launch_g<6>(p, s);
    case 7: return launch_g<7>(p, s);
    case 8: return launch_g<8>(p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sdllm
