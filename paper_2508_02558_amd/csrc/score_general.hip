// Saliency scoring (Sec. 3.3 second equation, aggregated as in Alg. 1) for the shapes score_mfma.hip does
// not take: fp32 tensors, head_dim 64, groups of more than eight heads or blocks of 32 query rows, raw logits of blocks that are not
// full, a few KV heads with one block each, rows too far apart for 32-bit offsets.  The softmax's row statistics come from attn_general_kernel (by-product
// of the dense step, or a statistics-only launch); this file reduces the columns.
//
// logits = Q K_tile^T with Q rows as the A operand, so a lane holds one candidate key against 16 query
// rows and sums their weights in registers.  A workgroup serves one (batch, KV head) and a few candidate
// tiles, one per wave at a time; the query rows of the group (blocks of 32 or 16 rows of every head, padded with copies of the
// last row, which count for nothing) sit in LDS, as many blocks at once as 64 KB hold.
// 2 x 8 heads of 64 x 1200 positions: what is left is latency (queries, statistics, one tile).
// A wave's first tile is requested behind the staging on purpose: held in registers meanwhile it costs a wave per SIMD, which is
// up to 1 % of a small cache-update step gained and 3 to 9 % lost where many workgroups share a CU (9 x 32 heads of 64 x 616
// positions 43.9 us, 45.8 with the tile first; fp32 2 x 8/1 x 1624 59.5, 65.4).
#include "general_tile.h"

namespace sdllm {

constexpr int kColWaves = 4;

template <typename T, int D>
constexpr int col_block_bytes() { return Ops<T, D>::kRows * (Ops<T, D>::kKRow + 8); }   // a block's query rows and their (max, 1/sum)
template <typename T, int D>
constexpr int col_blocks() { return 65536 / col_block_bytes<T, D>(); }                   // blocks held in LDS at once

template <typename T, int D>
__global__ __launch_bounds__(kColWaves * kWave) void score_cols_general_kernel(const ScoreParams p, const int rblocks, const Divisor by_rblocks) {
  using O = Ops<T, D>;
  constexpr int kBlocks = col_blocks<T, D>(), R = O::kRows, kQBytes = R * O::kKRow;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = lane / R, col = lane % R;
  const int bg = blockIdx.y, b = p.by_hkv.quotient(bg), g = bg - b * p.hkv;
  const int n_blk = p.group * rblocks;
  const int held = min(n_blk, kBlocks);
  uint8_t* lds_q = smem;
  float2* lds_ml = reinterpret_cast<float2*>(smem + held * kQBytes);
  uint8_t* lds_k = smem + held * col_block_bytes<T, D>() + wave * O::kKTile;

  // candidate tiles: prefix rows [0, n0), suffix rows from block_off + block_len on
  const int n0 = min(p.n_cand, p.block_off), n1 = p.n_cand - n0;
  const int tiles0 = (n0 + kTileKeys - 1) / kTileKeys, ntiles = tiles0 + (n1 + kTileKeys - 1) / kTileKeys;
  const int64_t stride = p.k_sr * (int64_t)sizeof(T);
  const char* k_base = (const char*)p.k + sizeof(T) * (b * p.k_sb + g * p.k_sh);
  const int step = gridDim.x * kColWaves;
  float* score_row = p.score + (size_t)bg * p.score_stride;
  const float inv_count = 1.f / (float)(p.group * p.nq);

  for (int blk0 = 0; blk0 < n_blk; blk0 += kBlocks) {
    const int here = min(kBlocks, n_blk - blk0);
    if (blk0) __syncthreads();   // the previous blocks are done with
    constexpr int kPerRow = O::kRow / 16;
    for (int i = tid; i < here * R * kPerRow; i += kColWaves * kWave) {
      const int c = i % kPerRow, r = i / kPerRow % R, k = i / kPerRow / R;
      const int hh = by_rblocks.quotient(blk0 + k), row = (blk0 + k - hh * rblocks) * R + r;
      const u32x4 v = *reinterpret_cast<const u32x4*>((const char*)p.q + sizeof(T) * (b * p.q_sb + (int64_t)(g * p.group + hh) * p.q_sh + min(row, p.nq - 1) * p.q_sr) + c * 16);
      *reinterpret_cast<u32x4*>(lds_q + k * kQBytes + r * O::kKRow + c * 16) = v;
    }
    if (p.softmax) {
      for (int i = tid; i < here * R; i += kColWaves * kWave) {
        const int r = i % R, k = i / R;
        const int hh = by_rblocks.quotient(blk0 + k), rb = blk0 + k - hh * rblocks;
        float m_tot = -INFINITY, l_tot = 0.f;
        const float* src = p.part_ml + (((size_t)b * p.hq + g * p.group + hh) * rblocks + rb) * p.n_stat_part * 2 * R + r;
#pragma unroll 8
        for (int s = 0; s < p.n_stat_part; ++s) {
          const float m_s = src[s * 2 * R], l_s = src[s * 2 * R + R], m_new = fmaxf(m_tot, m_s);
          if (m_new != -INFINITY) l_tot = l_tot * __builtin_amdgcn_exp2f(m_tot - m_new) + l_s * __builtin_amdgcn_exp2f(m_s - m_new);
          m_tot = m_new;
        }
        lds_ml[i] = make_float2(m_tot, rb * R + r < p.nq ? 1.f / l_tot : 0.f);   // the statistics of padding rows are the last row's too
      }
    }
    __syncthreads();
    for (int t = blockIdx.x * kColWaves + wave; t < ntiles; t += step) {
      const bool suf = t >= tiles0;
      const int first = (suf ? t - tiles0 : t) * kTileKeys;
      const int rows = min(kTileKeys, (suf ? n1 : n0) - first), cand0 = (suf ? n0 : 0) + first;
      const char* src = k_base + (int64_t)(suf ? p.block_off + p.block_len + first : first) * stride;
      u32x4 kreg[O::kLoads];
      g_load_rows<O, false>(src, rows, stride, lane, kreg);
      g_store_rows<O>(lds_k, O::kKRow, lane, kreg);
      wave_lds_sync();
      typename O::KTile keys;
      O::load_keys(lds_k, col, part, keys);
      float total[O::kKeysPerLane];
#pragma unroll
      for (int n = 0; n < O::kKeysPerLane; ++n) total[n] = 0.f;
      int row0 = (blk0 - by_rblocks.quotient(blk0) * rblocks) * R;   // of block k, in its head
      for (int k = 0; k < here; ++k) {
        float s[O::NS], sum[O::kKeysPerLane];
        O::score(lds_q + k * kQBytes, keys, col, part, s);
#pragma unroll
        for (int n = 0; n < O::kKeysPerLane; ++n) sum[n] = 0.f;
        if (p.softmax) {
#pragma unroll
          for (int i = 0; i < O::NS; ++i) {
            const float2 ml = lds_ml[k * R + O::query(i, part)];
            sum[O::key_slot(i)] += __builtin_amdgcn_exp2f(s[i] * p.scale_log2 - ml.x) * ml.y;
          }
        } else {
#pragma unroll
          for (int i = 0; i < O::NS; ++i) sum[O::key_slot(i)] += row0 + O::query(i, part) < p.nq ? s[i] : 0.f;
#pragma unroll
          for (int n = 0; n < O::kKeysPerLane; ++n) sum[n] *= p.scale;
        }
#pragma unroll
        for (int n = 0; n < O::kKeysPerLane; ++n) total[n] += sum[n];
        row0 = row0 + R < p.nq ? row0 + R : 0;
      }
#pragma unroll
      for (int n = 0; n < O::kKeysPerLane; ++n) {
        total[n] = parts_sum<O>(total[n]);
        const int key = n * R + col;
        if (part == 0 && key < rows) {
          if (blk0) total[n] += score_row[cand0 + key];   // left there by this same lane
          score_row[cand0 + key] = blk0 + here == n_blk ? total[n] * inv_count : total[n];
        }
      }
      wave_lds_sync();
    }
  }
}

template <typename T, int D>
static hipError_t launch_cols(const ScoreParams& p, hipStream_t s) {
  using O = Ops<T, D>;
  static LdsOptIn lds;
  constexpr int kBlocks = col_blocks<T, D>(), kBlockBytes = col_block_bytes<T, D>();
  const auto kernel = score_cols_general_kernel<T, D>;
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), kBlocks * kBlockBytes + kColWaves * O::kKTile);
  if (e != hipSuccess) return e;
  const int rblocks = (p.nq + O::kRows - 1) / O::kRows, rows = p.batch * p.hkv;
  if (rows > 65535) return hipErrorInvalidValue;
  const int n0 = p.n_cand < p.block_off ? p.n_cand : p.block_off;
  const int tiles = (n0 + kTileKeys - 1) / kTileKeys + (p.n_cand - n0 + kTileKeys - 1) / kTileKeys;
  const int held = p.group * rblocks < kBlocks ? p.group * rblocks : kBlocks;
  // a tile per wave while the workgroups stay within four per CU: staging the queries costs a workgroup about as much as two tiles
  int parts = (tiles + kColWaves - 1) / kColWaves;
  const int most = (4 * kNumCUs + rows - 1) / rows;
  if (parts > most) parts = most;
  const size_t bytes = (size_t)held * kBlockBytes + kColWaves * O::kKTile;
  return launch(kernel, dim3(parts, rows), dim3(kColWaves * kWave), bytes, s, p, rblocks, Divisor(rblocks));
}

hipError_t launch_score_cols_general(const ScoreParams& p, int dtype, hipStream_t s) {
  if (p.n_cand <= 0) return hipSuccess;
  if (dtype == 0) return p.d == 128 ? launch_cols<__bf16, 128>(p, s) : launch_cols<__bf16, 64>(p, s);
  return p.d == 128 ? launch_cols<float, 128>(p, s) : launch_cols<float, 64>(p, s);
}

}  // namespace sdllm
