// Full-sequence bidirectional attention (every one of the L query rows over all L keys, no mask)
// for bf16, head_dim 128: what cache states 0 and 1 run for the rows outside the current block
// (the mask predictor recomputes the whole sequence at those steps; Sec. 3.1 and the description of
// cache_state 0 in the cache-management appendix).  Compute-bound (2 L^2 d flops per head against
// 4 L d bytes), so this one is organised for the matrix cores rather than for HBM:
//   * a workgroup of 8 waves owns 256 consecutive query rows of one head, wave w the 32-row block w
//     (one 32x32 MFMA block, same fragment layout as the block-step kernels);
//   * all L keys stream through a double-buffered LDS stage of two 32-key tiles, loaded once per
//     workgroup with coalesced 16-byte loads and shared by the 8 waves: each K/V byte fetched from
//     L2 feeds 256 query rows; one workgroup barrier per 64 keys, the next stage's global loads in
//     flight meanwhile;
//   * each wave alternates one block of sixteen MFMAs (logits of tile t+1 interleaved with the PV
//     product of tile t) with one block of vector-ALU work (softmax of tile t+1), the LDS operand
//     reads for the next MFMA block requested in between: while one wave of a SIMD is in its MFMA
//     block the other one's softmax runs under it;
//   * the query-block workgroups of one head (and of the G heads of a KV group) are adjacent in the
//     grid and, after the XCD renumbering, share an L2.
#include "attn_tile_math.h"

namespace sdllm {

constexpr int kFullWaves = 8;
constexpr int kFullKvTileBytes = kTileBytes + kVTileBytes;             // K tile + V tile

// KS key groups: the 8 waves of a workgroup are 8/KS row blocks x KS groups, each group walking its own share of the
// keys.  A stage holds two tiles (KS = 1) or one tile of every group; four tiles of one group (KS = 2, two tiles each)
// took the staging registers beyond what two waves per SIMD have.
constexpr int full_stage_tiles(int ks) { return ks <= 2 ? 2 : 4; }
constexpr int full_rows_per_wg(int ks) { return kFullWaves / ks * 32; }
constexpr int full_stage_bytes(int ks) { return full_stage_tiles(ks) * kFullKvTileBytes; }
constexpr int kFullParkBytes = kWave * kRowBytes + 512;                // a wave's accumulators (padded lanes), (max, sum) per row
constexpr int full_lds_bytes(int ks) { return ks == 1 || 2 * full_stage_bytes(ks) > kFullWaves * kFullParkBytes ? 2 * full_stage_bytes(ks) : kFullWaves * kFullParkBytes; }

// 512 threads load one stage: thread tid takes 16-byte chunk tid%16 of row tid/16 of K and of V, of
// each of the stage's tiles.
template <int NT>
__device__ __forceinline__ void full_load_stage(const char* k_base, const char* v_base, uint32_t stride, int first_key,
                                                int n_keys, int tid, u32x4 (&kreg)[NT], u32x4 (&vreg)[NT]) {
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    int r = first_key + j * kTileKeys + (tid >> 4);
    r = r < n_keys ? r : n_keys - 1;          // past the end: re-read the last key, masked later
    const uint32_t off = (uint32_t)r * stride + ((tid & 15) << 4);
    kreg[j] = *reinterpret_cast<const u32x4*>(k_base + off);   // re-read by the other query blocks: keep in L2
    vreg[j] = *reinterpret_cast<const u32x4*>(v_base + off);
  }
}

template <int NT>
__device__ __forceinline__ void full_store_stage(uint8_t* stage, int tid, const u32x4 (&kreg)[NT], const u32x4 (&vreg)[NT]) {
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    *reinterpret_cast<u32x4*>(stage + j * kFullKvTileBytes + tile_off(tid >> 4, tid & 15)) = kreg[j];
    *reinterpret_cast<u32x4*>(stage + j * kFullKvTileBytes + kTileBytes + vtile_off(tid >> 4, tid & 15)) = vreg[j];
  }
}

__global__ __launch_bounds__(512) void dense_full_mfma_bf16_kernel(const DenseFullParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int col = lane & 31;

  // renumber workgroups so that consecutive ids (which go round-robin over the XCDs) of one head's
  // query blocks end up on the same XCD
  const int wg = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int qblocks = (p.seq_len + full_rows_per_wg(1) - 1) / full_rows_per_wg(1);
  const int qb = wg % qblocks;
  const int head = wg / qblocks;
  const int b = head / p.hq;
  const int h = head - b * p.hq;
  const int g = h / p.group;

  // rows past the end of the sequence compute on a copy of the last row and are not written back:
  // every wave then runs the same program, barriers included
  const int q_row = qb * full_rows_per_wg(1) + wave * 32 + col;
  const bool row_valid = q_row < p.seq_len;
  const int q_row_c = row_valid ? q_row : p.seq_len - 1;
  bf16x8 qf[8];
  load_q_frags((const char*)p.q + 2 * (b * p.q_sb + h * p.q_sh + (int64_t)q_row_c * p.q_sr), half, qf);

  const char* k_base = (const char*)p.k + 2 * (b * p.k_sb + g * p.k_sh);
  const char* v_base = (const char*)p.v + 2 * (b * p.k_sb + g * p.k_sh);
  const uint32_t stride = (uint32_t)(p.k_sr * 2);
  const int n_keys = p.seq_len;
  const int stage_keys = full_stage_tiles(1) * kTileKeys;
  const int nstages = (n_keys + stage_keys - 1) / stage_keys;
  const int ntiles = (n_keys + kTileKeys - 1) / kTileKeys;

  f32x16 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[e][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // Pipeline state between iterations: pb = softmax numerators of the current tile t (bf16), f = its V
  // fragments, a = the K fragments of tile t+1.  Iteration t issues one MFMA block (logits of t+1, PV
  // of t), requests the fragments the next block needs from LDS, and runs the softmax of t+1 while
  // they arrive.  Tile t lives in stage t/2; stage s+1 is published (and the barrier met) in the even
  // iteration 2s, after the last read of stage s (V of tile 2s+1) has been requested and before the
  // first read of stage s+1 (K of tile 2s+2).
  u32x4 kreg[full_stage_tiles(1)], vreg[full_stage_tiles(1)];
  full_load_stage(k_base, v_base, stride, 0, n_keys, tid, kreg, vreg);
  full_store_stage(smem, tid, kreg, vreg);
  __syncthreads();
  if (nstages > 1) full_load_stage(k_base, v_base, stride, stage_keys, n_keys, tid, kreg, vreg);

  bf16x8 a[8], pb[2];
  PvFrags f;
  f32x16 sn;
  tile_k_load(smem, half, col, a);
  __builtin_amdgcn_sched_barrier(0);
  tile_logits_mma(a, qf, sn);
  tile_pv_load(smem + kTileBytes, lane, f);
  if (ntiles > 1) tile_k_load(smem + kFullKvTileBytes, half, col, a);
  __builtin_amdgcn_sched_barrier(0);
  softmax_block(sn, min(kTileKeys, n_keys), p.scale_log2, half, m_run, l_run, acc, pb);

  for (int t = 0; t + 1 < ntiles; ++t) {   // t = current tile
    const int s = t >> 1;
    const bool even = (t & 1) == 0;
    const uint8_t* stage = smem + (s & 1) * full_stage_bytes(1);
    uint8_t* next_stage = smem + ((s + 1) & 1) * full_stage_bytes(1);
    __builtin_amdgcn_sched_barrier(0);
    mfma_block(a, qf, sn, f, pb, acc);
    __builtin_amdgcn_sched_barrier(0);
    // V of tile t+1: second tile of stage s (its last read) or first tile of stage s+1
    tile_pv_load((even ? stage + kFullKvTileBytes : next_stage) + kTileBytes, lane, f);
    if (even && s + 1 < nstages) {
      full_store_stage(next_stage, tid, kreg, vreg);
      __syncthreads();
      if (s + 2 < nstages) full_load_stage(k_base, v_base, stride, (s + 2) * stage_keys, n_keys, tid, kreg, vreg);
    }
    // K of tile t+2: first or second tile of stage s+1
    if (t + 2 < ntiles) tile_k_load(even ? next_stage : next_stage + kFullKvTileBytes, half, col, a);
    __builtin_amdgcn_sched_barrier(0);
    softmax_block(sn, min(kTileKeys, n_keys - (t + 1) * kTileKeys), p.scale_log2, half, m_run, l_run, acc, pb);
  }
  // PV product of the last tile
  __builtin_amdgcn_sched_barrier(0);
  pv_block(f, pb, acc);

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (row_valid) {
    char* out_row = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + (int64_t)q_row * p.o_sr);
    write_wave_result(acc, m_run, l_tot, lane, half, true, out_row, nullptr, nullptr);
  }
}

// The same with KS = 2 or 4 key groups, for sequences whose 256-row workgroups would leave CUs idle.  Group k walks
// tiles k, k + KS, ... through the pipeline above; all groups meet at the same barriers, one per tile, and their
// results are merged through LDS at the end.
template <int KS>
__global__ __launch_bounds__(512) void dense_split_mfma_bf16_kernel(const DenseFullParams p) {
  constexpr int NT = full_stage_tiles(KS), RB = kFullWaves / KS, kStage = full_stage_bytes(KS);
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, col = lane & 31;
  const int rb = wave % RB, kg = wave / RB;

  const int wg = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int qblocks = (p.seq_len + full_rows_per_wg(KS) - 1) / full_rows_per_wg(KS);
  const int qb = wg % qblocks;
  const int head = wg / qblocks;
  const int b = head / p.hq, h = head - b * p.hq, g = h / p.group;
  const int q_row = qb * full_rows_per_wg(KS) + rb * 32 + col;
  const bool row_valid = q_row < p.seq_len;
  bf16x8 qf[8];
  load_q_frags((const char*)p.q + 2 * (b * p.q_sb + h * p.q_sh + (int64_t)min(q_row, p.seq_len - 1) * p.q_sr), half, qf);

  const char* k_base = (const char*)p.k + 2 * (b * p.k_sb + g * p.k_sh);
  const char* v_base = (const char*)p.v + 2 * (b * p.k_sb + g * p.k_sh);
  const uint32_t stride = (uint32_t)(p.k_sr * 2);
  const int n_keys = p.seq_len;
  const int ntiles = (n_keys + kTileKeys - 1) / kTileKeys;
  const int nstages = (ntiles + NT - 1) / NT;
  const int n_mine = nstages - ((nstages - 1) * NT + kg < ntiles ? 0 : 1);   // the last stage may lack this group's tile
  auto tile_lds = [&](int j) { return smem + (j & 1) * kStage + kg * kFullKvTileBytes; };
  auto rows_of = [&](int j) { return min(kTileKeys, n_keys - (j * NT + kg) * kTileKeys); };

  f32x16 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[e][i] = 0.f;
  float m_run = kNoMax, l_run = 0.f;

  u32x4 kreg[NT], vreg[NT];
  full_load_stage<NT>(k_base, v_base, stride, 0, n_keys, tid, kreg, vreg);
  full_store_stage<NT>(smem, tid, kreg, vreg);
  if (nstages > 1) full_load_stage<NT>(k_base, v_base, stride, NT * kTileKeys, n_keys, tid, kreg, vreg);
  __syncthreads();

  bf16x8 a[8], pb[2];
  PvFrags f;
  f32x16 sn;
  // Publishes stage j: its buffer held stage j-2, whose last read every wave had requested, and waited for, before the
  // barrier of stage j-1.
  auto open_stage = [&](int j) {
    if (j >= nstages) return;
    full_store_stage<NT>(smem + (j & 1) * kStage, tid, kreg, vreg);
    __syncthreads();
    if (j + 1 < nstages) full_load_stage<NT>(k_base, v_base, stride, (j + 1) * NT * kTileKeys, n_keys, tid, kreg, vreg);
  };
  // tile j's logits are in sn: request V(j), open the next stage, request K(j+1), then the softmax of tile j
  auto after_logits = [&](int j) {
    if (j < n_mine) tile_pv_load(tile_lds(j) + kTileBytes, lane, f);
    open_stage(j + 1);
    if (j + 1 < n_mine) tile_k_load(tile_lds(j + 1), half, col, a);
    __builtin_amdgcn_sched_barrier(0);
    if (j < n_mine) softmax_block(sn, rows_of(j), p.scale_log2, half, m_run, l_run, acc, pb);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (n_mine > 0) {
    tile_k_load(tile_lds(0), half, col, a);
    __builtin_amdgcn_sched_barrier(0);
    tile_logits_mma(a, qf, sn);
  }
  after_logits(0);
  int j = 0;
  for (; j + 1 < n_mine; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    mfma_block(a, qf, sn, f, pb, acc);
    __builtin_amdgcn_sched_barrier(0);
    after_logits(j + 1);
  }
  if (n_mine > 0) pv_block(f, pb, acc);
  for (; j + 1 < nstages; ++j) open_stage(j + 2);   // the same barriers for every group

  // merge of the key groups of each row block
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  __syncthreads();                          // the stages are done with
  uint8_t* mine = smem + wave * kFullParkBytes;
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = {acc[e][i4 * 4], acc[e][i4 * 4 + 1], acc[e][i4 * 4 + 2], acc[e][i4 * 4 + 3]};
      *reinterpret_cast<f32x4*>(mine + lane * kRowBytes + (e * 4 + i4) * 16) = v;
    }
  if (lane < 32) {
    float* ml = reinterpret_cast<float*>(mine + kWave * kRowBytes);
    ml[lane] = m_run;
    ml[32 + lane] = l_tot;
  }
  __syncthreads();
  float f_w[KS], m_tot = -INFINITY, l_all = 0.f;
  auto parked = [&](int k) { return smem + (k * RB + rb) * kFullParkBytes; };
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    f_w[k] = reinterpret_cast<const float*>(parked(k) + kWave * kRowBytes)[col];
    m_tot = fmaxf(m_tot, f_w[k]);
  }
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    f_w[k] = __builtin_amdgcn_exp2f(f_w[k] - m_tot);   // a group without tiles: 0
    l_all += f_w[k] * reinterpret_cast<const float*>(parked(k) + kWave * kRowBytes)[32 + col];
  }
  const float inv = 1.f / l_all;
  char* out_row = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + (int64_t)q_row * p.o_sr);
#pragma unroll
  for (int j = 0; j < 16 / KS; ++j) {
    const int i = kg * (16 / KS) + j;
    f32x4 o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k) o4 += *reinterpret_cast<const f32x4*>(parked(k) + lane * kRowBytes + i * 16) * f_w[k];
    bf16x4 ob;
#pragma unroll
    for (int r = 0; r < 4; ++r) ob[r] = (__bf16)(o4[r] * inv);
    if (row_valid) *reinterpret_cast<bf16x4*>(out_row + out_col0(i >> 2, i & 3, half) * 2) = ob;
  }
}

template <int KS>
static hipError_t launch_full(const DenseFullParams& p, hipStream_t s) {
  static LdsOptIn lds;
  const auto kernel = [] {
    if constexpr (KS == 1) return dense_full_mfma_bf16_kernel;
    else return dense_split_mfma_bf16_kernel<KS>;
  }();
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), full_lds_bytes(KS));
  if (e != hipSuccess) return e;
  const int qblocks = (p.seq_len + full_rows_per_wg(KS) - 1) / full_rows_per_wg(KS);
  hipLaunchKernelGGL(kernel, dim3(qblocks * p.batch * p.hq), dim3(512), full_lds_bytes(KS), s, p);
  return hipGetLastError();
}

// Key groups per workgroup: what a workgroup takes for its tiles (us, fitted to 1 to 8 x 8 to 32 heads, 65 to 2049
// positions), times the rounds in which the CUs, one workgroup each, go through the grid.  28 heads: 200 positions
// 12.2 -> 8.5 us (4 groups), 400 18.1 -> 11.0 (4), 735 26.1 -> 19.2 (2); 24 heads x 1277 39.6 -> 28.6 (2); 8 heads x 1277
// 38.8 -> 18.9 (4).  28 heads x 1277 stay whole: 280 half workgroups need a second round (53.8 against 39.8 us).
int dense_full_key_groups(int heads, int seq_len) {
  const int tiles = (seq_len + kTileKeys - 1) / kTileKeys;
  int best = 1;
  double least = 0;
  for (int ks = 1; ks <= 4; ks *= 2) {
    const int64_t wgs = (int64_t)((seq_len + full_rows_per_wg(ks) - 1) / full_rows_per_wg(ks)) * heads;
    const int64_t rounds = (wgs + kNumCUs - 1) / kNumCUs;
    const int mine = (tiles + ks - 1) / ks;
    const double us = (double)rounds * (ks == 1 ? 4.3 + 0.9 * mine : ks == 2 ? 6.2 + 1.08 * mine : 5.8 + 1.3 * mine);
    if (ks == 1 || us < 0.95 * least) { best = ks; least = us; }
  }
  return best;
}

hipError_t launch_dense_full_mfma_bf16(const DenseFullParams& p, hipStream_t s) {
  switch (dense_full_key_groups(p.batch * p.hq, p.seq_len)) {
    case 2: return launch_full<2>(p, s);
    case 4: return launch_full<4>(p, s);
    default: return launch_full<1>(p, s);
  }
}

}  // namespace sdllm
