// Full-sequence bidirectional attention (every one of the L query rows over all L keys, no mask)
// for bf16, head_dim 128: what cache states 0 and 1 run for the rows outside the current block
// (the mask predictor recomputes the whole sequence at those steps; Sec. 3.1 and the description of
// cache_state 0 in the cache-management appendix).  Compute-bound (2 L^2 d flops per head against
// 4 L d bytes), so this one is organised for the matrix cores rather than for HBM:
//   * a workgroup of 8 waves owns 256 consecutive query rows of one head, wave w the 32-row block w
//     (one 32x32 MFMA block, same fragment layout as the block-step kernels); with KS key groups it owns
//     256 / KS rows and group k walks tiles k, k + KS, ...;
//   * all L keys stream through rings of tiles in LDS, fetched once per workgroup and shared by its
//     waves: each K/V byte from L2 feeds 256 / KS query rows;
//   * per tile a wave has 512 cycles of matrix work and 380 of vector issue.  Left alone the two waves of a SIMD
//     drift into the same phase (every barrier puts them there) and then queue for the matrix pipe and for the
//     vector ALU in turn: 1790 cycles per pair of tiles in the loop, by time stamps, 2026 of a whole launch of 256 heads x
//     4352 positions, by counters.  Here they are locked in opposite phases, with a barrier
//     at each change: while one wave issues its sixteen MFMAs (logits of tile t+1 interleaved with the PV product
//     of tile t), the LDS reads of the next operands and half of tile t's exponentials between them, the other
//     finds its row maxima and does the first half of its exponentials: 1600 and 1848 cycles (matrix pipe 50.5 -> 55.4 %
//     busy).  The clock falls meanwhile (2.0 -> 1.9 GHz): 2412 -> 2315 us in trains of calls, 2320 -> 2255 by kernel trace; 28
//     heads x 1181 positions, half the chip, 39.9 -> 37.0, x 735 with two key groups 19.1 -> 17.4.  The start costs 0.3 us
//     more, so that sequences of up to eight tiles go without (kStagedKeys);
//   * the query-block workgroups of one head (and of the G heads of a KV group) are adjacent in the
//     grid and, after the XCD renumbering, share an L2.
#include <type_traits>

#include "attn_tile_math.h"

namespace sdllm {

constexpr int kFullWaves = 8;
constexpr int kFullKvTileBytes = kTileBytes + kVTileBytes;             // K tile + V tile

// KS key groups: the 8 waves of a workgroup are 8/KS row blocks x KS groups, each group walking its own share of the
// keys.
constexpr int full_rows_per_wg(int ks) { return kFullWaves / ks * 32; }
constexpr int kFullParkBytes = kWave * kRowBytes + 512;                // a wave's accumulators (padded lanes), (max, sum) per row

// 512 threads load one stage (KS = 4): thread tid takes 16-byte chunk tid%16 of row tid/16 of K and of V, of
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

// Merge of the KS key groups of each row block through LDS (group k of row block rb is wave k * 8 / KS + rb).
template <int KS>
__device__ __forceinline__ void merge_key_groups(uint8_t* smem, const f32x16 (&acc)[4], float m_run, float l_tot, int wave, int lane,
                                                 int half, int col, bool row_valid, char* out_row) {
  constexpr int RB = kFullWaves / KS;
  const int rb = wave % RB, kg = wave / RB;
  __syncthreads();                          // the tiles are done with
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

// ---- one and two key groups: waves in opposite phases
// For sequences of more steps than the rings hold, that is beyond this many positions (why there: launch_dense_full_mfma_bf16).
constexpr int kStagedKeys = 256;
constexpr int phase_ring(int ks) { return ks == 1 ? 5 : 4; }   // steps held: 86 and 137 KB
static_assert((kStagedKeys / kTileKeys + 1) > phase_ring(1) && (kStagedKeys / kTileKeys + 2) / 2 > phase_ring(2), "the prologue fills the rings");
constexpr int phase_lds_bytes(int ks) {
  const int ring = phase_ring(ks) * ks * (kRingK + kRingV), parked = ks == 1 ? 0 : kFullWaves * kFullParkBytes;
  return ks == 1 ? ring + kFullWaves * kRingK : ring > parked ? ring : parked;
}

__device__ __forceinline__ i16x8 phase_v_frag(const uint8_t* at, int i) {
  typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
  at += (i >> 2) * 512 + (i & 3) * 64;
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)at);
  const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(at + 256));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Softmax numerators of registers 8 st + r and the one after it.
__device__ __forceinline__ void numerator_pair(f32x16& s, int st, int r, float scale_log2, float m_ref, float& l, bf16x8 (&pb)[2]) {
#pragma unroll
  for (int i = r; i < r + 2; ++i) {
    const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * st + i], scale_log2, -m_ref));
    l += x;
    pb[st][i] = (__bf16)x;
  }
}

// Vector phase of a tile: row maxima, the reference, numerators of keys 0-15.
__device__ __forceinline__ void softmax_first_half(f32x16& sn, int rows, float scale_log2, int half, float& m_ref, float& l_run,
                                                   f32x16 (&acc)[4], bf16x8 (&pb)[2]) {
  const float m_loc = tile_mask_max(sn, rows, scale_log2, half);
  move_reference(m_loc, m_ref, l_run, acc);
  float l = 0.f;
#pragma unroll
  for (int r = 0; r < 8; r += 2) numerator_pair(sn, 0, r, scale_log2, m_ref, l, pb);
  l_run += l;
}

// Matrix phase: logits of the next tile, PV of the current one, each operand register set reloaded for the
// next phase once it has been used; the current tile's second eight numerators are done between the first MFMAs.
__device__ __forceinline__ void matrix_phase(bf16x8 (&a)[8], const bf16x8 (&qf)[8], f32x16& sn, PvFrags& f, bf16x8 (&pb)[2], f32x16 (&acc)[4],
                                             const uint8_t* k_at, const uint8_t* v_at, float scale_log2, float m_ref, float& l_run) {
  f32x16 s = sn;
  float l = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) sn[i] = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], qf[i], sn, 0, 0, 0);
    acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.av[i >> 2][i & 3]), pb[i >> 2], acc[i & 3], 0, 0, 0);
    a[i] = shared_k_frag(k_at, i);
    f.av[i >> 2][i & 3] = phase_v_frag(v_at, i);
    if (i < 4) numerator_pair(s, 1, 2 * i, scale_log2, m_ref, l, pb);
    __builtin_amdgcn_sched_barrier(0);
  }
  l_run += l;
}

template <int KS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dense_phase_mfma_bf16_kernel(const DenseFullParams p) {
  constexpr int RB = kFullWaves / KS, N = phase_ring(KS), kStepK = KS * kRingK, kStepV = KS * kRingV, kV0 = N * kStepK;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, col = lane & 31;
  const int rb = wave % RB, kg = wave / RB;
  const bool late = wave >= kFullWaves / 2;   // waves w and w + 4 share a SIMD: the second four run one phase behind

  // renumber workgroups so that consecutive ids (which go round-robin over the XCDs) of one head's
  // query blocks end up on the same XCD
  const int wg = p.first_wg + xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int head = p.by_qblocks.quotient(wg), qb = wg - head * p.qblocks;
  if (qb * full_rows_per_wg(KS) >= p.seq_len) return;   // key groups of a part of the grid: a 256-row block may end in blocks without rows
  const int b = p.by_hq.quotient(head), h = head - b * p.hq, g = p.by_group.quotient(h);
  // rows past the end of the sequence compute on a copy of the last row and are not written back
  const int q_row = qb * full_rows_per_wg(KS) + rb * 32 + col;
  const bool row_valid = q_row < p.seq_len;
  // With one key group the query rows come whole rows at a time, through LDS of the wave's own (there is none left with two)
  bf16x8 qf[8];
  [[maybe_unused]] uint8_t* lds_q = smem + phase_ring(1) * (kRingK + kRingV) + wave * kRingK;
  if constexpr (KS == 1) {
#pragma unroll
    for (int c = 0; c < 8; ++c)
      fetch_to_lds(lds_address(lds_q) + (uint32_t)(c * kKGroup),
                   (const char*)p.q + 2 * (b * p.q_sb + h * p.q_sh + (int64_t)min(q_row - col + c + 8 * (lane >> 4), p.seq_len - 1) * p.q_sr) +
                       fetch_k_chunk(lane));
  } else {
    load_q_frags((const char*)p.q + 2 * (b * p.q_sb + h * p.q_sh + (int64_t)min(q_row, p.seq_len - 1) * p.q_sr), half, qf);
  }

  const char* k_base = (const char*)p.k + 2 * (b * p.k_sb + g * p.k_sh);
  const char* v_base = (const char*)p.v + 2 * (b * p.k_sb + g * p.k_sh);
  const uint32_t stride = (uint32_t)(p.k_sr * 2);
  const int n_keys = p.seq_len;
  const int ntiles = (n_keys + kTileKeys - 1) / kTileKeys;
  const int nsteps = (ntiles + KS - 1) / KS;                                 // step j: tiles j KS .. j KS + KS - 1, one per group; > N
  const int n_mine = nsteps - ((nsteps - 1) * KS + kg < ntiles ? 0 : 1);   // the last step may lack this group's tile

  // A step's fetch: wave w brings group w of every tile.  Rows past the last key re-read it (masked later), a step past the
  // last one likewise.
  const uint32_t lds0 = lds_address(smem), k_chunk = fetch_k_chunk(lane), v_chunk = fetch_v_chunk(lane);
  auto fetch = [&](const char* base, uint32_t chunk, int step, int i, int at) {
    const int row = min((step * KS + i) * kTileKeys + wave + 8 * (lane >> 4), n_keys - 1);
    fetch_to_lds(lds0 + (uint32_t)at, base, (uint32_t)row * stride + chunk);
  };
  auto fetch_k = [&](int step, int slot) {
#pragma unroll
    for (int i = 0; i < KS; ++i) fetch(k_base, k_chunk, step, i, slot + i * kRingK + wave * kKGroup);
  };
  auto fetch_v = [&](int step, int slot) {
#pragma unroll
    for (int i = 0; i < KS; ++i) fetch(v_base, v_chunk, step, i, kV0 + slot + i * kRingV + wave * kVGroup);
  };
  auto rows_of = [&](int j) { return min(kTileKeys, n_keys - (j * KS + kg) * kTileKeys); };
  const uint8_t* k_at = shared_k_at(smem + kg * kRingK, half, col);
  const uint8_t* v_at = shared_v_at(smem + kV0 + kg * kRingV, lane);

  f32x16 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[e][i] = 0.f;
  float m_run = kNoMax, l_run = 0.f;
  bf16x8 a[8], pb[2];
  PvFrags f;
  f32x16 sn;

  // Requests are counted, in the order K(0), V(0), K(1) (with the query rows), V(1), K(2), ..., V(N-1), K(N) and then V(t+N),
  // K(t+N+1) for t = 0, 1, ...  The empty statement (KS = 2) uses the query rows, so that the compiler waits for them now: its wait
  // is for everything requested by then.
  fetch_k(0, 0);
  fetch_v(0, 0);
  fetch_k(1, kStepK);
  in_issue_order();
  if constexpr (KS > 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(qf[i]));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if constexpr (KS == 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) qf[i] = shared_k_frag(shared_k_at(lds_q, half, col), i);
  }
  bare_barrier();
#pragma unroll
  for (int j = 1; j < N; ++j) {
    if (j > 1) fetch_k(j, j * kStepK);
    fetch_v(j, j * kStepV);
  }
  in_issue_order();
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = shared_k_frag(k_at, i);
  tile_logits_mma(a, qf, sn);
#pragma unroll
  for (int i = 0; i < 8; ++i) f.av[i >> 2][i & 3] = phase_v_frag(v_at, i);
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = shared_k_frag(k_at + kStepK, i);
  softmax_first_half(sn, rows_of(0), p.scale_log2, half, m_run, l_run, acc, pb);
  // What the early waves read before a wait of the late ones stands between has landed: K(2), K(3), V(1), V(2).
  if (KS == 1) asm volatile("s_waitcnt lgkmcnt(0) vmcnt(3)" ::: "memory");   // V(3), K(4), V(4)
  else asm volatile("s_waitcnt lgkmcnt(0) vmcnt(2)" ::: "memory");           // V(3)
  bare_barrier();
  fetch_k(N, 0);
  in_issue_order();
  if (late) bare_barrier();

  // Iteration t: matrix phase (logits of step t+1, PV of step t; reads K(t+2), V(t+1)), barrier, vector phase (softmax of step
  // t+1), barrier.  The late waves are one phase behind: vector phase t is the last that they end before the early ones'
  // matrix phase t+2, so what that reads, K(t+4) and V(t+3), has to have landed by then.  Requested behind those are V(t+N-1),
  // K(t+N) (KS = 1) and V(t+N), K(t+N+1): four requests either way.  A place in a ring is fetched into in vector phase t at the
  // earliest after the barrier that ends the late waves' vector phase t-1, at the end of which what they read there, in
  // matrix phase t-1, is in registers.
  static_assert(N == (KS == 1 ? 5 : 4), "the waits count on it");
  int t = 0, v_slot = kStepV, k_slot = 2 * kStepK, v_next = 0, k_next = kStepK;   // places of V(t+1), K(t+2), V(t+N), K(t+N+1)
  auto advance = [&](int& slot, int by) { slot = slot + by == N * by ? 0 : slot + by; };
  auto iteration = [&](auto fetches) {
    __builtin_amdgcn_s_setprio(1);
    matrix_phase(a, qf, sn, f, pb, acc, k_at + k_slot, v_at + v_slot, p.scale_log2, m_run, l_run);
    __builtin_amdgcn_s_setprio(0);
    bare_barrier();
    if (fetches) {
      fetch_v(t + N, v_next);
      fetch_k(t + N + 1, k_next);
    }
    in_issue_order();
    softmax_first_half(sn, rows_of(t + 1), p.scale_log2, half, m_run, l_run, acc, pb);
    in_issue_order();
    advance(v_slot, kStepV); advance(k_slot, kStepK); advance(v_next, kStepV); advance(k_next, kStepK);
    if (fetches) asm volatile("s_waitcnt lgkmcnt(0) vmcnt(4)" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0) vmcnt(0)" ::: "memory");
    bare_barrier();
  };
  for (; t + N < nsteps; ++t) iteration(std::true_type{});
  for (; t + 1 < n_mine; ++t) iteration(std::false_type{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land in LDS that is parked in, or another workgroup's
  float l = 0.f;
#pragma unroll
  for (int r = 0; r < 8; r += 2) numerator_pair(sn, 1, r, p.scale_log2, m_run, l, pb);
  l_run += l;
  pv_block(f, pb, acc);
  for (; t + 1 < nsteps; ++t) { bare_barrier(); bare_barrier(); }   // the same barriers for every group
  if (!late) bare_barrier();

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  char* out_row = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + (int64_t)q_row * p.o_sr);
  if constexpr (KS == 1) {
    if (row_valid) write_wave_result(acc, m_run, l_tot, lane, half, true, out_row, nullptr, nullptr);
  } else {
    merge_key_groups<KS>(smem, acc, m_run, l_tot, wave, lane, half, col, row_valid, out_row);
  }
}

// ---- short sequences: stages loaded through registers
// Two stages in LDS, of two tiles (KS = 1) or one tile per group; each wave alternates one block of sixteen MFMAs with the
// softmax, the LDS requests in between; a barrier per stage, at which all groups meet.  Always with four key groups, whose
// tiles leave no room for rings.
constexpr int split_stage_tiles(int ks) { return ks == 1 ? 2 : ks; }
constexpr int split_stage_bytes(int ks) { return split_stage_tiles(ks) * kFullKvTileBytes; }
constexpr int split_lds_bytes(int ks) {
  const int stages = 2 * split_stage_bytes(ks), parked = ks == 1 ? 0 : kFullWaves * kFullParkBytes;   // where the stages were
  return stages > parked ? stages : parked;
}

template <int KS>
__global__ __launch_bounds__(512) void dense_split_mfma_bf16_kernel(const DenseFullParams p) {
  constexpr int NT = split_stage_tiles(KS), T = NT / KS, RB = kFullWaves / KS, kStage = split_stage_bytes(KS);   // T tiles of a group
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, col = lane & 31;
  const int rb = wave % RB, kg = wave / RB;

  const int wg = p.first_wg + xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int head = p.by_qblocks.quotient(wg), qb = wg - head * p.qblocks;
  if (qb * full_rows_per_wg(KS) >= p.seq_len) return;   // key groups of a part of the grid: a 256-row block may end in blocks without rows
  const int b = p.by_hq.quotient(head), h = head - b * p.hq, g = p.by_group.quotient(h);
  const int q_row = qb * full_rows_per_wg(KS) + rb * 32 + col;
  const bool row_valid = q_row < p.seq_len;
  bf16x8 qf[8] = {};
  if (KS > 1 || q_row - col < p.seq_len)   // of eight row blocks a short sequence leaves up to seven without rows: they ask for none
    load_q_frags((const char*)p.q + 2 * (b * p.q_sb + h * p.q_sh + (int64_t)min(q_row, p.seq_len - 1) * p.q_sr), half, qf);

  const char* k_base = (const char*)p.k + 2 * (b * p.k_sb + g * p.k_sh);
  const char* v_base = (const char*)p.v + 2 * (b * p.k_sb + g * p.k_sh);
  const uint32_t stride = (uint32_t)(p.k_sr * 2);
  const int n_keys = p.seq_len;
  const int ntiles = (n_keys + kTileKeys - 1) / kTileKeys;
  const int nstages = (ntiles + NT - 1) / NT;
  const int n_mine = (ntiles - kg + KS - 1) / KS;                           // tiles kg, kg + KS, ...: the last stage may lack one
  auto tile_lds = [&](int j) { return smem + (j / T & 1) * kStage + (kg + j % T * KS) * kFullKvTileBytes; };
  auto rows_of = [&](int j) { return min(kTileKeys, n_keys - (j * KS + kg) * kTileKeys); };

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
  // Publishes stage s: its buffer held stage s-2, whose last read every wave had requested, and waited for, before the
  // barrier of stage s-1.
  auto open_stage = [&](int s) {
    if (s >= nstages) return;
    full_store_stage<NT>(smem + (s & 1) * kStage, tid, kreg, vreg);
    __syncthreads();
    if (s + 1 < nstages) full_load_stage<NT>(k_base, v_base, stride, (s + 1) * NT * kTileKeys, n_keys, tid, kreg, vreg);
  };
  // tile j's logits are in sn: request V(j), open the next stage if tile j was this one's last, request K(j+1), then the
  // softmax of tile j
  auto after_logits = [&](int j) {
    if (j < n_mine) tile_pv_load(tile_lds(j) + kTileBytes, lane, f);
    if ((j + 1) % T == 0) open_stage((j + 1) / T);
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
  if constexpr (KS > 1)
    for (; j + 1 < nstages; ++j) open_stage(j + 2);   // the same barriers for every group

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  char* out_row = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + (int64_t)q_row * p.o_sr);
  if constexpr (KS == 1) {
    if (row_valid) write_wave_result(acc, m_run, l_tot, lane, half, true, out_row, nullptr, nullptr);
  } else {
    merge_key_groups<KS>(smem, acc, m_run, l_tot, wave, lane, half, col, row_valid, out_row);
  }
}

// Workgroups [first, first + count) of those that `qblocks` of them per head make
template <int KS, bool PHASE>
static hipError_t launch_full(const DenseFullParams& p, int qblocks, int first, int count, hipStream_t s) {
  static LdsOptIn lds;
  constexpr int kLds = PHASE ? phase_lds_bytes(KS) : split_lds_bytes(KS);
  const auto kernel = [] {
    if constexpr (PHASE) return dense_phase_mfma_bf16_kernel<KS>;
    else return dense_split_mfma_bf16_kernel<KS>;
  }();
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), kLds);
  if (e != hipSuccess) return e;
  DenseFullParams q = p;
  q.qblocks = qblocks;
  q.first_wg = first;
  q.by_qblocks = Divisor(qblocks); q.by_hq = Divisor(p.hq); q.by_group = Divisor(p.group);
  return launch(kernel, dim3(count), dim3(512), kLds, s, q);
}

template <int KS, bool PHASE>
static hipError_t launch_full(const DenseFullParams& p, hipStream_t s) {
  const int qblocks = (p.seq_len + full_rows_per_wg(KS) - 1) / full_rows_per_wg(KS);
  return launch_full<KS, PHASE>(p, qblocks, 0, qblocks * p.batch * p.hq, s);
}

// Key groups per workgroup: what a workgroup takes for its tiles (us), times the rounds in which the CUs, one workgroup each, go
// through the grid.  The costs are fitted to the kernels on either side of kStagedKeys.  Beyond it (4 to 512 heads, 257 to 2049
// positions, 1 / 2 / 4 groups): 28 heads x 735 24.2 / 17.8 / 26.4 us, 8 x 1277 35.4 / 23.3 / 19.0, 8 x 2049 53.1 / 33.2 / 52.7, 24 x
// 1277 37.3 / 27.5 / 37.6, 56 x 1277 78.7 / 74.7 / 91.0; 28 x 1277 stay whole, as 280 half workgroups need a second round (37.7 /
// 48.7 / 54.8).  The choice is the fastest of the three or within 1 % of it at 645 of 665 sizes, within 8 % at the others.  Up to
// kStagedKeys 28 x 192 10.6 / 9.7 / 7.9; the fit misses up to a fifth with five tiles (28 x 160 9.4 / 9.4 / 7.9).
static int key_groups_throughout(int heads, int seq_len) {
  const int tiles = (seq_len + kTileKeys - 1) / kTileKeys;
  const bool rings = seq_len > kStagedKeys;
  int best = 1;
  double least = 0;
  for (int ks = 1; ks <= 4; ks *= 2) {
    const int64_t wgs = (int64_t)((seq_len + full_rows_per_wg(ks) - 1) / full_rows_per_wg(ks)) * heads;
    const int64_t rounds = (wgs + kNumCUs - 1) / kNumCUs;
    const int mine = (tiles + ks - 1) / ks;
    const double us = (double)rounds * (rings ? (ks == 1 ? 10.2 + 0.76 * mine : ks == 2 ? 8.9 + 0.86 * mine : 4.9 + 1.49 * mine)
                                              : (ks == 1 ? 4.3 + 0.9 * mine : ks == 2 ? 6.2 + 1.08 * mine : 5.8 + 1.3 * mine));
    if (ks == 1 || us < (rings ? 0.97 : 0.95) * least) { best = ks; least = us; }
  }
  return best;
}

// Whole workgroups in rounds of the chip leave a last round that may be nearly empty: 280 of them take as long as 512.  If at most half of a
// round is left, those rows run as a launch of their own with two key groups per workgroup, with four if it is a quarter, in less than a
// round's time: tiles x 0.27 - 3.5 or x 0.38 - 2 us gained.  Measured, before / with: 48 heads x 1364 positions (256 + 32 workgroups) 82.7 / 68.2 us, 64 x
// 1100 (+ 64) 69.2 / 59.4, 84 x 916 (+ 80) 60.7 / 55.0, 28 x 4700 (2 x 256 + 20) 388 / 339, 48 x 2985 (2 x 256 + 64) 259 / 229, 56 x 4078 (3 x
// 256 + 128) 469 / 450, 224 x 1174 (4 x 256 + 96) 194 / 187; where two groups throughout were the choice, 28 x 2393 119.5 / 108.3, 56 x 1200
// 69.9 / 62.7, but 192 x 600 58.9 / 60.4.  More than half a round left: 28 x 3684 (+ 164) 204 / 228.  Short: 364 x 513 (+ 68) 90.9 / 95.1.
// Nor where two groups throughout need no round more than the whole rounds do, as a last block of at most 128 rows is one of their workgroups
// instead of two: 24 x 2599 (504 of 512 half workgroups) 94.8 / 117.8, 56 x 1075 48.2 / 61.0, 112 x 1048 90.0 / 96.1,
// 60 x 3120 317 / 326.
DenseFullGroups dense_full_groups(int heads, int seq_len) {
  const int throughout = key_groups_throughout(heads, seq_len);
  const int tiles = (seq_len + kTileKeys - 1) / kTileKeys;
  const int64_t wgs = (int64_t)((seq_len + full_rows_per_wg(1) - 1) / full_rows_per_wg(1)) * heads;
  const int left = (int)(wgs % kNumCUs);
  if (seq_len <= kStagedKeys || throughout == 4 || wgs < kNumCUs || left == 0 || left > kNumCUs / 2) return {throughout, 0};
  const int groups = left <= kNumCUs / 4 ? 4 : 2;
  if (tiles < (throughout == 2 ? 32 : groups == 4 ? 9 : 24)) return {throughout, 0};
  const int64_t halves = (int64_t)((seq_len + full_rows_per_wg(2) - 1) / full_rows_per_wg(2)) * heads;
  if (throughout == 2 && halves <= 2 * (wgs - left)) return {throughout, 0};
  return {1, groups};
}

// Up to kStagedKeys positions one or two key groups load their stages through registers as well: locked phases cost half an iteration at the
// start and pay it back from some ten tiles on, and a wave without rows still fetches its share of the rings and of the queries.
// Phases / stages: 28 heads x 32 positions 4.07 / 3.60 us, x 64 5.49 / 4.82, x 96 6.76 / 6.55; 224 x 224 16.8 / 16.3; 256 x 128 11.65 /
// 11.08, x 256 20.7 / 20.3; two groups, 128 x 256 13.62 / 13.31.  Beyond, where 256-row workgroups come in twos: 256 x 288 34.9 / 35.2,
// 28 x 735 with two groups 17.6 / 19.2.
hipError_t launch_dense_full_mfma_bf16(const DenseFullParams& p, hipStream_t s) {
  const auto [ks, tail] = dense_full_groups(p.batch * p.hq, p.seq_len);
  if (p.seq_len <= kStagedKeys)
    return ks == 4 ? launch_full<4, false>(p, s) : ks == 2 ? launch_full<2, false>(p, s) : launch_full<1, false>(p, s);
  if (tail == 0) return ks == 4 ? launch_full<4, false>(p, s) : ks == 2 ? launch_full<2, true>(p, s) : launch_full<1, true>(p, s);
  const int qblocks = (p.seq_len + full_rows_per_wg(1) - 1) / full_rows_per_wg(1), all = qblocks * p.batch * p.hq;
  const int whole = all / kNumCUs * kNumCUs;
  const hipError_t e = launch_full<1, true>(p, qblocks, 0, whole, s);
  if (e != hipSuccess) return e;
  return tail == 2 ? launch_full<2, true>(p, qblocks * 2, whole * 2, (all - whole) * 2, s)
                   : launch_full<4, false>(p, qblocks * 4, whole * 4, (all - whole) * 4, s);
}

}  // namespace sdllm
