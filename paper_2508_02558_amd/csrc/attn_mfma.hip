// Block-query attention over Concat(cache, block) for bf16, head_dim 128, 32 query rows
// (Alg. 3 of the paper, cache_state == 2; the same kernel run over the full sequence is the
// dense block-row attention of cache states 0 and 1).
//
// Design for gfx950.  The 32 query rows of one head make exactly one 32x32 MFMA block, so a
// wavefront owns whole 32-key tiles: logits^T = K_tile * Q^T (K rows as the A operand, so each
// lane ends up holding 16 logits of ONE query row and the softmax row reduction stays in
// registers), then O^T += V_tile^T * P^T.  With 32 queries per 8 KB of K the kernel is bound by
// HBM (about 31 flop/byte), so the structure is chosen for bytes in flight, not for MFMA rate:
//   * each wave streams its own tiles; there is no workgroup barrier in the main loop;
//   * global loads are full-row coalesced (16 lanes x 16 B per 256-byte row), held in registers
//     for one tile of look-ahead, then written to a wave-private, row-padded LDS tile from
//     which the MFMA operand fragments are read without bank conflicts;
//   * the V^T operands come straight out of the row-major V tile through the transposing LDS read
//     (ds_read_b64_tr_b16), four MFMAs covering the 128 columns (MFMA e produces columns 32e + m);
//   * up to 8 waves per workgroup (the planner picks 4 or 5 for unsplit MHA heads) split the keys of
//     one head and merge their running (max, sum, numerator) through LDS; more workgroups per head
//     (split-KV) write fp32 partials that a small combine kernel merges.
#include <type_traits>

#include "attn_tile_math.h"

namespace sdllm {

constexpr int kWaveLds = kTileBytes + kVTileBytes;    // K tile, V tile; later 64 lanes x 272 B of accumulators and 512 B of (max, sum)
static_assert(kWaveLds >= 64 * kRowBytes + 512 && kVTileBytes >= kRingK, "what shares a wave's LDS");

// Whether the queries have LDS of their own: where a CU holds one workgroup anyway.  With two or four to a CU they come by
// way of wave 0's V tile.
__host__ __device__ inline bool queries_apart(int waves, int wgs) { return waves > 4 || wgs <= kNumCUs; }

static size_t attn_mfma_lds_bytes(int waves, int wgs) { return (size_t)waves * kWaveLds + (queries_apart(waves, wgs) ? kRingK : 0); }

// NSEG = 2: keys are Concat(cache, block) (sparse step); NSEG = 1: one key tensor (dense step, or a
// sparse step with an empty cache).  The two instantiations also show up as separate kernels in a
// profile, which keeps sparse and dense launches apart.
// STATS (dense launches of the cache-update step only): also accumulate each query row's (max, sum)
// over the candidate keys, so the scoring pass that follows need not stream K for them again.
// DEEP: prefetch K and V of the next tile together (one memory latency per tile instead of two, twice
// the bytes in flight).  Chosen for small grids, which are latency-bound; large grids saturate HBM and
// run faster with the shallower alternating scheme.
// SHARED_KV: the G query heads of a KV group run as separate workgroups (grouped-query attention on
// a small grid); their K/V reads are then plain loads so that the siblings hit in L2.  K is also read
// with plain loads by the statistics launches: the scoring that follows (the column sweep at the end of
// this kernel, or the scoring kernel) reads the same rows again and finds part of them in L2 and the
// memory-side cache (B=8 LLaDA shape, cache-update step: 234 -> 226 us).
// SHARED_Q: the query rows come once per workgroup, through LDS.  As fragments that every wave loads from memory they are 32
// rows x 32 bytes an instruction and keep the CU's address path from the first keys for about 1 us (28 heads x 69 tiles in 8
// splits 11.4 -> 11.0 us, 32 x 21 in 3 10.1 -> 9.6, 336 x 11 11.2 -> 10.1, dense rows of 96 heads x 72 24.8 -> 23.6).  Multi-head calls
// without key splits stay with the fragments: the barrier that the other way takes holds their waves' streams together
// (64 heads x 21 tiles 11.5 against 11.8 us, 224 x 8 8.7 against 9.0, 256 x 69 45.1 against 45.3).
template <int NSEG, bool STATS, bool DEEP, bool SHARED_KV, bool BY_SPLIT, bool SHARED_Q>
__global__ __launch_bounds__(512) void attn_mfma_bf16_kernel(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int half = lane >> 5;
  const int col = lane & 31;

  // Consecutive workgroup ids go round-robin over the 8 XCDs; renumber so that neighbours sit on one XCD and share its L2:
  // the query heads of one KV group and key split, which read the same keys, or (BY_SPLIT) the splits of one head.
  const int wg = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int group = SHARED_KV && !BY_SPLIT ? p.group : 1;
  const int pair = wg / group;
  const int split = pair % p.n_split;
  const int bg = pair / p.n_split;
  const int b = bg / (BY_SPLIT ? p.hq : p.hkv);
  const int g_or_h = bg - b * (BY_SPLIT ? p.hq : p.hkv);
  const int h = BY_SPLIT ? g_or_h : g_or_h * group + wg - pair * group;
  const int g = BY_SPLIT ? h / p.group : g_or_h;
  const int head = b * p.hq + h;

  const SegPtrs sp = seg_ptrs(p, b, g, NSEG == 2);
  const int ntiles = sp.tiles0 + (sp.n1 + kTileKeys - 1) / kTileKeys;
  const int t_begin = split * p.tiles_per_split;
  const int t_end = min(ntiles, t_begin + p.tiles_per_split);

  // Q^T fragments (B operand): lane (col = query row, half) holds head-dim [16t + 8 half, +8)
  bf16x8 qf[8];
  const bool q_apart = queries_apart(nw, gridDim.x);
  uint8_t* lds_q = smem + (q_apart ? nw * kWaveLds : kTileBytes);
  if (SHARED_Q) request_queries<false>(p, b, h, lds_q, wave, nw, lane);
  else load_q_frags((const char*)p.q + 2 * (b * p.q_sb + h * p.q_sh + col * p.q_sr), half, qf);

  uint8_t* lds_k = smem + wave * kWaveLds;
  uint8_t* lds_v = lds_k + kTileBytes;

  f32x16 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[e][i] = 0.f;
  float m_run = -INFINITY;   // softmax reference of the row (log2 domain, within 8 of the running max), same in both halves
  float l_run = 0.f;         // running row sum over the keys this half-lane has seen
  float mc_run = -INFINITY, lc_run = 0.f;   // the same over candidate keys only (STATS)

  // Shallow scheme: one staging register set, used alternately for the K and the V tile, so a wave
  // keeps exactly one 8 KB tensor tile in flight (40-64 KB per CU with 5-8 waves).  Measured on MI355X, a
  // streaming read is fastest with 32-64 KB outstanding per CU and loses ~5 % at 128 KB, so K(t+1)
  // flies under the PV product of tile t and V(t) under its logits/softmax.
  u32x4 reg[8], reg2[DEEP ? 8 : 1];
  int t = t_begin + wave;
  uint32_t stride = 0;
  TileSrc ts{};
  if (t < t_end) {
    ts = tile_src(sp, t, stride);
    load_rows<!(SHARED_KV || STATS)>(ts.k, ts.rows, stride, lane, reg);
    if (DEEP) load_rows<!SHARED_KV>(ts.v, ts.rows, stride, lane, reinterpret_cast<u32x4(&)[8]>(reg2));
  }
  if (SHARED_Q) {
    in_issue_order();   // the queries are there when only the first tile's requests are left
    if (t >= t_end) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (DEEP) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    bare_barrier();
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = shared_k_frag(shared_k_at(lds_q, half, col), kk);
    if (!q_apart) {     // before wave 0's V tile goes there
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      bare_barrier();
    }
  }

  for (; t < t_end; t += nw) {
    const int rows = ts.rows;
    const int tn = t + nw;
    store_rows(lds_k, lane, reg);
    if (DEEP) {
      store_rows_v(lds_v, lane, reinterpret_cast<u32x4(&)[8]>(reg2));
      wave_lds_sync();
      if (tn < t_end) {                              // both tensors of tile t+1 fly during tile t
        ts = tile_src(sp, tn, stride);
        load_rows<!(SHARED_KV || STATS)>(ts.k, ts.rows, stride, lane, reg);
        load_rows<!SHARED_KV>(ts.v, ts.rows, stride, lane, reinterpret_cast<u32x4(&)[8]>(reg2));
      }
    } else {
      wave_lds_sync();
      load_rows<!SHARED_KV>(ts.v, ts.rows, stride, lane, reg);   // V(t) flies during the logits and the softmax
    }

    // logits^T[key, query] = K_tile Q^T (raw), row max in the scaled log2 domain
    f32x16 s;
    const float m_loc = tile_logits(lds_k, qf, rows, p.scale_log2, half, col, s);
    const int key0 = half * 4;
    if (STATS) {
      // single segment: register i is absolute position 32 t + key; the block's own keys (and, for
      // prefix-only eviction, the suffix) are not candidates
      const int pos0 = t * kTileKeys + key0;
      float sc[16];
      float mc_loc = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int pos = pos0 + (i >> 2) * 8 + (i & 3);
        sc[i] = (pos < p.cand0_end || pos >= p.cand1_begin) ? s[i] * p.scale_log2 : -INFINITY;
        mc_loc = fmaxf(mc_loc, sc[i]);
      }
      mc_loc = fmaxf(mc_loc, __shfl_xor(mc_loc, 32));
      const float mc_new = fmaxf(mc_run, mc_loc);
      if (mc_new != -INFINITY) {
        float lc_loc = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) lc_loc += __builtin_amdgcn_exp2f(sc[i] - mc_new);
        lc_run = lc_run * __builtin_amdgcn_exp2f(mc_run - mc_new) + lc_loc;
        mc_run = mc_new;
      }
    }
    tile_softmax(s, m_loc, p.scale_log2, m_run, l_run, acc);

    if (!DEEP) {
      store_rows_v(lds_v, lane, reg);
      wave_lds_sync();
      if (tn < t_end) {                              // K(t+1) flies during the PV product
        ts = tile_src(sp, tn, stride);
        load_rows<!(SHARED_KV || STATS)>(ts.k, ts.rows, stride, lane, reg);
      }
    }

    tile_pv(lds_v, s, lane, acc);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  float l_tot = l_run + __shfl_xor(l_run, 32);
  const float lc_tot = lc_run + __shfl_xor(lc_run, 32);
  const size_t slot = (size_t)head * p.n_split + split;

  if (nw == 1) {
    // a single wave owns the whole result: straight from registers
    if (STATS && lane < 32) {
      p.cand_ml[slot * 64 + lane] = mc_run;
      p.cand_ml[slot * 64 + 32 + lane] = lc_tot;
    }
    write_wave_result(acc, m_run, l_tot, lane, half, p.n_split == 1,
                      (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + col * p.o_sr), p.part_o + (slot * 32 + col) * 128,
                      p.part_ml + slot * 64);
    return;
  }

  // Merge the waves of the workgroup, all waves working: every wave parks its 64 accumulator
  // registers per lane in its own LDS region ([lane][e][i], lane stride 272 B) together with its
  // row (max, sum); after one barrier wave w reduces the 4-register slots w, w+nw, ... (of 16) over all waves.
  // All LDS reads of a slot are issued before any is used, so the merge costs a few hundred cycles.
  {
    uint8_t* mine = smem + wave * kWaveLds;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 v = {acc[e][i4 * 4], acc[e][i4 * 4 + 1], acc[e][i4 * 4 + 2], acc[e][i4 * 4 + 3]};
        *reinterpret_cast<f32x4*>(mine + lane * kRowBytes + (e * 4 + i4) * 16) = v;
      }
    float* my_ml = reinterpret_cast<float*>(mine + 64 * kRowBytes);
    if (lane < 32) {
      my_ml[lane] = m_run; my_ml[32 + lane] = l_tot;
      if (STATS) { my_ml[64 + lane] = mc_run; my_ml[96 + lane] = lc_tot; }
    }
  }
  __syncthreads();
  if (STATS && wave == 0 && lane < 32) {
    float mc = -INFINITY, lc = 0.f;
    for (int w = 0; w < nw; ++w)
      mc = fmaxf(mc, reinterpret_cast<const float*>(smem + w * kWaveLds + 64 * kRowBytes)[64 + lane]);
    for (int w = 0; w < nw; ++w) {
      const float* ml = reinterpret_cast<const float*>(smem + w * kWaveLds + 64 * kRowBytes);
      if (ml[64 + lane] != -INFINITY) lc += ml[96 + lane] * __builtin_amdgcn_exp2f(ml[64 + lane] - mc);
    }
    p.cand_ml[slot * 64 + lane] = mc;
    p.cand_ml[slot * 64 + 32 + lane] = lc;
    if (p.score_out) {   // merged statistics for the column sweep below, in wave 0's own slots
      float* st = reinterpret_cast<float*>(smem + 64 * kRowBytes) + 64;
      st[lane] = mc;
      st[32 + lane] = 1.f / lc;
    }
  }
  // With the wave count a compile-time constant every LDS read of the merge (the waves' (max, sum) and the
  // up to ceil(16 / NW) slots this wave reduces) is requested before the first is used: one LDS round trip
  // instead of one per slot.
  auto merge = [&](auto nw_tag) {
    constexpr int NW = decltype(nw_tag)::value;
    constexpr int NJ = (16 + NW - 1) / NW;
    float m_w[NW], l_w[NW], f_w[NW];
    f32x4 part[NJ][NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* ml = reinterpret_cast<const float*>(smem + w * kWaveLds + 64 * kRowBytes);
      m_w[w] = ml[col];
      l_w[w] = ml[32 + col];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int i = min(wave + j * NW, 15);   // past the last slot (some waves, last round): re-read slot 15, not stored
#pragma unroll
      for (int w = 0; w < NW; ++w)
        part[j][w] = *reinterpret_cast<const f32x4*>(smem + w * kWaveLds + lane * kRowBytes + i * 16);
    }
    __builtin_amdgcn_sched_barrier(0);
    float m_tot = -INFINITY, l_all = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_tot = fmaxf(m_tot, m_w[w]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      // a wave that saw no tile parked (-inf, 0, 0): factor 0
      f_w[w] = m_w[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_w[w] - m_tot);
      l_all += f_w[w] * l_w[w];
    }
    const float inv = 1.f / l_all;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int i = wave + j * NW;
      if (i < 16) {
        f32x4 o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) o4 += part[j][w] * f_w[w];
        const int d0 = out_col0(i >> 2, i & 3, half);   // slot i = (e, i4): four consecutive output columns
        if (p.n_split == 1) {
          bf16x4 ob;
#pragma unroll
          for (int r = 0; r < 4; ++r) ob[r] = (__bf16)(o4[r] * inv);
          char* op = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + col * p.o_sr);
          *reinterpret_cast<bf16x4*>(op + d0 * 2) = ob;
        } else {
          *reinterpret_cast<f32x4*>(p.part_o + (slot * 32 + col) * 128 + d0) = o4;
        }
      }
    }
    if (p.n_split > 1 && wave == 0 && lane < 32) {
      p.part_ml[slot * 64 + lane] = m_tot;
      p.part_ml[slot * 64 + 32 + lane] = l_all;
    }
  };
  switch (nw) {
    case 2: merge(std::integral_constant<int, 2>{}); break;
    case 3: merge(std::integral_constant<int, 3>{}); break;
    case 4: merge(std::integral_constant<int, 4>{}); break;
    case 5: merge(std::integral_constant<int, 5>{}); break;
    case 6: merge(std::integral_constant<int, 6>{}); break;
    case 7: merge(std::integral_constant<int, 7>{}); break;
    default: merge(std::integral_constant<int, 8>{}); break;
  }

  // Column sweep (cache-update step, MHA, no key splits): with the row statistics of the scoring softmax
  // final, the workgroup walks its head's keys once more, LAST TILE FIRST (the most recently read K rows
  // are the ones the memory-side cache may still hold), and leaves each candidate key's softmax-mean
  // saliency score (Alg. 1 steps 5-6).  Same fragments as the attention, operands swapped: Q rows as the A
  // operand, so a lane holds ONE key (lane % 32) against 16 query rows (8*(i/4) + 4*half + i%4).
  if (STATS && p.score_out) {
    __syncthreads();   // statistics visible; every wave is done with the parked accumulators
    const float* st = reinterpret_cast<const float*>(smem + 64 * kRowBytes) + 64;
    float row_m[16], row_il[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = (i >> 2) * 8 + half * 4 + (i & 3);
      row_m[i] = st[row];
      row_il[i] = st[32 + row];
    }
    float* score_row = p.score_out + (size_t)(b * p.hkv + g) * p.score_stride;
    const int gap = p.cand1_begin - p.cand0_end;
    int tc = ntiles - 1 - wave;
    if (tc >= 0) {
      ts = tile_src(sp, tc, stride);
      load_rows<true>(ts.k, ts.rows, stride, lane, reg);
    }
    for (; tc >= 0; tc -= nw) {
      const int rows = ts.rows;
      store_rows(lds_k, lane, reg);
      wave_lds_sync();
      if (tc - nw >= 0) {
        ts = tile_src(sp, tc - nw, stride);
        load_rows<true>(ts.k, ts.rows, stride, lane, reg);
      }
      bf16x8 a[8];
      tile_k_load(lds_k, half, col, a);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 sc;
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[kk], a[kk], sc, 0, 0, 0);
      float total = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) total += __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i], p.scale_log2, -row_m[i])) * row_il[i];
      total += __shfl_xor(total, 32);
      const int pos = tc * kTileKeys + col;
      const bool cand = pos < p.cand0_end || pos >= p.cand1_begin;
      if (half == 0 && col < rows && cand) score_row[pos < p.cand0_end ? pos : pos - gap] = total * p.score_inv_count;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

template <int NSEG, bool STATS, bool DEEP, bool SHARED_KV, bool SHARED_Q, bool BY_SPLIT = false>
static hipError_t launch_variant(const AttnParams& p, hipStream_t s) {
  const int nwg = p.batch * p.hq * p.n_split;
  static LdsOptIn lds;
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(attn_mfma_bf16_kernel<NSEG, STATS, DEEP, SHARED_KV, BY_SPLIT, SHARED_Q>),
                                  (int)attn_mfma_lds_bytes(kMaxWavesPerWg, 0));
  if (e != hipSuccess) return e;
  return launch(attn_mfma_bf16_kernel<NSEG, STATS, DEEP, SHARED_KV, BY_SPLIT, SHARED_Q>, dim3(nwg), dim3(p.waves * kWave),
                     attn_mfma_lds_bytes(p.waves, nwg), s, p);
}

template <int NSEG, bool STATS>
static hipError_t launch_nseg(const AttnParams& p, hipStream_t s) {
  // at most half the CUs busy: latency-bound, take the deep prefetch
  const bool deep = p.batch * p.hq * p.n_split <= kNumCUs / 2;
  // Splits of a head side by side: key splits of 24 tiles or more on more than half the chip, over one segment up to 40 (28
  // heads, sparse, 300 tiles 19.6 -> 19.0 us; 56 x 260 26.6 -> 25.7; 32 heads, dense rows, 242 tiles 17.5 -> 17.0).  Shorter ones
  // gain 0 to 8 % from heads side by side (16 heads x 34 tiles 10.1 -> 9.4 us), fewer workgroups 1 to 4 % (16 x 1000 tiles 38.1
  // -> 36.5), longer dense rows 1 to 4 % (28 x 700 tiles 31.2 -> 30.2).
  if constexpr (!STATS)
    if (p.group > 1 && !deep && p.n_split > 1 && p.tiles_per_split >= 24 && (NSEG == 2 || p.tiles_per_split < 40))
      return launch_variant<NSEG, false, false, true, true, true>(p, s);
  if (p.group > 1) return deep ? launch_variant<NSEG, STATS, true, true, true>(p, s) : launch_variant<NSEG, STATS, false, true, true>(p, s);
  // Multi-head sparse steps whose splits have five waves (nine or ten tiles, two to a wave) lose by the shared rows what those of
  // four, seven and eight gain: 32 heads x 66 tiles 13.6 us with fragments, 14.0, x 80 14.4, 14.8, 16 heads x 27 10.0, 10.3 (against
  // 13.3, 13.1 for 32 x 64, four waves, and 16.75, 16.45 for 32 x 105, seven).
  const bool shared_q = p.n_split > 1 && !(NSEG == 2 && p.waves == 5);
  if (shared_q) return deep ? launch_variant<NSEG, STATS, true, false, true>(p, s) : launch_variant<NSEG, STATS, false, false, true>(p, s);
  return deep ? launch_variant<NSEG, STATS, true, false, false>(p, s) : launch_variant<NSEG, STATS, false, false, false>(p, s);
}

hipError_t launch_attn_mfma_bf16(const AttnParams& p, hipStream_t s) {
  if (p.seg[0].n > 0 && p.seg[1].n > 0) return launch_nseg<2, false>(p, s);
  if (p.seg[1].n > 0) {   // empty cache: the block is the only key tensor
    AttnParams q = p;
    q.seg[0] = p.seg[1];
    q.seg[1].n = 0;
    return launch_nseg<1, false>(q, s);
  }
  return p.cand_ml ? launch_nseg<1, true>(p, s) : launch_nseg<1, false>(p, s);
}

}  // namespace sdllm
