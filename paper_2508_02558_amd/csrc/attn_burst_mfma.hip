// Block-query attention of small calls (bf16, head_dim 128, 32 query rows): Alg. 3, cache_state == 2, and the dense block
// rows of state 0, where a workgroup per head and key split has at most nine tiles of 32 keys.
//
// Nothing of such a call is throughput: it is one chain of latencies.  The kernels that stream tiles pay a round trip to memory
// per tile of a wave and merge whole accumulators (16 KB a wave through LDS) at the end.  Here
//   * every byte that the workgroup reads is requested before anything is waited for: 9 x 16 KB of keys and values and the query
//     rows, straight into LDS, which they fill;
//   * a wave per tile takes logits and softmax numerators relative to the tile's own row maxima, and leaves the numerators as bf16
//     operands where its K tile was;
//   * then the waves share out the output instead of the keys: wave w multiplies 32 columns of V with the numerators of 16 query
//     rows over all tiles and weighs the tiles' products as their maxima say, so that there is nothing to merge; its V operands
//     come from LDS under the exponentials.
// 28 heads x 69 tiles in 8 splits, by time stamps when the tiles still shared one reference per row: 1.7 us for the launch, 1.1 until all has
// landed, 0.5 logits, 0.6 numerators, 0.6 products, 0.9 until the partials are out, and 3.3 for the merge.  Calls, before and after (replayed
// graphs, each layer with keys of its own): 28 heads x 69 tiles 10.45 -> 9.35 us, x 40 9.34 -> 7.85, x 7 5.95 -> 4.99, x 2 4.56 -> 3.53; 32 x 21 9.64 ->
// 9.23; 4 x 72 10.45 -> 7.34; 224 x 6 6.17 -> 5.24; 128 x 7 (multi-head) 7.77 -> 7.09; geometric mean over 313 sizes 1.23, none slower
// (profiles/small_calls_sweep.txt).  Where the line to the other kernels lies: burst_splits in api.hip.
// Tried, not kept: the same in chunks of eight tiles, K of the next requested behind the operand reads of the last (2.2 us a chunk against 1.3 of
// the streaming kernels: what stands between two barriers of everybody adds up); non-temporal fetches for multi-head calls (level, also where the
// keys come from memory); V operands read behind the barrier of the numerators
// (+0.15 us); all kernel arguments loaded first (level).  Indexes divided by the compiler instead of by Divisor cost 0.15 to 0.3 us.
#include <type_traits>

#include "attn_tile_math.h"

namespace sdllm {

constexpr int kBurstSlot = kRingK + kRingV;                  // a tile of K and one of V
constexpr int kBurstOutWaves = 8;                            // 4 x 32 columns, 2 x 16 query rows
// What a tile's wave leaves in the K tile's place for the others: row maxima and sums, numerators
constexpr int kBurstMax = 0, kBurstSum = 128, kBurstP = 256;
constexpr int burst_lds_bytes(int tiles) { return tiles * kBurstSlot + kRingK; }
static_assert(burst_lds_bytes(kBurstMaxTiles) <= 160 * 1024, "the workgroup's tiles and query rows fill LDS");

// 16 bytes of a V row in LDS: as in mfma_tile.h, but with 32-byte halves swapped in rows 16 to 31, which the transposing
// read of 16x16x32 operands takes together with rows 0 to 15.
__device__ __forceinline__ uint32_t burst_v_chunk(int lane) { return (uint32_t)((lane & 15) ^ ((lane >> 5) << 1)) << 4; }

struct BurstDivisors { Divisor group, n_split, hkv; };

template <int NSEG>
__global__ __launch_bounds__(kBurstMaxTiles * kWave) void attn_burst_mfma_bf16_kernel(const AttnParams p, const BurstDivisors by) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = p.waves;
  const int half = lane >> 5, col = lane & 31;

  // workgroups of one KV group and key split sit on one XCD and share its L2
  const int wg = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int pair = by.group.quotient(wg);
  const int bg = by.n_split.quotient(pair);
  const int split = pair - bg * p.n_split;
  const int b = by.hkv.quotient(bg), g = bg - b * p.hkv;
  const int h = g * p.group + wg - pair * p.group, head = b * p.hq + h;

  const SegPtrs sp = seg_ptrs(p, b, g, NSEG == 2);
  const int ntiles = sp.tiles0 + (sp.n1 + kTileKeys - 1) / kTileKeys;
  const int t_begin = split * p.tiles_per_split;
  const int nt = min(p.tiles_per_split, ntiles - t_begin);   // 1 .. kBurstMaxTiles, at most one per wave
  const bool mine = wave < nt;

  uint8_t* q_lds = smem + p.tiles_per_split * kBurstSlot;
  uint8_t* k_lds = smem + wave * kBurstSlot;                 // this wave's tile
  request_queries<false>(p, b, h, q_lds, wave, nw, lane);
  int rows = 0;
  if (mine) {
    uint32_t stride;
    const TileSrc ts = tile_src(sp, t_begin + wave, stride);
    rows = ts.rows;
    const uint32_t at = lds_address(k_lds), kc = fetch_k_chunk(lane), vc = burst_v_chunk(lane);
    const int r8 = 8 * (lane >> 4);
#pragma unroll
    for (int c = 0; c < 8; ++c)   // rows past the end re-read the last key; masked later
      fetch_to_lds(at + c * kKGroup, ts.k, (uint32_t)min(c + r8, rows - 1) * stride + kc);
#pragma unroll
    for (int c = 0; c < 8; ++c)
      fetch_to_lds(at + kRingK + c * kVGroup, ts.v, (uint32_t)min(c + r8, rows - 1) * stride + vc);
    in_issue_order();
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");        // the query rows
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  bare_barrier();

  f32x16 s;
  float m_row;
  if (mine) {
    bf16x8 qf[8], a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) qf[i] = shared_k_frag(shared_k_at(q_lds, half, col), i);
    in_issue_order();
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");         // K
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = shared_k_frag(shared_k_at(k_lds, half, col), i);
    __builtin_amdgcn_sched_barrier(0);
    tile_logits_mma(a, qf, s);
    const float m_loc = tile_mask_max(s, rows, p.scale_log2, half);
    m_row = fmaxf(kNoMax, fmaxf(m_loc, __shfl_xor(m_loc, 32)));
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // V as well
  bare_barrier();

  // O^T[32 e + 16 j + m, 16 qh + n]: 16x16x32 MFMAs whose k-th eight keys (k = lane / 16) are those of unit (k % 2, k / 2)
  const int e = wave & 3, qh = wave >> 2;
  const int k4 = lane >> 4, s16 = lane & 15, st = k4 & 1, hf = k4 >> 1, row = qh * 16 + s16;
  const size_t slot = (size_t)head * p.n_split + split;
  auto stat = [&](int t, int what, int r) { return *reinterpret_cast<const float*>(smem + t * kBurstSlot + what + r * 4); };
  auto finish = [&](auto tiles) {
    constexpr int NT = decltype(tiles)::value;
    // this wave's V operands come now, under the exponentials
    const uint8_t* v_at = smem + kRingK + (hf * 4 + (s16 >> 2)) * kVGroup + st * 512 + e * 64 + (s16 & 3) * 8;
    i16x8 vf[NT][2];
    if (wave < kBurstOutWaves) {
      typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint8_t* at = v_at + t * kBurstSlot + ((j ^ st) << 5);
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)at);
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(at + 256));
          vf[t][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (mine) {
      bf16x8 pb[2];
      float l = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], p.scale_log2, -m_row));
        l += x;
        pb[i >> 3][i & 7] = (__bf16)x;
      }
      const float l_row = l + __shfl_xor(l, 32);
      // unit (step, half) of a query row: the numerators of keys 16 step + 4 half + {0..3, 8..11}
#pragma unroll
      for (int i = 0; i < 2; ++i) *reinterpret_cast<bf16x8*>(k_lds + kBurstP + i * 1024 + lane * 16) = pb[i];
      if (lane < 32) {
        *reinterpret_cast<float*>(k_lds + kBurstMax + lane * 4) = m_row;
        *reinterpret_cast<float*>(k_lds + kBurstSum + lane * 4) = l_row;
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bare_barrier();
    if (wave >= kBurstOutWaves) return;

    bf16x8 pf[NT];
    float m_t[NT], l_t[NT], m_run = kNoMax, l_tot = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) m_t[t] = stat(t, kBurstMax, row);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      pf[t] = *reinterpret_cast<const bf16x8*>(smem + t * kBurstSlot + kBurstP + st * 1024 + (hf * 32 + row) * 16);
#pragma unroll
    for (int t = 0; t < NT; ++t) l_t[t] = stat(t, kBurstSum, row);
    __builtin_amdgcn_sched_barrier(0);
    // With a reference per tile and row the largest numerators are 1, which bf16 has exactly.  Mean error against 64 bits over 12 sizes 1.92e-3,
    // 2.12e-3 with one reference for the workgroup, 2.06e-3 in the kernels that stream tiles.  32 heads x 21 tiles 8.58 -> 8.33 us without the
    // exchange of maxima, a block of 28 heads x 69 to 76 tiles 312 -> 314.
#pragma unroll
    for (int t = 0; t < NT; ++t) m_run = fmaxf(m_run, m_t[t]);
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float f = __builtin_amdgcn_exp2f(m_t[t] - m_run);
      l_tot = __builtin_fmaf(f, l_t[t], l_tot);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[t][j]), pf[t], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][r] = __builtin_fmaf(f, o[r], acc[j][r]);
      }
    }

    const int d0 = 32 * e + 4 * k4;
    if (p.n_split == 1) {
      char* out_row = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + row * p.o_sr);
      const float inv = 1.f / l_tot;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (__bf16)(acc[j][r] * inv);
        *reinterpret_cast<bf16x4*>(out_row + (d0 + 16 * j) * 2) = o;
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<f32x4*>(p.part_o + (slot * 32 + row) * 128 + d0 + 16 * j) = acc[j];
    if (e == 0) {
      if (lane < 16) {
        p.part_ml[slot * 64 + row] = m_run;
        p.part_ml[slot * 64 + 32 + row] = l_tot;
      }
    }
  };
  switch (nt) {
    case 1: finish(std::integral_constant<int, 1>{}); break;
    case 2: finish(std::integral_constant<int, 2>{}); break;
    case 3: finish(std::integral_constant<int, 3>{}); break;
    case 4: finish(std::integral_constant<int, 4>{}); break;
    case 5: finish(std::integral_constant<int, 5>{}); break;
    case 6: finish(std::integral_constant<int, 6>{}); break;
    case 7: finish(std::integral_constant<int, 7>{}); break;
    case 8: finish(std::integral_constant<int, 8>{}); break;
    default: finish(std::integral_constant<int, kBurstMaxTiles>{}); break;
  }
}

template <int NSEG>
static hipError_t launch_nseg(const AttnParams& p, hipStream_t s) {
  static LdsOptIn lds;
  const auto kernel = attn_burst_mfma_bf16_kernel<NSEG>;
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), burst_lds_bytes(kBurstMaxTiles));
  if (e != hipSuccess) return e;
  const int nwg = p.n_split * p.batch * p.hq;
  if (p.tiles_per_split < 1 || p.tiles_per_split > kBurstMaxTiles || p.waves > kBurstMaxTiles) return hipErrorInvalidValue;
  if (p.waves < kBurstOutWaves || p.waves < p.tiles_per_split) return hipErrorInvalidValue;
  const BurstDivisors by{Divisor(p.group), Divisor(p.n_split), Divisor(p.hkv)};
  return launch(kernel, dim3(nwg), dim3(p.waves * kWave), burst_lds_bytes(p.tiles_per_split), s, p, by);
}

hipError_t launch_attn_burst_mfma_bf16(const AttnParams& p, hipStream_t s) {
  if (p.seg[0].n > 0 && p.seg[1].n > 0) return launch_nseg<2>(p, s);
  if (p.seg[1].n > 0) {   // empty cache: the block is the only key tensor
    AttnParams q = p;
    q.seg[0] = p.seg[1];
    q.seg[1].n = 0;
    return launch_nseg<1>(q, s);
  }
  return launch_nseg<1>(p, s);
}

}  // namespace sdllm
