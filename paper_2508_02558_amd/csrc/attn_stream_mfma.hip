// Block-query attention with tiles fetched straight into LDS (bf16, head_dim 128, 32 query rows): Alg. 3,
// cache_state == 2, and the dense block rows of states 0/1, for grouped-query heads and for small calls.
//
// One workgroup per query head (and key split), each wave streaming its own 32-key tiles, as in
// attn_mfma.hip.  There the heads of a KV group read the same keys side by side, so what a CU fetches comes
// from L2, not from HBM, and the kernel is bound by what happens between the fetch and the matrix cores: a
// tile went to registers, from there to LDS and back, with one tensor tile in flight per wave.  Here the fetch
// writes LDS itself: no staging registers, half the LDS instructions, and K and V of the next tile in flight
// while a tile is computed (K's buffer is refilled as soon as its operands are in registers, V's likewise), so
// a wave waits for a fetch only if it takes longer than the other tensor's products and the softmax.  The
// 16 KB a wave needs for its two tiles let eight waves sit on a CU, which is why the buffers are single.
// What bounds it now: 8 waves x 16 KB per 1.3 us and CU (12.6 KB/us per wave), a chain of LDS reads, eight
// dependent logits products, softmax and eight independent products per tile at two waves per SIMD.
// Measured against the kernels it took over from: 8 x 28/4 heads, 4608 keys, dense rows 39.9 -> 33.9 us (shared-tile
// kernel, key splits and combine launch before), 2336 keys 20.6 -> 19.4 us.  Small calls, where eight or fewer waves
// of one workgroup now do what key splits and a combine launch did: 56/8 heads x 28 tiles 12.9 -> 10.5 us, 32 heads x 14
// tiles 10.4 -> 8.0 us.
#include <type_traits>

#include "attn_tile_math.h"

namespace sdllm {

constexpr int kRawTile = kTileKeys * 256;               // a 32-key tile of one tensor as it lies in LDS
constexpr int kParkBytes = 64 * 256;                    // a wave's accumulators: 64 lanes x 16 slots of 16 bytes
constexpr int kStreamWaveLds = kParkBytes + 512;

// ---- tiles fetched straight into LDS -------------------------------------------------------------
// One load instruction moves 64 lanes x 16 bytes to 1 KB of consecutive LDS (four rows of a tile); which
// 16-byte chunk of its row a lane fetches is free, so the chunks of a row are permuted to keep the operand
// reads off each other's banks: row r holds chunk c of K in place c ^ (r & 15), of V in place
// c ^ ((r & 3) << 2).
template <bool V>
__device__ __forceinline__ void fetch_tile(const char* base, int rows, uint32_t stride, uint8_t* lds_tile, int lane) {
  typedef __attribute__((address_space(1))) const void gvoid;
  typedef __attribute__((address_space(3))) void lvoid;
  const uint32_t r0 = lane >> 4, place = lane & 15;
  auto chunk = [&](int j) { return V ? place ^ (r0 << 2) : place ^ r0 ^ (uint32_t)((j & 3) << 2); };
  if (rows == kTileKeys) {   // wave-uniform
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const char* src = base + (size_t)(j * 4) * stride + (r0 * stride + (chunk(j) << 4));
      __builtin_amdgcn_global_load_lds((gvoid*)src, (lvoid*)(lds_tile + j * 1024), 16, 0, 0);
    }
  } else {                   // rows past the end re-read the last key; masked later
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const char* src = base + ((uint32_t)min(j * 4 + (int)r0, rows - 1) * stride + (chunk(j) << 4));
      __builtin_amdgcn_global_load_lds((gvoid*)src, (lvoid*)(lds_tile + j * 1024), 16, 0, 0);
    }
  }
}

__device__ __forceinline__ void read_k_frags(const uint8_t* tile, int half, int col, bf16x8 (&a)[8]) {
  const uint32_t at = (uint32_t)(col * 256 + ((half ^ (col & 15)) << 4));
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) a[kk] = *reinterpret_cast<const bf16x8*>(tile + (at ^ (uint32_t)(kk * 32)));
}

// The reads and their wait are one block: as builtins the compiler would have them wait for every fetch into
// LDS that is in flight, K's next tile included.
__device__ __forceinline__ void read_v_frags(const uint8_t* tile, int lane, PvFrags& f) {
  const int half = lane >> 5, grp = (lane >> 4) & 1, s16 = lane & 15;
  const uint32_t at = (uint32_t)((half * 4 + (s16 >> 2)) * 256 + ((s16 >> 2) << 6) + grp * 32 + (s16 & 3) * 8);
  typedef __attribute__((address_space(3))) const uint8_t lds_u8;
  const uint32_t base = (uint32_t)(uintptr_t)(lds_u8*)tile;
  const uint32_t a0 = base + at, a1 = base + (at ^ 64u), a2 = base + (at ^ 128u), a3 = base + (at ^ 192u);
  i16x4 r[16];   // [step][e][lo, hi]
  asm volatile(
      "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:2048\n\t"
      "ds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:2048\n\t"
      "ds_read_b64_tr_b16 %4, %18\n\tds_read_b64_tr_b16 %5, %18 offset:2048\n\t"
      "ds_read_b64_tr_b16 %6, %19\n\tds_read_b64_tr_b16 %7, %19 offset:2048\n\t"
      "ds_read_b64_tr_b16 %8, %16 offset:4096\n\tds_read_b64_tr_b16 %9, %16 offset:6144\n\t"
      "ds_read_b64_tr_b16 %10, %17 offset:4096\n\tds_read_b64_tr_b16 %11, %17 offset:6144\n\t"
      "ds_read_b64_tr_b16 %12, %18 offset:4096\n\tds_read_b64_tr_b16 %13, %18 offset:6144\n\t"
      "ds_read_b64_tr_b16 %14, %19 offset:4096\n\tds_read_b64_tr_b16 %15, %19 offset:6144\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
        "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11]), "=&v"(r[12]), "=&v"(r[13]), "=&v"(r[14]), "=&v"(r[15])
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
      : "memory");
#pragma unroll
  for (int i = 0; i < 8; ++i) f.av[i >> 2][i & 3] = __builtin_shufflevector(r[2 * i], r[2 * i + 1], 0, 1, 2, 3, 4, 5, 6, 7);
}

// Likewise; `at` is the lane's place of shared_k_at.
__device__ __forceinline__ void read_q_frags(uint32_t at, bf16x8 (&q)[8]) {
  asm volatile(
      "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:32\n\tds_read_b128 %2, %8 offset:64\n\tds_read_b128 %3, %8 offset:96\n\t"
      "ds_read_b128 %4, %8 offset:128\n\tds_read_b128 %5, %8 offset:160\n\tds_read_b128 %6, %8 offset:192\n\t"
      "ds_read_b128 %7, %8 offset:224\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3]), "=&v"(q[4]), "=&v"(q[5]), "=&v"(q[6]), "=&v"(q[7])
      : "v"(at)
      : "memory");
}

template <int NSEG, bool STATS, bool TOUCH>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_stream_mfma_bf16_kernel(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int half = lane >> 5, col = lane & 31;

  // workgroups of one KV group and key split sit on one XCD and share its L2
  const int wg = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int pair = wg / p.group;
  const int split = pair % p.n_split;
  const int bg = pair / p.n_split;
  const int b = bg / p.hkv, g = bg - b * p.hkv;
  const int h = g * p.group + wg - pair * p.group, head = b * p.hq + h;

  const SegPtrs sp = seg_ptrs(p, b, g, NSEG == 2);
  const int ntiles = sp.tiles0 + (sp.n1 + kTileKeys - 1) / kTileKeys;
  const int t_begin = split * p.tiles_per_split + wave;                   // this wave's tiles: t_begin, t_begin + nw, ...
  const int t_end = min(ntiles, (split + 1) * p.tiles_per_split);
  const int n_mine = max(0, (t_end - t_begin + nw - 1) / nw);

  // Visiting order (STATS; one key segment): tiles [x0, x0 + n_mixed) hold keys that are not candidates
  // and are visited last, positions [n_pure, ntiles) of the order.
  int x0 = 0, n_mixed = 0;
  if (STATS) {
    x0 = p.cand0_end / kTileKeys;
    n_mixed = max(min(ntiles, (p.cand1_begin + kTileKeys - 1) / kTileKeys) - x0, 0);
  }
  const int n_pure = ntiles - n_mixed;
  auto tile_of = [&](int t) { return !STATS || t < x0 ? t : (t < n_pure ? t + n_mixed : x0 + (t - n_pure)); };
  auto pos_of = [&](int j) { return t_begin + j * nw; };                  // j-th tile of this wave, in visiting order

  uint8_t* k_lds = smem + wave * kParkBytes;
  uint8_t* v_lds = k_lds + kRawTile;
  auto fetch_k = [&](int j) {
    uint32_t stride;
    const TileSrc ts = tile_src(sp, tile_of(pos_of(j)), stride);
    fetch_tile<false>(ts.k, ts.rows, stride, k_lds, lane);
  };
  auto fetch_v = [&](int j) {
    uint32_t stride;
    const TileSrc ts = tile_src(sp, tile_of(pos_of(j)), stride);
    fetch_tile<true>(ts.v, ts.rows, stride, v_lds, lane);
  };
  auto rows_of = [&](int j) {
    const int t = tile_of(pos_of(j));
    return t < sp.tiles0 ? min(kTileKeys, sp.n0 - t * kTileKeys) : min(kTileKeys, sp.n1 - (t - sp.tiles0) * kTileKeys);
  };
  // Each of the group's heads brings every group-th tile into L2 four tiles ahead of the others and itself, one request
  // per 128-byte line (its first word, to LDS that nobody reads): the siblings run in step, so without it all of
  // them wait for the same line from memory (8 x 28/4 heads x 4608 keys 42.5 -> 39.0 us with the keys in HBM, 36.0
  // -> 34.3 us with them in the memory-side cache; three or five tiles ahead are the same, seven lose half of it).
  constexpr int kAhead = 4;
  auto touch = [&](int j) {
    typedef __attribute__((address_space(1))) const void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    uint32_t stride;
    const TileSrc ts = tile_src(sp, tile_of(pos_of(j)), stride);
    const uint32_t off = (uint32_t)min(lane >> 1, ts.rows - 1) * stride + ((lane & 1) << 7);
    uint8_t* unread = smem + nw * kParkBytes + wave * 512;   // the statistics' place in the merge
    __builtin_amdgcn_global_load_lds((gvoid*)(ts.k + off), (lvoid*)unread, 4, 0, 0);
    __builtin_amdgcn_global_load_lds((gvoid*)(ts.v + off), (lvoid*)(unread + 256), 4, 0, 0);
  };
  int touch_next = 0;                                        // this head's next tile j: (wave + j) % group == h % group
  if (TOUCH) {
    touch_next = (h + 8 * p.group - wave) % p.group;
    while (touch_next < 2) touch_next += p.group;
  }
  bool touched = false;                                      // two requests more after the last K tile's
  auto touch_up_to = [&](int j) {
    if (!TOUCH) return;
    touched = touch_next <= j && touch_next < n_mine;
    if (touched) { touch(touch_next); touch_next += p.group; }
  };
  // The waits below count requests, so they hang on the order of issue: K(0), V(0), K(1), touch, and from then on for each
  // tile K(j+2), touch, V(j+1), every one of them whole before the next begins.  in_issue_order between
  // them keeps the compiler from interleaving requests whose LDS destinations it can tell apart.
  auto landed = [&](bool all) {   // every fetch of this wave is in LDS, or all but the eight (and the touch) requested last
    if (all) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (TOUCH && touched) asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    wave_lds_sync();
  };

  // The query rows come once per workgroup, through LDS: as fragments straight from memory (32 rows x 32 bytes an
  // instruction, the same for every wave) they kept the CU's address path from the first keys for about 1 us (8 heads x 11
  // tiles 7.25 -> 6.5 us, 84 x 21 9.55 -> 8.45, 224 x 73 18.5 -> 17.2 and, with the keys in HBM, 24.0 -> 22.6).
  uint8_t* q_lds = smem + nw * kStreamWaveLds;
  request_queries<true>(p, b, h, q_lds, wave, nw, lane);
  in_issue_order();
  if (n_mine > 0) {
    fetch_k(0);
    in_issue_order();
    fetch_v(0);
    in_issue_order();
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  bare_barrier();
  bf16x8 qf[8];
  read_q_frags(lds_address(shared_k_at(q_lds, half, col)), qf);

  f32x16 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[e][i] = 0.f;
  float m_run = kNoMax, l_run = 0.f;
  float mc_run = -INFINITY, lc_run = 0.f;   // the same over candidate keys only (STATS)

  bf16x8 a[8], pb[2];
  PvFrags f;
  f32x16 sn;
  auto softmax = [&](int j) {
    if (STATS) {
      const int pos = pos_of(j);
      if (pos >= n_pure) {
        // first tile with other keys: what the attention has accumulated so far covers candidates only
        if (j == 0 || pos - nw < n_pure) { mc_run = m_run; lc_run = l_run; }
        tile_candidate_stats(sn, tile_of(pos) * kTileKeys + half * 4, p, mc_run, lc_run);
      }
    }
    softmax_block(sn, rows_of(j), p.scale_log2, half, m_run, l_run, acc, pb);
  };
  // logits of tile j from LDS; K's buffer is free again once the operands are in registers
  auto logits = [&](int j) {
    read_k_frags(k_lds, half, col, a);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (j + 1 < n_mine) fetch_k(j + 1);
    in_issue_order();
    touch_up_to(j + kAhead);
    in_issue_order();
    tile_logits_mma(a, qf, sn);
    __builtin_amdgcn_sched_barrier(0);
  };

  if (n_mine > 0) {
    landed(false);                          // K(0)
    logits(0);
    softmax(0);
    for (int j = 0; j + 1 < n_mine; ++j) {
      // K(j+1); V(j) may still fly, except that V(0) was requested before K(1)
      if (TOUCH && j == 0 && touched) { asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); wave_lds_sync(); }
      else landed(j == 0);
      logits(j + 1);
      landed(j + 2 >= n_mine);              // V(j); K(j+2), if there is one, may still fly
      read_v_frags(v_lds, lane, f);
      fetch_v(j + 1);
      in_issue_order();
      pv_block(f, pb, acc);
      __builtin_amdgcn_sched_barrier(0);
      softmax(j + 1);
    }
    landed(true);
    read_v_frags(v_lds, lane, f);
    pv_block(f, pb, acc);
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (STATS && (n_mine == 0 || pos_of(n_mine - 1) < n_pure)) { mc_run = m_run; lc_run = l_run; }   // candidates only
  const float lc_tot = lc_run + __shfl_xor(lc_run, 32);
  const size_t out_slot = (size_t)head * p.n_split + split;
  char* out_row = (char*)p.out + 2 * (b * p.o_sb + h * p.o_sh + col * p.o_sr);

  if (nw == 1) {   // this wave owns the whole result
    if (STATS && lane < 32) {
      p.cand_ml[out_slot * 64 + lane] = mc_run;
      p.cand_ml[out_slot * 64 + 32 + lane] = lc_tot;
    }
    write_wave_result(acc, m_run, l_tot, lane, half, p.n_split == 1, out_row, p.part_o + (out_slot * 32 + col) * 128,
                      p.part_ml + out_slot * 64);
    return;
  }

  // Merge of the waves: every wave parks its accumulators (slot i of lane l in place i ^ (l & 15)) and its rows'
  // statistics; the waves then share out the 16 slots.
  uint8_t* mine = smem + wave * kParkBytes;
  auto stat_of = [&](int w) { return reinterpret_cast<float*>(smem + nw * kParkBytes + w * 512); };
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = {acc[e][i4 * 4], acc[e][i4 * 4 + 1], acc[e][i4 * 4 + 2], acc[e][i4 * 4 + 3]};
      *reinterpret_cast<f32x4*>(mine + lane * 256 + (((e * 4 + i4) ^ (lane & 15)) << 4)) = v;
    }
  if (lane < 32) {
    float* ml = stat_of(wave);
    ml[lane] = m_run; ml[32 + lane] = l_tot;
    if (STATS) { ml[64 + lane] = mc_run; ml[96 + lane] = lc_tot; }
  }
  __syncthreads();
  if (STATS && wave == 0 && lane < 32) {
    float mc = -INFINITY, lc = 0.f;
    for (int s = 0; s < nw; ++s) mc = fmaxf(mc, stat_of(s)[64 + lane]);
    for (int s = 0; s < nw; ++s) {
      const float* ml = stat_of(s);
      if (ml[64 + lane] != -INFINITY) lc += ml[96 + lane] * __builtin_amdgcn_exp2f(ml[64 + lane] - mc);
    }
    p.cand_ml[out_slot * 64 + lane] = mc;
    p.cand_ml[out_slot * 64 + 32 + lane] = lc;
  }
  auto merge = [&](auto nw_tag) {
    constexpr int KS = decltype(nw_tag)::value;
    constexpr int NJ = (16 + KS - 1) / KS;
    float m_s[KS], l_s[KS], f_s[KS];
    f32x4 part[NJ][KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const float* ml = stat_of(s);
      m_s[s] = ml[col];
      l_s[s] = ml[32 + col];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int i = min(wave + j * KS, 15);   // past the last: re-read, not stored
#pragma unroll
      for (int s = 0; s < KS; ++s)
        part[j][s] = *reinterpret_cast<const f32x4*>(smem + s * kParkBytes + lane * 256 + ((i ^ (lane & 15)) << 4));
    }
    __builtin_amdgcn_sched_barrier(0);
    float m_tot = -INFINITY, l_all = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) m_tot = fmaxf(m_tot, m_s[s]);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      f_s[s] = __builtin_amdgcn_exp2f(m_s[s] - m_tot);   // a wave that saw no tile: 0
      l_all += f_s[s] * l_s[s];
    }
    const float inv = 1.f / l_all;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int i = wave + j * KS;
      if (i < 16) {
        f32x4 o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) o4 += part[j][s] * f_s[s];
        const int d0 = out_col0(i >> 2, i & 3, half);
        if (p.n_split == 1) {
          bf16x4 ob;
#pragma unroll
          for (int r = 0; r < 4; ++r) ob[r] = (__bf16)(o4[r] * inv);
          *reinterpret_cast<bf16x4*>(out_row + d0 * 2) = ob;
        } else {
          *reinterpret_cast<f32x4*>(p.part_o + (out_slot * 32 + col) * 128 + d0) = o4;
        }
      }
    }
    if (p.n_split > 1 && wave == 0 && lane < 32) {
      p.part_ml[out_slot * 64 + lane] = m_tot;
      p.part_ml[out_slot * 64 + 32 + lane] = l_all;
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
}

template <int NSEG, bool STATS, bool TOUCH>
static hipError_t launch_touch(const AttnParams& p, hipStream_t s) {
  static LdsOptIn lds;
  const auto kernel = attn_stream_mfma_bf16_kernel<NSEG, STATS, TOUCH>;
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), kMaxWavesPerWg * kStreamWaveLds + kRingK);
  if (e != hipSuccess) return e;
  if (p.waves < 1 || p.waves > kMaxWavesPerWg) return hipErrorInvalidValue;
  return launch(kernel, dim3(p.n_split * p.batch * p.hq), dim3(p.waves * kWave), p.waves * kStreamWaveLds + kRingK, s, p);
}

template <int NSEG, bool STATS>
static hipError_t launch_variant(const AttnParams& p, hipStream_t s) {
  return stream_touches_ahead(p.group, p.tiles_per_split, p.waves) ? launch_touch<NSEG, STATS, true>(p, s) : launch_touch<NSEG, STATS, false>(p, s);
}

hipError_t launch_attn_stream_mfma_bf16(const AttnParams& p, hipStream_t s) {
  if (p.seg[0].n > 0 && p.seg[1].n > 0) return launch_variant<2, false>(p, s);
  if (p.seg[1].n > 0) {   // empty cache: the block is the only key tensor
    AttnParams q = p;
    q.seg[0] = p.seg[1];
    q.seg[1].n = 0;
    return launch_variant<1, false>(q, s);
  }
  return p.cand_ml ? launch_variant<1, true>(p, s) : launch_variant<1, false>(p, s);
}

}  // namespace sdllm
