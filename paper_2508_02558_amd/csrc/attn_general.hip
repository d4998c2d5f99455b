// Attention for every shape that the 32-row, head_dim 128 bf16 kernels do not take: fp32 tensors, head_dim
// 64, block lengths other than 32, rows too far apart for 32-bit offsets, and all rows of a sequence in
// those types (Alg. 3 over one or two key segments, as in attn_mfma.hip).
//
// A workgroup owns a block of consecutive query rows of one head (32 with bf16, 16 with fp32 tensors; rows
// past the last compute on a copy of it and are not stored) and a range of 32-key tiles; its waves take the
// tiles in turn, each with a wave-private LDS tile and no barrier in the loop, and merge through LDS at the
// end.  K and V of the next tile are requested together before a tile is computed: these calls are mostly
// small, so what bounds them is the number of memory round trips in a row, not bytes.  Few rows: the keys are
// split over workgroups as well (fp32 partials, combine launch).  The blocks of a longer head read the same
// keys from L2.
// Measured, against one wave per query row with its dot products on the vector ALU and each lane reading
// whole key rows: dense rows of a 64-token block (batch 2, 32 heads of 128, 1280 keys, bf16) with row
// statistics 417 + 299 -> 18 us.  All 1092 rows of 2 x 8 heads: head_dim 64
// bf16 23.5 us (208 TFLOP/s), head_dim 128 fp32 155 us (63 TFLOP/s; 197 us with 32-row blocks, one wave per SIMD).
// fp32 at head_dim 128 fills its 256 registers: the variant that also leaves statistics spills 12 bytes per lane.
#include "attn_merge.h"
#include "general_tile.h"

namespace sdllm {

// What a launch leaves behind.
enum { kOut = 0, kOutAndStats = 1, kStatsOnly = 2 };   // attention output; the candidates' softmax (max, sum) per row

template <typename T, int D>
constexpr int g_wave_lds() {
  using O = Ops<T, D>;
  const int tiles = O::kKTile + O::kVTile, parked = kWave * (O::NACC * 4 + 16);
  return (tiles > parked ? tiles : parked) + 512;
}

// What a workgroup finds its place with.  The fp32 kernels multiply, which makes calls of 5 to 14 us 1 to 4 % shorter.  The bf16 ones
// divide as the compiler does: with multiplications 64 heads x 2 row blocks x 19 tiles gained 2 % (13.85 -> 13.6 us), 16 x 2 x 9 and
// 16 x 2 x 23 lost 3 % (8.05 -> 8.35, 11.2 -> 11.55), by the order in which the first requests then come; the arguments alone cost
// 0.06 us there.
template <typename T>
struct RowBlocks { int n; };
template <>
struct RowBlocks<float> { int n; Divisor by[4]; };   // per_key, n_split, hkv, n

template <typename T, int D, int MODE>
__global__ __launch_bounds__(kGeneralMaxWaves * kWave) void attn_general_kernel(const AttnParams p, const RowBlocks<T> blocks) {
  using O = Ops<T, D>;
  constexpr int R = O::kRows, NS = O::NS, kWaveBytes = g_wave_lds<T, D>(), kPark = O::NACC * 4 + 16, kUnits = O::NACC / 4;
  constexpr float kSlack = 8.f;   // as in attn_tile_math.h: the softmax reference moves when a maximum exceeds it by more
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int part = lane / R, col = lane % R;

  // workgroups that read the same keys (the query heads of a KV group, their row blocks) sit on one XCD
  const int wg = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int rblocks = blocks.n, per_key = p.group * rblocks;
  auto quotient = [&](int n, int d, int i) {
    if constexpr (sizeof(T) == 4) return blocks.by[i].quotient(n);
    else return n / d;
  };
  const int pair = quotient(wg, per_key, 0);
  const int bg = quotient(pair, p.n_split, 1), split = pair - bg * p.n_split;
  const int b = quotient(bg, p.hkv, 2), g = bg - b * p.hkv;
  const int vhead = bg * per_key + wg - pair * per_key;   // (batch, query head, block of R rows)
  const int head = quotient(vhead, rblocks, 3), h = head - b * p.hq;
  const int row = (vhead - head * rblocks) * R + col;
  const bool row_valid = row < p.nq;

  const KvSegment s0 = p.seg[0], s1 = p.seg[1];
  const int tiles0 = (s0.n + kTileKeys - 1) / kTileKeys, ntiles = tiles0 + (s1.n + kTileKeys - 1) / kTileKeys;
  const int t_begin = split * p.tiles_per_split, t_end = min(ntiles, t_begin + p.tiles_per_split);
  const int64_t at0 = (b * s0.sb + g * s0.sh) * (int64_t)sizeof(T), at1 = (b * s1.sb + g * s1.sh) * (int64_t)sizeof(T);

  u32x4 kreg[O::kLoads];
  typename O::V vreg;
  int rows = 0, rows_next = 0;
  const char* v_at = nullptr;
  int64_t stride = 0;
  auto locate = [&](int t, const char*& k_at) {      // all wave-uniform
    const int seg = t < tiles0 ? 0 : 1;
    const int first = (t - (seg ? tiles0 : 0)) * kTileKeys;
    stride = (seg ? s1.sr : s0.sr) * (int64_t)sizeof(T);
    const int64_t at = (seg ? at1 : at0) + first * stride;
    k_at = (const char*)(seg ? s1.k : s0.k) + at;
    v_at = (const char*)(seg ? s1.v : s0.v) + at;
    rows_next = min(kTileKeys, (seg ? s1.n : s0.n) - first);
  };
  int t = t_begin + wave;
  if (t < t_end) {
    const char* k_at;
    locate(t, k_at);
    g_load_rows<O, false>(k_at, rows_next, stride, lane, kreg);
    if (MODE != kStatsOnly) g_v_load<D>(v_at, rows_next, stride, lane, vreg);
  }
  typename O::Frag qf[O::NP];
  g_row_pieces<O>((const T*)p.q + b * p.q_sb + h * p.q_sh + (int64_t)min(row, p.nq - 1) * p.q_sr, part, qf);

  uint8_t* lds_k = smem + wave * kWaveBytes;
  uint8_t* lds_v = lds_k + O::kKTile;
  typename O::Acc acc[O::NE];
  constexpr int kAccRegs = O::NACC / O::NE;
#pragma unroll
  for (int e = 0; e < O::NE; ++e)
#pragma unroll
    for (int i = 0; i < kAccRegs; ++i) acc[e][i] = 0.f;
  float m_run = kNoMax, l_run = 0.f;      // softmax reference of the row; sum over the keys this lane has seen
  float mc_run = -INFINITY, lc_run = 0.f;    // over candidate keys only

  for (; t < t_end; t += nw) {
    rows = rows_next;
    const bool more = t + nw < t_end;
    g_store_rows<O>(lds_k, O::kKRow, lane, kreg);
    if (MODE != kStatsOnly) g_v_publish<D>(lds_v, lane, vreg);
    wave_lds_sync();
    if (more) {
      const char* k_at;
      locate(t + nw, k_at);
      g_load_rows<O, false>(k_at, rows_next, stride, lane, kreg);
      if (MODE != kStatsOnly && O::kVTile > 0) g_v_load<D>(v_at, rows_next, stride, lane, vreg);
    }
    float s[NS];
    O::logits(lds_k, qf, col, part, s);
    if (rows < kTileKeys) {   // only the last tile of a segment is ragged
#pragma unroll
      for (int i = 0; i < NS; ++i) s[i] = O::key(i, part) < rows ? s[i] : -INFINITY;
    }
    if (MODE != kOut) {   // one key segment: register i is position 32 t + key
      float sc[NS], mc_loc = -INFINITY;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int pos = t * kTileKeys + O::key(i, part);
        sc[i] = pos < p.cand0_end || pos >= p.cand1_begin ? s[i] * p.scale_log2 : -INFINITY;
        mc_loc = fmaxf(mc_loc, sc[i]);
      }
      const float mc_new = fmaxf(mc_run, parts_max<O>(mc_loc));
      if (mc_new != -INFINITY) {
        float lc_loc = 0.f;
#pragma unroll
        for (int i = 0; i < NS; ++i) lc_loc += __builtin_amdgcn_exp2f(sc[i] - mc_new);
        lc_run = lc_run * __builtin_amdgcn_exp2f(mc_run - mc_new) + lc_loc;
        mc_run = mc_new;
      }
    }
    if (MODE != kStatsOnly) {
      float m_loc = s[0];
#pragma unroll
      for (int i = 1; i < NS; ++i) m_loc = fmaxf(m_loc, s[i]);
      m_loc *= p.scale_log2;
      if (__ballot(m_loc > m_run + kSlack) != 0) {   // always taken on a wave's first tile
        const float m_new = fmaxf(m_run, parts_max<O>(m_loc));
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int e = 0; e < O::NE; ++e)
#pragma unroll
          for (int i = 0; i < kAccRegs; ++i) acc[e][i] *= alpha;
      }
      float l_loc = 0.f;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        s[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], p.scale_log2, -m_run));
        l_loc += s[i];
      }
      l_run += l_loc;
      g_pv<D>(lds_v, vreg, s, lane, acc);
      if (O::kVTile == 0 && more) g_v_load<D>(v_at, rows_next, stride, lane, vreg);   // fp32: flies under the next tile's logits
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  const float l_tot = parts_sum<O>(l_run), lc_tot = parts_sum<O>(lc_run);
  const size_t slot = (size_t)vhead * p.n_split + split;

  // merge of the waves: each parks its results ([lane][unit of four columns]) and its rows' statistics
  uint8_t* mine = smem + wave * kWaveBytes;
  float* my_ml = reinterpret_cast<float*>(mine + kWave * kPark);
  if (MODE != kStatsOnly) {
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < O::NE; ++e)
#pragma unroll
        for (int i = 0; i < kAccRegs; ++i)
          if (O::flat(e, i) >> 2 == u) v[O::flat(e, i) & 3] = acc[e][i];
      *reinterpret_cast<f32x4*>(mine + lane * kPark + u * 16) = v;
    }
  }
  if (lane < R) {
    my_ml[lane] = m_run; my_ml[32 + lane] = l_tot;
    if (MODE != kOut) { my_ml[64 + lane] = mc_run; my_ml[96 + lane] = lc_tot; }
  }
  __syncthreads();
  auto stat_of = [&](int w) { return reinterpret_cast<const float*>(smem + w * kWaveBytes + kWave * kPark); };
  if (MODE != kOut && wave == 0 && lane < R) {
    float mc = -INFINITY, lc = 0.f;
    for (int w = 0; w < nw; ++w) mc = fmaxf(mc, stat_of(w)[64 + lane]);
    for (int w = 0; w < nw; ++w)
      if (stat_of(w)[64 + lane] != -INFINITY) lc += stat_of(w)[96 + lane] * __builtin_amdgcn_exp2f(stat_of(w)[64 + lane] - mc);
    p.cand_ml[slot * 2 * R + lane] = mc;
    p.cand_ml[slot * 2 * R + R + lane] = lc;
  }
  if (MODE == kStatsOnly) return;
  // a wave that saw no tile parked (kNoMax, 0, 0), one that is not there counts for nothing
  float f_w[kGeneralMaxWaves], l_w[kGeneralMaxWaves], m_tot = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int w = 0; w < kGeneralMaxWaves; ++w) {
    const float* st = stat_of(min(w, nw - 1));
    f_w[w] = w < nw ? st[col] : -INFINITY;
    l_w[w] = st[32 + col];
    m_tot = fmaxf(m_tot, f_w[w]);
  }
#pragma unroll
  for (int w = 0; w < kGeneralMaxWaves; ++w) {
    f_w[w] = f_w[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(f_w[w] - m_tot);
    l_all += f_w[w] * l_w[w];
  }
  const float inv = 1.f / l_all;
  for (int u = wave; u < kUnits; u += nw) {
    f32x4 o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kGeneralMaxWaves; ++w)
      if (w < nw) o4 += *reinterpret_cast<const f32x4*>(smem + w * kWaveBytes + lane * kPark + u * 16) * f_w[w];
    const int d0 = O::unit_col(u, part);
    if (p.n_split > 1) {
      *reinterpret_cast<f32x4*>(p.part_o + (slot * R + col) * D + d0) = o4;
    } else if (row_valid) {
      T* out = (T*)p.out + b * p.o_sb + h * p.o_sh + (int64_t)row * p.o_sr + d0;
      if constexpr (sizeof(T) == 2) {
        bf16x4 ob;
#pragma unroll
        for (int r = 0; r < 4; ++r) ob[r] = (__bf16)(o4[r] * inv);
        *reinterpret_cast<bf16x4*>(out) = ob;
      } else {
        *reinterpret_cast<f32x4*>(out) = o4 * inv;
      }
    }
  }
  if (p.n_split > 1 && wave == 0 && lane < R) {
    p.part_ml[slot * 2 * R + lane] = m_tot;
    p.part_ml[slot * 2 * R + R + lane] = l_all;
  }
}

// The split-KV merge as a launch of its own (combine_block in attn_merge.h does the work).
template <typename T, int TPI>
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(const AttnParams p) {
  combine_block<T, TPI>(p, blockIdx.x);
}

template <int MAX>
__global__ __launch_bounds__(kCombineThreads) void attn_combine32_kernel(const AttnParams p) {
  combine32_block<MAX>(p, blockIdx.y, blockIdx.x >> 2, blockIdx.x & 3);
}

template <typename T, int D, int MODE>
static hipError_t launch_mode(const AttnParams& p, hipStream_t s) {
  static LdsOptIn lds;
  constexpr int kWaveBytes = g_wave_lds<T, D>();
  const auto kernel = attn_general_kernel<T, D, MODE>;
  const hipError_t e = lds.ensure(reinterpret_cast<const void*>(kernel), kGeneralMaxWaves * kWaveBytes);
  if (e != hipSuccess) return e;
  const int rblocks = (p.nq + Ops<T, D>::kRows - 1) / Ops<T, D>::kRows;
  const int64_t nwg = (int64_t)p.batch * p.hq * rblocks * p.n_split;
  if (nwg > INT32_MAX || p.waves < 1 || p.waves > kGeneralMaxWaves) return hipErrorInvalidValue;
  RowBlocks<T> blocks{rblocks};
  if constexpr (sizeof(T) == 4) {
    const int by[4] = {p.group * rblocks, p.n_split, p.hkv, rblocks};
    for (int i = 0; i < 4; ++i) blocks.by[i] = Divisor(by[i]);
  }
  return launch(kernel, dim3((unsigned)nwg), dim3(p.waves * kWave), p.waves * kWaveBytes, s, p, blocks);
}

template <typename T, int D>
static hipError_t launch_t(const AttnParams& p, bool stats_only, hipStream_t s) {
  if (stats_only) return launch_mode<T, D, kStatsOnly>(p, s);
  return p.cand_ml ? launch_mode<T, D, kOutAndStats>(p, s) : launch_mode<T, D, kOut>(p, s);
}

hipError_t launch_attn_general(const AttnParams& p, int dtype, bool stats_only, hipStream_t s) {
  if (dtype == 0) return p.d == 128 ? launch_t<__bf16, 128>(p, stats_only, s) : launch_t<__bf16, 64>(p, stats_only, s);
  return p.d == 128 ? launch_t<float, 128>(p, stats_only, s) : launch_t<float, 64>(p, stats_only, s);
}

hipError_t launch_attn_combine(const AttnParams& p, int dtype, hipStream_t s) {
  return with_combine32(p, p.batch <= 65535 ? dtype : -1, [&](auto max) {
    constexpr int MAX = decltype(max)::value;
    if constexpr (MAX > 0) {
      return launch(attn_combine32_kernel<MAX>, dim3((unsigned)(4 * p.hq), (unsigned)p.batch), dim3(kCombineThreads), 0, s, p);
    } else {
      const bool four = combine_tpi(p.n_split) == 4;
      if (dtype != 0 && four) return hipErrorInvalidValue;   // fp32 has plan_general's splits, eight at most
      const auto kernel = dtype != 0 ? attn_combine_kernel<float, 1> : four ? attn_combine_kernel<__bf16, 4> : attn_combine_kernel<__bf16, 1>;
      return launch(kernel, dim3((unsigned)combine_blocks(p)), dim3(kCombineThreads), 0, s, p);
    }
  });
}

}  // namespace sdllm
