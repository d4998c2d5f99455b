// C-ABI entry points: argument validation, launch planning and dispatch.  No arithmetic of the
// method lives here except the retained-count rule and the cache-state schedule, which are host
// logic by nature (Alg. 1 step 9; Alg. 2 / Alg. 5).
#include <math.h>
#include <stdlib.h>

#include <algorithm>

#include "sdllm.h"
#include "sdllm_bench.h"
#include "sdllm_internal.h"

using namespace sdllm;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline int elem_size(int dtype) { return dtype == SDLLM_BF16 ? 2 : 4; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int32_t quota(int32_t n, double r, int32_t rounding) {
  const double x = r * (double)n;
  const double k = rounding == SDLLM_CEIL ? ceil(x - 1e-9) : floor(x + 1e-9);
  if (k < 0) return 0;
  if (k > n) return n;
  return (int32_t)k;
}

struct Counts { int32_t n_pre, n_suf, n_cand, k_total, k_pre, k_suf; };

Counts counts_of(const sdllm_shape_t& s) {
  Counts c;
  c.n_pre = s.block_off;
  c.n_suf = s.seq_len - s.block_off - s.block_len;
  c.n_cand = c.n_pre + c.n_suf;
  if (s.evict_scope == SDLLM_EVICT_PREFIX_ONLY) {
    c.k_pre = quota(c.n_pre, s.retention, s.k_rounding);
    c.k_suf = c.n_suf;
    c.k_total = c.k_pre + c.k_suf;
  } else if (s.select_mode == SDLLM_PER_SEGMENT) {
    c.k_pre = quota(c.n_pre, s.retention, s.k_rounding);
    c.k_suf = quota(c.n_suf, s.retention, s.k_rounding);
    c.k_total = c.k_pre + c.k_suf;
  } else {
    c.k_total = quota(c.n_cand, s.retention, s.k_rounding);
    c.k_pre = c.k_suf = -1;
  }
  return c;
}

bool strides_ok(const int64_t* st, int esize) {
  for (int i = 0; i < 3; ++i)
    if (st[i] < 0 || (st[i] * esize) % 16 != 0) return false;
  return true;
}

int32_t check_shape(const sdllm_shape_t* s) {
  if (!s) return SDLLM_ERR_INVALID_ARG;
  if (s->batch < 1 || s->n_kv_heads < 1 || s->n_q_heads < 1 || s->n_q_heads % s->n_kv_heads != 0)
    return SDLLM_ERR_INVALID_ARG;
  if (s->dtype != SDLLM_BF16 && s->dtype != SDLLM_F32) return SDLLM_ERR_INVALID_ARG;
  if (s->block_len < 1 || s->block_off < 0 || s->seq_len < 1 ||
      (int64_t)s->block_off + s->block_len > s->seq_len)
    return SDLLM_ERR_INVALID_ARG;
  if (!(s->retention >= 0.0 && s->retention <= 1.0)) return SDLLM_ERR_INVALID_ARG;
  if (s->pool_kernel < 1 || s->pool_kernel % 2 == 0) return SDLLM_ERR_INVALID_ARG;
  if (s->score_mode != SDLLM_SOFTMAX_MEAN && s->score_mode != SDLLM_LOGIT_MEAN) return SDLLM_ERR_INVALID_ARG;
  if (s->select_mode != SDLLM_PER_SEGMENT && s->select_mode != SDLLM_JOINT) return SDLLM_ERR_INVALID_ARG;
  if (s->k_rounding != SDLLM_CEIL && s->k_rounding != SDLLM_FLOOR) return SDLLM_ERR_INVALID_ARG;
  if (s->pool_mode != SDLLM_MAX_POOL && s->pool_mode != SDLLM_AVG_POOL) return SDLLM_ERR_INVALID_ARG;
  if (s->evict_scope != SDLLM_EVICT_BIDIRECTIONAL && s->evict_scope != SDLLM_EVICT_PREFIX_ONLY)
    return SDLLM_ERR_INVALID_ARG;
  if (!(s->softmax_scale >= 0.f) || !isfinite(s->softmax_scale) || s->reserved != 0) return SDLLM_ERR_INVALID_ARG;
  const int es = elem_size(s->dtype);
  if (!strides_ok(s->q_stride, es) || !strides_ok(s->kv_stride, es) || !strides_ok(s->blk_stride, es) ||
      !strides_ok(s->cache_stride, es) || !strides_ok(s->out_stride, es))
    return SDLLM_ERR_INVALID_ARG;
  if (s->head_dim != 64 && s->head_dim != 128) return SDLLM_ERR_UNSUPPORTED;
  if (s->block_len > 64) return SDLLM_ERR_UNSUPPORTED;
  return SDLLM_OK;
}

bool row_stride_ok(const int64_t* st, int d) { return st[2] >= d; }

float scale_of(const sdllm_shape_t& s) {
  return s.softmax_scale > 0.f ? s.softmax_scale : 1.0f / sqrtf((float)s.head_dim);
}

constexpr float kLog2e = 1.4426950408889634f;

// ---------------------------------------------------------------- attention planning
struct AttnPlan {
  bool mfma;  // one of the kernels for bf16, head_dim 128, 32 query rows; otherwise the general one
  bool gqa;   // grouped-query kernel: one workgroup per (batch, KV head), wave = query head
  bool stream;   // one workgroup per head with tiles fetched straight into LDS
  bool burst;    // at most nine tiles per workgroup, all of them fetched at once
  int n_split, tiles_per_split, waves;
  size_t part_o_bytes, part_ml_bytes;
  size_t ws_bytes() const { return part_o_bytes + part_ml_bytes; }
};

bool seg_fits_u32(int64_t row_stride, int32_t n, int esize) {
  return n <= 0 || ((int64_t)(n - 1) * row_stride + 128) * esize < (int64_t)1 << 31;
}

// Whether sdllm_dense_attn runs the bf16 kernel for whole sequences; otherwise the general one.
bool dense_full_takes(const sdllm_shape_t& s) {
  return s.dtype == SDLLM_BF16 && s.head_dim == 128 && seg_fits_u32(s.kv_stride[2], s.seq_len, 2);
}

// Whether an attention call of the block's rows runs one of the kernels for bf16, head_dim 128, 32 rows.
bool takes_mfma(const sdllm_shape_t& s, int32_t n0, int64_t sr0, int32_t n1, int64_t sr1) {
  return s.dtype == SDLLM_BF16 && s.head_dim == 128 && s.block_len == 32 && seg_fits_u32(sr0, n0, 2) && seg_fits_u32(sr1, n1, 2);
}

int row_blocks(const sdllm_shape_t& s, int32_t rows) { return (rows + block_rows(s.dtype) - 1) / block_rows(s.dtype); }

// The general kernel: one workgroup per (head, block of query rows) and key split.
void plan_general(AttnPlan& pl, const sdllm_shape_t& s, int32_t nq, int tiles, bool may_split) {
  const int64_t vheads = (int64_t)s.batch * s.n_q_heads * row_blocks(s, nq);
  const int most_waves = kGeneralMaxWaves;
  // Tiles from which splitting a head's keys repays the second launch, and the fewest a split is left with.  Sparse steps,
  // split against unsplit: bf16, head_dim 128, 8 or 28 row blocks x 14 tiles 10.4 / 9.2 us, x 24 10.4 / 11.2; 64 x 24
  // 12.0 / 11.5, x 36 12.2 / 14.3; 128 x 36 16.7 / 17.1 (two blocks of a head) and 19.5 / 17.4 (one); head_dim 64,
  // whose tiles are half as long, 8 or 28 x 24 9.7 / 8.3, x 48 9.7 / 11.8, 128 x 48 15.0 / 13.6, x 75 19.0 / 18.8.  fp32, where
  // a tile is 0.5 or 1 us of a SIMD's matrix work, head_dim 64, 16 x 14 10.2 / 10.2, x 24 10.6 / 13.4; head_dim 128,
  // 16 x 14 13.1 / 16.3.
  const bool f32 = s.dtype == SDLLM_F32, d64 = s.head_dim == 64;
  const int from = f32 ? (d64 ? 16 : 12) : d64 ? (vheads <= 64 ? 36 : 76) : vheads <= 32 ? 20 : vheads <= 64 ? 28 : 40;
  const int least = f32 ? (d64 ? 8 : 4) : vheads <= 32 ? 7 : 11;
  int n_split = 1;
  if (may_split && vheads <= kNumCUs / 2 && tiles >= from) {
    // within one workgroup per CU, which also keeps the partials of every plan below SDLLM_STATIC_SCRATCH_BYTES
    // (256 x 16.25 KB)
    n_split = (int)(kNumCUs / vheads);
    if (n_split > 8) n_split = 8;
    if (n_split > tiles / least) n_split = tiles / least;
    if (n_split < 1) n_split = 1;
  }
  pl.tiles_per_split = (tiles + n_split - 1) / n_split;
  pl.n_split = pl.tiles_per_split > 0 ? (tiles + pl.tiles_per_split - 1) / pl.tiles_per_split : 1;
  // Waves per workgroup: a CU holds `cu_waves` of them (registers), as one workgroup or several, so `w` waves take
  // ceil(workgroups / (CUs x cu_waves / w)) rounds of ceil(tiles / w) tiles each; the fewest win (560 workgroups x 35
  // tiles of head_dim 64, bf16, all rows of a sequence: 28 us with two waves, 23 us with four), the smaller merge
  // among equals.
  const int cu_waves = s.head_dim == 64 ? 12 : 8;
  int64_t fewest = INT64_MAX;
  for (int w = 2; w <= most_waves; w *= 2) {
    const int64_t slots = (int64_t)kNumCUs * (cu_waves / w);
    const int64_t cost = ((vheads * pl.n_split + slots - 1) / slots) * ((pl.tiles_per_split + w - 1) / w);
    if (cost < fewest) { fewest = cost; pl.waves = w; }
  }
  if (pl.waves > pl.tiles_per_split) pl.waves = pl.tiles_per_split;
  if (pl.waves < 1) pl.waves = 1;
  while (pl.waves > 1 && vheads * pl.n_split * pl.waves * kWave > UINT32_MAX) pl.waves /= 2;   // threads of one launch
  if (pl.n_split > 1) {
    pl.part_o_bytes = align_up((size_t)vheads * pl.n_split * block_rows(s.dtype) * s.head_dim * sizeof(float));
    pl.part_ml_bytes = align_up((size_t)vheads * pl.n_split * 2 * block_rows(s.dtype) * sizeof(float));
  }
}

// Key splits of the shared-tile kernel: as many as keep the grid within what the CUs hold at once (a few workgroups more
// would wait for a whole round), but never fewer than 4 tiles (two LDS stages) each.  Four-wave workgroups: two per CU.
// Two-wave workgroups: four fit, three per CU measured best (G = 4, 768 heads: 79.6 -> 63.9 us with 2 splits; G = 2, 1024
// heads: 90 us with 1 split, 108 with 2).
int shared_splits(int rows, int group, int tiles) {
  const int wg_waves = attn_gqa_waves_per_wg(group);
  int n = (wg_waves >= 4 ? 2 : 3) * kNumCUs / (rows * ((group + wg_waves - 1) / wg_waves));   // workgroups per KV head and split
  if (n > tiles / 4) n = tiles / 4;
  return n < 1 ? 1 : n;
}

// Whether the shared-tile kernel (K/V read once per group, one wave per head, key splits merged through fp32 partials and a
// second launch) beats one workgroup per query head and key split (n_split of them, as without it).
//
// Two waves per workgroup (G = 2, 4), measured for sparse and dense steps: 256 heads lose (G = 4: 28/51 us per head
// against 34/50 us shared), 384 heads win (G = 4: 46/82 against 42/68 us; G = 2: 54/97 against 50/80 us), 512 heads tie,
// 640 win.
//
// Four waves (G = 7, 8; sparse steps and dense rows alike, keys from HBM).  It starts 12 us behind (splits, partials, merge)
// and then takes less per tile, the less of the chip the other kernels fill the more:
// * up to one workgroup of theirs per CU, from 60 tiles each plus 0.4 per workgroup on: 140 heads from 118 tiles (130: 31.4
//   against 34.9 us), 168 from 125, 192 from 136 (150: 37.1 against 38.6), 224 from 155, 256 from 165 (150: 43.2 against
//   41.7, 200: 51.9 against 53.4); with key splits, tiles of one split: 96 heads x 2 from 140, 84 x 3 from 160 (600 tiles in all
//   57.2 against 58.7), 64 x 4 from 165, 16 x 8 from 112;
// * up to two per CU (four waves each): 272 heads from 68 tiles (84: 34.7 against 38.5), 320 from 62, 392 from 70, 448 from
//   76, 512 from 84;
// * up to four per CU (two waves each): from 40 tiles if its own waves take more than three quarters of the chip's 2048
//   (532 heads x 3 splits: 46 tiles 37.0 against 38.9 us; 640 x 3: 42 tiles 36.3 against 38.3; 896 x 2: 46 tiles 47.4 against
//   49.5), else from 50 (616 x 2: 42 tiles 40.2 against 37.9, 52 tiles 44.1 against 44.4; 768 x 2: 42 tiles 41.9 against
//   39.8).  At a cache-update step, where the merge is free and the others mask every tile for the statistics, from 30
//   (whole step, 544 heads x 42 tiles 63.7 against 66.6 us, 896 x 30 70.6 against 72.6) and 46 (616 heads: 42 tiles 72.9
//   against 72.3, 46 tiles 76.3 against 76.5);
// * beyond that the others need another round and lose from the first tiles on (1036 heads: 4 tiles 16.8 against 13.1 us,
//   28 tiles 47.8 against 37.9; 1984: 12 tiles 38.1 against 27.8).
// Below the sizes of the last line its partials, up to 34 MB, would make sdllm_sparse_attn_noalloc refuse calls.
bool shared_tile_pays(int heads, int rows, int tiles, int n_split, bool update) {
  const int group = heads / rows;
  const int64_t wave_tiles = (int64_t)heads * tiles;
  if (!attn_gqa_supports_group(group)) return false;
  if (attn_gqa_waves_per_wg(group) < 4) return heads >= 320 && wave_tiles >= 26000;
  const int own = shared_splits(rows, group, tiles);
  bool pays;
  if (heads <= kNumCUs) pays = 5 * (int64_t)tiles >= (int64_t)n_split * (300 + 2 * heads * n_split);
  else if (heads <= 2 * kNumCUs) pays = tiles >= 66 && 6 * tiles >= heads;
  else if (heads <= 4 * kNumCUs) pays = tiles >= (heads * own > 6 * kNumCUs ? (update ? 30 : 40) : (update ? 46 : 50));
  else pays = true;
  return pays && (own == 1 || wave_tiles >= 30000 || (tiles >= 512 && wave_tiles >= 22000) || (heads >= 128 && wave_tiles >= 18000));
}

// Room for the key splits' partials of a kernel for 32 rows
void size_partials(AttnPlan& pl, const sdllm_shape_t& s) {
  if (pl.n_split == 1) return;
  const size_t slots = (size_t)s.batch * s.n_q_heads * pl.n_split;
  pl.part_o_bytes = align_up(slots * s.block_len * s.head_dim * sizeof(float));
  pl.part_ml_bytes = align_up(slots * 2 * s.block_len * sizeof(float));
}

// update: the dense rows of a cache-update step, where the merge of key splits costs no launch of its own (it runs in the
// compaction's) and the kernel mostly leaves the scoring's row statistics as well.
// scratch: the workspace there is.  A shared-tile kernel that does not fit gives way to the others up to 80 MB of keys and
// values (5000 tiles; it is a matter of speed there, and sdllm_sparse_attn_noalloc has 8 MB); beyond, the call is refused.
AttnPlan plan_streams(const sdllm_shape_t& s, int32_t n0, int64_t sr0, int32_t n1, int64_t sr1, bool update = false,
                      size_t scratch = SIZE_MAX) {
  AttnPlan pl{};
  pl.mfma = takes_mfma(s, n0, sr0, n1, sr1);
  pl.n_split = 1;
  pl.tiles_per_split = 0;
  pl.waves = 1;
  if (!pl.mfma) {
    plan_general(pl, s, s.block_len, (n0 + kTileKeys - 1) / kTileKeys + (n1 + kTileKeys - 1) / kTileKeys, true);
    return pl;
  }
  const int tiles = (n0 + kTileKeys - 1) / kTileKeys + (n1 + kTileKeys - 1) / kTileKeys;
  const int64_t wave_tiles = (int64_t)s.batch * s.n_q_heads * tiles;
  const int group = s.n_q_heads / s.n_kv_heads;
  const int heads = s.batch * s.n_q_heads, rows = s.batch * s.n_kv_heads;
  const auto partials = [&] { size_partials(pl, s); };
  // Key splits of the kernels with one workgroup per head, only while the grid is small: as many as keep
  // it within one workgroup per CU (an eight-wave workgroup fills a CU's LDS, so workgroup
  // number 257 waits for a whole round: 56 heads x 4 splits 15.1 us, x 5 splits 22.3 us), at most 8
  // (28 heads, replayed as a HIP graph so that only GPU time counts: 69 tiles 12.6 us with 6 splits and
  // 12.15 us with 8, 137 tiles 16.85 -> 15.2 us, 261 tiles 20.3 -> 18.5 us), and a minimum of tiles per
  // workgroup.  Batch-1 shapes are pure latency and a wave with
  // one or two tiles beats a longer chain (28/4 heads x 4352 keys: 17.2 -> 15.0 us with 6 or 7 splits
  // instead of 4).  From 129 heads on there is one workgroup per head.
  // A split costs fp32 partials and a second launch of about 4 us: with up to 32 heads (where three or
  // more splits fit) seven tiles per workgroup repay it, one tile per wave or two (32 heads x 21 tiles,
  // sparse step 12.1 -> 11.6 us, dense step over 41 tiles 14.0 -> 12.9 us with 3 splits); from 64 heads
  // on it takes eleven (128 heads x 21 tiles: 14.5 us unsplit, 15.9 us with 2 splits).
  int n_split = kNumCUs / heads;
  const int most = 8;
  if (n_split > most) n_split = most;
  const int max_split = tiles / (heads <= 32 ? 7 : 11);
  if (n_split > max_split) n_split = max_split;
  if (n_split < 1) n_split = 1;
  if (shared_tile_pays(heads, rows, tiles, n_split, update)) {
    const int n_shared = shared_splits(rows, group, tiles);
    pl.gqa = true;
    pl.tiles_per_split = (tiles + n_shared - 1) / n_shared;
    pl.n_split = (tiles + pl.tiles_per_split - 1) / pl.tiles_per_split;
    pl.waves = group;
    partials();
    if (pl.ws_bytes() <= scratch || (int64_t)rows * tiles > 5000) return pl;
    pl.gqa = false;
    pl.part_o_bytes = pl.part_ml_bytes = 0;
  }
  // The kernel that fetches tiles straight into LDS (attn_stream_mfma.hip) takes
  // * grouped-query heads with one workgroup per head: always with 129 to 256 heads (8 x 28/4 heads: 28 tiles
  //   11.8 -> 11.3 us, 75 tiles 20.9 -> 19.5 us, 144 tiles 37.1 -> 29.0 us).  With more, where its four-wave workgroups fit two
  //   to a CU as the other kernel's do, for groups of 7 and 8: up to 280 heads from 36 tiles on (40 tiles 22.3 -> 20.5 us; at
  //   336 heads 23.8 against 24.8), and for groups of 8 from 52 tiles on (416 heads 31.3 -> 30.1 us); with
  //   the statistics of a cache-update step always from 36 (whole step, 448 heads x 52 tiles 65.3 ->
  //   62.7 us, 616 x 42 77.9 -> 72.3);
  // * fewer grouped-query heads instead of key splits, up to the tile count at which two or more workgroups per head
  //   repay the combine launch: 8 to 32 heads 20 tiles 9.6 to 10.7 -> 9.2 us, 22 tiles level, 24 tiles 9.3 to 10.1 against 10.2;
  //   48 to 80 heads 30 tiles 13.1 -> 11.4 us, 36 tiles 11.6 to 12.7 against 12.3; 96 to 128 heads, groups of 6 to 8, 46 tiles
  //   15.1 to 15.7 -> 13.9 us, 52 tiles level, and groups of 3 and 4, whose keys are more bytes, 34 tiles 13.8 to 16.0 -> 12.6 to
  //   14.6, 42 tiles 15.8 to 17.2 against 16.4 to 17.3.  Where the merge rides on another launch there is nothing to save
  //   (cache-update step, 28 heads x 26 tiles 25.8 us split against 27.8; 12 heads, raw-logit scores 20.2 against 24.1),
  //   except for the split itself with more than 85 heads (128 heads x 22 tiles 29.7 -> 28.7, 112 x 30 30.4 against 31.3);
  // * split grouped-query heads at the cache-update step, where the other kernel masks every tile for the scoring's
  //   statistics, if its waves get three tiles or more (28 heads x 1040 tiles, whole step 88.4 -> 85.8 us); without
  //   statistics the two are within 2 % of each other up to 60 tiles a split;
  // * multi-head calls instead of splits up to 8 MB of keys and values, thirty-two of which (layers) fit the memory-side
  //   cache: 16 heads x 21 tiles 10.4 -> 9.3 us, 32 heads x 14 10.4 -> 8.0 us, 64 x 8 7.7 -> 6.8 us.  Beyond that a decoder's
  //   layers evict each other and the keys come from HBM, where 32 heads x 21 tiles take 11.2 us split and
  //   11.7 us unsplit (replayed as a graph 10.7 against 11.8; 10.7 against 9.6 if the cache holds them); the
  //   non-temporal streams of attn_mfma.hip also keep the dense rows of calls that they leave unsplit (they then
  //   sweep the scores as well).
  const bool unsplit_pays = n_split == 1 || (update ? heads > 85 && tiles <= 26
                                                    : tiles <= (heads <= 32 ? 22 : heads <= 85 ? 33 : group >= 6 ? 48 : 38));
  const bool stats = update && s.score_mode == SDLLM_SOFTMAX_MEAN;
  if (group > 1 && heads <= kNumCUs)
    pl.stream = unsplit_pays || (stats && tiles >= 24 * n_split);
  else if (group > 1)
    pl.stream = (group == 7 || group == 8) && tiles >= 36 && (stats || heads <= 280 || (heads <= 2 * kNumCUs && group == 8 && tiles >= 52));
  else
    pl.stream = heads <= 128 && wave_tiles <= 512 && unsplit_pays && (n1 > 0 || n_split > 1);
  if (pl.stream && unsplit_pays) n_split = 1;
  pl.tiles_per_split = (tiles + n_split - 1) / n_split;
  pl.waves = pl.tiles_per_split < kMaxWavesPerWg ? pl.tiles_per_split : kMaxWavesPerWg;
  // split workgroups: two tiles per wave when there are fewer than sixteen (28 heads x 69 tiles in 6
  // splits: 12.6 -> 12.35 us with six waves instead of eight; the in-workgroup merge is smaller)
  if (n_split > 1) { const int w2 = (pl.tiles_per_split + 1) / 2; pl.waves = w2 < kMaxWavesPerWg ? w2 : kMaxWavesPerWg; }
  // One workgroup per head: fewer, longer-running waves measured faster than eight (smaller merge at
  // the end, 40-48 KB instead of 64 KB of loads in flight per CU).  With more heads than CUs four
  // waves let two workgroups share a CU, so one streams while the other merges and writes, and no
  // workgroup waits for a second round (B=16 LLaDA shape: 94 -> 89 us; B=8: 47.5 -> 46.3 us with
  // five waves; 280 grouped-query heads, G = 7: 41.4 -> 36.0 us; 320 heads, G = 4: 48.6 -> 43.6 us).
  // With more than two heads per CU, two waves, so that four workgroups fit (544 heads, MHA:
  // 117.9 -> 106.0 us; 640 heads: 134.5 -> 113.8 us; 768 heads of G = 3: 88.8 -> 75.0 us).
  // Up to one head per CU the grouped-query heads keep eight waves: there they are short of
  // arithmetic throughput, not of bandwidth (B=8 Dream shape: 22 -> 26 us with fewer).
  if (n_split == 1) {
    const int cap = heads > 2 * kNumCUs ? 2 : heads > kNumCUs ? 4 : (group == 1 ? 5 : kMaxWavesPerWg);
    if (pl.waves > cap) pl.waves = cap;
  }
  // Fetching into LDS: few tiles are done soonest by waves that take three or four each (28 heads: 8 tiles 6.7 us with
  // four waves and 7.8 with eight, 14 tiles 8.0 with five and 9.0, 21 tiles 9.3 with six and 10.2, 45 tiles 13.5
  // and 13.9, 60 tiles 16.4 and 15.6).
  if (pl.stream) {
    const int w = heads > kNumCUs ? 4 : n_split > 1 || tiles > 50 ? kMaxWavesPerWg : tiles > 16 ? 6 : tiles > 9 ? 5 : 4;
    pl.waves = w < pl.tiles_per_split ? w : pl.tiles_per_split;
  }
  pl.n_split = (tiles + pl.tiles_per_split - 1) / pl.tiles_per_split;   // no empty split
  partials();
  return pl;
}

// Key splits with which the kernel that fetches all of a workgroup's tiles at once (attn_burst_mfma.hip) takes a call ahead of the
// kernels above, 0 if it does not.  It wins as long as its workgroups fit one to a CU, except (other kernel / this one, us, calls one after
// the other on 32 layers' keys and values, which come from memory where they are more than the memory-side cache holds)
// * unsplit multi-head heads, whose keys are all different, from some 20 MB on, where streams of a wave's tiles keep memory busier than one
//   burst: 136 heads x 9 tiles 8.35 / 8.29, 144 x 9 8.41 / 8.50, 224 x 9 9.26 / 10.3; 176 x 8 8.46 / 8.39, 192 x 8 8.53 / 8.76; 216 x 7 8.57 /
//   8.53 (dense rows 8.74 / 8.92), 232 x 7 8.72 / 8.90; 240 x 5 7.61 / 7.62, 256 x 5 7.73 / 7.88; 216 x 4 6.82 / 6.79, 256 x 4 7.03 / 7.21; 256 x
//   6 8.63 / 8.67, x 3 6.6 / 6.24;
// * where the others go unsplit and it would have to split: multi-head 20 heads x 10 6.72 / 6.51, 28 x 12 7.24 / 6.94, but x 13 7.25 / 7.52, 32 x
//   13 7.57 / 7.80, x 15 8.40 / 7.94, 34 x 13 7.55 / 7.91, 40 x 11 7.42 / 7.59, x 12 7.99 / 7.81, 48 x 14 9.09 / 9.32, x 15 9.63 / 9.14, 64 x 15
//   9.98 / 10.2, x 16 10.4 / 10.25, 72 x 20 11.6 / 11.8, x 21 12.05 / 11.95, x 23 12.1 / 12.1 (dense rows 11.6 / 12.3); grouped-query 28 x 11
//   7.18 / 6.64, 40 x 13 7.36 / 7.58, x 15 7.63 / 7.49, 48 x 17 7.93 / 7.90 (two heads to a group 7.94 / 8.23), 56 x 17 7.94 / 8.08, x 18 8.19 /
//   8.20, 64 x 24 9.5 / 8.9, 80 x 10 6.3 / 7.5, x 27 9.5 / 9.8; so not with more than 64 heads;
// * split multi-head heads with more than 18 of them, from 1280 tiles (21 MB) or from where the others take another split on (33 and 44 tiles):
//   all tiles come at once, but the arithmetic waits for the last of them, where streams compute meanwhile.  20 x 71 11.34 / 11.33 (dense rows x
//   65 10.88 / 11.17), 24 x 59 11.20 / 11.18, x 68 11.68 / 12.16, 28 x 47 10.95 / 10.88 (dense rows x 50 11.31 / 11.52), x 50 11.18 / 11.27, x 68
//   12.16 / 13.05, 32 x 41 11.31 / 10.81 (dense rows 10.91 / 11.13), x 44 11.22 / 11.52, x 68 12.79 / 13.82, 40 x 41 12.82 / 12.00, x 44 12.13 /
//   12.61, 48 x 32 13.16 / 11.47, x 35 12.09 / 12.24, 64 x 32 13.58 / 13.13, x 35 13.42 / 14.07.  (With three layers' keys in the memory-side
//   cache it is 8 to 12 % the faster one at these.)
// More than one round of workgroups, whose second round waits for the first, is a quarter to a half slower (28 x 90 11.1 / 13.8).
// The splits are those of least modelled time: a tile in a workgroup 0.22 us, the ninth 0.08 more (a third wave on one SIMD), four
// splits to fold 0.16, and 0.94 for 16 KB of partials on each of 100 workgroups, fitted to 460 calls of 2 to 96 heads x 10 to 280
// tiles (rms 0.2 us; half a per cent lost to the best count on average, 5 % at 2 of 130 sizes).  The merge folds as many as it is
// instantiated for: 1 head x 40 tiles in 20 splits (as 24) 6.96 us, in 14 (as 16) 6.48.
// most: no more of them.
int burst_splits(int heads, int tiles, int group, int most) {
  static constexpr int kMostMultiHead[kBurstMaxTiles + 1] = {kNumCUs, kNumCUs, kNumCUs, kNumCUs, 216, 240, kNumCUs, 200, 176, 136};   // by tiles
  if (tiles <= kBurstMaxTiles) return heads <= (group > 1 ? kNumCUs : kMostMultiHead[tiles]) ? 1 : 0;
  if (heads > 64) return 0;
  const int from = heads <= 20 ? 10 : heads <= 30 || (group > 1 && heads <= 36) ? 11
                   : group > 1 ? (heads <= 40 ? 15 : heads <= 48 ? (group == 2 ? 18 : 17) : heads <= 56 ? 18 : 24)
                               : (heads <= 38 ? 15 : heads <= 44 ? 12 : heads <= 56 ? 15 : 16);
  if (tiles < from) return 0;
  if (group == 1 && heads > 25 && (tiles == 13 || tiles == 14) && heads <= 38) return 0;
  if (group == 1 && heads > 18 && tiles > (heads <= 32 ? 1280 / heads : heads <= 42 ? 43 : 32)) return 0;
  int best = 0, least = INT32_MAX;
  for (int n = (tiles + kBurstMaxTiles - 1) / kBurstMaxTiles; n <= most && n * heads <= kNumCUs; ++n) {
    const int mine = (tiles + n - 1) / n;
    const int fours = n <= 16 ? (n + 3) / 4 : n <= 24 ? 6 : 8;   // with_combine32
    const int cost = 22 * mine + (mine > kMaxWavesPerWg ? 8 : 0) + 16 * fours + 15 * heads * n / 16;   // 0.01 us
    if (cost < least) { least = cost; best = n; }
  }
  return best;
}

// Whether that kernel takes a call without by-products (pl is the plan then), given `scratch` bytes of workspace aligned to 16.  It
// makes do with fewer splits where those of the rule do not fit, and leaves the call to the kernels above where even those are too
// many: sdllm_workspace_bytes asks for the room (4.3 MB at most), but calls that bring no more than the kernels above need are taken too.
constexpr size_t kBurstPartialBytes = 32 * (128 + 2) * sizeof(float);
bool plan_burst(AttnPlan& pl, const sdllm_shape_t& s, int32_t n0, int64_t sr0, int32_t n1, int64_t sr1, size_t scratch) {
  if (!takes_mfma(s, n0, sr0, n1, sr1)) return false;
  const int64_t heads = (int64_t)s.batch * s.n_q_heads;
  const int tiles = (n0 + kTileKeys - 1) / kTileKeys + (n1 + kTileKeys - 1) / kTileKeys;
  if (heads > kNumCUs) return false;
  const size_t fit = scratch / (heads * kBurstPartialBytes);
  const int n = burst_splits((int)heads, tiles, s.n_q_heads / s.n_kv_heads, fit < 32 ? (int)fit : 32);
  if (n == 0) return false;
  pl = AttnPlan{};
  pl.mfma = pl.burst = true;
  pl.tiles_per_split = (tiles + n - 1) / n;
  pl.n_split = (tiles + pl.tiles_per_split - 1) / pl.tiles_per_split;
  pl.waves = pl.tiles_per_split > kMaxWavesPerWg ? pl.tiles_per_split : kMaxWavesPerWg;
  size_partials(pl, s);
  return pl.ws_bytes() <= scratch;   // two buffers, each a multiple of 256 bytes
}

// Workspace with which a call without by-products runs that kernel with the splits of its rule, 0 if it does not run it
size_t burst_bytes(const sdllm_shape_t& s, int32_t n0, int64_t sr0, int32_t n1, int64_t sr1) {
  AttnPlan pl;
  return plan_burst(pl, s, n0, sr0, n1, sr1, SIZE_MAX) ? pl.ws_bytes() : 0;
}

// Whether the dense launch of a cache-update step can also leave the saliency scores: multi-head attention
// (one query head per KV head) on the one-workgroup-per-head kernel, no key splits, at least two waves.
bool fuses_columns(const AttnPlan& pl, const sdllm_shape_t& s) {
  return pl.mfma && !pl.gqa && !pl.stream && pl.n_split == 1 && pl.waves >= 2 && s.n_q_heads == s.n_kv_heads;
}

// cand_ml != null (dense MFMA launches only): also emit the scoring pass's row statistics over the
// candidate keys, n_split partials per query row.
// deferred != null: when the keys are split over workgroups, leave the merge of the splits to the caller
// (it gets the launch parameters in *deferred and must run launch_compact_combine or launch_attn_combine on
// the same stream before the partials' workspace is reused); deferred->n_split == 1 says nothing is left.
int32_t run_attn(const sdllm_shape_t& s, const void* q, const KvSegment& a, const KvSegment& b, void* out, void* ws,
                 size_t ws_bytes, hipStream_t stream, bool update = false, float* cand_ml = nullptr, int cand0_end = 0,
                 int cand1_begin = 0, AttnParams* deferred = nullptr, float* score_out = nullptr, int score_stride = 0) {
  AttnPlan pl = plan_streams(s, a.n, a.sr, b.n, b.sr, update, ws ? ws_bytes : 0);
  const bool fits = ws && ws_bytes >= pl.ws_bytes();
  // also where the next kernel, with fewer splits, would make do with less: what a call has to bring depends on its sizes only
  if (pl.ws_bytes() > 0 && pl.mfma && !fits) return SDLLM_ERR_WORKSPACE;
  if (AttnPlan at_once; !update && !cand_ml && plan_burst(at_once, s, a.n, a.sr, b.n, b.sr, ws && aligned16(ws) ? ws_bytes : 0)) pl = at_once;
  if (pl.ws_bytes() > 0 && !pl.mfma && !(fits && aligned16(ws))) {
    // the general kernel works without a usable workspace too: one workgroup per block of rows walks all keys
    plan_general(pl, s, s.block_len, (a.n + kTileKeys - 1) / kTileKeys + (b.n + kTileKeys - 1) / kTileKeys, false);
  }
  AttnParams p{};
  p.q = q;
  p.out = out;
  p.seg[0] = a;
  p.seg[1] = b;
  p.q_sb = s.q_stride[0]; p.q_sh = s.q_stride[1]; p.q_sr = s.q_stride[2];
  p.o_sb = s.out_stride[0]; p.o_sh = s.out_stride[1]; p.o_sr = s.out_stride[2];
  p.batch = s.batch; p.hq = s.n_q_heads; p.hkv = s.n_kv_heads; p.group = s.n_q_heads / s.n_kv_heads;
  p.nq = s.block_len; p.d = s.head_dim;
  p.scale_log2 = scale_of(s) * kLog2e;
  p.n_split = pl.n_split; p.tiles_per_split = pl.tiles_per_split; p.waves = pl.waves;
  p.part_o = (float*)ws;
  p.part_ml = (float*)((char*)ws + pl.part_o_bytes);
  p.cand_ml = cand_ml;
  p.cand0_end = cand0_end;
  p.cand1_begin = cand1_begin;
  // the column sweep rides on the statistics launch of the one-workgroup-per-head kernel (fuses_columns below)
  p.score_out = p.cand_ml ? score_out : nullptr;
  p.score_stride = score_stride;
  p.score_inv_count = 1.f / (float)(s.block_len * (s.n_q_heads / s.n_kv_heads));
  hipError_t e;
  if (pl.mfma) {
    e = pl.burst ? launch_attn_burst_mfma_bf16(p, stream) : pl.stream ? launch_attn_stream_mfma_bf16(p, stream)
        : pl.gqa ? launch_attn_gqa_mfma_bf16(p, stream) : launch_attn_mfma_bf16(p, stream);
  } else {
    e = launch_attn_general(p, s.dtype, false, stream);
  }
  if (deferred) *deferred = p;
  if (e == hipSuccess && pl.n_split > 1 && !deferred) e = launch_attn_combine(p, s.dtype, stream);
  return e == hipSuccess ? SDLLM_OK : SDLLM_ERR_HIP;
}

// ---------------------------------------------------------------- scoring planning
struct ScorePlan {
  bool mfma;
  int n_scored;       // candidates that get a score
  int n_part, tiles_per_part, waves;
  // workspace: scores, softmax row statistics and, for segments too long for one workgroup, the selection's
  // key buffer, thresholds, bin lists and chunk offsets
  size_t score_bytes, ml_bytes, keys_bytes, sorted_bytes, bins_bytes;
  size_t ws_bytes() const { return score_bytes + ml_bytes + keys_bytes + sorted_bytes + bins_bytes; }
};

// The ranked segments and the unconditional tail of the selection for this shape (Alg. 1 steps 8-10;
// Alg. 4 keeps the suffix whole).
void fill_segments(const sdllm_shape_t& s, const Counts& c, SelectParams& q) {
  q.rows = s.batch * s.n_kv_heads;
  q.n_cand = c.n_cand;
  q.k_total = c.k_total;
  q.pool_half = (s.pool_kernel - 1) / 2;
  q.avg_pool = s.pool_mode == SDLLM_AVG_POOL;
  q.block_off = s.block_off; q.block_len = s.block_len;
  if (s.evict_scope == SDLLM_EVICT_PREFIX_ONLY) {
    q.n_seg = 1;
    q.seg_begin[0] = 0; q.seg_len[0] = c.n_pre; q.seg_k[0] = c.k_pre; q.seg_out[0] = 0;
    q.tail_begin = c.n_pre; q.tail_len = c.n_suf; q.tail_out = c.k_pre;
  } else if (s.select_mode == SDLLM_PER_SEGMENT) {
    q.n_seg = 2;
    q.seg_begin[0] = 0; q.seg_len[0] = c.n_pre; q.seg_k[0] = c.k_pre; q.seg_out[0] = 0;
    q.seg_begin[1] = c.n_pre; q.seg_len[1] = c.n_suf; q.seg_k[1] = c.k_suf; q.seg_out[1] = c.k_pre;
  } else {
    q.n_seg = 1;
    q.seg_begin[0] = 0; q.seg_len[0] = c.n_cand; q.seg_k[0] = c.k_total; q.seg_out[0] = 0;
  }
}

// Workgroups per row of the 32-row kernels' column pass, their tiles and waves
void plan_columns(size_t rows, int tiles, int& waves, int& n_part, int& tiles_per_part) {
  if (tiles < 1) tiles = 1;
  int waves_per_row = (int)((kNumCUs * kMaxWavesPerWg + rows - 1) / rows);
  if (waves_per_row > tiles) waves_per_row = tiles;
  if (waves_per_row < 1) waves_per_row = 1;
  waves = waves_per_row < kMaxWavesPerWg ? waves_per_row : kMaxWavesPerWg;
  n_part = (waves_per_row + waves - 1) / waves;
  // never a few workgroups more than there are CUs: with several heads' Q staged in LDS a CU holds
  // one scoring workgroup, and the extra ones would wait for a whole round
  if (rows < (size_t)kNumCUs && n_part > kNumCUs / (int)rows) n_part = kNumCUs / (int)rows;
  tiles_per_part = (tiles + n_part - 1) / n_part;
  n_part = (tiles + tiles_per_part - 1) / tiles_per_part;   // no empty part
}

// Tiles of the candidates that get a score, per KV head
int scored_tiles(const sdllm_shape_t& s) {
  const Counts c = counts_of(s);
  const int n1 = s.evict_scope == SDLLM_EVICT_PREFIX_ONLY ? 0 : c.n_suf;
  return (c.n_pre + kTileKeys - 1) / kTileKeys + (n1 + kTileKeys - 1) / kTileKeys;
}

ScorePlan plan_score(const sdllm_shape_t& s) {
  const Counts c = counts_of(s);
  ScorePlan pl{};
  pl.n_scored = s.evict_scope == SDLLM_EVICT_PREFIX_ONLY ? c.n_pre : c.n_cand;
  const size_t rows = (size_t)s.batch * s.n_kv_heads;
  pl.score_bytes = align_up(rows * c.n_cand * sizeof(float));
  {
    SelectParams q{};
    fill_segments(s, c, q);
    const SelectWorkspace sw = select_workspace(q);
    pl.keys_bytes = align_up(sw.keys * sizeof(uint32_t));
    pl.sorted_bytes = align_up(sw.sorted * sizeof(uint32_t));
    pl.bins_bytes = align_up(sw.bins * sizeof(uint32_t));
  }
  pl.mfma = s.dtype == SDLLM_BF16 && s.head_dim == 128 && s.block_len == 32 &&
            score_mfma_supports_group(s.n_q_heads / s.n_kv_heads) && seg_fits_u32(s.kv_stride[2], s.seq_len, 2);
  pl.n_part = 1;
  pl.tiles_per_part = 0;
  pl.waves = 1;
  if (pl.mfma) {
    plan_columns(rows, scored_tiles(s), pl.waves, pl.n_part, pl.tiles_per_part);
  } else {
    // row statistics: a statistics-only run of the general attention kernel over the whole sequence
    AttnPlan st{};
    plan_general(st, s, s.block_len, (s.seq_len + kTileKeys - 1) / kTileKeys, true);
    pl.n_part = st.n_split; pl.tiles_per_part = st.tiles_per_split; pl.waves = st.waves;
  }
  pl.ml_bytes = align_up((size_t)s.batch * s.n_q_heads * row_blocks(s, s.block_len) * pl.n_part * 2 * block_rows(s.dtype) * sizeof(float));
  return pl;
}

// Whether the column pass of a block length other than 32 runs the kernels for 32 rows: every block of 32 rows of a head as a head of its
// own, rows that are not there with no weight (of a softmax; raw logits take full blocks).  Those keep a tile's keys in registers and
// fetch tiles for all heads at once, where the general kernel reads queries and keys from LDS for each.  Cache-update steps, general / as
// heads: block of 64, 2 x 32 heads x 1280 positions 38.9 / 37.9 us, 1 x 8 x 1100 26.0 / 23.2, 1 x 8/2 x 600 31.0 / 22.6, 8 x 32/8 x 4000 220 / 173;
// block of 16, 1 x 14/2 x 600 27.0 / 21.8, 8 x 28/4 x 3000 84 / 68, 4 x 32 x 2000 72.1 / 70.4, but one block per KV head and few of them, where the
// general kernel's smaller workgroups are more: KV heads x positions, each layer with keys of its own, 64 x 200 22.5 / 22.1, x 600 30.3 / 29.8,
// x 2600 61.6 / 56.6, 128 x 600 36.3 / 35.3, x 1300 60.2 / 55.6, 48 x 600 level, 32 x 600 28.5 / 27.6, x 1800 31.6 / 32.8, x 2600 38.1 / 39.3, 16 x 900
// 23.8 / 24.8.  (With all keys and values in the memory-side cache 64 x 1300 and 128 x 600 lose 3 to 6 %.)
bool blocks_as_heads(const sdllm_shape_t& s) {
  const int group = row_blocks(s, s.block_len) * (s.n_q_heads / s.n_kv_heads);
  return s.dtype == SDLLM_BF16 && s.head_dim == 128 && (s.block_len % 32 == 0 || s.score_mode == SDLLM_SOFTMAX_MEAN) &&
         s.batch * (int64_t)s.n_kv_heads <= 65535 && seg_fits_u32(s.kv_stride[2], s.seq_len, 2) &&
         score_mfma_supports_group(group) && (group > 1 || s.batch * (int64_t)s.n_kv_heads >= 64);
}

// The position from which keys are scored again after the prefix: past the block, or never (prefix-only eviction).
int candidates_resume(const sdllm_shape_t& s) {
  return s.evict_scope == SDLLM_EVICT_PREFIX_ONLY ? s.seq_len : s.block_off + s.block_len;
}

int32_t check_q(const sdllm_shape_t& s, const void* q) {
  if (!q || !aligned16(q) || !row_stride_ok(s.q_stride, s.head_dim)) return SDLLM_ERR_INVALID_ARG;
  return SDLLM_OK;
}

// Alg. 1 steps 2-10.  ext_ml != null: the softmax row statistics over the candidates were already
// produced (ext_parts partials per row) and only the column reduction and the selection run.
// in_step: called by a cache-update step (ext_ml only there, for softmax scores).
// scores_ready: the scores are in the workspace's score buffer already; only the selection runs.
int32_t score_select_impl(const sdllm_shape_t& s, const void* q_blk, const void* k_full, int32_t* idx_out,
                          float* pooled_out, float* score_out, void* ws, size_t ws_bytes, hipStream_t hs,
                          float* ext_ml, int ext_parts, bool in_step = false, bool scores_ready = false) {
  const Counts c = counts_of(s);
  const ScorePlan pl = plan_score(s);
  if (!ws || ws_bytes < pl.ws_bytes() || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0) return SDLLM_ERR_WORKSPACE;
  if (c.n_cand == 0) return SDLLM_OK;
  {
    SelectParams probe{};
    fill_segments(s, c, probe);
    for (int i = 0; i < probe.n_seg; ++i)
      if (probe.seg_len[i] > select_max_segment()) return SDLLM_ERR_UNSUPPORTED;   // beyond the selection's per-segment tables
  }

  char* at = (char*)ws;
  float* score = score_out ? score_out : (float*)at;
  at += pl.score_bytes;
  float* ml = (float*)at;
  at += pl.ml_bytes;
  uint32_t* keys = pl.keys_bytes ? (uint32_t*)at : nullptr;
  at += pl.keys_bytes;
  uint32_t* sorted = pl.sorted_bytes ? (uint32_t*)at : nullptr;
  at += pl.sorted_bytes;
  uint32_t* bins = pl.bins_bytes ? (uint32_t*)at : nullptr;

  ScoreParams sp{};
  sp.q = q_blk; sp.k = k_full;
  sp.q_sb = s.q_stride[0]; sp.q_sh = s.q_stride[1]; sp.q_sr = s.q_stride[2];
  sp.k_sb = s.kv_stride[0]; sp.k_sh = s.kv_stride[1]; sp.k_sr = s.kv_stride[2];
  sp.batch = s.batch; sp.hq = s.n_q_heads; sp.hkv = s.n_kv_heads; sp.group = s.n_q_heads / s.n_kv_heads;
  sp.by_hkv = Divisor(s.n_kv_heads);
  sp.inv_count = 1.f / (float)(sp.group * s.block_len);
  sp.nq = s.block_len; sp.d = s.head_dim;
  sp.block_off = s.block_off; sp.block_len = s.block_len;
  sp.n_cand = pl.n_scored;
  sp.score_stride = c.n_cand;
  sp.softmax = s.score_mode == SDLLM_SOFTMAX_MEAN;
  sp.scale = scale_of(s);
  sp.scale_log2 = sp.scale * kLog2e;
  sp.score = score;
  sp.n_part = pl.n_part; sp.tiles_per_part = pl.tiles_per_part; sp.waves = pl.waves;
  sp.part_ml = ext_ml ? ext_ml : ml;
  sp.n_stat_part = ext_ml ? ext_parts : pl.n_part;
  sp.skip_stats = ext_ml != nullptr;
  sp.in_step = in_step;
  // scores_ready: the dense attention of this step already left the scores in the workspace's score buffer
  hipError_t e = hipSuccess;
  if (!scores_ready && pl.mfma) {
    e = launch_score_mfma_bf16(sp, hs);
  } else if (!scores_ready) {
    if (sp.softmax && !ext_ml && sp.n_cand > 0) {
      AttnParams p{};
      p.q = q_blk;
      p.q_sb = sp.q_sb; p.q_sh = sp.q_sh; p.q_sr = sp.q_sr;
      p.seg[0] = KvSegment{k_full, nullptr, sp.k_sb, sp.k_sh, sp.k_sr, s.seq_len};
      p.batch = sp.batch; p.hq = sp.hq; p.hkv = sp.hkv; p.group = sp.group; p.nq = sp.nq; p.d = sp.d;
      p.scale_log2 = sp.scale_log2;
      p.n_split = pl.n_part; p.tiles_per_split = pl.tiles_per_part; p.waves = pl.waves;
      p.cand_ml = ml;
      p.cand0_end = s.block_off;
      p.cand1_begin = candidates_resume(s);
      e = launch_attn_general(p, s.dtype, true, hs);
    }
    if (e == hipSuccess && blocks_as_heads(s)) {
      // blocks of 32 rows are heads to the column pass, and their statistics lie as it reads them
      sp.q_shift = row_blocks(s, s.block_len) - 1;
      sp.hq <<= sp.q_shift; sp.group <<= sp.q_shift;
      sp.skip_stats = 1;
      plan_columns((size_t)s.batch * s.n_kv_heads, scored_tiles(s), sp.waves, sp.n_part, sp.tiles_per_part);
      e = launch_score_mfma_bf16(sp, hs);
    } else if (e == hipSuccess) {
      e = launch_score_cols_general(sp, s.dtype, hs);
    }
  }
  if (e != hipSuccess) return SDLLM_ERR_HIP;

  SelectParams q{};
  fill_segments(s, c, q);
  q.score = score; q.pooled = pooled_out; q.idx = idx_out;
  q.keys = keys; q.sorted = sorted; q.bins = bins;
  e = launch_select(q, hs);
  return e == hipSuccess ? SDLLM_OK : SDLLM_ERR_HIP;
}

// Argument checks and launch parameters of the gather (k_total > 0).
int32_t compact_params(const sdllm_shape_t& s, const void* k_full, const void* v_full, const int32_t* idx, void* k_cache,
                       void* v_cache, CompactParams& p) {
  if (!k_full || !v_full || !idx || !k_cache || !v_cache) return SDLLM_ERR_INVALID_ARG;
  if (!aligned16(k_full) || !aligned16(v_full) || !aligned16(k_cache) || !aligned16(v_cache))
    return SDLLM_ERR_INVALID_ARG;
  if (!row_stride_ok(s.kv_stride, s.head_dim) || !row_stride_ok(s.cache_stride, s.head_dim))
    return SDLLM_ERR_INVALID_ARG;
  const int es = elem_size(s.dtype);
  p.k = k_full; p.v = v_full; p.idx = idx; p.kc = k_cache; p.vc = v_cache;
  p.s_sb = s.kv_stride[0] * es; p.s_sh = s.kv_stride[1] * es; p.s_sr = s.kv_stride[2] * es;
  p.c_sb = s.cache_stride[0] * es; p.c_sh = s.cache_stride[1] * es; p.c_sr = s.cache_stride[2] * es;
  p.batch = s.batch; p.hkv = s.n_kv_heads; p.k_total = counts_of(s).k_total; p.seq_len = s.seq_len;
  p.row_bytes = s.head_dim * es;
  return SDLLM_OK;
}

// Workspace of sdllm_block_step: [0, base) is shared by the attention partials and the scoring
// buffers (used one after the other on the stream); the fused row statistics of the cache-update
// step live behind it because they are written by the attention and read by the scoring.
// With split keys at the cache-update step the merge of the splits runs in the compaction's launch, so
// the attention partials stay alive through scoring and selection: those then work behind them (score_off).  Also for
// the general kernels (2 x 32 heads, block of 64, 1280 positions 43.2 -> 41.0 us, 2 x 8 of head_dim 64, 1200 positions 24.3 -> 21.7),
// whose partials may as well be merged before the scoring: with a workspace that has no room for both (beside = false).
struct BlockStepWs {
  size_t base, stats_bytes, score_off;
  int stats_parts;
  bool fuse, fuse_cols;
  size_t bytes() const { return base + stats_bytes; }
};

BlockStepWs plan_block_step(const sdllm_shape_t& s, bool beside = true) {
  const Counts c = counts_of(s);
  const AttnPlan full = plan_streams(s, s.seq_len, s.kv_stride[2], 0, 0);
  const AttnPlan dense = plan_streams(s, s.seq_len, s.kv_stride[2], 0, 0, c.k_total > 0);   // of a cache-update step
  const AttnPlan sparse = plan_streams(s, c.k_total, s.cache_stride[2], s.block_len, s.blk_stride[2]);
  const ScorePlan sc = plan_score(s);
  BlockStepWs w{};
  w.score_off = (beside || dense.mfma) && dense.n_split > 1 && c.k_total > 0 ? align_up(dense.ws_bytes()) : 0;
  w.base = dense.ws_bytes();
  if (full.ws_bytes() > w.base) w.base = full.ws_bytes();
  if (sparse.ws_bytes() > w.base) w.base = sparse.ws_bytes();
  if (w.score_off + sc.ws_bytes() > w.base) w.base = w.score_off + sc.ws_bytes();
  w.base = align_up(w.base);
  w.fuse = s.score_mode == SDLLM_SOFTMAX_MEAN && c.n_cand > 0;
  w.stats_parts = dense.n_split;
  w.fuse_cols = w.fuse && fuses_columns(dense, s);
  w.stats_bytes = w.fuse ? align_up((size_t)s.batch * s.n_q_heads * row_blocks(s, s.block_len) * dense.n_split * 2 * block_rows(s.dtype) * sizeof(float)) : 0;
  return w;
}

}  // namespace

// ---------------------------------------------------------------- static scratch (sdllm_sparse_attn_noalloc)
// The array is part of the device image: one copy per GPU, at its own address, alive until the
// process ends.  In host code the name `scratch` is only a handle for hipGetSymbolAddress; kernels
// and launch parameters get the per-device address resolved here.  The declaration carries no `used`
// attribute on purpose: the compiler gives a static device variable that host code refers to external
// linkage in the device image, which is how the runtime finds it, and leaves a `used` one local (the
// runtime then aborts in hipGetSymbolAddress).
static __device__ __align__(256) unsigned char scratch[SDLLM_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Address of the current device's copy of `scratch` (resolved once per device, with that device current).
hipError_t static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // concurrent first calls resolve the same address
  }
  *out = ptr;
  return hipSuccess;
}

}  // namespace

// ================================================================ exported functions
extern "C" {

const char* sdllm_error_string(int32_t status) {
  switch (status) {
    case SDLLM_OK: return "ok";
    case SDLLM_ERR_INVALID_ARG: return "invalid argument";
    case SDLLM_ERR_UNSUPPORTED: return "unsupported shape or type";
    case SDLLM_ERR_WORKSPACE: return "workspace missing or too small";
    case SDLLM_ERR_HIP: return "HIP launch failed";
    case SDLLM_ERR_STATIC_LIMIT: return "request exceeds the static scratch of sdllm_sparse_attn_noalloc";
    default: return "unknown status";
  }
}

int32_t sdllm_version(void) { return 100; }

int32_t sdllm_retained_count(const sdllm_shape_t* shape, int32_t* k_total, int32_t* k_pre, int32_t* k_suf) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const Counts c = counts_of(*shape);
  if (k_total) *k_total = c.k_total;
  if (k_pre) *k_pre = c.k_pre;
  if (k_suf) *k_suf = c.k_suf;
  return SDLLM_OK;
}

int32_t sdllm_cache_state(int32_t step_in_block, int32_t delay, int32_t* state) {
  if (!state || step_in_block < 0 || delay < 0) return SDLLM_ERR_INVALID_ARG;
  *state = step_in_block > delay ? SDLLM_STATE_REUSE : (step_in_block == delay ? SDLLM_STATE_UPDATE : SDLLM_STATE_FULL);
  return SDLLM_OK;
}

int32_t sdllm_workspace_bytes(const sdllm_shape_t* shape, int32_t op, int32_t n_cached, size_t* bytes) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  if (!bytes) return SDLLM_ERR_INVALID_ARG;
  const sdllm_shape_t& s = *shape;
  size_t need = 0;
  switch (op) {
    case SDLLM_OP_SCORE_SELECT: need = plan_score(s).ws_bytes(); break;
    case SDLLM_OP_COMPACT_KV: need = 0; break;
    case SDLLM_OP_SPARSE_ATTN:
      if (n_cached < 0) return SDLLM_ERR_INVALID_ARG;
      need = std::max(plan_streams(s, n_cached, s.cache_stride[2], s.block_len, s.blk_stride[2]).ws_bytes(),
                      burst_bytes(s, n_cached, s.cache_stride[2], s.block_len, s.blk_stride[2]));
      break;
    case SDLLM_OP_BLOCK_STEP:   // sdllm_block_step refuses less than the first only
      need = std::max({plan_block_step(s).bytes(), burst_bytes(s, counts_of(s).k_total, s.cache_stride[2], s.block_len, s.blk_stride[2]),
                       burst_bytes(s, s.seq_len, s.kv_stride[2], 0, 0)});
      break;
    default: return SDLLM_ERR_INVALID_ARG;
  }
  *bytes = need > 0 ? need : kAlign;   // never zero, so callers can always allocate
  return SDLLM_OK;
}

int32_t sdllm_score_select(const sdllm_shape_t* shape, const void* q_blk, const void* k_full, int32_t* idx_out,
                           float* pooled_out, float* score_out, void* ws, size_t ws_bytes, void* stream) {
  int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const sdllm_shape_t& s = *shape;
  if ((st = check_q(s, q_blk)) != SDLLM_OK) return st;
  if (!k_full || !aligned16(k_full) || !row_stride_ok(s.kv_stride, s.head_dim)) return SDLLM_ERR_INVALID_ARG;
  if (counts_of(s).k_total > 0 && !idx_out) return SDLLM_ERR_INVALID_ARG;
  return score_select_impl(s, q_blk, k_full, idx_out, pooled_out, score_out, ws, ws_bytes, (hipStream_t)stream, nullptr, 0);
}

int32_t sdllm_compact_kv(const sdllm_shape_t* shape, const void* k_full, const void* v_full, const int32_t* idx,
                         void* k_cache, void* v_cache, void* stream) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  if (counts_of(*shape).k_total == 0) return SDLLM_OK;
  CompactParams p{};
  const int32_t sp = compact_params(*shape, k_full, v_full, idx, k_cache, v_cache, p);
  if (sp != SDLLM_OK) return sp;
  return launch_compact(p, (hipStream_t)stream) == hipSuccess ? SDLLM_OK : SDLLM_ERR_HIP;
}

int32_t sdllm_sparse_attn(const sdllm_shape_t* shape, const void* q_blk, const void* k_cache, const void* v_cache,
                          int32_t n_cached, const void* k_blk, const void* v_blk, void* out, void* ws,
                          size_t ws_bytes, void* stream) {
  int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const sdllm_shape_t& s = *shape;
  if ((st = check_q(s, q_blk)) != SDLLM_OK) return st;
  if (n_cached < 0) return SDLLM_ERR_INVALID_ARG;
  if (n_cached > 0 && (!k_cache || !v_cache || !aligned16(k_cache) || !aligned16(v_cache) ||
                       !row_stride_ok(s.cache_stride, s.head_dim)))
    return SDLLM_ERR_INVALID_ARG;
  if (!k_blk || !v_blk || !out || !aligned16(k_blk) || !aligned16(v_blk) || !aligned16(out) ||
      !row_stride_ok(s.blk_stride, s.head_dim) || !row_stride_ok(s.out_stride, s.head_dim))
    return SDLLM_ERR_INVALID_ARG;
  KvSegment a{k_cache, v_cache, s.cache_stride[0], s.cache_stride[1], s.cache_stride[2], n_cached};
  KvSegment b{k_blk, v_blk, s.blk_stride[0], s.blk_stride[1], s.blk_stride[2], s.block_len};
  return run_attn(s, q_blk, a, b, out, ws, ws_bytes, (hipStream_t)stream);
}

int32_t sdllm_sparse_attn_noalloc(const sdllm_shape_t* shape, const void* q_blk, const void* k_cache,
                                  const void* v_cache, int32_t n_cached, const void* k_blk, const void* v_blk,
                                  void* out, void* stream) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  if (n_cached < 0) return SDLLM_ERR_INVALID_ARG;
  const sdllm_shape_t& s = *shape;
  const size_t need = plan_streams(s, n_cached, s.cache_stride[2], s.block_len, s.blk_stride[2], false, SDLLM_STATIC_SCRATCH_BYTES).ws_bytes();
  if (need > SDLLM_STATIC_SCRATCH_BYTES) return SDLLM_ERR_STATIC_LIMIT;
  void* ptr = nullptr;
  if (static_scratch(&ptr) != hipSuccess) return SDLLM_ERR_HIP;
  return sdllm_sparse_attn(shape, q_blk, k_cache, v_cache, n_cached, k_blk, v_blk, out, ptr, SDLLM_STATIC_SCRATCH_BYTES, stream);
}

int32_t sdllm_block_step(const sdllm_shape_t* shape, int32_t step_in_block, int32_t delay, const void* q_blk,
                         const void* k_in, const void* v_in, int32_t* idx, void* k_cache, void* v_cache, void* out,
                         void* ws, size_t ws_bytes, void* stream, int32_t* state_out) {
  int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const sdllm_shape_t& s = *shape;
  int32_t state;
  if ((st = sdllm_cache_state(step_in_block, delay, &state)) != SDLLM_OK) return st;
  BlockStepWs w = plan_block_step(s);
  if (ws_bytes < w.bytes()) w = plan_block_step(s, false);
  const size_t need = w.bytes() > 0 ? w.bytes() : kAlign;
  if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0) return SDLLM_ERR_WORKSPACE;
  if ((st = check_q(s, q_blk)) != SDLLM_OK) return st;
  if (!k_in || !v_in || !out || !aligned16(k_in) || !aligned16(v_in) || !aligned16(out) ||
      !row_stride_ok(s.out_stride, s.head_dim))
    return SDLLM_ERR_INVALID_ARG;
  const Counts c = counts_of(s);
  if (state_out) *state_out = state;

  if (state == SDLLM_STATE_REUSE) {
    return sdllm_sparse_attn(shape, q_blk, k_cache, v_cache, c.k_total, k_in, v_in, out, ws, ws_bytes, stream);
  }
  // states 0/1: the block's rows of dense attention over all L keys of this step
  if (!row_stride_ok(s.kv_stride, s.head_dim)) return SDLLM_ERR_INVALID_ARG;
  if (state == SDLLM_STATE_UPDATE && c.k_total > 0 && (!idx || !k_cache || !v_cache)) return SDLLM_ERR_INVALID_ARG;
  KvSegment a{k_in, v_in, s.kv_stride[0], s.kv_stride[1], s.kv_stride[2], s.seq_len};
  KvSegment b{nullptr, nullptr, 0, 0, 0, 0};
  AttnParams pending{};           // split-KV merge still to run (cache-update step only)
  pending.n_split = 1;
  const bool update = state == SDLLM_STATE_UPDATE && c.k_total > 0;
  AttnParams* defer = update && w.score_off > 0 ? &pending : nullptr;
  if (state == SDLLM_STATE_FULL || !w.fuse)
    st = run_attn(s, q_blk, a, b, out, ws, ws_bytes, (hipStream_t)stream, update, nullptr, 0, 0, defer);
  else {
    // cache-update step: the dense attention also leaves the scoring softmax's row statistics
    // ... and, where one workgroup owns a head, the saliency scores themselves (first buffer of the scoring workspace)
    st = run_attn(s, q_blk, a, b, out, ws, w.base, (hipStream_t)stream, update, (float*)((char*)ws + w.base), s.block_off, candidates_resume(s),
                  defer, w.fuse_cols ? (float*)((char*)ws + w.score_off) : nullptr, c.n_cand);
  }
  if (st != SDLLM_OK || state == SDLLM_STATE_FULL) return st;
  // from here on a pending merge must run whatever else fails: `out` is not complete without it
  auto finish_pending = [&](int32_t status) {
    if (pending.n_split > 1 && launch_attn_combine(pending, s.dtype, (hipStream_t)stream) != hipSuccess && status == SDLLM_OK)
      return (int32_t)SDLLM_ERR_HIP;
    return status;
  };
  if (!row_stride_ok(s.q_stride, s.head_dim)) return finish_pending(SDLLM_ERR_INVALID_ARG);
  st = score_select_impl(s, q_blk, k_in, idx, nullptr, nullptr, (char*)ws + w.score_off, w.base - w.score_off,
                         (hipStream_t)stream, w.fuse ? (float*)((char*)ws + w.base) : nullptr, w.stats_parts, true, w.fuse_cols);
  if (st != SDLLM_OK) return finish_pending(st);
  if (pending.n_split == 1) return sdllm_compact_kv(shape, k_in, v_in, idx, k_cache, v_cache, stream);
  CompactParams cp{};
  if ((st = compact_params(s, k_in, v_in, idx, k_cache, v_cache, cp)) != SDLLM_OK) return finish_pending(st);
  return launch_compact_combine(cp, pending, s.dtype, (hipStream_t)stream) == hipSuccess ? SDLLM_OK : SDLLM_ERR_HIP;
}

int32_t sdllm_dense_attn(const sdllm_shape_t* shape, const void* q_full, const int64_t* q_full_stride,
                         const void* k_full, const void* v_full, void* out_full, const int64_t* out_full_stride,
                         void* stream) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const sdllm_shape_t& s = *shape;
  if (!q_full || !k_full || !v_full || !out_full || !q_full_stride || !out_full_stride) return SDLLM_ERR_INVALID_ARG;
  if (!aligned16(q_full) || !aligned16(k_full) || !aligned16(v_full) || !aligned16(out_full)) return SDLLM_ERR_INVALID_ARG;
  const int es = elem_size(s.dtype);
  if (!strides_ok(q_full_stride, es) || !strides_ok(out_full_stride, es) || !row_stride_ok(q_full_stride, s.head_dim) ||
      !row_stride_ok(out_full_stride, s.head_dim) || !row_stride_ok(s.kv_stride, s.head_dim))
    return SDLLM_ERR_INVALID_ARG;
  const float scale_log2 = scale_of(s) * kLog2e;
  hipError_t e;
  if (dense_full_takes(s)) {
    DenseFullParams p{};
    p.q = q_full; p.k = k_full; p.v = v_full; p.out = out_full;
    p.q_sb = q_full_stride[0]; p.q_sh = q_full_stride[1]; p.q_sr = q_full_stride[2];
    p.k_sb = s.kv_stride[0]; p.k_sh = s.kv_stride[1]; p.k_sr = s.kv_stride[2];
    p.o_sb = out_full_stride[0]; p.o_sh = out_full_stride[1]; p.o_sr = out_full_stride[2];
    p.batch = s.batch; p.hq = s.n_q_heads; p.hkv = s.n_kv_heads; p.group = s.n_q_heads / s.n_kv_heads;
    p.seq_len = s.seq_len; p.d = s.head_dim;
    p.scale_log2 = scale_log2;
    e = launch_dense_full_mfma_bf16(p, (hipStream_t)stream);
  } else {
    AttnPlan pl{};
    plan_general(pl, s, s.seq_len, (s.seq_len + kTileKeys - 1) / kTileKeys, false);
    AttnParams p{};
    p.q = q_full; p.out = out_full;
    p.seg[0] = KvSegment{k_full, v_full, s.kv_stride[0], s.kv_stride[1], s.kv_stride[2], s.seq_len};
    p.seg[1] = KvSegment{nullptr, nullptr, 0, 0, 0, 0};
    p.q_sb = q_full_stride[0]; p.q_sh = q_full_stride[1]; p.q_sr = q_full_stride[2];
    p.o_sb = out_full_stride[0]; p.o_sh = out_full_stride[1]; p.o_sr = out_full_stride[2];
    p.batch = s.batch; p.hq = s.n_q_heads; p.hkv = s.n_kv_heads; p.group = s.n_q_heads / s.n_kv_heads;
    p.nq = s.seq_len; p.d = s.head_dim;
    p.scale_log2 = scale_log2;
    p.n_split = 1; p.tiles_per_split = pl.tiles_per_split; p.waves = pl.waves;
    e = launch_attn_general(p, s.dtype, false, (hipStream_t)stream);
  }
  return e == hipSuccess ? SDLLM_OK : SDLLM_ERR_HIP;
}

int32_t sdllm_launch_plan(const sdllm_shape_t* shape, int32_t call, int32_t n_cached, sdllm_launch_plan_t* plan) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const sdllm_shape_t& s = *shape;
  if (!plan || call < SDLLM_CALL_SPARSE || call > SDLLM_CALL_DENSE || n_cached < 0) return SDLLM_ERR_INVALID_ARG;
  *plan = sdllm_launch_plan_t{};
  if (call == SDLLM_CALL_DENSE && dense_full_takes(s)) {
    plan->kernel = SDLLM_KERNEL_DENSE;
    plan->key_splits = 1;
    plan->waves = kMaxWavesPerWg;
    plan->key_groups = dense_full_groups(s.batch * s.n_q_heads, s.seq_len).main;
    return SDLLM_OK;
  }
  AttnPlan pl{};
  if (call == SDLLM_CALL_SPARSE) pl = plan_streams(s, n_cached, s.cache_stride[2], s.block_len, s.blk_stride[2]);
  else if (call == SDLLM_CALL_DENSE) plan_general(pl, s, s.seq_len, (s.seq_len + kTileKeys - 1) / kTileKeys, false);
  else pl = plan_streams(s, s.seq_len, s.kv_stride[2], 0, 0, call == SDLLM_CALL_UPDATE && counts_of(s).k_total > 0);
  plan->kernel = !pl.mfma ? SDLLM_KERNEL_GENERAL : pl.gqa ? SDLLM_KERNEL_SHARED_TILE : pl.stream ? SDLLM_KERNEL_STREAM : SDLLM_KERNEL_PER_HEAD;
  plan->key_splits = pl.n_split;
  plan->waves = pl.waves;
  plan->touches_ahead = pl.stream && stream_touches_ahead(s.n_q_heads / s.n_kv_heads, pl.tiles_per_split, pl.waves);
  return SDLLM_OK;
}

int32_t sdllm_burst_splits(const sdllm_shape_t* shape, int32_t call, int32_t n_cached, int32_t* splits) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  const sdllm_shape_t& s = *shape;
  if (!splits || call < SDLLM_CALL_SPARSE || call > SDLLM_CALL_DENSE || n_cached < 0) return SDLLM_ERR_INVALID_ARG;
  AttnPlan pl;
  const bool taken = call == SDLLM_CALL_SPARSE ? plan_burst(pl, s, n_cached, s.cache_stride[2], s.block_len, s.blk_stride[2], SIZE_MAX)
                                               : call == SDLLM_CALL_FULL && plan_burst(pl, s, s.seq_len, s.kv_stride[2], 0, 0, SIZE_MAX);
  *splits = taken ? pl.n_split : 0;
  return SDLLM_OK;
}

int32_t sdllm_column_kernel(const sdllm_shape_t* shape, int32_t* kernel) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  if (!kernel) return SDLLM_ERR_INVALID_ARG;
  *kernel = plan_score(*shape).mfma ? SDLLM_COLUMNS_32 : blocks_as_heads(*shape) ? SDLLM_COLUMNS_BLOCKS : SDLLM_COLUMNS_GENERAL;
  return SDLLM_OK;
}

int32_t sdllm_dense_tail_groups(const sdllm_shape_t* shape, int32_t* groups) {
  const int32_t st = check_shape(shape);
  if (st != SDLLM_OK) return st;
  if (!groups) return SDLLM_ERR_INVALID_ARG;
  *groups = dense_full_takes(*shape) ? dense_full_groups(shape->batch * shape->n_q_heads, shape->seq_len).tail : 0;
  return SDLLM_OK;
}

int32_t sdllm_stream_read_probe(const void* src, size_t bytes, void* sink, void* stream) {
  if (!src || !aligned16(src)) return SDLLM_ERR_INVALID_ARG;
  return launch_stream_read(src, bytes, (uint32_t*)sink, (hipStream_t)stream) == hipSuccess ? SDLLM_OK : SDLLM_ERR_HIP;
}

}  // extern "C"
