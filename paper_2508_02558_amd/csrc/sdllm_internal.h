// Internal declarations shared by the C-ABI dispatcher and the kernel launchers.
// Nothing here is exported; the public surface is include/sdllm.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace sdllm {

constexpr int kWave = 64;            // CDNA wavefront
constexpr int kTileKeys = 32;        // keys per MFMA tile (one 32x32 block of logits)
constexpr int kMaxWavesPerWg = 8;    // attention / scoring workgroups hold up to 8 waves
constexpr int kNumCUs = 256;         // MI355X
constexpr int kNumXCDs = 8;
// query rows per workgroup of the general kernels (general_tile.h), also of the 32-row bf16 kernels
constexpr int kGeneralRowsBf16 = 32, kGeneralRowsF32 = 16;
constexpr int kGeneralMaxWaves = 8;
inline int block_rows(int dtype) { return dtype == 0 ? kGeneralRowsBf16 : kGeneralRowsF32; }

// Workgroup ids are dealt round-robin over the 8 XCDs, each with its own L2.  This renumbering gives
// every XCD one contiguous range of the result instead (XCD x gets the ids it was dealt, in order,
// placed after those of the XCDs before it), for any grid size, so that neighbours in the new
// numbering - the query heads of a KV group, the key splits of a head - share an L2.
__host__ __device__ inline int xcd_contiguous_id(int dealt, int n) {
  const int x = dealt % kNumXCDs, q = n / kNumXCDs, r = n % kNumXCDs;
  return x * q + (x < r ? x : r) + dealt / kNumXCDs;
}

// Exact n / d of 0 <= n < 2^31 by a d in [1, 2^31) that the host knows: with 2^(l-1) < d <= 2^l and mul = ceil(2^(31+l) / d), that is
// 2^(31+l) / d plus less than 1, n mul / 2^(31+l) exceeds n / d by less than n / 2^(31+l), and so by less than 1 / d.  Three scalar
// instructions where the compiler's division by a kernel parameter is some thirty vector ones in a chain.  In front of a kernel's
// first load that is worth 1 to 4 % of calls of 6 to 14 us (general fp32 kernels 13.4 -> 13.1, full-sequence attention of
// 28 heads x 100 positions 6.8 -> 6.7).  Not so in attn_mfma.hip, 2 to 5 % slower with it (28 heads x 69 tiles 10.2 -> 10.4,
// 256 x 8 8.8 -> 9.2), in the general bf16 kernels, 3 % slower to 2 % faster, and level in the other two kernels of block queries:
// they divide as the compiler does.
struct Divisor {
  uint32_t mul, shift;
  Divisor() = default;
  constexpr explicit Divisor(uint32_t d) : mul(0), shift(31) {
    while (((uint64_t)1 << (shift - 31)) < d) ++shift;
    mul = (uint32_t)((((uint64_t)1 << shift) + d - 1) / d);
  }
  __host__ __device__ constexpr int quotient(int n) const { return (int)(((uint64_t)(uint32_t)n * mul) >> shift); }
};
static_assert(Divisor(1).quotient(INT32_MAX) == INT32_MAX && Divisor(7).quotient(48) == 6 && Divisor(7).quotient(49) == 7 &&
                  Divisor(3).quotient(INT32_MAX) == INT32_MAX / 3 && Divisor(INT32_MAX).quotient(INT32_MAX - 1) == 0 &&
                  Divisor(INT32_MAX).quotient(INT32_MAX) == 1 && Divisor(1 << 30).quotient(INT32_MAX) == 1,
              "exact at the ends");

// Kernels that need more than the default 64 KB of dynamic LDS have to opt in, once per device (the
// attribute belongs to the device's copy of the kernel).  One object per kernel remembers which
// devices are done; concurrent host threads at worst both set the same value.
class LdsOptIn {
 public:
  hipError_t ensure(const void* kernel, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool tracked = dev >= 0 && dev < 64;
    const uint64_t bit = tracked ? uint64_t{1} << dev : 0;
    if (tracked && (done_.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && tracked) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

template <class T> struct AsIs { using type = T; };

// Launches a kernel.  hipLaunchKernelGGL goes through a pushed and popped launch configuration and takes 2.5 us of the host, this 2.25;
// arguments are converted to the kernel's own parameter types.  An error is returned and not left for the next call to find.
template <class... P>
hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s, const typename AsIs<P>::type&... args) {
  void* at[] = {const_cast<void*>(static_cast<const void*>(&args))...};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, at, lds_bytes, s);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

// One source of keys/values: rows of a [B, Hkv, n, d] tensor given by element strides.
struct KvSegment {
  const void* k;
  const void* v;
  int64_t sb, sh, sr;  // element strides: batch, head, row
  int32_t n;           // rows per (batch, head)
};

// Attention of nq query rows per head over Concat(seg[0], seg[1]) (Alg. 3, state 2; with a
// single full-sequence segment it is the dense block-row attention of states 0/1).
struct AttnParams {
  const void* q;
  void* out;
  KvSegment seg[2];
  int64_t q_sb, q_sh, q_sr;
  int64_t o_sb, o_sh, o_sr;
  int32_t batch, hq, hkv, group, nq, d;
  float scale_log2;     // softmax scale * log2(e)
  // split-KV plan
  int32_t n_split;          // workgroups per head
  int32_t tiles_per_split;  // 32-key tiles each workgroup owns
  int32_t waves;            // waves per workgroup
  // per block of R query rows (R = block_rows(dtype), N = ceil(nq / R) blocks per head, one for the 32-row kernels):
  float* part_o;            // [B*Hq, N, n_split, R, d] fp32 partial numerators (n_split > 1)
  float* part_ml;           // [B*Hq, N, n_split, 2, R] running max (log2 domain) and denominator
  // Optional by-product of a dense (single-segment) launch: the softmax row statistics of the
  // scoring pass, i.e. (max, sum) per query row over the CANDIDATE keys only, which are the keys
  // outside [cand0_end, cand1_begin).  Layout [B*Hq, N, n_split, 2, R], the layout the scoring
  // kernels read their partial statistics in.  Null: not produced.
  float* cand_ml;
  int32_t cand0_end, cand1_begin;
  // Optional second by-product of such a launch (one workgroup per head, no key splits, MHA): the
  // softmax-mean saliency score of every candidate key (Alg. 1 steps 5-6), [B*Hkv, score_stride] floats,
  // written by a second sweep over K that each workgroup runs once its row statistics are final.
  // Null: not produced.
  float* score_out;
  int32_t score_stride;
  float score_inv_count;    // 1 / (block queries x query heads per KV head)
};

// Scoring of the candidates K_f = Concat[K_{:o}, K_{o+b:}] against the block's queries.
struct ScoreParams {
  const void* q;
  const void* k;        // full-sequence keys
  int64_t q_sb, q_sh, q_sr;
  int64_t k_sb, k_sh, k_sr;
  int32_t batch, hq, hkv, group, nq, d;
  int32_t q_shift;      // kernels for blocks of 32 rows: 1 if hq and group count blocks, two to a head of 33 to 64 query rows; else 0
  float inv_count;      // 1 / (query rows x heads of a group)
  int32_t block_off, block_len;
  int32_t n_cand;       // candidates scored (N, or N_pre for prefix-only eviction)
  int32_t softmax;      // 1: SOFTMAX_MEAN, 0: LOGIT_MEAN
  float scale;          // softmax scale
  float scale_log2;     // scale * log2(e)
  float* score;         // [B*Hkv, score_stride], the first n_cand of each row written
  int32_t score_stride;
  // row statistics of the softmax (pass 1 -> pass 2)
  int32_t n_part;       // workgroups per (batch, KV head) row of the scoring kernels
  int32_t tiles_per_part;
  float* part_ml;       // [B*Hq, N, n_stat_part, 2, R]
  int32_t n_stat_part;  // partial (max, sum) pairs per query row in part_ml
  int32_t skip_stats;   // 1: part_ml was already filled (by the dense attention of the same step)
  int32_t in_step;      // 1: between the other launches of a cache-update step
  Divisor by_hkv;
  int32_t cols_follow;  // set by the launcher: the statistics kernel runs the column pass itself (n_part == 1)
  int32_t waves;
};

struct SelectParams {
  const float* score;   // [rows, n_cand]
  float* pooled;        // optional [rows, n_cand]: the pooled scores (only when the caller wants them)
  int32_t* idx;         // [rows, k_total]
  int32_t rows;         // B * Hkv
  int32_t n_cand;
  int32_t n_seg;        // 1 or 2 ranked segments
  int32_t seg_begin[2], seg_len[2], seg_k[2], seg_out[2];
  int32_t k_total;
  int32_t pool_half;    // (s-1)/2
  int32_t avg_pool;
  int32_t block_off, block_len;
  // candidates appended unconditionally after the ranked ones (prefix-only eviction keeps the
  // whole suffix): candidate indices [tail_begin, tail_begin + tail_len)
  int32_t tail_begin, tail_len, tail_out;
  // workspace of the path for segments too long for one workgroup (sizes: select_workspace()), else null
  uint32_t* keys;       // [rows, n_cand] order-preserving integer image of the pooled scores, in position order
  uint32_t* sorted;     // [rows, n_cand] the same keys, every chunk of 1024 ordered by leading bits
  uint32_t* bins;       // [rows, 2, chunks] lists of the non-empty leading-bit bins of every chunk
  int32_t chunks;       // set by the launcher: chunks of the longest ranked segment
};

struct SelectWorkspace { size_t keys, sorted, bins; };   // in 32-bit words

struct CompactParams {
  const void* k;
  const void* v;
  const int32_t* idx;
  void* kc;
  void* vc;
  int64_t s_sb, s_sh, s_sr;  // source strides in BYTES
  int64_t c_sb, c_sh, c_sr;  // cache strides in BYTES
  int32_t batch, hkv, k_total, seq_len;
  int32_t row_bytes;
  Divisor by_hkv, by_row_blocks;   // set by the launcher: KV heads, blocks per row of the index set
  int32_t row_blocks, first_block;
};

// Full-sequence bidirectional attention: L query rows per head over all L keys.
struct DenseFullParams {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  int64_t q_sb, q_sh, q_sr;
  int64_t k_sb, k_sh, k_sr;
  int64_t o_sb, o_sh, o_sr;
  int32_t batch, hq, hkv, group, seq_len, d;
  float scale_log2;
  int32_t qblocks, first_wg;              // set by the launcher: workgroups per head, number of the first one
  Divisor by_qblocks, by_hq, by_group;
};

// kernel launchers (each returns hipGetLastError() after its launches)
hipError_t launch_attn_mfma_bf16(const AttnParams& p, hipStream_t s);
hipError_t launch_attn_gqa_mfma_bf16(const AttnParams& p, hipStream_t s);
hipError_t launch_attn_stream_mfma_bf16(const AttnParams& p, hipStream_t s);
constexpr int kBurstMaxTiles = 9;    // tiles per workgroup of the next: 9 x 16.75 KB and the query rows fill the 160 KB of LDS
hipError_t launch_attn_burst_mfma_bf16(const AttnParams& p, hipStream_t s);   // no statistics, no scores
// Touching tiles ahead (attn_stream_mfma.hip) pays from about a dozen tiles per wave on (8 x 28/4 heads: 144 tiles 36.0 -> 34.3 us,
// 74 tiles 19.8 -> 20.8) and for groups that share the requests out thinly (6 x 32/8 heads x 243 tiles, every fourth tile
// each: 70.1 -> 71.6 us).
inline bool stream_touches_ahead(int group, int tiles_per_split, int waves) { return group >= 7 && tiles_per_split >= 12 * waves; }
bool attn_gqa_supports_group(int group);
int attn_gqa_waves_per_wg(int group);
// any type, head_dim and row count; stats_only: nothing but cand_ml
hipError_t launch_attn_general(const AttnParams& p, int dtype, bool stats_only, hipStream_t s);
hipError_t launch_attn_combine(const AttnParams& p, int dtype, hipStream_t s);
hipError_t launch_score_mfma_bf16(const ScoreParams& p, hipStream_t s);
bool score_mfma_supports_group(int group);
hipError_t launch_score_cols_general(const ScoreParams& p, int dtype, hipStream_t s);   // part_ml filled before (softmax)
hipError_t launch_select(const SelectParams& p, hipStream_t s);
SelectWorkspace select_workspace(const SelectParams& p);
int select_max_segment();
hipError_t launch_compact(const CompactParams& p, hipStream_t s);
// the gather plus the split-KV merge of an attention launch whose partials are still in the workspace
hipError_t launch_compact_combine(const CompactParams& p, const AttnParams& a, int dtype, hipStream_t s);
hipError_t launch_dense_full_mfma_bf16(const DenseFullParams& p, hipStream_t s);
// Key groups that its workgroups are divided into: all of them, or all but those of a last round that is a launch of its own (tail: that
// one's groups, 0 without it).
struct DenseFullGroups { int main, tail; };
DenseFullGroups dense_full_groups(int heads, int seq_len);
hipError_t launch_stream_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t s);

}  // namespace sdllm
