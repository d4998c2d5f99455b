// Gather-compaction of the retained K/V rows into the dense sparse cache (Sec. 3.3 fourth
// equation; Alg. 1 steps 12-14).  Pure byte movement: each thread copies one 16-byte chunk of two
// consecutive cache rows of K and of V, so a wavefront reads and writes whole rows with 16-byte
// non-temporal accesses and has 4 loads in flight per lane (more in flight measured slower).
//
// At the cache-update step of a shape whose dense attention was split over the keys, the merge of those
// splits has nothing to do with the gather and is only needed once the step returns: one launch then
// runs both (compact_combine_kernel: the first blocks merge, the rest copy), which saves a launch
// boundary and hides the merge under the copy.
#include "attn_merge.h"
#include "sdllm_internal.h"

namespace sdllm {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr int kRowsPerThread = 2;
constexpr int kCompactThreads = 256;
static_assert(kCompactThreads == kCombineThreads, "the fused launch runs both bodies with one block size");

// Rows of the index set that a block copies
inline int compact_rows(const CompactParams& p) { return kRowsPerThread * kCompactThreads / (p.row_bytes >> 4); }

// Block block_id of [batch, KV head] x row_blocks: no thread divides.  Two 64-bit divisions of indexes stood in front of a thread's
// loads; with the merge of 8 splits, 4 KV heads x 2160 rows 3.4 -> 2.85 us, x 8320 rows 7.3 -> 6.8 (kernel trace); the 256 x 2160 rows
// of a batch are bound by memory either way.
__device__ __forceinline__ void compact_block(const CompactParams& p, int block_id) {
  const int bg = p.by_row_blocks.quotient(block_id), b = p.by_hkv.quotient(bg), g = bg - b * p.hkv;
  const int shift = __builtin_ctz(p.row_bytes) - 4;   // a row is 8, 16 or 32 chunks of 16 bytes
  const int c16 = (threadIdx.x & ((1 << shift) - 1)) << 4;
  const int j0 = ((block_id - bg * p.row_blocks) * (kCompactThreads >> shift) + (threadIdx.x >> shift)) * kRowsPerThread;
  if (j0 >= p.k_total) return;
  const int* idx = p.idx + (int64_t)bg * p.k_total;

  const char* src_k[kRowsPerThread]; const char* src_v[kRowsPerThread];
  char* dst_k[kRowsPerThread]; char* dst_v[kRowsPerThread];
  bool ok[kRowsPerThread];
#pragma unroll
  for (int u = 0; u < kRowsPerThread; ++u) {
    ok[u] = j0 + u < p.k_total;
    const int j = min(j0 + u, p.k_total - 1);
    int pos = idx[j];
    pos = min(max(pos, 0), p.seq_len - 1);   // never leave the source tensor, whatever idx holds
    const int64_t so = b * p.s_sb + g * p.s_sh + (int64_t)pos * p.s_sr + c16;
    const int64_t co = b * p.c_sb + g * p.c_sh + (int64_t)j * p.c_sr + c16;
    src_k[u] = (const char*)p.k + so; src_v[u] = (const char*)p.v + so;
    dst_k[u] = (char*)p.kc + co; dst_v[u] = (char*)p.vc + co;
  }
  u32x4 kv[kRowsPerThread], vv[kRowsPerThread];
#pragma unroll
  for (int u = 0; u < kRowsPerThread; ++u) {
    kv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src_k[u]));
    vv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src_v[u]));
  }
#pragma unroll
  for (int u = 0; u < kRowsPerThread; ++u) {
    if (ok[u]) {
      __builtin_nontemporal_store(kv[u], reinterpret_cast<u32x4*>(dst_k[u]));
      __builtin_nontemporal_store(vv[u], reinterpret_cast<u32x4*>(dst_v[u]));
    }
  }
}

__global__ __launch_bounds__(kCompactThreads) void compact_kernel(const CompactParams p) { compact_block(p, p.first_block + (int)blockIdx.x); }

// blocks [0, n_combine): split-KV merge of the attention described by `a` (output of type T); the rest: the gather.
// MAX > 0: combine32_block, else combine_block with TPI threads per item
template <typename T, int TPI, int MAX>
__global__ __launch_bounds__(kCompactThreads) void compact_combine_kernel(const CompactParams p, const AttnParams a,
                                                                          const Divisor by_hq, const int n_combine) {
  if ((int)blockIdx.x < n_combine) {
    if constexpr (MAX > 0) {
      const int head = blockIdx.x >> 2, b = by_hq.quotient(head);
      combine32_block<MAX>(a, b, head - b * a.hq, blockIdx.x & 3);
    } else {
      combine_block<T, TPI>(a, blockIdx.x);
    }
  } else {
    compact_block(p, (int)blockIdx.x - n_combine);
  }
}

// Blocks of the gather, whose split over the grid is left in p
static int64_t plan_compact(CompactParams& p) {
  const int per_block = compact_rows(p);
  p.row_blocks = (p.k_total + per_block - 1) / per_block;
  p.by_row_blocks = Divisor(p.row_blocks > 0 ? p.row_blocks : 1);
  p.by_hkv = Divisor(p.hkv);
  return (int64_t)p.batch * p.hkv * p.row_blocks;
}

// A launch has fewer than 2^32 threads.  With few rows per (batch, KV head), a block or a part of one for each, the blocks can be more.
constexpr int64_t kMostBlocks = UINT32_MAX / kCompactThreads;

static hipError_t launch_blocks(CompactParams& p, int64_t first, int64_t blocks, hipStream_t s) {
  for (; first < blocks; first += kMostBlocks) {
    p.first_block = (int)first;
    const hipError_t e = launch(compact_kernel, dim3((unsigned)(blocks - first < kMostBlocks ? blocks - first : kMostBlocks)), dim3(kCompactThreads), 0, s, p);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_compact(const CompactParams& p, hipStream_t s) {
  CompactParams c = p;
  const int64_t blocks = plan_compact(c);
  return blocks > INT32_MAX ? hipErrorInvalidValue : launch_blocks(c, 0, blocks, s);
}

hipError_t launch_compact_combine(const CompactParams& p, const AttnParams& a, int dtype, hipStream_t s) {
  const bool four = combine_tpi(a.n_split) == 4;
  if (dtype != 0 && four) return hipErrorInvalidValue;   // fp32 has plan_general's splits, eight at most
  return with_combine32(a, dtype, [&](auto max) {
    constexpr int MAX = decltype(max)::value;
    const int64_t n_combine = MAX > 0 ? (int64_t)4 * a.batch * a.hq : combine_blocks(a);
    CompactParams c = p;
    const int64_t blocks = plan_compact(c);
    if (blocks > INT32_MAX || n_combine > kMostBlocks) return hipErrorInvalidValue;
    const int64_t beside = blocks < kMostBlocks - n_combine ? blocks : kMostBlocks - n_combine;   // of the gather in the merge's launch
    const auto kernel = [&] {
      if constexpr (MAX > 0) return compact_combine_kernel<__bf16, 1, MAX>;
      else return dtype != 0 ? compact_combine_kernel<float, 1, 0> : four ? compact_combine_kernel<__bf16, 4, 0> : compact_combine_kernel<__bf16, 1, 0>;
    }();
    const hipError_t e = launch(kernel, dim3((unsigned)(n_combine + beside)), dim3(kCompactThreads), 0, s, c, a, Divisor(a.hq), (int)n_combine);
    return e == hipSuccess ? launch_blocks(c, beside, blocks, s) : e;
  });
}

}  // namespace sdllm
