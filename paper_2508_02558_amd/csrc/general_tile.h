// Per-tile building blocks of the general kernels (attn_general.hip, score_general.hip): a block of query rows
// against a 32-key tile for fp32 or bf16 tensors and head_dim 64 or 128, on the matrix cores.
//
// A wavefront addresses a row (of K, of Q) as 16-byte pieces: lane (col = lane % kRows, part = lane / kRows)
// holds pieces kParts * t + part of row `col`.  The order in which the head dimension is contracted is free,
// so the same pieces serve both types: a bf16 piece is one operand of v_mfma_f32_32x32x16_bf16 (32 query
// rows, 2 parts), an fp32 piece four operands of v_mfma_f32_16x16x4_f32 (16 query rows, 4 parts; exact fp32
// products and sums).  fp32 takes 16 rows because its matrix instructions are sixteen times slower: the
// chain a wave walks for one tile is half as long as with 32, and the registers of head_dim 128 still
// leave two waves per SIMD.
//   logits^T = K_tile Q^T: register i of a lane is key Ops::key(i, part) for query row `col`.
//   O^T += V_tile^T P^T: results 4u .. 4u+3 of a lane are four output columns from Ops::unit_col(u, part) on.
// fp32 probabilities throughout: with bf16 tensors they enter the second product as the sum of three bf16 parts, which
// together hold all 24 significand bits.  Against two parts, 16 bits, that takes 2 to 8 % more of a sparse step and 4 to 16 %
// more over all rows of a sequence (head_dim 64: 8 heads x 300 rows 5.9 -> 6.2 us, 2 x 8 x 1092 21.4 -> 23.5, 28 heads x 4000
// 260 -> 303), the last step of g_bf16_parts included.
#pragma once

#include "mfma_tile.h"

namespace sdllm {

typedef short gi16x4 __attribute__((ext_vector_type(4)));

template <typename T, int D>
struct Ops;

template <int D>
struct Ops<__bf16, D> {
  using Frag = bf16x8;
  using Acc = f32x16;
  static constexpr int kRows = kGeneralRowsBf16, kParts = 2;
  static constexpr int NS = 16;                          // logits per lane and tile
  static constexpr int NE = D / 32;                      // accumulators: MFMAs per step of the second product
  static constexpr int NACC = NE * 16;                   // results per lane
  static constexpr int NP = D / 16;                      // 16-byte pieces of a row per lane
  static constexpr int kRow = D * 2;                     // bytes of a row
  static constexpr int kKRow = kRow + 16;                // LDS row of a K (or Q) tile: an odd number of 16-byte pieces, so that
                                                         // sixteen rows' pieces of one column lie on different banks
  static constexpr int kVRow = kRow + 64;                // LDS row of a V tile: four rows x 64 bytes of a transposing read on 64 banks
  static constexpr int kKTile = kTileKeys * kKRow;
  static constexpr int kVTile = kTileKeys * kVRow;
  static constexpr int kLoads = kRow / 32;               // 16-byte loads per lane and tensor tile
  struct V { u32x4 r[kLoads]; };                         // a V tile on its way to LDS

  static __device__ __forceinline__ int key(int i, int part) { return 8 * (i >> 2) + 4 * part + (i & 3); }
  static __device__ __forceinline__ int flat(int e, int i) { return e * 16 + i; }   // position of register (e, i) among a lane's results
  static __device__ __forceinline__ int unit_col(int u, int part) { return 32 * (u >> 2) + 8 * (u & 3) + 4 * part; }

  // s = rows of an LDS tile x `fixed`
  static __device__ __forceinline__ void logits(const uint8_t* tile, const Frag (&fixed)[NP], int col, int part, float (&s)[NS]) {
    Frag a[NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) a[t] = *reinterpret_cast<const Frag*>(tile + col * kKRow + (t * 2 + part) * 16);
    Acc c;
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
    for (int t = 0; t < NP; ++t) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], fixed[t], c, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = c[i];
  }

  // Scoring, operands swapped: one 32-row block of queries in LDS x a key tile held as fragments.  Register
  // i: query row key(i, part), candidate col.
  struct KTile { Frag f[NP]; };
  static constexpr int kKeysPerLane = 1;
  static __device__ __forceinline__ void load_keys(const uint8_t* tile, int col, int part, KTile& k) {
#pragma unroll
    for (int t = 0; t < NP; ++t) k.f[t] = *reinterpret_cast<const Frag*>(tile + col * kKRow + (t * 2 + part) * 16);
  }
  static __device__ __forceinline__ void score(const uint8_t* queries, const KTile& k, int col, int part, float (&s)[NS]) {
    logits(queries, k.f, col, part, s);
  }
  static __device__ __forceinline__ int query(int i, int part) { return key(i, part); }
  static __device__ __forceinline__ int key_slot(int) { return 0; }          // which of the lane's keys register i belongs to
};

template <int D>
struct Ops<float, D> {
  using Frag = f32x4;
  using Acc = f32x4;
  static constexpr int kRows = kGeneralRowsF32, kParts = 4;
  static constexpr int NS = 8;
  static constexpr int NE = D / 16;
  static constexpr int NACC = NE * 4;
  static constexpr int NP = D / 16;
  static constexpr int kRow = D * 4;
  static constexpr int kKRow = kRow + 16;
  static constexpr int kKTile = kTileKeys * kKRow;
  static constexpr int kVTile = 0;                       // V operands come straight from memory
  static constexpr int kLoads = kRow / 32;
  struct V { f32x4 r[NS][NE / 4]; };                     // register i: key row key(i, part), columns 64c + 4 col .. + 3

  static __device__ __forceinline__ int key(int i, int part) { return 16 * (i >> 2) + 4 * part + (i & 3); }
  // lane m feeds columns 64c + 4m + e' to MFMA 4c + e': register (e, i) is column 64 (e/4) + 4 (4 part + i) + e%4
  static __device__ __forceinline__ int flat(int e, int i) { return (e >> 2) * 16 + i * 4 + (e & 3); }
  static __device__ __forceinline__ int unit_col(int u, int part) { return 64 * (u >> 2) + 16 * part + 4 * (u & 3); }

  static __device__ __forceinline__ void logits(const uint8_t* tile, const Frag (&fixed)[NP], int col, int part, float (&s)[NS]) {
    Frag a[2][NP];
    Acc c[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < NP; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) a[h][t] = *reinterpret_cast<const Frag*>(tile + (16 * h + col) * kKRow + (t * 4 + part) * 16);
#pragma unroll
    for (int t = 0; t < NP; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) c[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][t][i], fixed[t][i], c[h], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = c[i >> 2][i & 3];
  }

  // Register i: query row 4 part + i%4, candidate 16 (i/4) + col.
  struct KTile { Frag f[2][NP]; };
  static constexpr int kKeysPerLane = 2;
  static __device__ __forceinline__ void load_keys(const uint8_t* tile, int col, int part, KTile& k) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < NP; ++t) k.f[h][t] = *reinterpret_cast<const Frag*>(tile + (16 * h + col) * kKRow + (t * 4 + part) * 16);
  }
  static __device__ __forceinline__ void score(const uint8_t* queries, const KTile& k, int col, int part, float (&s)[NS]) {
    Acc c[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const Frag q = *reinterpret_cast<const Frag*>(queries + col * kKRow + (t * 4 + part) * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) c[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[i], k.f[h][t][i], c[h], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = c[i >> 2][i & 3];
  }
  static __device__ __forceinline__ int query(int i, int part) { return 4 * part + (i & 3); }
  static __device__ __forceinline__ int key_slot(int i) { return i >> 2; }
};

// A value of a row over the lanes that share it (the parts of a row sit kRows lanes apart).
template <typename O, typename F>
__device__ __forceinline__ float over_parts(float v, const F& f) {
#pragma unroll
  for (int o = O::kRows; o < kWave; o <<= 1) v = f(v, __shfl_xor(v, o));
  return v;
}
template <typename O>
__device__ __forceinline__ float parts_max(float v) { return over_parts<O>(v, [](float a, float b) { return fmaxf(a, b); }); }
template <typename O>
__device__ __forceinline__ float parts_sum(float v) { return over_parts<O>(v, [](float a, float b) { return a + b; }); }

// Rows [0, rows) of a tile, `stride` bytes apart, as 16-byte pieces (whole rows per group of lanes).  Rows
// past the end re-read the last one (ZERO: are zero).
template <typename O, bool ZERO>
__device__ __forceinline__ void g_load_rows(const char* base, int rows, int64_t stride, int lane, u32x4 (&reg)[O::kLoads]) {
  constexpr int kPerRow = O::kRow / 16, kRowsPerLoad = kWave / kPerRow;
  const int c = lane % kPerRow, r0 = lane / kPerRow;
#pragma unroll
  for (int j = 0; j < O::kLoads; ++j) {
    const int r = j * kRowsPerLoad + r0;
    const u32x4 v = *reinterpret_cast<const u32x4*>(base + (int64_t)min(r, rows - 1) * stride + c * 16);
    reg[j] = ZERO && r >= rows ? u32x4{0u, 0u, 0u, 0u} : v;
  }
}

template <typename O>
__device__ __forceinline__ void g_store_rows(uint8_t* tile, int row_bytes, int lane, const u32x4 (&reg)[O::kLoads]) {
  constexpr int kPerRow = O::kRow / 16, kRowsPerLoad = kWave / kPerRow;
#pragma unroll
  for (int j = 0; j < O::kLoads; ++j)
    *reinterpret_cast<u32x4*>(tile + (j * kRowsPerLoad + lane / kPerRow) * row_bytes + (lane % kPerRow) * 16) = reg[j];
}

// This lane's pieces of one row in memory.
template <typename O>
__device__ __forceinline__ void g_row_pieces(const void* row, int part, typename O::Frag (&f)[O::NP]) {
#pragma unroll
  for (int t = 0; t < O::NP; ++t)
    f[t] = *reinterpret_cast<const typename O::Frag*>((const char*)row + (t * O::kParts + part) * 16);
}

// V tile: requested from memory (g_v_load), made readable (g_v_publish: bf16 only), multiplied (g_pv).  Rows
// past the end are zero, so that a probability of zero meets no infinity there.
template <int D>
__device__ __forceinline__ void g_v_load(const char* base, int rows, int64_t stride, int lane, typename Ops<__bf16, D>::V& v) {
  g_load_rows<Ops<__bf16, D>, true>(base, rows, stride, lane, v.r);
}
template <int D>
__device__ __forceinline__ void g_v_load(const char* base, int rows, int64_t stride, int lane, typename Ops<float, D>::V& v) {
  using O = Ops<float, D>;
  const int part = lane / O::kRows, col = lane % O::kRows;
#pragma unroll
  for (int i = 0; i < O::NS; ++i) {
    const int r = O::key(i, part);
    const char* at = base + (int64_t)min(r, rows - 1) * stride + col * 16;
#pragma unroll
    for (int c = 0; c < O::NE / 4; ++c) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(at + c * 256);
      v.r[i][c] = r < rows ? x : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
}

template <int D>
__device__ __forceinline__ void g_v_publish(uint8_t* tile, int lane, const typename Ops<__bf16, D>::V& v) {
  g_store_rows<Ops<__bf16, D>>(tile, Ops<__bf16, D>::kVRow, lane, v.r);
}
template <int D>
__device__ __forceinline__ void g_v_publish(uint8_t*, int, const typename Ops<float, D>::V&) {}

// Eight probabilities as the sum of three bf16 operands.  Each part is what the one before left, cut off after eight
// bits instead of rounded: the sum is exact, and no part of a positive value is negative.  None is zero either (2^-126
// takes its place), so that an infinity in V stays one: 0 to 5 % of a call.  Finding out afterwards that a result is no
// number and walking the tiles once more costs small calls as much (the second loop's instructions have to be fetched), a
// branch around the instructions 5 to 40 % (scratch at head_dim 128).
__device__ __forceinline__ void g_bf16_parts(const float* p, bf16x8 (&part)[3]) {
  u32x4 out[3];
  const auto cut = [](float x) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & 0xffff0000u); };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float x[2] = {p[2 * j], p[2 * j + 1]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      out[k][j] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, x[1]), __builtin_bit_cast(uint32_t, x[0]), 0x07060302u);
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = __builtin_amdgcn_fmed3f(x[i] - cut(x[i]), x[i], 0x1p-126f);   // zero stays zero
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) part[k] = __builtin_bit_cast(bf16x8, out[k]);
}

// bf16: V^T operands through the transposing LDS read (lane s of a 16-lane group points at key row s/4 and
// column piece s%4 and receives four consecutive keys of one column)
template <int D>
__device__ __forceinline__ void g_pv(const uint8_t* tile, const typename Ops<__bf16, D>::V&, const float (&p)[16], int lane,
                                     f32x16 (&acc)[D / 32]) {
  using O = Ops<__bf16, D>;
  typedef __attribute__((address_space(3))) gi16x4 lds_i16x4;
  const int part = lane >> 5, grp = (lane >> 4) & 1, s16 = lane & 15;
  const uint8_t* base = tile + (part * 4 + (s16 >> 2)) * O::kVRow + (grp * 16 + (s16 & 3) * 4) * 2;
  bf16x8 av[2][O::NE];
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int e = 0; e < O::NE; ++e) {
      const gi16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(base + st * 16 * O::kVRow + e * 64));
      const gi16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(base + (st * 16 + 8) * O::kVRow + e * 64));
      av[st][e] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
    }
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    bf16x8 parts[3];
    g_bf16_parts(p + st * 8, parts);
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int e = 0; e < O::NE; ++e) acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[st][e], parts[k], acc[e], 0, 0, 0);
  }
}
// fp32: step i contracts the four keys that the parts of a row hold in register i
template <int D>
__device__ __forceinline__ void g_pv(const uint8_t*, const typename Ops<float, D>::V& v, const float (&p)[8], int, f32x4 (&acc)[D / 16]) {
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int e = 0; e < D / 16; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v.r[i][e >> 2][e & 3], p[i], acc[e], 0, 0, 0);
}

}  // namespace sdllm
