// Device helpers shared by the bf16 MFMA kernels: vector types, the padded LDS tile layout and the
// coalesced 32-key tile load.
#pragma once

#include "sdllm_internal.h"

namespace sdllm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
// native vectors (not the HIP uint4 struct) so that register arrays of them are promoted to VGPRs
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kRowBytes = 256 + 16;               // 128 bf16 + one 16-byte pad: rows rotate over the banks
constexpr int kTileBytes = kTileKeys * kRowBytes; // one 32 x 128 bf16 tile in LDS

// V tiles use 320-byte rows: the transposing LDS read of the PV product touches four consecutive
// rows x 64 bytes per 32 lanes, and a row offset of 64 bytes (mod 256) puts those on 64 distinct banks.
constexpr int kVRowBytes = 256 + 64;
constexpr int kVTileBytes = kTileKeys * kVRowBytes;

__device__ __forceinline__ uint32_t vtile_off(int row, int chunk) { return (uint32_t)(row * kVRowBytes + (chunk << 4)); }

__device__ __forceinline__ uint32_t tile_off(int row, int chunk) {
  // padded rows: the sixteen lanes that read one chunk column of sixteen rows hit sixteen different
  // 16-byte bank groups, and every address is a per-lane base plus a compile-time constant
  return (uint32_t)(row * kRowBytes + (chunk << 4));
}

// Rows [0, rows) of a tile starting at `base` (wave-uniform), `stride` bytes apart: lane l loads the
// 16-byte chunk l%16 of rows l/16, l/16 + 4, ...  Rows past the end re-read the last valid row.
// NT: non-temporal loads for data that is streamed once per launch (they keep the tiles from
// displacing reusable lines in L2/MALL and measured ~12 % faster on MI355X); plain loads when sibling
// workgroups re-read the same rows (query heads of one KV group served by separate workgroups).
// A full tile (the common case, wave-uniform test) is addressed as base + j * (4 rows) (scalar) plus ONE
// per-lane offset, so the eight loads cost the vector ALU one multiply and eight adds instead of
// eight clamps, eight multiplies and eight adds (with two such calls per tile the address arithmetic
// was half of the vector-ALU time of an attention tile).
template <bool NT = true>
__device__ __forceinline__ void load_rows(const char* base, int rows, uint32_t stride, int lane, u32x4 (&reg)[8]) {
  const uint32_t c16 = (lane & 15) << 4;
  if (rows == kTileKeys) {
    const uint32_t lane_off = (uint32_t)(lane >> 4) * stride + c16;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const u32x4* src = reinterpret_cast<const u32x4*>(base + (size_t)(j * 4) * stride + lane_off);
      reg[j] = NT ? __builtin_nontemporal_load(src) : *src;
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    int r = j * 4 + (lane >> 4);
    r = r < rows ? r : rows - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(base + (uint32_t)r * stride + c16);
    reg[j] = NT ? __builtin_nontemporal_load(src) : *src;
  }
}

__device__ __forceinline__ void store_rows(uint8_t* lds_tile, int lane, const u32x4 (&reg)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j)
    *reinterpret_cast<u32x4*>(lds_tile + tile_off(j * 4 + (lane >> 4), lane & 15)) = reg[j];
}

__device__ __forceinline__ void store_rows_v(uint8_t* lds_tile, int lane, const u32x4 (&reg)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j)
    *reinterpret_cast<u32x4*>(lds_tile + vtile_off(j * 4 + (lane >> 4), lane & 15)) = reg[j];
}

// ---- tiles that several waves share, fetched straight into LDS
// A tile lies there as eight groups of four rows (r, r + 8, r + 16, r + 24 in group r), each as one fetch instruction
// leaves it, the groups a little more than 1 KB apart: the operand reads then need one lane address per tensor plus constants,
// and meet no bank conflict (K: eight rows 32 bytes apart modulo 256, the 16-byte chunks of two rows of a group swapped;
// V: four rows 64 bytes apart).
constexpr int kKGroup = 1024 + 32, kVGroup = 1024 + 64;
constexpr int kRingK = 8 * kKGroup, kRingV = 8 * kVGroup;   // one tile

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is a reserved register: named so that no use of it is moved across
// 64 lanes x 16 bytes from base + off to 1 KB of LDS at `at` (an LDS byte address; it and base wave-uniform).  In assembly because with
// the builtin the compiler makes every LDS read wait for all fetches in flight; the caller counts the requests.  m0 holds the
// LDS address.
__device__ __forceinline__ void fetch_to_lds(uint32_t at, const char* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(at), "v"(off), "s"(base) : "memory", "m0");
}
// The same from an address per lane.
__device__ __forceinline__ void fetch_to_lds(uint32_t at, const char* lane_src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(at), "v"(lane_src) : "memory", "m0");
}
#pragma clang diagnostic pop
// A wave-uniform address in scalar registers, where the compiler would keep it in vector registers.
__device__ __forceinline__ const char* in_scalars(const char* p) {
  const uint64_t a = (uint64_t)p;
  return (const char*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32);
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  typedef __attribute__((address_space(3))) const uint8_t lds_u8;
  return (uint32_t)(uintptr_t)(lds_u8*)p;
}
// Which 16 bytes of its row a lane of a fetch brings, and where a lane's operands of a tile begin (K operand i: 32 i bytes on).
__device__ __forceinline__ uint32_t fetch_k_chunk(int lane) { return (uint32_t)((lane & 15) ^ ((lane >> 4) & 1)) << 4; }
__device__ __forceinline__ uint32_t fetch_v_chunk(int lane) { return (uint32_t)(lane & 15) << 4; }
__device__ __forceinline__ const uint8_t* shared_k_at(const uint8_t* tile, int half, int col) {
  return tile + (col & 7) * kKGroup + (col >> 3) * 256 + ((half ^ ((col >> 3) & 1)) << 4);
}
__device__ __forceinline__ const uint8_t* shared_v_at(const uint8_t* tile, int lane) {
  return tile + ((lane >> 5) * 4 + ((lane & 15) >> 2)) * kVGroup + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
}
__device__ __forceinline__ bf16x8 shared_k_frag(const uint8_t* at, int i) { return *reinterpret_cast<const bf16x8*>(at + i * 32); }

// Memory and scheduling barrier for the compiler: what is requested before it is issued before what comes after.
__device__ __forceinline__ void in_issue_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// Workgroup barrier without the compiler's waits: the caller has waited for what the others are to see.
__device__ __forceinline__ void bare_barrier() {
  in_issue_order();
  __builtin_amdgcn_s_barrier();
  in_issue_order();
}

// Softmax reference of a row before its first key of finite logit.  Finite itself: against -inf the numerators of a tile
// whose logits are all -inf would be exp2(-inf + inf).  Everything scaled by exp2(kNoMax - m) is zero, as with -inf.
constexpr float kNoMax = -3.0e38f;

// make this wave's LDS writes visible to its own later reads (wave-private tiles need no s_barrier)
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace sdllm
