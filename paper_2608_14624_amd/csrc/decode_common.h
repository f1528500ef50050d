// What the decode kernels in ranges (paged_decode_attn.hip) and the cascade's
// (cascade_ranges.hip) share: vector types, the plan's arithmetic and the load
// of one 32-key chunk.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave_ops.h"

namespace cs {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
typedef const __attribute__((address_space(4))) int32_t* ScalarInts;

constexpr int kBlock = 16;
constexpr int kChunk = 32;           // keys per wave step (2 pool blocks)
constexpr int kMaxGroup = 16;
constexpr float kLog2e = 1.4426950408889634f;

// keys are planned in units of one chunk
constexpr int kUnitKeys = kChunk;
constexpr int kUnitBlocks = kUnitKeys / kBlock;

// one-wave work-groups per CU that a plan deals its units to (the reasons
// stand at decode_ranges_kernel)
constexpr int kRangeGroupsPerCu128 = 3;
constexpr int kRangeGroupsPerCu64 = 4;

// word 3 of a raw buffer descriptor (32-bit data format, no swizzle), and the
// cache policy bit of a non-temporal buffer load
constexpr int kRawBufferWord3 = 0x00020000;
constexpr int kNonTemporal = 2;

__device__ __forceinline__ int units_of(int len) { return (max(len, 0) + kUnitKeys - 1) / kUnitKeys; }

__device__ __forceinline__ int wave_total(int x) { return __builtin_amdgcn_readlane(wave_scan(x), 63); }

// The four lanes j, j + 16, j + 32 and j + 48 hold one query's values: their
// maximum and sum with two VALU lane swaps instead of LDS permutes.
// v_permlane32_swap exchanges the upper half of its first operand with the
// lower half of its second, v_permlane16_swap the odd rows of 16 of the first
// with the even ones of the second; with both operands holding x, the two then
// hold a lane's own value and its partner's.  (The clang builtins of this ROCm
// return the first operand for both results; the s_nops cover the hazard of a
// VALU write before a permlane read, which the compiler cannot see in asm.)
__device__ __forceinline__ void swap32(float x, float& a, float& b) {
  a = x;
  b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap16(float x, float& a, float& b) {
  a = x;
  b = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float quad_max(float x) {
  float a, b, e, f;
  swap16(x, a, b);
  swap32(fmaxf(a, b), e, f);
  return fmaxf(e, f);
}
__device__ __forceinline__ float quad_sum(float x) {
  float a, b, e, f;
  swap16(x, a, b);
  swap32(a + b, e, f);
  return e + f;
}

// K fragments (A operand of the 16x16x32 MFMA) and V rows of one chunk, the
// tiles of blocks id0 and id1 (of the KV head that the pools start at), through
// buffer descriptors over the tiles: the per-lane offsets are the same for every
// tile.  The descriptor of a negative block id is empty, so its K and V are 0, as
// in paged_decode_attn_kernel, and nothing outside the pools is read.
template <int D, int kVPolicy>
__device__ __forceinline__ void load_chunk_tiles(const uint16_t* k_pool, const uint16_t* v_pool, int id0, int id1,
                                                 size_t slot_elems, int lane, bf16x8 (&kreg)[2][D / 32],
                                                 bf16x8 (&vreg)[kChunk * D / 8 / 64]) {
  constexpr int kTileBytes = kBlock * D * 2;
  constexpr int kVPerBlock = kChunk * D / 8 / 64 / 2;
  const int k_off = 2 * ((lane & 15) * D + 8 * (lane >> 4));
  const int v_off = 16 * lane;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const int id = mt ? id1 : id0;
    const size_t at = (size_t)id * slot_elems;
    const int bytes = id < 0 ? 0 : kTileBytes;
    const __amdgpu_buffer_rsrc_t krs =
        __builtin_amdgcn_make_buffer_rsrc((void*)(k_pool + at), (short)0, bytes, kRawBufferWord3);
    const __amdgpu_buffer_rsrc_t vrs =
        __builtin_amdgcn_make_buffer_rsrc((void*)(v_pool + at), (short)0, bytes, kRawBufferWord3);
#pragma unroll
    for (int dc = 0; dc < D / 32; ++dc)
      kreg[mt][dc] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(krs, k_off + 64 * dc, 0, 0));
#pragma unroll
    for (int v = 0; v < kVPerBlock; ++v)
      vreg[mt * kVPerBlock + v] =
          __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(vrs, v_off + 1024 * v, 0, kVPolicy));
  }
}

}  // namespace
}  // namespace cs
