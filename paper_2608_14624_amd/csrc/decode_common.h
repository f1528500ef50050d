// What the decode kernels in ranges (paged_decode_attn.hip) and the cascade's
// (cascade_ranges.hip) share: vector types, the plan's arithmetic, the load of
// one 32-key chunk and the merge of partial results.
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

// V tile of one wave in LDS: 32 keys x D, rows padded by 32 B so that the 32
// lanes of a transposing read (8 keys x 32 B) fall on distinct banks.
constexpr int v_tile_stride(int head_dim) { return head_dim + 16; }

// The V rows of keys key0 .. into the wave's tile; rows past the `len` keys (inside
// the last block, or the other half of a shared prefix's last unit) as zeros: their
// probabilities are 0, but 0 times a stale NaN or Inf in the pool is NaN.
template <int D>
__device__ __forceinline__ void store_v_tile(const bf16x8 (&vreg)[kChunk * D / 8 / 64], int lane, int key0, int len,
                                             uint16_t* tile) {
  constexpr int kRowChunks = D / 8;
  constexpr int kVLoads = kChunk * kRowChunks / 64;
#pragma unroll
  for (int v = 0; v < kVLoads; ++v) {
    const int cc = lane + 64 * v;
    *reinterpret_cast<bf16x8*>(&tile[(cc / kRowChunks) * v_tile_stride(D) + (cc % kRowChunks) * 8]) = vreg[v];
  }
  if (key0 + kChunk > len) {
#pragma unroll
    for (int v = 0; v < kVLoads; ++v) {
      const int cc = lane + 64 * v;
      if (key0 + cc / kRowChunks >= len)
        *reinterpret_cast<bf16x8*>(&tile[(cc / kRowChunks) * v_tile_stride(D) + (cc % kRowChunks) * 8]) = bf16x8{};
    }
  }
}

// V^T fragment (16 dims x 32 keys) for output tile dt: the slot s of lane
// group qd is key 16*(s/4) + 4*qd + s%4, matching the S^T accumulator
// layout (tile s/4, register s%4).  ds_read_b64_tr_b16 hands lane j of a
// 16-lane group M[4e + j/4][j%4] of the 8-byte rows its lanes address; lane
// 16*qd + i addresses key 4*qd + i/4, dims 16*dt + 4*(i%4).
template <int D>
__device__ __forceinline__ bf16x8 v_fragment(const uint16_t* tile, int lane, int dt) {
  const int j = lane & 15, qd = lane >> 4;
  const uint16_t* base = tile + (4 * qd + (j >> 2)) * v_tile_stride(D) + 4 * (j & 3) + 16 * dt;
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(base));
  const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(base + 16 * v_tile_stride(D)));
  const i16x4 lohi[2] = {lo, hi};
  return __builtin_bit_cast(bf16x8, lohi);
}

// The merge of a launch in ranges: one work-group combines the partial results
// (O relative to m, m and l) of the `group` rows of a sequence and KV head.  A
// thread holds four features of one row; as many teams of threads as fit and
// have work share the row's pieces(hj) pieces, each taking kMergeStep at a time so
// that their loads are in flight together, and the teams' results meet in LDS.
// Piece k of row hj is partial row at(hj, k); pieces is called first.
// The launch is one chain of memory latencies (lengths and plan, pieces, output),
// so what counts is that there are few of them: steps of 8 with the last piece read
// again past the end took 9.4 us where this takes 6.5 (128 sequences, 8 KV heads),
// all 32 teams that fit one query head of 64 features 9.4 us a call of 16 pairs of
// 560 keys where as many as have work take 8.5.
constexpr int kMergeStep = 4;
constexpr int kMergeThreads = 512;     // kMaxGroup * 128 / 4
template <int D, typename Pieces, typename At, typename Store>
__device__ __forceinline__ void merge_pieces(const float* ws_o, const float* ws_ml, int group, float c, Pieces&& pieces,
                                             At&& at_of, Store&& store) {
  __shared__ f32x4 team_acc[kMergeThreads];
  __shared__ float2 team_md[kMergeThreads];
  const int elems = group * (D / 4);   // threads of a team
  const int team = threadIdx.x / elems;
  const int idx = threadIdx.x - team * elems;
  const int hj = idx / (D / 4);
  const int d = idx % (D / 4) * 4;
  const int n = pieces(hj);
  const int teams = min(kMergeThreads / elems, max(1, ceil_div(n, kMergeStep)));
  float mx = -INFINITY, den = 0.f;
  f32x4 acc = f32x4{};
  if (team < teams) {
    for (int i = team; i < n; i += kMergeStep * teams) {
      float2 ml[kMergeStep];
      f32x4 o[kMergeStep];
#pragma unroll
      for (int x = 0; x < kMergeStep; ++x) {
        ml[x] = make_float2(-INFINITY, 0.f);
        o[x] = f32x4{};
        if (i + x * teams >= n) continue;
        const size_t at = at_of(hj, i + x * teams);
        ml[x] = *reinterpret_cast<const float2*>(ws_ml + 2 * at);
        o[x] = *reinterpret_cast<const f32x4*>(ws_o + at * D + d);
      }
      float m_new = mx;
#pragma unroll
      for (int x = 0; x < kMergeStep; ++x) m_new = fmaxf(m_new, ml[x].x);
      const float alpha = __builtin_amdgcn_exp2f((mx - m_new) * c);
      mx = m_new;
      acc *= alpha;
      den *= alpha;
#pragma unroll
      for (int x = 0; x < kMergeStep; ++x) {
        const float wt = __builtin_amdgcn_exp2f((ml[x].x - mx) * c);      // 0 past the last piece
        acc += wt * o[x];
        den += wt * ml[x].y;
      }
    }
  }
  team_acc[threadIdx.x] = acc;
  team_md[threadIdx.x] = make_float2(mx, den);
  __syncthreads();
  if (team != 0) return;
  float m_all = mx;
  for (int t = 1; t < teams; ++t) m_all = fmaxf(m_all, team_md[t * elems + idx].x);
  const float w_first = __builtin_amdgcn_exp2f((mx - m_all) * c);
  acc *= w_first;
  den *= w_first;
  for (int t = 1; t < teams; ++t) {
    const float2 md = team_md[t * elems + idx];
    const float wt = __builtin_amdgcn_exp2f((md.x - m_all) * c);      // 0 for a team without pieces
    acc += wt * team_acc[t * elems + idx];
    den += wt * md.y;
  }
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[e] / den);
  store(hj, d, o);
}

}  // namespace
}  // namespace cs
