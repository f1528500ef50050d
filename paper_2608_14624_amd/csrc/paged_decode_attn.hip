// Paged decode attention for gfx950: one new token per sequence attends over
// all keys of its sequence in the paged pool.
//
// This is the one-token case of the prefix-reuse attention (arXiv
// 2608.14624, Sec. 2.1: a request reuses the cached KV of its prefix; the
// per-turn latency the paper reports includes the decode that follows the
// prefill, Sec. 5): the query of sequence r is its last position L_r - 1 and
// sees every key 0 .. L_r - 1.  Decode reads each key once per KV head and
// does G = Hq / Hkv dot products with it, so it is bound by HBM bandwidth,
// not by the matrix cores.
//
// Kernel design
//   * One work-group = W wave64s = one (sequence, KV head), W = 12 (4 in
//     cascade mode); the G query heads of the group are the N = 16 columns
//     of v_mfma_f32_16x16x32_bf16 (G <= 16).
//   * The W waves split the key range in 32-key chunks (wave w takes chunks
//     w, w+W, ...) and run independent online softmaxes, so there is no
//     synchronisation in the loop; the W partial results are merged in LDS
//     at the end (log-sum-exp weights), so no workspace is needed.
//   * S^T = K Q^T with K fragments loaded from HBM straight into the MFMA A
//     operand (16 B per lane), Q^T kept in VGPRs.  O^T = V^T P^T reads V^T
//     with ds_read_b64_tr_b16 from a per-wave LDS tile that the wave itself
//     wrote (LDS operations of one wave complete in order, so no barrier).
//   * The K/V loads of a wave's next chunk are issued before the math of the
//     current one, so each wave keeps 16 KiB in flight.
//   * Work-groups are ordered KV head fastest, so each XCD serves one head.
//
// Cascade mode (the launches that cascade_ranges.hip does not take): a sequence
// belongs to a group whose shared prefix (its first
// shared_len keys) is attended by the stacked prefill kernel, which leaves
// one partial result (O relative to its running max m, the max m and the sum
// l) per 1024-key chunk in a workspace.  Here a work-group takes one KV head
// and one 1024-key segment of a sequence's own keys shared_len .. L - 1, so
// a long history spreads over several work-groups, and leaves its partial
// in the workspace too; cascade_merge_kernel then combines every partial of
// a row with log-sum-exp weights exp2((m_i - max) * c).
#include "decode_common.h"
#include "internal.h"

#include <float.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

namespace cs {
namespace {

// waves per work-group: 12 for plain decode (one work-group fills a CU at
// three waves per SIMD, so a CU's last, longest sequence runs on all of its
// wave slots instead of a third of them), 4 for the cascade's 1024-key
// segments
constexpr int kDecodeWaves = 12;
constexpr int kCascadeWaves = 4;
constexpr int kThreads = 256;        // the merge kernel
// plain decode batches up to this size run longest sequence first
constexpr int kLptMaxBatch = 1024;

struct DecParams {
  const uint16_t* q;          // [B][Hq][D]
  const uint16_t* k_pool;
  const uint16_t* v_pool;
  const int32_t* block_tables;
  const int32_t* seq_lens;
  uint16_t* out;              // [B][Hq][D]
  int max_blocks_per_seq;
  int num_q_heads;
  int num_kv_heads;
  int group;
  float scale_log2;
  // decode in ranges (decode_ranges_kernel): work-groups per KV head, partials
  // per KV head in ws_o / ws_ml, and the plan ({aligned, units per piece})
  int ranges;
  int aligned_ranges;
  int slots;
  int2* plan;
  // cascade mode only
  const int32_t* cu_groups;     // [num_groups + 1], cu_groups[0] = 0, last = batch
  const int32_t* shared_lens;   // [num_groups]
  int num_groups;
  int batch;
  int chunk_keys;               // keys per partial of the shared prefix
  int chunks;                   // shared-prefix partials per row (upper bound)
  int segments;                 // own-key partials per row (upper bound)
  float* ws_o;                  // [chunks + segments][batch * num_q_heads][D]
  float* ws_ml;                 // [chunks + segments][batch * num_q_heads][2]
  int ws_rows;
};

// first key of sequence r that its group does not share
__device__ __forceinline__ int shared_len_of(const DecParams& p, int r) {
  int lo = 0, hi = p.num_groups - 1;   // the last group gr with cu_groups[gr] <= r
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (p.cu_groups[mid] <= r) lo = mid; else hi = mid - 1;
  }
  return p.shared_lens[lo];
}

template <int D, int W>
struct DecLds {
  static constexpr int vStride = v_tile_stride(D);
  union {
    uint16_t v[W][kChunk * vStride];
    struct {
      float m[W][kMaxGroup];
      float l[W][kMaxGroup];
      float o[W][kMaxGroup][D];
    } merge;
  };
};

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

template <int D, bool kCascade>
__global__ __launch_bounds__(64 * (kCascade ? kCascadeWaves : kDecodeWaves)) void paged_decode_attn_kernel(DecParams p) {
  constexpr int kWaves = kCascade ? kCascadeWaves : kDecodeWaves;
  constexpr int kWGThreads = 64 * kWaves;
  __shared__ DecLds<D, kWaves> sm;
  constexpr int vStride = DecLds<D, kWaves>::vStride;
  constexpr int DC = D / 32;         // 32-wide k-steps of the QK^T product
  constexpr int DT = D / 16;         // 16-row output tiles over the head dim
  constexpr int kRowChunks = D / 8;  // 16-byte chunks per key row
  constexpr int kVLoads = kChunk * kRowChunks / 64;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15;           // MFMA column: query head within the group
  const int qd = lane >> 4;          // lane group: k-slots 8*qd .. +7

  const int g = blockIdx.x % p.num_kv_heads;
  int r, seg = 0;
  if constexpr (kCascade) {
    r = (blockIdx.x / p.num_kv_heads) % p.batch;
    seg = blockIdx.x / p.num_kv_heads / p.batch;
  } else {
    // Longest sequence first: the work-groups of one wave of dispatch take
    // the sequences of ranks w / num_kv_heads in decreasing length (ties by
    // index), so the last of the launch's rounds holds the shortest ones
    // and the CUs run out of work together.  Every work-group ranks the
    // lengths itself (each thread a few candidates against all of them, in
    // LDS): the order is a permutation whatever the lengths hold, so every
    // (sequence, head) is still computed exactly once, and each output is
    // the same as in any other order.
    r = blockIdx.x / p.num_kv_heads;
    if (p.batch <= kLptMaxBatch) {
      __shared__ int lens[kLptMaxBatch];
      __shared__ int pick;
      for (int s = threadIdx.x; s < p.batch; s += kWGThreads) lens[s] = p.seq_lens[s];
      if (threadIdx.x == 0) pick = r;
      __syncthreads();
      for (int s = threadIdx.x; s < p.batch; s += kWGThreads) {
        const int ls = lens[s];
        int rank = 0;
        for (int t = 0; t < p.batch; ++t) {
          const int lt = lens[t];
          rank += (lt > ls) || (lt == ls && t < s);
        }
        if (rank == r) pick = s;
      }
      __syncthreads();
      r = pick;
    }
  }
  const int L = p.seq_lens[r];
  int start = 0;       // keys start .. end - 1 are this work-group's
  int end = L;
  if constexpr (kCascade) {
    start = shared_len_of(p, r) + seg * kCascadeSegmentKeys;
    end = min(L, start + kCascadeSegmentKeys);
    if (start >= end) return;          // nothing of this sequence's own here
  }
  const int n_blk = (end + kBlock - 1) / kBlock;
  const int first_chunk = start / kChunk;
  const int ch_end = (end + kChunk - 1) / kChunk;
  const size_t tile_elems = (size_t)kBlock * D;
  const size_t slot_elems = (size_t)p.num_kv_heads * tile_elems;
  const uint16_t* kbase = p.k_pool + (size_t)g * tile_elems;
  const uint16_t* vbase = p.v_pool + (size_t)g * tile_elems;
  const __attribute__((address_space(4))) int32_t* bt =
      (const __attribute__((address_space(4))) int32_t*)(p.block_tables +
                                                          (size_t)r * p.max_blocks_per_seq);

  // ---- Q^T operand: column j = query head g*G + j, dims 32*dc + 8*qd .. +7
  const bool head_valid = j < p.group;
  const int h = g * p.group + (head_valid ? j : 0);
  bf16x8 qreg[DC];
#pragma unroll
  for (int dc = 0; dc < DC; ++dc) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (head_valid)
      v = *reinterpret_cast<const uint4*>(p.q + ((size_t)r * p.num_q_heads + h) * D + 32 * dc + 8 * qd);
    qreg[dc] = as_bf16x8(v);
  }

  // ---- loads of one chunk: K fragments (A operand) and V rows (to LDS) --
  uint4 kreg[2][DC];
  uint4 vreg[kVLoads];
  auto load_chunk = [&](int ch) {
    const int b0 = 2 * ch;
    const int id0 = b0 < n_blk ? bt[b0] : -1;
    const int id1 = b0 + 1 < n_blk ? bt[b0 + 1] : -1;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const int id = mt ? id1 : id0;
#pragma unroll
      for (int dc = 0; dc < DC; ++dc) {
        kreg[mt][dc] = make_uint4(0, 0, 0, 0);
        if (id >= 0)
          kreg[mt][dc] = *reinterpret_cast<const uint4*>(kbase + (size_t)id * slot_elems + j * D + 32 * dc + 8 * qd);
      }
    }
#pragma unroll
    for (int u = 0; u < kVLoads; ++u) {
      const int c = lane + 64 * u;
      const int key = c / kRowChunks;           // 0..31, uniform block per u
      const int id = key < kBlock ? id0 : id1;
      vreg[u] = make_uint4(0, 0, 0, 0);
      if (id >= 0)
        vreg[u] = *reinterpret_cast<const uint4*>(vbase + (size_t)id * slot_elems + (key % kBlock) * D + (c % kRowChunks) * 8);
    }
  };

  const uint16_t* vt = sm.v[wave];
  f32x4 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) oacc[dt] = f32x4{};
  float m_run = -INFINITY;
  float l_run = 0.f;
  const float c = p.scale_log2;

  int ch = first_chunk + wave;
  if (ch < ch_end) load_chunk(ch);
  for (; ch < ch_end; ch += kWaves) {
    // V rows of this chunk into the wave's LDS tile
#pragma unroll
    for (int u = 0; u < kVLoads; ++u) {
      const int cc = lane + 64 * u;
      *reinterpret_cast<uint4*>(&sm.v[wave][(cc / kRowChunks) * vStride + (cc % kRowChunks) * 8]) = vreg[u];
    }
    // rows past the end of the sequence (inside its last block) overwritten
    // with zeros: their probabilities are 0, but 0 times a stale NaN or Inf
    // in the pool is NaN
    if ((ch + 1) * kChunk > end) {
#pragma unroll
      for (int u = 0; u < kVLoads; ++u) {
        const int cc = lane + 64 * u;
        if (ch * kChunk + cc / kRowChunks >= end)
          *reinterpret_cast<uint4*>(&sm.v[wave][(cc / kRowChunks) * vStride + (cc % kRowChunks) * 8]) =
              make_uint4(0, 0, 0, 0);
      }
    }
    // S^T = K Q^T: two 16-key tiles
    f32x4 s[2] = {f32x4{}, f32x4{}};
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int dc = 0; dc < DC; ++dc)
        s[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kreg[mt][dc]), qreg[dc], s[mt], 0, 0, 0);
    if (ch + kWaves < ch_end) load_chunk(ch + kWaves);     // in flight during the math

    // mask keys past the end; register r of tile mt holds key 32*ch + 16*mt + 4*qd + r
    const int kbase_idx = ch * kChunk;
    float mloc = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int key = kbase_idx + 16 * mt + 4 * qd + rr;
        s[mt][rr] = (key < end && key >= start) ? s[mt][rr] : -INFINITY;
        mloc = fmaxf(mloc, s[mt][rr]);
      }
    mloc = fmaxf(mloc, __shfl_xor(mloc, 16));
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
    const float m_new = fmaxf(m_run, mloc);
    const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt] *= alpha;
    const float mc = m_new * c;
    bf16x8 pb;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][rr], c, -mc));
        pb[4 * mt + rr] = (__bf16)e;
        l_run += (float)pb[4 * mt + rr];
      }
    // O^T += V^T P^T
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v_fragment<D>(vt, lane, dt), pb, oacc[dt], 0, 0, 0);
  }

  // ---- merge the waves' partial softmaxes -----------------------------
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  __syncthreads();                     // every wave is done with its V tile
  if (qd == 0) {
    sm.merge.m[wave][j] = m_run;
    sm.merge.l[wave][j] = l_run;
  }
  // accumulator register rr of tile dt holds dim 16*dt + 4*qd + rr of head j
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) sm.merge.o[wave][j][16 * dt + 4 * qd + rr] = oacc[dt][rr];
  __syncthreads();
  for (int idx = threadIdx.x; idx < p.group * D; idx += kWGThreads) {
    const int hj = idx / D;
    const int d = idx % D;
    const size_t row = (size_t)r * p.num_q_heads + g * p.group + hj;
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, sm.merge.m[w][hj]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float wt = __builtin_amdgcn_exp2f((sm.merge.m[w][hj] - mx) * c);   // 0 for idle waves
      num += wt * sm.merge.o[w][hj][d];
      den += wt * sm.merge.l[w][hj];
    }
    if constexpr (kCascade) {
      // this segment's partial: O relative to mx, mx, and the sum
      const size_t widx = (size_t)(p.chunks + seg) * p.ws_rows + row;
      p.ws_o[widx * D + d] = num;
      if (d == 0) {
        p.ws_ml[2 * widx] = mx;
        p.ws_ml[2 * widx + 1] = den;
      }
    } else {
      p.out[row * D + d] = __builtin_bit_cast(uint16_t, (__bf16)(num / den));
    }
  }
}

// ---- decode in ranges ----------------------------------------------------
//
// One wave per work-group, a few per CU, p.ranges of them per KV head whatever
// the batch holds.  The sequences' keys are counted in units of 32 (one chunk),
// and every wave works the plan out itself from the lengths (wave-wide scans),
// so the host needs no lengths and no tight bound of them.
//   * Nothing shared: the sequences' units are laid end to end in batch order
//     and dealt in equal contiguous ranges of ceil(total / ranges) units.
//   * Where enough of the batch shares prefixes (counted by the pool block at
//     index kProbeBlock of the block tables): every sequence is cut at the same
//     positions, multiples of ceil(total / (aligned_rounds ranges)) units, and the
//     waves take the first pieces of all sequences, then the second ones, ..., so
//     that sequences with the same blocks read them at about the same time and
//     most find them in L2.
// A piece of a sequence that is not the whole of it leaves a partial result (O
// relative to its running max m, the max m and the sum l) in a slot of the
// workspace, and decode_ranges_merge_kernel combines a sequence's pieces.  The
// slot of a contiguous piece is r + w (sequence r, range w: both grow from piece
// to piece, so slots are unique), of an aligned piece its index among all.
//
// What bounds it is HBM, and how it is asked: 4 KiB (block, head) tiles at
// scattered places.  More requests in flight than the memory needs make some
// waves starve (first loads served after 60 us of a 90 us launch) while the
// slowest range sets the time, and ordinary loads wash the whole stream through
// the last-level cache.  128 sequences of 6000-9000 keys, 32 / 8 heads of 128:
// twelve waves per CU as work-groups of four 659 us, with non-temporal loads
// 612, four single-wave work-groups per CU and non-temporal loads 574, three
// 571 (6.7 TB/s; one 12-wave work-group per sequence and KV head: 642).  Three
// per CU at head_dim 128 (two: 1% slower, five: 6%), four at 64, where a wave's
// chunk is half the bytes (three: 5% slower).  K and V both non-temporal is up
// to 4% faster than V alone, but 17% slower where the pools were written just
// before (4 GB of them: 875 us against 749; ordinary loads 797).  Sequences that
// share want ordinary loads and more waves, at head_dim 128 eight per CU with two
// pieces each (128 sequences of 8 agents 317 us, four and four 355), at 64, where
// a unit is half the bytes, sixteen with one (256 sequences of 8 agents, 8 / 2
// heads, 86 us; eight and two 97, one work-group per sequence and KV head 89).
//
// For sequences with blocks of their own the aligned pieces are the slower ones
// (many waves, ordinary loads): 128 of 6000-9000 keys, two of them on one anchor,
// 32 / 8 heads of 128, 592 us in ranges, 676 in pieces, one work-group each 648.
// And short launches lose in pieces what the order saves: the pieces' ends do not
// meet the work of the waves.  Pieces are therefore taken where at least a
// quarter of the sequences are on a block counted before (kSharingPart), and that
// share times the units of an equal range is at least kSharedUnits.  us a call,
// ranges and pieces, at share times units: 4 / 1 heads of 64, 128 sequences of one
// agent 18.5 and 22.7 (11), 500 of 16 45.3 and 48.3 (29), 256 of 8 61 and 54 (52);
// 8 / 2 of 64, 128 of one 25.1 and 26.4 (21), 500 of 16 68 and 61 (57), 128 of 64
// 32 and 38 (11); 32 / 8 of 64, 24 of 3 18.3 and 19.8 (11), 64 of 4 47.8 and 42.2
// (42); 32 / 8 of 128, 16 of 2 46.9 and 48.4 (31), 64 of 4 75 and 67 (56); of 128
// sequences of 6000-9000 keys 64 in pairs (a quarter counted: 67) 555 and 532 at
// 128, 269 and 281 at 64, and 48 in pairs 565 and 568, 273 and 302.
// Pieces per CU and KV head, and how many of them a wave takes:
constexpr int kAlignedPiecesPerCu = 16;
constexpr int aligned_rounds(int head_dim) { return head_dim == 64 ? 1 : 2; }
constexpr int kSharingPart = 4;
constexpr int kSharedUnits = 36;
constexpr int kProbeBlock = 31;
constexpr int kProbeTable = 2 * kRangeMaxBatch;
constexpr int kPlanRounds = kRangeMaxBatch / 64;

// f(0), f(1), ... over the rounds of 64 sequences that a batch takes, or up to
// twice as many (past the batch f has nothing to do): a small batch passes the
// code of the other rounds in one jump, where a test per round and loop took 1.3
// us of a 14 us call in instruction fetches.
template <int kFrom = 0, typename F>
__device__ __forceinline__ void plan_rounds(int batch, F&& f) {
  constexpr int kTo = kFrom == 0 ? 1 : 2 * kFrom;
#pragma unroll
  for (int i = kFrom; i < kTo; ++i) f(i);
  if constexpr (kTo < kPlanRounds) {
    if (batch > 64 * kTo) plan_rounds<kTo>(batch, f);
  }
}

// How many of the batch's sequences hold the pool block at index kProbeBlock that
// another one counted before them holds (one wave; ids: the lane's sequences',
// -1 where there is none): a hash table of the blocks in LDS, at most half full.
// The count is that of all less the different ones, so it does not depend on the
// order in which the lanes meet.
__device__ __forceinline__ int count_sharing(const int (&ids)[kPlanRounds], int batch, int lane, int* table) {
  for (int i = lane; i < kProbeTable; i += 64) table[i] = -1;
  __syncthreads();
  int dups = 0;
  plan_rounds(batch, [&](int i) __attribute__((always_inline)) {
    const int id = ids[i];
    bool dup = false;
    if (id >= 0) {
      unsigned h = ((unsigned)id * 2654435761u) >> 16;
      for (int tries = 0; tries < kProbeTable; ++tries) {
        h %= kProbeTable;
        const int old = atomicCAS(&table[h], -1, id);
        if (old == -1) break;
        if (old == id) {
          dup = true;
          break;
        }
        ++h;
      }
    }
    dups += __builtin_popcountll(__builtin_amdgcn_ballot_w64(dup));
  });
  __syncthreads();
  return dups;
}

// A position in a wave's list of pieces.
struct RangeCursor {
  int r;          // sequence
  int len;        // its keys
  int x, xe;      // unit within the sequence, end of the piece
  int slot;       // where the piece's partial goes, -1: the piece is the whole sequence
  bool valid;
};

template <int D>
__global__ __launch_bounds__(64) void decode_ranges_kernel(DecParams p) {
  constexpr int vStride = v_tile_stride(D);
  constexpr int DC = D / 32;
  constexpr int DT = D / 16;
  constexpr int kVLoads = kChunk * D / 8 / 64;
  constexpr int kManyUnits = 0xffff;
  __shared__ union {
    struct {
      uint16_t v[kChunk * vStride];
      uint16_t units[kRangeMaxBatch];    // of every sequence (kManyUnits: that many or more)
    };
    int probe[kProbeTable];
  } sm;

  const int lane = threadIdx.x;
  const int j = lane & 15;
  const int qd = lane >> 4;
  const int g = blockIdx.x % p.num_kv_heads;
  const int w = blockIdx.x / p.num_kv_heads;
  const ScalarInts lens_c = (ScalarInts)p.seq_lens;

  // ---- the plan.  All lengths and probed blocks are asked for at once, and the
  // units then kept in LDS: read from memory again for every piece, a batch of
  // 256 spent longer on finding its last pieces than on a short piece itself.
  int n_of[kPlanRounds], ids_probed[kPlanRounds];
  const bool probes = p.batch > 1 && p.max_blocks_per_seq > kProbeBlock;
  plan_rounds(p.batch, [&](int i) __attribute__((always_inline)) {
    const int s = 64 * i + lane;
    n_of[i] = s < p.batch ? p.seq_lens[s] : 0;
    ids_probed[i] = probes && s < p.batch ? p.block_tables[(size_t)s * p.max_blocks_per_seq + kProbeBlock] : -1;
  });
  int total = 0, longest = 0;
  plan_rounds(p.batch, [&](int i) __attribute__((always_inline)) {
    if (n_of[i] <= kProbeBlock * kBlock) ids_probed[i] = -1;      // an entry past its last block
    n_of[i] = units_of(n_of[i]);
    total += wave_total(n_of[i]);
    longest = max(longest, wave_max(n_of[i]));
  });
  bool aligned = false;
  if (p.batch > 1 && total >= kSharedUnits * p.ranges) {
    const int sharing = count_sharing(ids_probed, p.batch, lane, sm.probe);
    aligned = kSharingPart * sharing >= p.batch &&
              (long long)sharing * total >= (long long)kSharedUnits * p.batch * p.ranges;
  }
  plan_rounds(p.batch, [&](int i) __attribute__((always_inline)) {
    sm.units[64 * i + lane] = (uint16_t)min(n_of[i], kManyUnits);
  });
  __syncthreads();
  auto units_at = [&](int s) {           // of sequence s (a lane's), 0 past the batch
    if (s >= p.batch) return 0;
    const int n = sm.units[s];
    return n == kManyUnits ? units_of(p.seq_lens[s]) : n;
  };
  const int ranges = aligned ? p.aligned_ranges : p.ranges;     // waves that take part
  // With few KV heads there are more waves than the merge has use for: few
  // sequences in pieces of one unit leave it hundreds of partials each.  Past
  // 16 pieces of the longest sequence a range has up to 4 units (8 / 1 heads,
  // one sequence of 7000 keys 27.3 -> 13.9 us, 3 of 2000-6000 23.3 -> 14.6; 8 of
  // 100-500 9.8 with 1, 11.3 with 4).  Aligned pieces are longer by their rule.
  const int shortest = min(4, ceil_div(longest, 16));
  const int per = max(max(1, shortest), ceil_div(total, aligned ? aligned_rounds(D) * ranges : ranges));
  if (blockIdx.x == 0 && lane == 0) *p.plan = make_int2(aligned, per);

  // the sequence's slots: its pieces are numbered from here
  auto piece_base = [&](int r) {
    int t = 0;
    for (int s = 0; s < r; s += 64) t += wave_total(s + lane < r ? ceil_div(units_at(s + lane), per) : 0);
    return t;
  };
  // aligned pieces in order of (piece, sequence): the wave's are w, w + ranges, ...
  int rank = 0, piece = 0;
  auto aligned_piece = [&](RangeCursor& c) {
    for (;; ++piece) {
      int count = 0;
      for (int s = 0; s < p.batch; s += 64)
        count += __builtin_popcountll(__builtin_amdgcn_ballot_w64(units_at(s + lane) > piece * per));
      if (count == 0) {
        c.valid = false;
        return;
      }
      if (rank < count) break;
      rank -= count;
    }
    int before = 0;
    for (int s = 0; s < p.batch; s += 64) {
      const unsigned long long mask = __builtin_amdgcn_ballot_w64(units_at(s + lane) > piece * per);
      const int n = __builtin_popcountll(mask);
      if (rank < before + n) {
        const int mine = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
        const bool hit = ((mask >> lane) & 1) && mine == rank - before;
        c.r = s + __builtin_ctzll(__builtin_amdgcn_ballot_w64(hit));
        break;
      }
      before += n;
    }
    c.len = lens_c[c.r];
    c.x = piece * per;
    c.xe = min(units_of(c.len), c.x + per);
    c.slot = units_of(c.len) <= per ? -1 : piece_base(c.r) + piece;
    c.valid = true;
  };
  // contiguous ranges: `left` units of the range lie past the cursor's piece
  int left = 0;
  auto contiguous_piece = [&](RangeCursor& c) {      // from unit c.x of sequence c.r on
    const int n = units_of(c.len);
    c.xe = min(n, c.x + left);
    left -= c.xe - c.x;
    c.slot = (c.x == 0 && c.xe == n) ? -1 : c.r + w;
    c.valid = true;
  };

  RangeCursor ids{};
  if (w >= ranges) return;
  if (aligned) {
    rank = w;
    aligned_piece(ids);
  } else {
    const int u = w * per;
    left = min(total, u + per) - u;
    if (left > 0) {
      int first = 0;                                    // first unit of sequence ids.r
      for (int s = 0;; s += 64) {
        const int n = units_at(s + lane);
        const int incl = wave_scan(n);
        const unsigned long long past = __builtin_amdgcn_ballot_w64(first + incl > u);
        if (past != 0) {
          const int l = __builtin_ctzll(past);
          ids.r = s + l;
          first += __builtin_amdgcn_readlane(incl - n, l);
          break;
        }
        first += __builtin_amdgcn_readlane(incl, 63);
      }
      ids.len = lens_c[ids.r];
      ids.x = u - first;
      contiguous_piece(ids);
    }
  }
  if (!ids.valid) return;
  // the unit after the cursor's: in its piece, or the first of the next one
  auto advance = [&](RangeCursor& c, auto tag) {
    if (++c.x < c.xe) return;
    if constexpr (decltype(tag)::value) {
      rank += ranges;
      aligned_piece(c);
      return;
    }
    if (left <= 0) {
      c.valid = false;
      return;
    }
    do c.len = lens_c[++c.r];
    while (c.len <= 0);
    c.x = 0;
    contiguous_piece(c);
  };

  const size_t tile_elems = (size_t)kBlock * D;
  const size_t slot_elems = (size_t)p.num_kv_heads * tile_elems;
  const uint16_t* kbase = p.k_pool + (size_t)g * tile_elems;
  const uint16_t* vbase = p.v_pool + (size_t)g * tile_elems;
  const bool head_valid = j < p.group;
  const int h = g * p.group + (head_valid ? j : 0);
  const float c = p.scale_log2;
  // a unit whose logits are all -inf weighs 0 relative to this, not NaN
  const float lowest = -FLT_MAX / fmaxf(c, 1.f);

  bf16x8 kreg[2][DC];
  bf16x8 vreg[kVLoads];
  // K fragments and V rows of the blocks id0, id1.  Where each block is read
  // once V is loaded non-temporally, so that half the stream leaves the
  // last-level cache alone
  auto load_chunk = [&](int id0, int id1, auto tag) {
    load_chunk_tiles<D, decltype(tag)::value ? 0 : kNonTemporal>(kbase, vbase, id0, id1, slot_elems, lane, kreg, vreg);
  };
  // block ids of a cursor's unit; past the sequence's end its last block again
  // (its keys there are masked, its V rows zeroed)
  auto ids_of = [&](const RangeCursor& cu, int& id0, int& id1) {
    const ScalarInts bt = (ScalarInts)(p.block_tables + (size_t)cu.r * p.max_blocks_per_seq);
    const int b0 = cu.x * kUnitBlocks;
    id0 = bt[b0];
    id1 = bt[min(b0 + 1, (cu.len - 1) / kBlock)];
  };
  bf16x8 qreg[DC];
  auto load_q = [&](int r) {
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) {
      qreg[dc] = bf16x8{};
      if (head_valid)
        qreg[dc] = *reinterpret_cast<const bf16x8*>(p.q + ((size_t)r * p.num_q_heads + h) * D + 32 * dc + 8 * qd);
    }
  };

  f32x4 oacc[DT];
  float m_run, l_run;
  auto reset = [&]() {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt] = f32x4{};
    m_run = -INFINITY;
    l_run = 0.f;
  };

  // three cursors: the unit being computed, the one whose loads are in flight
  // behind it, and the one whose block ids are being read
  auto run = [&](auto tag) __attribute__((always_inline)) {
    RangeCursor cur = ids;
    int id0, id1;
    ids_of(cur, id0, id1);
    load_q(cur.r);
    load_chunk(id0, id1, tag);
    reset();
    advance(ids, tag);
    RangeCursor nxt = ids;
    if (nxt.valid) ids_of(nxt, id0, id1);

    for (;;) {
      const int key0 = cur.x * kUnitKeys;
      store_v_tile<D>(vreg, lane, key0, cur.len, sm.v);
      f32x4 s[2] = {f32x4{}, f32x4{}};
  #pragma unroll
      for (int mt = 0; mt < 2; ++mt)
  #pragma unroll
        for (int dc = 0; dc < DC; ++dc)
          s[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kreg[mt][dc], qreg[dc], s[mt], 0, 0, 0);
      // the next unit's loads, in flight during the math; block ids one further
      if (nxt.valid) {
        load_chunk(id0, id1, tag);
        advance(ids, tag);
        if (ids.valid) ids_of(ids, id0, id1);
      }
      float mloc = -INFINITY;
  #pragma unroll
      for (int mt = 0; mt < 2; ++mt)
  #pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int key = key0 + 16 * mt + 4 * qd + rr;
          s[mt][rr] = key < cur.len ? s[mt][rr] : -INFINITY;
          mloc = fmaxf(mloc, s[mt][rr]);
        }
      // A unit's probabilities are relative to its own maximum and its O is
      // rescaled in fp32: the largest of every 32 are then exact in bf16, where
      // against the running maximum of a whole range only a few were.  Relative
      // error against float64, 128 sequences of 4.2k-10.8k keys: 0.00227 with
      // running maxima, 0.00218 with one per wave of a 12-wave work-group, 0.00202
      // so, in the same time (the 64 FMAs of a unit hide behind its loads).
      const float m_unit = fmaxf(quad_max(mloc), lowest);
      const float m_new = fmaxf(m_run, m_unit);
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
      const float beta = __builtin_amdgcn_exp2f((m_unit - m_new) * c);
      m_run = m_new;
      const float mc = m_unit * c;
      bf16x8 pb;
      float l_unit = 0.f;
  #pragma unroll
      for (int mt = 0; mt < 2; ++mt)
  #pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][rr], c, -mc));
          pb[4 * mt + rr] = (__bf16)e;
          l_unit += (float)pb[4 * mt + rr];
        }
      l_run = __builtin_fmaf(l_run, alpha, l_unit * beta);
  #pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const f32x4 o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v_fragment<D>(sm.v, lane, dt), pb, f32x4{}, 0, 0, 0);
  #pragma unroll
        for (int e = 0; e < 4; ++e) oacc[dt][e] = __builtin_fmaf(oacc[dt][e], alpha, o[e] * beta);
      }

      if (cur.x + 1 == cur.xe) {
        // the piece ends: lane (j, qd) holds dims 16 dt + 4 qd .. +3 of head j
        if (nxt.valid) load_q(nxt.r);
        l_run = quad_sum(l_run);
        if (head_valid) {
          if (cur.slot < 0) {
            uint16_t* orow = p.out + ((size_t)cur.r * p.num_q_heads + h) * D;
  #pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
              bf16x4 o;
  #pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = (__bf16)(oacc[dt][e] / l_run);
              *reinterpret_cast<uint2*>(orow + 16 * dt + 4 * qd) = __builtin_bit_cast(uint2, o);
            }
          } else {
            const size_t at = ((size_t)g * p.slots + cur.slot) * p.group + j;
  #pragma unroll
            for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4*>(p.ws_o + at * D + 16 * dt + 4 * qd) = oacc[dt];
            if (qd == 0) *reinterpret_cast<float2*>(p.ws_ml + 2 * at) = make_float2(m_run, l_run);
          }
        }
        if (!nxt.valid) return;
        reset();
      }
      cur = nxt;
      nxt = ids;
    }
  };
  if (aligned)
    run(std::true_type{});
  else
    run(std::false_type{});
}

// One work-group per (sequence, KV head): combines the pieces that
// decode_ranges_kernel left of a sequence (a sequence of one piece has its
// output already).
template <int D>
__global__ __launch_bounds__(kMergeThreads) void decode_ranges_merge_kernel(DecParams p) {
  const int lane = threadIdx.x & 63;
  const int g = blockIdx.x % p.num_kv_heads;
  const int r = blockIdx.x / p.num_kv_heads;
  const int2 plan = *p.plan;
  const bool aligned = plan.x != 0;
  const int per = plan.y;
  // units before r, or (aligned) pieces before r
  int before = 0;
  for (int s = 0; s < r; s += 64) {
    const int x = s + lane < r ? units_of(p.seq_lens[s + lane]) : 0;
    before += wave_total(aligned ? ceil_div(x, per) : x);
  }
  const int units = units_of(p.seq_lens[r]);
  int first, n;                          // the sequence's first slot, and its pieces
  if (aligned) {
    first = before;
    n = ceil_div(units, per);
  } else {
    const int w0 = before / per;
    first = r + w0;
    n = (before + units - 1) / per - w0 + 1;
  }
  // a sequence of one piece has its output; one without keys gets NaN here, as
  // from one work-group per pair
  if (units == 0) n = 0;
  if (n == 1) return;
  const size_t base = ((size_t)g * p.slots + first) * p.group;
  const size_t row = (size_t)r * p.num_q_heads + g * p.group;
  merge_pieces<D>(
      p.ws_o, p.ws_ml, p.group, p.scale_log2, [&](int) { return n; },
      [&](int hj, int k) { return base + (size_t)k * p.group + hj; },
      [&](int hj, int d, bf16x4 o) { *reinterpret_cast<uint2*>(p.out + (row + hj) * D + d) = __builtin_bit_cast(uint2, o); });
}

// One work-group per (sequence, KV head): the final output of cascade decode
// from every partial of the row (shared-prefix chunks, own-key segments).
// The maxima and sums of all partials are gathered into LDS by all threads
// at once, turned into per-partial weights, and every thread then sums its
// output elements over the partials with the loads issued together.
template <int D>
__global__ __launch_bounds__(kThreads) void cascade_merge_kernel(DecParams p) {
  extern __shared__ float wsm[];            // [group][parts]: maxima, then weights
  const int g = blockIdx.x % p.num_kv_heads;
  const int r = blockIdx.x / p.num_kv_heads;
  const int L = p.seq_lens[r];
  const int shared = shared_len_of(p, r);
  const int n_shared = (shared + p.chunk_keys - 1) / p.chunk_keys;
  const int n_own = (L - shared + kCascadeSegmentKeys - 1) / kCascadeSegmentKeys;
  const int n = n_shared + n_own;
  const int stride = p.chunks + p.segments;     // row length of wsm
  float* m_s = wsm;
  float* l_s = wsm + p.group * stride;
  const float c = p.scale_log2;
  const size_t row0 = (size_t)r * p.num_q_heads + g * p.group;
  auto part_of = [&](int i) { return i < n_shared ? i : p.chunks + (i - n_shared); };
  for (int t = threadIdx.x; t < p.group * n; t += kThreads) {
    const int hj = t / n, i = t % n;
    const float2 ml = *reinterpret_cast<const float2*>(p.ws_ml + 2 * ((size_t)part_of(i) * p.ws_rows + row0 + hj));
    m_s[hj * stride + i] = ml.x;
    l_s[hj * stride + i] = ml.y;
  }
  __syncthreads();
  if ((int)threadIdx.x < p.group) {
    const int hj = threadIdx.x;
    float mx = -INFINITY;
    for (int i = 0; i < n; ++i) mx = fmaxf(mx, m_s[hj * stride + i]);
    float den = 0.f;
    for (int i = 0; i < n; ++i) {
      const float wt = __builtin_amdgcn_exp2f((m_s[hj * stride + i] - mx) * c);
      m_s[hj * stride + i] = wt;              // the maximum becomes the weight
      den += wt * l_s[hj * stride + i];
    }
    const float inv = 1.f / den;
    for (int i = 0; i < n; ++i) m_s[hj * stride + i] *= inv;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < p.group * D; idx += kThreads) {
    const int hj = idx / D;
    const int d = idx % D;
    const size_t row = row0 + hj;
    float acc = 0.f;
    int i = 0;
    for (; i + 4 <= n; i += 4) {
      float o[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) o[u] = p.ws_o[((size_t)part_of(i + u) * p.ws_rows + row) * D + d];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc += m_s[hj * stride + i + u] * o[u];
    }
    for (; i < n; ++i) acc += m_s[hj * stride + i] * p.ws_o[((size_t)part_of(i) * p.ws_rows + row) * D + d];
    p.out[row * D + d] = __builtin_bit_cast(uint16_t, (__bf16)acc);
  }
}

}  // namespace

// Ranges or one work-group per (sequence, KV head): ranges win from a few
// hundred keys on, at every batch.  us a call back to back, one work-group per pair
// -> ranges with their merge: 32 / 8 heads of 128, 2 sequences of 84-140 keys 11.1 ->
// 8.2, 3 of 2000-6000 49 -> 14, 24 of 500-9000 115 -> 67, 128 of 100-500 67 -> 35, 128 of
// 4200-10800 676 -> 616; 32 / 8 heads of 64, 128 of 2000-6000 210 -> 181.
// At head_dim 64 up to 512 keys, while the pairs fit one round, the merge launch is
// not paid for (8 sequences of 100-500 keys 8.5 -> 8.6).  Past 512 a full round of
// pairs of nearly equal lengths still loses up to 1.3 us to it, ragged ones gain (32
// sequences, 32 / 8 heads: 448-560 keys 10.6 -> 11.4, 112-560 9.9 -> 9.6, 1600-2000
// 23.9 -> 24.8, 400-2000 20.4 -> 19.5).
DecodeGeometry decode_geometry(int batch, int max_seq_len, int num_kv_heads, int head_dim, int cus) {
  DecodeGeometry geo = {};
  if (batch < 1 || batch > kRangeMaxBatch || max_seq_len <= 128) return geo;
  if (head_dim == 64 && max_seq_len <= 512 && (long long)batch * num_kv_heads <= cus) return geo;
  const int groups_per_cu = head_dim == 128 ? kRangeGroupsPerCu128 : kRangeGroupsPerCu64;
  geo.ranges = std::max(1, groups_per_cu * cus / num_kv_heads);
  const int rounds = aligned_rounds(64) * aligned_rounds(128);     // a whole number of waves at both
  const int pieces = rounds * std::max(1, kAlignedPiecesPerCu / rounds * cus / num_kv_heads);
  geo.aligned_ranges = pieces / aligned_rounds(head_dim);
  geo.slots = std::max(geo.ranges, pieces) + batch;
  return geo;
}

hipError_t launch_paged_decode_attn(const DecodeLaunch& a, hipStream_t stream) {
  DecParams p = {};
  p.q = a.q;
  p.k_pool = a.k_pool;
  p.v_pool = a.v_pool;
  p.block_tables = a.block_tables;
  p.seq_lens = a.seq_lens;
  p.out = a.out;
  p.max_blocks_per_seq = a.max_blocks_per_seq;
  p.num_q_heads = a.num_q_heads;
  p.num_kv_heads = a.num_kv_heads;
  p.group = a.num_q_heads / a.num_kv_heads;
  p.scale_log2 = a.scale * kLog2e;
  p.batch = a.batch;
  const unsigned rows = (unsigned)((long long)a.batch * a.num_kv_heads);
  if (a.ranges > 0) {
    p.ranges = a.ranges;
    p.aligned_ranges = a.aligned_ranges;
    p.slots = a.slots;
    p.ws_o = static_cast<float*>(a.workspace);
    p.ws_ml = p.ws_o + (size_t)a.slots * a.num_q_heads * a.head_dim;
    p.plan = reinterpret_cast<int2*>(p.ws_ml + (size_t)a.slots * a.num_q_heads * 2);
    const dim3 grid((unsigned)(std::max(a.ranges, a.aligned_ranges) * a.num_kv_heads)), block(64);
    if (a.head_dim == 128) {
      hipLaunchKernelGGL(decode_ranges_kernel<128>, grid, block, 0, stream, p);
      hipLaunchKernelGGL(decode_ranges_merge_kernel<128>, dim3(rows), dim3(kMergeThreads), 0, stream, p);
    } else {
      hipLaunchKernelGGL(decode_ranges_kernel<64>, grid, block, 0, stream, p);
      hipLaunchKernelGGL(decode_ranges_merge_kernel<64>, dim3(rows), dim3(kMergeThreads), 0, stream, p);
    }
    return hipGetLastError();
  }
  const dim3 grid(rows), block(64 * kDecodeWaves);
  if (a.head_dim == 128) {
    hipLaunchKernelGGL((paged_decode_attn_kernel<128, false>), grid, block, 0, stream, p);
  } else {
    hipLaunchKernelGGL((paged_decode_attn_kernel<64, false>), grid, block, 0, stream, p);
  }
  return hipGetLastError();
}

hipError_t launch_cascade_decode_rest(const CascadeLaunch& a, hipStream_t stream) {
  const CascadeGeometry geo = cascade_geometry(a.num_groups, a.max_group_seqs, a.max_shared_len,
                                               a.max_rest_len, a.num_q_heads, a.num_kv_heads);
  DecParams p = {};
  p.q = a.q;
  p.k_pool = a.k_pool;
  p.v_pool = a.v_pool;
  p.block_tables = a.block_tables;
  p.seq_lens = a.seq_lens;
  p.out = a.out;
  p.max_blocks_per_seq = a.max_blocks_per_seq;
  p.num_q_heads = a.num_q_heads;
  p.num_kv_heads = a.num_kv_heads;
  p.group = a.num_q_heads / a.num_kv_heads;
  p.scale_log2 = a.scale * kLog2e;
  p.cu_groups = a.cu_groups;
  p.shared_lens = a.shared_lens;
  p.num_groups = a.num_groups;
  p.batch = a.batch;
  p.chunk_keys = geo.chunk_keys;
  p.chunks = geo.chunks;
  p.segments = geo.segments;
  p.ws_o = a.ws_o;
  p.ws_ml = a.ws_ml;
  p.ws_rows = a.batch * a.num_q_heads;
  const long long rows = (long long)a.batch * a.num_kv_heads;
  if (geo.segments > 0) {
    const dim3 grid((unsigned)(rows * geo.segments)), block(64 * kCascadeWaves);
    if (a.head_dim == 128) {
      hipLaunchKernelGGL((paged_decode_attn_kernel<128, true>), grid, block, 0, stream, p);
    } else {
      hipLaunchKernelGGL((paged_decode_attn_kernel<64, true>), grid, block, 0, stream, p);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const size_t lds = 2 * sizeof(float) * (size_t)p.group * (geo.chunks + geo.segments);
  if (a.head_dim == 128) {
    hipLaunchKernelGGL(cascade_merge_kernel<128>, dim3((unsigned)rows), dim3(kThreads), lds, stream, p);
  } else {
    hipLaunchKernelGGL(cascade_merge_kernel<64>, dim3((unsigned)rows), dim3(kThreads), lds, stream, p);
  }
  return hipGetLastError();
}

}  // namespace cs
