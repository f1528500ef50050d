// Cascade decode in ranges for gfx950: the shared prefixes of the groups and
// the sequences' own keys in one launch, dealt evenly to one-wave work-groups.
//
// The operation is cascade decode (arXiv 2608.14624, Sec. 2.1 "Agent anchor",
// Sec. 2.2: every invocation of an agent reads its anchor's blocks): a group of
// sequences shares the keys 0 .. shared_len - 1, which are read once for all of
// its queries; each sequence then has keys of its own.
//
// Kernel design
//   * Both kinds of work are lists of 32-key units over which some query rows
//     attend: a group's shared prefix with the stacked rows of all its
//     sequences and of the KV head's query heads (in column blocks of p.width
//     rows, 16 to 64), and a sequence's own keys with its p.group rows.  The
//     lists are laid end to end, shared prefixes first, and dealt in
//     contiguous ranges of `per` units to p.ranges waves per KV head, as in
//     decode_ranges_kernel; every wave makes the plan from the device metadata.
//   * A wave holds up to four tiles of 16 rows (the columns of
//     v_mfma_f32_16x16x32_bf16): K and V are loaded once per unit and each V
//     fragment read from LDS once for all tiles, so a prefix shared by 64 rows
//     crosses the memory once.
//   * Every piece of a list in a range leaves partial results (O relative to
//     the running max m, m, the sum l) for its rows in the workspace, and
//     cascade_ranges_merge_kernel combines a row's pieces.  `per` is at least
//     what keeps all partials inside the workspace, whose size is that of the
//     chunks and segments of 1024 keys of the other cascade launches.
//
// What bounds it is HBM (the plan's equal ranges keep every wave streaming to
// the end; why few waves, and V non-temporal: at decode_ranges_kernel).
// 128 sequences of 8 agents, shared prefixes of 4-8k, own keys 128-4096 (0.72
// GB of distinct K/V), 32 / 8 heads of 128: the three launches of the other
// path 172 us (shared prefixes 48 us at 4.1 TB/s, own keys 116 us at 4.6, merge
// 9), these two 138 us (126 us at 5.7 TB/s, and 6.5 us).  Four waves per CU at
// head_dim 128 (all that the registers of four tiles allow; three 151 us), eight
// at 64 (six 80 us, eight 77).  Ranges of equal cost instead of equal units, a
// unit of four tiles counted up to twice, were slower (147 to 153 us): the
// waves at the shared prefixes are not the last.
#include "decode_common.h"
#include "internal.h"

#include <float.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

namespace cs {
namespace {

constexpr int kTileRows = 16;
constexpr int kMaxTiles = 4;

struct CascadeParams {
  const uint16_t* q;          // [B][Hq][D]
  const uint16_t* k_pool;
  const uint16_t* v_pool;
  const int32_t* block_tables;
  const int32_t* seq_lens;
  const int32_t* cu_groups;     // [num_groups + 1]
  const int32_t* shared_lens;   // [num_groups]
  uint16_t* out;
  int batch;
  int max_blocks_per_seq;
  int num_groups;
  int num_q_heads;
  int num_kv_heads;
  int group;
  float scale_log2;
  int ranges;                   // waves per KV head
  int width;                    // rows of a column block of a shared prefix
  int rows;                     // partial rows per KV head in the workspace
  float* ws_o;                  // [num_kv_heads][rows][D]
  float* ws_ml;                 // [num_kv_heads][rows][2]
  // the plan, for the merge: kPlanHead values {units per range, first row of
  // the own partials, ranges wholly before the own keys}, then kPlanSeq per
  // sequence {its index in its group, units of the shared prefix, units before
  // it, column blocks before it, units before its own keys, own units}
  int32_t* plan;
};
constexpr int kPlanHead = 8;
constexpr int kPlanSeq = 6;

// A position in a wave's list of pieces.
struct CascadeCursor {
  int x, xe;      // unit within the list, end of the piece
  int len;        // keys of the list
  int row;        // block-table row
  int block;      // its block of the list's first key
  int seq;        // first sequence of the list's rows
  int rho;        // first row: query head rho % group of sequence seq + rho / group
  int rows;       // rows of the list (a column block has at most p.width)
  int at;         // partial row of the first row
  bool valid;
};

template <int D>
__global__ __launch_bounds__(64, D == 64 ? 2 : 1) void cascade_ranges_kernel(CascadeParams p) {
  constexpr int vStride = v_tile_stride(D);
  constexpr int DC = D / 32;
  constexpr int DT = D / 16;
  constexpr int kVLoads = kChunk * D / 8 / 64;
  __shared__ uint16_t vt[kChunk * vStride];
  // lengths of the sequences' own keys; first sequence and shared keys of the groups
  __shared__ int own_len[kRangeMaxBatch];
  __shared__ int group_at[kRangeMaxBatch + 1], group_len[kRangeMaxBatch];

  const int lane = threadIdx.x;
  const int j = lane & 15;
  const int qd = lane >> 4;
  const int g = blockIdx.x % p.num_kv_heads;
  const int w = blockIdx.x / p.num_kv_heads;
  const ScalarInts lens_c = (ScalarInts)p.seq_lens;
  const bool writes_plan = blockIdx.x == 0;

  // ---- the plan.  The lengths are asked for before the groups are waited for.
  int len_next = lane < p.batch ? p.seq_lens[lane] : 0;
  for (int i = lane; i < p.num_groups; i += 64) {
    group_at[i] = p.cu_groups[i];
    group_len[i] = p.shared_lens[i];
  }
  if (lane == 0) group_at[p.num_groups] = p.batch;
  __syncthreads();
  auto group_rows = [&](int gr) { return (group_at[gr + 1] - group_at[gr]) * p.group; };
  // units and column blocks of a lane's group (none where nothing is shared)
  auto group_lists = [&](int gr, int& units, int& blocks) {
    units = blocks = 0;
    if (gr < p.num_groups && group_at[gr + 1] > group_at[gr] && group_len[gr] > 0) {
      units = units_of(group_len[gr]);
      blocks = ceil_div(group_rows(gr), p.width);
    }
  };
  int shared_end = 0, col_blocks = 0;    // units and column blocks of the shared prefixes
  for (int b = 0; b < p.num_groups; b += 64) {
    int units, blocks;
    group_lists(b + lane, units, blocks);
    const int incl = wave_scan(blocks * units), incl_b = wave_scan(blocks);
    // a group's part of the plan, at its first sequence; the others take it from there
    if (writes_plan && b + lane < p.num_groups && group_at[b + lane + 1] > group_at[b + lane]) {
      int32_t* rec = p.plan + kPlanHead + kPlanSeq * group_at[b + lane];
      rec[1] = units;
      rec[2] = shared_end + incl - blocks * units;
      rec[3] = col_blocks + incl_b - blocks;
    }
    shared_end += __builtin_amdgcn_readlane(incl, 63);
    col_blocks += __builtin_amdgcn_readlane(incl_b, 63);
  }
  if (writes_plan) __syncthreads();
  int total = shared_end;
  for (int b = 0; b < p.batch; b += 64) {
    const int s = b + lane;
    const int len = len_next;
    int first = 0;                         // of the sequence's group
    len_next = s + 64 < p.batch ? p.seq_lens[s + 64] : 0;
    int own = 0;
    if (s < p.batch) {
      int lo = 0, hi = p.num_groups - 1;   // the last group that starts at or before s
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (group_at[mid] <= s) lo = mid; else hi = mid - 1;
      }
      first = group_at[lo];
      own = max(len - max(group_len[lo], 0), 0);
      own_len[s] = own;
    }
    const int units = units_of(own);
    const int incl = wave_scan(units);
    if (writes_plan && s < p.batch) {
      int32_t* rec = p.plan + kPlanHead + kPlanSeq * s;
      const int32_t* of_group = p.plan + kPlanHead + kPlanSeq * first;
      rec[0] = s - first;
      rec[1] = of_group[1];
      rec[2] = of_group[2];
      rec[3] = of_group[3];
      rec[4] = total + incl - units;
      rec[5] = units;
    }
    total += __builtin_amdgcn_readlane(incl, 63);
  }
  __syncthreads();
  // A list of n units is cut into at most n / per + 2 pieces, so `per` must be
  // large enough that the partials of all of them fit the workspace.
  const long long fixed = (long long)(col_blocks + 2) * p.width + (long long)(p.batch + 2) * p.group;
  const long long partials = (long long)shared_end * p.width + (long long)(total - shared_end) * p.group;
  const int room = max(1, p.rows - (int)fixed);
  int per = max(1, ceil_div(total, p.ranges));
  if (partials > (long long)per * room) per = (int)((partials + room - 1) / room);
  const int own_w = shared_end / per;                                // first range with own keys
  const int own_at = (col_blocks + own_w + 1) * p.width;             // their first partial row
  if (writes_plan && lane == 0) {
    p.plan[0] = per;
    p.plan[1] = own_at;
    p.plan[2] = own_w;
  }

  // this range: units begin .. end - 1
  const int begin = w * per;
  const int end = min(total, begin + per);
  if (begin >= end) return;

  // the list the wave is at: column block cb of group gr, or sequence r's own
  // keys; the units before it
  int gr = 0, cb = 0, cb_index = 0, r = -1, list_at = 0;
  bool own = false;
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  // the list's units from x on that are in the range
  auto take = [&](CascadeCursor& c, int x) {
    c.x = x;
    c.xe = min(units_of(c.len), end - list_at);
    c.valid = true;
  };
  auto at_shared = [&](CascadeCursor& c) {
    const int s0 = uniform(group_at[gr]);
    c.len = uniform(group_len[gr]);
    c.row = s0;
    c.block = 0;
    c.seq = s0;
    c.rho = cb * p.width;
    c.rows = min(uniform(group_rows(gr)) - c.rho, p.width);
    c.at = (cb_index + w) * p.width;
  };
  auto at_own = [&](CascadeCursor& c) {
    c.len = uniform(own_len[r]);
    c.row = r;
    c.block = (lens_c[r] - c.len) / kBlock;
    c.seq = r;
    c.rho = 0;
    c.rows = p.group;
    c.at = own_at + (r + w - own_w) * p.group;
  };
  // the unit after the cursor's: in its piece, or the first of the next list
  // if that starts in the range
  auto advance = [&](CascadeCursor& c) {
    if (++c.x < c.xe) return;
    list_at += units_of(c.len);
    if (list_at >= end) {
      c.valid = false;
      return;
    }
    if (!own) {
      ++cb_index;
      if ((cb + 1) * p.width < uniform(group_rows(gr))) {
        ++cb;
      } else {
        cb = 0;
        do ++gr;
        while (gr < p.num_groups && (uniform(group_len[gr]) <= 0 || uniform(group_rows(gr)) <= 0));
        own = gr >= p.num_groups;
      }
    }
    if (own) {
      do ++r;
      while (uniform(own_len[r]) <= 0);
      at_own(c);
    } else {
      at_shared(c);
    }
    take(c, 0);
  };

  CascadeCursor ids{};
  if (begin < shared_end) {
    for (int b = 0;; b += 64) {
      int units, blocks;
      group_lists(b + lane, units, blocks);
      const int incl = wave_scan(blocks * units), incl_b = wave_scan(blocks);
      const unsigned long long past = __builtin_amdgcn_ballot_w64(list_at + incl > begin);
      if (past != 0) {
        const int l = __builtin_ctzll(past);
        gr = b + l;
        const int n = __builtin_amdgcn_readlane(units, l);
        list_at += __builtin_amdgcn_readlane(incl - blocks * units, l);
        cb = (begin - list_at) / n;
        cb_index += __builtin_amdgcn_readlane(incl_b - blocks, l) + cb;
        list_at += cb * n;
        at_shared(ids);
        break;
      }
      list_at += __builtin_amdgcn_readlane(incl, 63);
      cb_index += __builtin_amdgcn_readlane(incl_b, 63);
    }
  } else {
    own = true;
    list_at = shared_end;
    for (int b = 0;; b += 64) {
      const int n = b + lane < p.batch ? units_of(own_len[b + lane]) : 0;
      const int incl = wave_scan(n);
      const unsigned long long past = __builtin_amdgcn_ballot_w64(list_at + incl > begin);
      if (past != 0) {
        const int l = __builtin_ctzll(past);
        r = b + l;
        list_at += __builtin_amdgcn_readlane(incl - n, l);
        at_own(ids);
        break;
      }
      list_at += __builtin_amdgcn_readlane(incl, 63);
    }
  }
  take(ids, begin - list_at);

  const size_t tile_elems = (size_t)kBlock * D;
  const size_t slot_elems = (size_t)p.num_kv_heads * tile_elems;
  const uint16_t* kbase = p.k_pool + (size_t)g * tile_elems;
  const uint16_t* vbase = p.v_pool + (size_t)g * tile_elems;
  const float c = p.scale_log2;
  const float drop = 8.f / c;
  // a unit whose logits are all -inf weighs 0 relative to this, not NaN
  const float lowest = -FLT_MAX / fmaxf(c, 1.f);

  bf16x8 kreg[2][DC];
  bf16x8 vreg[kVLoads];
  auto load_chunk = [&](int id0, int id1) {
    load_chunk_tiles<D, kNonTemporal>(kbase, vbase, id0, id1, slot_elems, lane, kreg, vreg);
  };
  // block ids of a cursor's unit; past the list's end its last block again (its
  // keys there are masked, its V rows zeroed)
  auto ids_of = [&](const CascadeCursor& cu, int& id0, int& id1) {
    const ScalarInts bt = (ScalarInts)(p.block_tables + (size_t)cu.row * p.max_blocks_per_seq + cu.block);
    const int b0 = cu.x * kUnitBlocks;
    id0 = bt[b0];
    id1 = bt[min(b0 + 1, (cu.len - 1) / kBlock)];
  };
  // three cursors: the unit being computed, the one whose loads are in flight
  // behind it, and the one whose block ids are being read
  CascadeCursor cur = ids;
  int id0, id1;
  ids_of(cur, id0, id1);
  load_chunk(id0, id1);
  advance(ids);
  CascadeCursor nxt = ids;
  if (nxt.valid) ids_of(nxt, id0, id1);

  // One piece of a list whose rows fill NT tiles of 16, the tiles' independent
  // chains interleaved (with a branch per tile instead, a unit of four tiles
  // took 10 us); rows past the list's last hold q = 0.
  auto run_piece = [&](auto nt_tag) __attribute__((always_inline)) {
    constexpr int NT = decltype(nt_tag)::value;
    constexpr int kEvery = NT == 1 ? 1 : 8;
    // Q^T operands: column j of tile t is row rho + 16 t + j of the list
    bf16x8 qreg[NT][DC];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int i = t * kTileRows + j;
      const int rho = cur.rho + (i < cur.rows ? i : 0);
      const uint16_t* src = p.q + ((size_t)(cur.seq + rho / p.group) * p.num_q_heads + g * p.group + rho % p.group) * D;
#pragma unroll
      for (int dc = 0; dc < DC; ++dc) {
        qreg[t][dc] = bf16x8{};
        if (i < cur.rows) qreg[t][dc] = *reinterpret_cast<const bf16x8*>(src + 32 * dc + 8 * qd);
      }
    }
    f32x4 oacc[NT][DT];
    float m_run[NT], m_max[NT], l_run[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) oacc[t][dt] = f32x4{};
      m_run[t] = m_max[t] = -INFINITY;
      l_run[t] = 0.f;
    }
    for (;;) {
      const int key0 = cur.x * kUnitKeys;
      store_v_tile<D>(vreg, lane, key0, cur.len, vt);
      f32x4 s[NT][2];
#pragma unroll
      for (int t = 0; t < NT; ++t) s[t][0] = s[t][1] = f32x4{};
#pragma unroll
      for (int dc = 0; dc < DC; ++dc)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int t = 0; t < NT; ++t)
            s[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kreg[mt][dc], qreg[t][dc], s[t][mt], 0, 0, 0);
      // the next unit's loads, in flight during the math; block ids one further
      if (nxt.valid) {
        load_chunk(id0, id1);
        advance(ids);
        if (ids.valid) ids_of(ids, id0, id1);
      }
      // mask keys past the end; register rr of tile mt holds key 16 mt + 4 qd + rr
      if (key0 + kChunk > cur.len) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
              s[t][mt][rr] = key0 + 16 * mt + 4 * qd + rr < cur.len ? s[t][mt][rr] : -INFINITY;
      }
      // The reference maximum of the probabilities moves where a row's max grew by
      // more than 2^8, and every kEvery units to the unit's own (but never 2^8
      // below the largest so far): the largest probabilities of those units are
      // then exact in bf16.  Relative error against float64, with a reference that
      // only grew, now, and in chunks and segments: 128 sequences of 8 agents
      // 0.00234, 0.00228, 0.00231 in the same time (154 us); 48 with 1000 shared
      // and up to 4000 own keys 0.00232, 0.00221, 0.00226.  Every unit for own
      // keys is free; for stacked rows every fourth costs 1-2%, every unit 2-8%.
      float mloc[NT];
      bool grow = false;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        mloc[t] = fmaxf(quad_max(fmaxf(fmaxf(fmaxf(s[t][0][0], s[t][0][1]), fmaxf(s[t][0][2], s[t][0][3])),
                                       fmaxf(fmaxf(s[t][1][0], s[t][1][1]), fmaxf(s[t][1][2], s[t][1][3])))),
                        lowest);
        m_max[t] = fmaxf(m_max[t], mloc[t]);
        grow |= (mloc[t] - m_run[t]) * c > 8.f;      // true for every row at a piece's first unit
      }
      if (cur.x % kEvery == 0 || __builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float m_new = fmaxf(mloc[t], m_max[t] - drop);
          const float alpha = __builtin_amdgcn_exp2f((m_run[t] - m_new) * c);
          m_run[t] = m_new;
          l_run[t] *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) oacc[t][dt] *= alpha;
        }
      }
      bf16x8 pb[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float mc = m_run[t] * c;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr)
            pb[t][4 * mt + rr] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[t][mt][rr], c, -mc));
        // row sum over the same bf16 probabilities the PV product uses
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
        l_run[t] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t], pb[t], 0, 1), ones, l_run[t], false);
        l_run[t] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t], pb[t], 2, 3), ones, l_run[t], false);
        l_run[t] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t], pb[t], 4, 5), ones, l_run[t], false);
        l_run[t] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t], pb[t], 6, 7), ones, l_run[t], false);
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const bf16x8 v = v_fragment<D>(vt, lane, dt);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          oacc[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pb[t], oacc[t][dt], 0, 0, 0);
      }
      if (cur.x + 1 == cur.xe) break;
      cur = nxt;
      nxt = ids;
    }
    // the partial: lane (j, qd) holds dims 16 dt + 4 qd .. +3 of row j of a tile
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float l = quad_sum(l_run[t]);
      if (t * kTileRows + j < cur.rows) {
        const size_t at = (size_t)g * p.rows + cur.at + t * kTileRows + j;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4*>(p.ws_o + at * D + 16 * dt + 4 * qd) = oacc[t][dt];
        if (qd == 0) *reinterpret_cast<float2*>(p.ws_ml + 2 * at) = make_float2(m_run[t], l);
      }
    }
    cur = nxt;
    nxt = ids;
  };
  while (cur.valid) {
    if (cur.rows <= kTileRows)
      run_piece(std::integral_constant<int, 1>{});
    else if (cur.rows <= 2 * kTileRows)
      run_piece(std::integral_constant<int, 2>{});
    else
      run_piece(std::integral_constant<int, 4>{});
  }
}

// One work-group per (sequence, KV head): combines the pieces of its group's
// shared prefix and of its own keys.
template <int D>
__global__ __launch_bounds__(kMergeThreads) void cascade_ranges_merge_kernel(CascadeParams p) {
  const int g = blockIdx.x % p.num_kv_heads;
  const int r = blockIdx.x / p.num_kv_heads;
  const ScalarInts plan = (ScalarInts)p.plan;
  const int per = plan[0], own_at = plan[1], own_w = plan[2];
  const ScalarInts rec = plan + kPlanHead + kPlanSeq * r;
  const int index = rec[0], n_units = rec[1], group_first = rec[2], group_cb = rec[3];
  const int own_first = rec[4], own_units = rec[5];
  const int w_own = own_first / per;
  const int n_own = own_units > 0 ? (own_first + own_units - 1) / per - w_own + 1 : 0;
  // row hj's column block of the shared prefix, its pieces there
  const size_t row = (size_t)r * p.num_q_heads + g * p.group;
  const int own_row = own_at + (r + w_own - own_w) * p.group;
  int n_shared = 0, shared_row = 0;
  auto pieces = [&](int hj) {
    const int rho = index * p.group + hj;
    const int cb = rho / p.width;
    const int cb_first = group_first + cb * n_units;
    const int w_cb = cb_first / per;
    n_shared = n_units > 0 ? (cb_first + n_units - 1) / per - w_cb + 1 : 0;
    shared_row = (group_cb + cb + w_cb) * p.width + rho % p.width;
    return n_shared + n_own;
  };
  merge_pieces<D>(
      p.ws_o, p.ws_ml, p.group, p.scale_log2, pieces,
      [&](int hj, int k) {
        return (size_t)g * p.rows +
               (k < n_shared ? shared_row + k * p.width : own_row + hj + (k - n_shared) * p.group);
      },
      [&](int hj, int d, bf16x4 o) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const __bf16 x = o[e];
          p.out[(row + hj) * D + d + e] = __builtin_bit_cast(uint16_t, x);
        }
      });
}

}  // namespace

// one-wave work-groups per CU: at head_dim 128 four fit (registers)
constexpr int kCascadeGroupsPerCu128 = 4;
constexpr int kCascadeGroupsPerCu64 = 8;

// Ranges need room: besides a piece per range, every list may be cut once more,
// and the plan itself takes some rows; what is left bounds the number of pieces,
// so a small batch's workspace may allow only ranges `stretch` times as long as an
// equal share.  And a prefix is streamed once for every column block of its
// group, by other waves at other times, in units of up to four tiles.
// The host knows the bounds of the lengths alone, so it compares two estimates,
// with prefixes at their bound and own parts at 0.4 of theirs.  In us, for
// shared, own and distinct shared (once per group) units per range, fitted to 296
// calls (32 / 8, 64 / 8, 16 / 16 and 8 / 2 heads at 64 and 128, 8 to 160 sequences
// of 1 to 12 agents, prefixes of 1000 to 10000 keys, own bounds of 200 to 4000):
// chunks 21 + 1.1 shared + 3 own + 2.5 distinct, ranges (0.8 + 1.2 x tiles / 4 x
// share of shared units) x units per range + 1.5 (own + distinct).  Ranges are
// taken where they come out 5% ahead: on average 1% slower than the better of the
// two, where a rule on the stretch alone (3) was 6%.  us a call, chunks -> ranges:
//   128 sequences of 8 agents, 32 / 8 heads of 128       190 -> 154   taken
//   16 of 4 agents, prefixes of 10000, own 4000           85 -> 59    taken
//   128 of one agent, 64 / 8, 8000, own 2500             185 -> 169   taken
//   64 of one agent, 32 / 8, 8000, own 600                56 -> 90
//   128 of one agent, 64 / 8, 2300, own 600               67 -> 115
//   160 of 4 agents, 32 / 8 of 64, 8000, own 600          59 -> 84
//   96 of 3 agents, 64 / 8, 10000, own 1200               97 -> 106   taken
//   128 of 8 agents, 32 / 8, 10000, own 200              105 -> 88
// With one query head per KV head, whose partials are small, long ranges end
// late: at a stretch of 2.4, 32 sequences of 8 agents, 16 / 16 heads, 183 -> 266.
CascadeRanges cascade_ranges(int batch, int num_groups, int max_group_seqs, int max_shared_len,
                             int max_rest_len, int num_q_heads, int num_kv_heads, int head_dim,
                             long long parts, int cus) {
  CascadeRanges geo = {};
  if (batch > kRangeMaxBatch) return geo;
  const int group = num_q_heads / num_kv_heads;
  const long long plan_rows = (kPlanSeq * (long long)batch + kPlanHead + 1) / 2;   // of 8 bytes in ws_ml
  const long long rows = (parts * batch * num_q_heads - plan_rows) / num_kv_heads;
  const int width = (int)std::min<long long>(kMaxTiles * kTileRows,
                                             ((long long)max_group_seqs * group + kTileRows - 1) / kTileRows * kTileRows);
  const long long col_blocks = (long long)batch * group / width + num_groups;
  const long long fixed = (col_blocks + 2) * width + (batch + 2LL) * group;
  const long long room = rows - fixed;
  if (room <= 0 || rows > 0x7fffffffLL) return geo;
  const int ranges = std::max(1, (head_dim == 128 ? kCascadeGroupsPerCu128 : kCascadeGroupsPerCu64) * cus / num_kv_heads);
  const double per_unit = 1. / ((double)kUnitKeys * ranges);
  const double shared = per_unit * (((long long)batch * group + width - 1) / width) * max_shared_len;
  const double distinct = std::min(shared, per_unit * num_groups * max_shared_len);
  const double own = per_unit * 0.4 * batch * max_rest_len;
  const double share = shared + own;
  const double stretch = share > 0. ? (shared * width + own * group) * ranges / (share * room) : 1.;
  if (stretch > (group == 1 ? 2. : 3.)) return geo;
  const double chunks_us = 21. + 1.1 * shared + 3. * own + 2.5 * distinct;
  const double ranges_us = std::max(stretch, 1.) * (0.8 * share + 1.2 * width / (kMaxTiles * kTileRows) * shared) +
                           1.5 * (own + distinct);
  if (ranges_us > 0.95 * chunks_us) return geo;
  geo.ranges = ranges;
  geo.width = width;
  geo.rows = (int)rows;
  return geo;
}

hipError_t launch_cascade_ranges(const CascadeLaunch& a, const CascadeRanges& geo, hipStream_t stream) {
  CascadeParams p;
  p.q = a.q;
  p.k_pool = a.k_pool;
  p.v_pool = a.v_pool;
  p.block_tables = a.block_tables;
  p.seq_lens = a.seq_lens;
  p.cu_groups = a.cu_groups;
  p.shared_lens = a.shared_lens;
  p.out = a.out;
  p.batch = a.batch;
  p.max_blocks_per_seq = a.max_blocks_per_seq;
  p.num_groups = a.num_groups;
  p.num_q_heads = a.num_q_heads;
  p.num_kv_heads = a.num_kv_heads;
  p.group = a.num_q_heads / a.num_kv_heads;
  p.scale_log2 = a.scale * kLog2e;
  p.ranges = geo.ranges;
  p.width = geo.width;
  p.rows = geo.rows;
  p.ws_o = a.ws_o;
  p.ws_ml = a.ws_ml;
  p.plan = reinterpret_cast<int32_t*>(a.ws_ml + 2 * (size_t)geo.rows * a.num_kv_heads);
  const dim3 grid((unsigned)(geo.ranges * a.num_kv_heads)), rows((unsigned)(a.batch * a.num_kv_heads));
  if (a.head_dim == 128) {
    hipLaunchKernelGGL(cascade_ranges_kernel<128>, grid, dim3(64), 0, stream, p);
    hipLaunchKernelGGL(cascade_ranges_merge_kernel<128>, rows, dim3(kMergeThreads), 0, stream, p);
  } else {
    hipLaunchKernelGGL(cascade_ranges_kernel<64>, grid, dim3(64), 0, stream, p);
    hipLaunchKernelGGL(cascade_ranges_merge_kernel<64>, rows, dim3(kMergeThreads), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace cs
