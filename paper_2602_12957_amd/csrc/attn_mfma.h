// Verification attention on the matrix cores (bf16 MFMA 32x32x16, fp32 online softmax).
//
// What it computes (paper Section 3.2, Eq. 8 in the chain case of the tree-ancestry mask): draft row r of
// sequence s at absolute position p attends to the cached positions 0..p of s -- the accepted prefix plus
// the rows before it in its own block, which the QKV epilogue appended to the pages just before.
//
// Work split.  A workgroup owns one (sequence, kv head, tile of query rows).  A wave holds 32 queries of one query head
// (lane l <-> query l % 32); the waves of a workgroup are the query heads that share the kv head (GQA) and/or further 32-row
// sub-tiles, so every 128-key K/V stage in LDS is used by all of them: 4 waves for region-level batches (many short
// blocks, Eq. 2), 8 for page-level ones (few long blocks, Eq. 4: twice the reuse of each stage).
//
// One row's arithmetic is the same in every variant and every batch: its keys are visited in 64-key groups at
// absolute positions, even groups by one accumulator set and odd groups by another ("parity"), in ascending order, and the
// two sets are folded at the end (even first).  Verification of a block and token-by-token decoding therefore give
// the same bits.
//
// Orientation.  Both products are computed transposed so that a lane owns ONE query:
//   S^T = K Q^T   (MFMA i = key, j = query)  -> the lane's 32 registers per step are 32 keys of its query;
//   O^T = V^T P^T (MFMA i = head dim, j = query) -> a correction factor is a per-lane scalar.
// P^T is fed straight from the S^T registers as the B operand.  Register v of lane half h holds key
// 8*(v/4) + 4h + v%4, so the contraction slots of a 16-key step are keys {4h..4h+3, 8+4h..8+4h+3}; the V
// pages are stored transposed and in exactly that token order ([dim][perm(token)], see kv_v_slot), hence the
// A operand of the second product is one 16-byte LDS read per lane and no transpose is ever done here.
//
// What bounds it, and why a wave holds both parities.  A group of 64 keys is 16 matrix instructions (32 cycles each), eight small
// ones (8 cycles) for the row sums, and 32 exponentials and 16 conversions per lane.  The matrix pipe and the vector unit run
// side by side only if independent work of both kinds is in the instruction stream: microbenchmark, one wave per SIMD, ns per
// group: products alone 225, vector part alone 190, both interleaved 230 to 260.  With one parity to a wave, four waves per SIMD
// in step behind a barrier a stage, each waited for its own chain of reads, products, maximum, exponentials and products: 577 ns
// a group (four pages of 8193 rows: 1907 us a layer).  Here, in every turn, the exponentials of one parity run beside the
// products of the other, in an order fixed by hand; what the exponentials need beside (maximum, subtraction, rescaling) is taken
// out of the common case (attn_reference: a pass over those pages takes 68 ms, and 72 with queries and keys scaled by 8, where
// most reference points are not 0; 105 when such groups had to subtract and went through the general rule), and the keys and
// values are requested by LDS-direct loads, so that staging takes no registers and no store instructions.  On the way (us a
// layer at that size): no running maximum 1757; both parities in a wave 1779; row sums without v_dot2 1731; the order pinned 1594.
// 16 regions of 17 to 257 rows on 1055 keys: 29.7 -> 26.2.  What is left there: the matrix pipe is busy for 64 % of the launch, 10 %
// of it is its last tasks, and 28 % of a wave's time are waits for LDS reads and at barriers.
//
// The key loop has two forms.  Stages whose every key is visible to every query of the workgroup (the bulk of a
// cached prefix) run with no mask and no validity checks; the last one or two stages of a
// workgroup (the diagonal of the causal mask, the tree-ancestry mask, the partly filled last page) run the
// checked form.
#pragma once

#include "common.h"
#include "gemm_mfma.h"
#include "misc_kernels.h"

namespace hsd {

constexpr int kAttnKeys = 128;            // keys per LDS stage: 8 pages; keys 0-63 are parity 0's, 64-127 parity 1's
// LDS: three stages of K rows, then two of V^T pages (a stage's V is wanted half a stage after its K, and its K may have to be
// read a second time); 80 KB, so that two workgroups of four waves share a compute unit (eight waves of 242 registers or more fill it)
constexpr int kAttnHalfStage = kAttnKeys * kHd * 2;
constexpr int kAttnKStages = 3, kAttnVStages = 2;
constexpr size_t kAttnLdsBytes = (kAttnKStages + kAttnVStages) * kAttnHalfStage;

// What a workgroup needs to know about its task -- one (query tile, kv head group) -- resolved once per pass instead
// of by every workgroup of every layer (a binary search and four dependent reads before the first K/V request
// could go out).
struct __attribute__((aligned(32))) AttnTile {
  int32_t seq;          // batch index of the sequence, -1: no task (padding of the launch)
  int32_t tile_in_seq;  // index of the tile among the sequence's tiles
  int32_t slot;         // state row (seq_len / block_table row)
  int32_t S, base, Lq;  // cached length, first row and number of rows of the sequence's block
  int32_t y;            // kv head * (head groups per kv head) + head group
  int32_t pack;         // k_attn_wide only: 4 * (index of the set among the tile's head sets) + log2(heads per set)
};

// Query sets of k_attn_wide.  A set is 32 columns: 2^lhp query heads of 32 >> lhp rows each, as many heads as the rows of
// the sequence leave room for, so that short blocks read K and V once for several heads.  g4 = query heads of a kv head
// among the sets of a tile (1, 2 or 4); a tile of 32 rows (or the whole short block) is g4 >> lhp sets, and the sets of a
// sequence are numbered tile by tile.
__host__ __device__ inline int attn_wide_lhp(int Lq, int g4) { return (g4 == 4 && Lq <= 8) ? 2 : (g4 >= 2 && Lq <= 16) ? 1 : 0; }
__host__ __device__ inline int attn_wide_sets(int Lq, int g4) { return ((Lq + 31) / 32) * (g4 >> attn_wide_lhp(Lq, g4)); }

constexpr int kAttnMaxGroups = 1024;   // task groups placed by the balancing pass (more: plain order)
// Workgroups in the launch for `max_tiles` query tiles (an upper bound known on the host), `n_y` head groups and
// groups of `sub_tiles` tiles: 8 lists of equal length with room for the unevenness the placement can leave.
__host__ __device__ inline int attn_grid_size(int max_tiles, int n_y, int sub_tiles) {
  return 8 * ((max_tiles * n_y + 7) / 8 + sub_tiles);
}

// Task table of an attention launch: tasks[i] is the task of workgroup i, for i < n_wg = attn_grid_size(...).
// wide_g4 = 0: a task is a tile of q_tile rows.  wide_g4 > 0 (k_attn_wide): a task is a query set (see attn_wide_lhp);
// "tile" below then means a set, q_tile is 32.
//
// Placement.  Workgroup i runs on XCD i % 8 (workgroups go to the 8 XCDs round robin), and each XCD has its own L2.
// The tiles of one sequence and kv head read the same K/V, so they should meet in one L2: tasks are grouped by
// (sequence, head group, run of `sub_tiles` consecutive tiles), every group goes to ONE XCD as a whole, and the
// groups are dealt to the XCDs heaviest first, each to the XCD with the least work so far (work = 128-key stages a
// task walks) among those whose list still has room, which keeps the 8 lists level.  Inside a group the tile with
// the most keys comes first, and heavy groups come first in every list, so the long tasks of a ragged batch start
// early instead of forming the tail.  List x's j-th task becomes workgroup 8 j + x; workgroups past the end of a
// list find seq = -1.  Batches with more than kAttnMaxGroups groups are even enough by sheer number: they keep the
// plain order (sequence by sequence, heaviest tile first).
// The placement moves work between compute units and changes no result.  One block of 1024 threads; `lds`: kAttnTilesLds
// ints, 8-byte aligned.
constexpr int kAttnTilesLds = HSD_MAX_SEQ + 16 + 8 * kAttnMaxGroups;
__device__ inline void attn_tiles_block(const PassSetup &ps, int *lds) {
  int *s_cnt = lds;                        // per sequence: groups (or tiles) before it, after the scan
  int *s_part = lds + HSD_MAX_SEQ;
  uint64_t *g_sort = reinterpret_cast<uint64_t *>(s_part + 16);   // (heaviest task, work, lower index) of a group, larger first
  int *g_work = reinterpret_cast<int *>(g_sort + kAttnMaxGroups), *g_n = g_work + kAttnMaxGroups;
  int *o_group = g_n + kAttnMaxGroups, *o_nw = o_group + kAttnMaxGroups;   // the groups in dealing order; tasks and work
  int *g_bin = g_work, *g_pos = g_n;       // where a group went (the work and task counts have been copied by then)
  const int32_t *__restrict__ cu_q = ps.cu_q, *__restrict__ seq_slot = ps.seq_slot, *__restrict__ seq_len = ps.seq_len;
  const int n_seq = ps.n_seq, n_slots = ps.n_slots, q_tile = ps.q_tile, n_y = ps.n_y, sub_tiles = ps.sub_tiles, n_wg = ps.n_wg,
            wide_g4 = ps.wide_g4;
  AttnTile *__restrict__ tasks = ps.tasks;
  const int t = threadIdx.x;
  const AttnTile none{-1, 0, 0, 0, 0, 0, 0, 0};
  auto tiles_of = [&](int Lq) { return wide_g4 > 0 ? attn_wide_sets(Lq, wide_g4) : (Lq + q_tile - 1) / q_tile; };
  auto task_of = [&](int s, int tile, int slot, int S, int base, int Lq, int y) {
    if (wide_g4 <= 0) return AttnTile{s, tile, slot, S, base, Lq, y, 0};
    const int lhp = attn_wide_lhp(Lq, wide_g4), sets = wide_g4 >> lhp;
    return AttnTile{s, tile / sets, slot, S, base, Lq, y, 4 * (tile % sets) + lhp};
  };
  for (int i = t; i < n_wg; i += blockDim.x) tasks[i] = none;
  for (int s = t; s < n_seq; s += blockDim.x) {
    const int tiles = tiles_of(cu_q[s + 1] - cu_q[s]);
    s_cnt[s] = n_y * ((tiles + sub_tiles - 1) / sub_tiles);
  }
  __syncthreads();   // also: the padding above is complete before any task is written
  const int n_groups = block_exclusive_scan_4096(s_cnt, n_seq, s_part);
  if (n_groups > kAttnMaxGroups) {
    __syncthreads();
    for (int s = t; s < n_seq; s += blockDim.x) s_cnt[s] = tiles_of(cu_q[s + 1] - cu_q[s]);
    __syncthreads();
    block_exclusive_scan_4096(s_cnt, n_seq, s_part);
    for (int s = t; s < n_seq; s += blockDim.x) {
      const int slot = slot_of(seq_slot, s, n_slots), base = cu_q[s], Lq = cu_q[s + 1] - base;
      const int tiles = tiles_of(Lq), S = seq_len[slot];
      for (int k = 0; k < tiles; ++k)
        for (int y = 0; y < n_y; ++y) {
          const int i = (s_cnt[s] + k) * n_y + y;
          if (i < n_wg) tasks[i] = task_of(s, tiles - 1 - k, slot, S, base, Lq, y);
        }
    }
    return;
  }
  // group t of the batch: sequence s, head group y = local % n_y, tiles [t0, t1) with t0 = (local / n_y) * sub_tiles
  int gs = 0, gy = 0, t0 = 0, t1 = 0, slot = 0, S = 0, base = 0, Lq = 0;
  auto stages_of = [&](int tile) {
    const int rt = wide_g4 > 0 ? tile / (wide_g4 >> attn_wide_lhp(Lq, wide_g4)) : tile;
    return (S + min((rt + 1) * q_tile, Lq) + kAttnKeys - 1) / kAttnKeys;
  };
  if (t < n_groups) {
    int lo = 0, hi = n_seq - 1;   // last sequence whose first group is <= t (every sequence has at least one)
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_cnt[mid] <= t) lo = mid; else hi = mid - 1;
    }
    gs = lo;
    const int local = t - s_cnt[gs];
    gy = local % n_y;
    slot = slot_of(seq_slot, gs, n_slots);
    S = seq_len[slot];
    base = cu_q[gs];
    Lq = cu_q[gs + 1] - base;
    t0 = (local / n_y) * sub_tiles;
    t1 = min(t0 + sub_tiles, tiles_of(Lq));
    int w = 0;
    for (int tile = t0; tile < t1; ++tile) w += stages_of(tile);
    g_work[t] = w;
    g_n[t] = t1 - t0;
    // heaviest task first, then more work first, then lower index (stages below 2^26, work below 2^28)
    g_sort[t] = (static_cast<uint64_t>(stages_of(t1 - 1)) << 38) | (static_cast<uint64_t>(w) << 10) | (1023 - t);
  } else if (t < kAttnMaxGroups) {
    g_sort[t] = 0;
  }
  __syncthreads();
  if (t < n_groups) {
    int rank = 0;
    const uint64_t mine = g_sort[t];
    for (int o = 0; o < n_groups; o += 8) {
#pragma unroll
      for (int j = 0; j < 8; ++j) rank += g_sort[o + j] > mine;   // (0 past the last group)
    }
    o_group[rank] = t;
    o_nw[rank] = (g_work[t] << 4) | g_n[t];   // a group has at most 8 tasks
  }
  __syncthreads();
  if (t < kWave) {
    // One wave deals the groups; lane x < 8 keeps list x's work and length in registers.  Eight groups at a time: the
    // heaviest to the list with the least work, the second to the next ... (one group at a time cost 0.2 us each, 57 us for
    // 64 sequences).  The lists hold n_wg / 8 tasks each and the tasks number at most 8 * (n_wg / 8 - sub_tiles), so some
    // list always has room for one more group of at most sub_tiles tasks: a round in which a list might overflow is dealt
    // one group after the other, each to the list with the least work among those with room.
    const int cap = n_wg / 8;
    int load = 0, count = 0;
    for (int r0 = 0; r0 < n_groups; r0 += 8) {
      const int m = min(8, n_groups - r0);
      if (__any(t < 8 && count + sub_tiles > cap)) {
        for (int j = 0; j < m; ++j) {
          const int nw = o_nw[r0 + j], n = nw & 15;
          int key = (t < 8 && count + n <= cap) ? ((load << 3) | t) : 0x7fffffff;
          key = min(key, __builtin_amdgcn_update_dpp(0x7fffffff, key, 0xB1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
          key = min(key, __builtin_amdgcn_update_dpp(0x7fffffff, key, 0x4E, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
          key = min(key, __builtin_amdgcn_update_dpp(0x7fffffff, key, 0x141, 0xf, 0xf, false));   // row_half_mirror
          const int best = __builtin_amdgcn_readfirstlane(key) & 7;
          if (t == best) {
            const int g = o_group[r0 + j];
            g_bin[g] = t;
            g_pos[g] = count;
            load += nw >> 4;
            count += n;
          }
        }
      } else {
        int place = 0;   // of this lane's list among the eight, least work first
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int other = __builtin_amdgcn_readlane(load, x);
          place += (other < load) || (other == load && x < t);
        }
        if (t < 8 && place < m) {
          const int g = o_group[r0 + place], nw = o_nw[r0 + place];
          g_bin[g] = t;
          g_pos[g] = count;
          load += nw >> 4;
          count += nw & 15;
        }
      }
    }
  }
  __syncthreads();
  if (t < n_groups) {
    for (int k = 0; k < t1 - t0; ++k) {   // heaviest tile first
      const int i = 8 * (g_pos[t] + k) + g_bin[t];
      if (i < n_wg) tasks[i] = task_of(gs, t1 - 1 - k, slot, S, base, Lq, gy);
    }
  }
}

// Key split.  With `chunk_keys` > 0 the keys of every sequence are cut at the absolute positions chunk_keys,
// 2*chunk_keys, ... (a multiple of the 128-key stage; chunk kAttnMaxChunks - 1 is open ended) and each chunk of a
// query tile goes to a workgroup of its own (grid z), which leaves its un-normalised (max, sum, O^T) in `part_*`;
// k_attn_merge folds the chunks of a row in ascending order.  The cut points depend on absolute positions only,
// never on the batch, so a row gets the same bits whether it is scored in a long block or alone; what changes
// against the unsplit kernel is the grouping of the fp32 sums, i.e. rounding.
// Short contexts with few query tiles (region-level drafts) gain the workgroups they need to fill the chip; the
// price is 264 bytes written and read again per (row, head, chunk).
constexpr int kAttnMaxChunks = 8;
struct AttnSplit {
  int chunk_keys, total_q;
  float *part_o;     // [kAttnMaxChunks][n_q_heads][total_q][64] un-normalised O rows
  float2 *part_ml;   // [kAttnMaxChunks][n_q_heads][total_q] (integer reference point, sum)
};

union Frag8 {
  uint4 u;
  bf16x8 v;
  uint16_t h[8];
};

// Softmax.  q comes scaled by log2(e) / sqrt(64) (EpiQKV::kQScale), so a score is an exponent of two and a probability is
// exp2(score - m) with a reference point m of the query.  m needs to keep sums and probabilities in range, no more: fp32 and
// bf16 are as precise at 2^60 as at 1.  It is an INTEGER, so that every correction factor is an exact power of two.  It is set
// at the first group of 64 keys that holds a visible one, to 0 where that group's largest score lies within +-kAttnZeroRange and
// to the score rounded up otherwise, and moves (to a group's largest score rounded up) only at a group with a score kAttnMoveAt
// above it.  Largest probability of the first group: 2^-65 at least, 2^64 at most, so what falls below the smallest number is less
// than 2^-61 of the row; of any: 2^96, which leaves 2^31 for the values and the number of keys.  The subtraction is free: the
// products start from -m instead of 0.  So a group at which no point is set or moved needs no maximum and no rescaling, whatever
// the scores, and its test is one comparison: a probability of 2^96 or more makes the group's sum as large.
// Each kernel applies the rule group by group, in ascending order over both parities: a row's numbers do not depend on the
// kernel.
constexpr float kAttnZeroRange = 64.f, kAttnMoveAt = 96.f;
// Below 2^kAttnMoveAt by more than the errors of the exponential and of a score, which rounds differently from -m and from 0: by
// less than 0.1 up to kAttnShiftRange.  Queries with a point beyond that never skip the rule.
constexpr float kAttnSumLimit = 0x1p95f, kAttnShiftRange = 0x1p16f;
__device__ __forceinline__ float attn_reference(float m, float mx) {
  if (m == -INFINITY) {
    const float c = ceilf(mx);
    return fabsf(c) <= kAttnZeroRange ? 0.f : c;   // -inf while no key is visible
  }
  return mx - m >= kAttnMoveAt ? ceilf(mx) : m;
}

// Row sums are fp32 sums of the probabilities as the second product sees them, ROUNDED to bf16: the rounding then cancels in
// the quotient, and a row whose probability lies on one key gets that key's value to the last bit.  (Sums of the unrounded
// values hold more bits, but the quotient loses: a row with one key is off by up to 2^-8.)  They are taken by
// v_mfma_f32_4x4x4_16b_bf16 with ones as A: every lane is a column of its own, so four of its probabilities are added to its
// accumulator and no row sees another's infinities or NaN.  Order: a lane half's eight keys of a page, the group's pages 0 and
// 2 in one chain, 1 and 3 in another, their sum, then the groups one after the other.
// ns a group beside the 16 products and the exponentials, one / two waves a SIMD (microbenchmark): no sums 306 / 236; 32 fp32
// additions of the unrounded values 358 / 282; these 331 / 299; the rounded values unpacked and added 461 / 336; 16
// v_dot2_f32_bf16 about 500.
__device__ __forceinline__ floatx4 attn_add_4(uint2 p, floatx4 sum) {
  typedef short short4v __attribute__((ext_vector_type(4)));
  const short4v ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(short4v, p), sum, 0, 0, 0);
}
__device__ __forceinline__ floatx4 attn_add_page(const bf16x8 &p, floatx4 sum) {
  const uint4 w = __builtin_bit_cast(uint4, p);
  return attn_add_4(make_uint2(w.z, w.w), attn_add_4(make_uint2(w.x, w.y), sum));
}

typedef __attribute__((address_space(3))) unsigned char *AttnLds;
// s_waitcnt vmcnt(N) with the other counters left alone (N < 64), also for the compiler's eyes: no LDS access moves across it
#define HSD_ATTN_VMCNT(N)                                                                             \
  do {                                                                                               \
    asm volatile("" ::: "memory");                                                                   \
    __builtin_amdgcn_s_waitcnt(((N) & 15) | (7 << 4) | (15 << 8) | (((N) >> 4) << 14));              \
    asm volatile("" ::: "memory");                                                                   \
  } while (0)
// A page of 2 KB (uniform address) to LDS (uniform) in two LDS-direct loads: lane l's 16 bytes at byte off0 of the page go to
// dst + 16 l, those at off1 to dst + 1024 + 16 l.  In asm: the compiler would otherwise wait for every load in flight before
// each LDS read.  No register is written; the reads wait by HSD_ATTN_VMCNT and a barrier.  m0, which the loads take their LDS
// address from, is a register the compiler keeps for itself and does not save around asm: it is put back as it was found.
__device__ __forceinline__ void attn_load_page(const bf16 *page, AttnLds dst, int off0, int off1) {
  const uint32_t d = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst)));
  const uint64_t p = reinterpret_cast<uint64_t>(page);
  const uint64_t up = (static_cast<uint64_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p >> 32))) << 32) |
                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p)));
  uint32_t m0;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, %4\n\t"
      "s_add_u32 m0, m0, 0x400\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %3, %4\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(m0)
      : "s"(d), "v"(off0), "v"(off1), "s"(up)
      : "memory", "scc");
}

// QS = query sets (waves; 32 queries x one head each) per workgroup: 4 (region-level) or 8 (page-level).
// G4 = query heads of one kv head among them (1, 2 or 4); QS/G4 row sub-tiles of 32 queries.
// TREE selects the tree-ancestry mask (row_end = packed index one past each row's subtree) instead of the causal one.
// SPLIT: grid z = key chunk (see AttnSplit); results go to the partial buffers instead of `out`.
// grid: (attn_grid_size(...) tasks, 1, chunks), block 64*QS, dynamic LDS kAttnLdsBytes.
template <int G4, int QS, bool TREE, bool SPLIT>
__global__ void __launch_bounds__(64 * QS, 2) k_attn_mfma(int n_q_heads, const AttnTile *__restrict__ tiles, PagedKV kv,
                                                               const bf16 *__restrict__ q, bf16 *__restrict__ out,
                                                               const int32_t *__restrict__ row_end, AttnSplit sp) {
  constexpr int NP = 8 / QS;                      // pages of a stage that a wave requests: 2 or 1
  static_assert(QS == 4 || QS == 8, "a stage's 8 pages are requested by 4 or 8 waves");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  constexpr int SUB = QS / G4, QT = 32 * SUB;

  // the tile's descriptor comes through the scalar unit in one read (constant address space: written by an
  // earlier kernel, never during this one)
  typedef const int32_t __attribute__((address_space(4))) *ConstI32;
  const ConstI32 td = (ConstI32)(reinterpret_cast<const int32_t *>(tiles + blockIdx.x));
  const int s = td[0];
  if (s < 0) return;  // uniform for the whole workgroup
  const int tile_in_seq = td[1], slot = td[2], S = td[3], base = td[4], Lq = td[5], ty = td[6];

  const int group = n_q_heads / kv.n_kv_heads, hb = (group + G4 - 1) / G4;
  const int kvh = ty / hb, hgrp = ty % hb;
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5, qj = lane & 31;
  const int wq = __builtin_amdgcn_readfirstlane(t >> 6);           // query-set index
  const int head = kvh * group + hgrp * G4 + (wq % G4);
  const int row0_wg = tile_in_seq * QT;
  const int row0 = row0_wg + (wq / G4) * 32;                       // first query row (within the block) of this wave
  const bool wave_active = row0 < Lq;
  const int my_row = min(row0 + qj, Lq - 1);
  const int pos_j = S + my_row;                                    // absolute position of the lane's query
  const int wave_keys = S + min(row0 + 32, Lq);                    // keys any query of this wave can see
  const int wg_keys = S + min(row0_wg + QT, Lq);                   // ... of this workgroup
  const int n_valid = S + Lq;                                      // positions holding data of this round
  // stages kt0 .. kt1-1 of 128 keys are this workgroup's
  int key_lo = 0, key_hi = wg_keys;
  if constexpr (SPLIT) {
    key_lo = static_cast<int>(blockIdx.z) * sp.chunk_keys;
    if (key_lo >= wg_keys) return;  // uniform for the whole workgroup: no query of the tile reaches this chunk
    if (blockIdx.z + 1 < kAttnMaxChunks) key_hi = min(wg_keys, key_lo + sp.chunk_keys);
  }
  const int kt0 = key_lo / kAttnKeys, kt1 = (key_hi + kAttnKeys - 1) / kAttnKeys;
  // stages before kt_plain need no mask and no checks: every key lies in the cached prefix (tree) or at or before
  // the workgroup's first query (chain), hence holds data and is visible to every query of the workgroup
  const int kt_plain = min(kt1, (TREE ? S : S + row0_wg + 1) / kAttnKeys);
  const int qdim = n_q_heads * kHd;

  // ---- requests.  Page pg of a stage is fetched by wave pg % QS, K and V in two loads of 1 KB each that write LDS directly:
  // lane l's 16 bytes land at 16 l.  K (16 rows of 128 bytes): the 16-byte piece p of row r lies at position
  // p ^ ((r >> 1) & 7) of its row; V^T (64 dims of 32 bytes): half h of dim d lies at h ^ ((d >> 3) & 1): the reads of 16
  // rows, or dims, cover all 64 banks once.  The page ids of many stages are read at once, a lane each.
  // An id that is out of range (a page beyond the data of this round, a damaged table) reads block 0 instead; every
  // position such a page could stand for is masked (and its V zeroed) by the checked form of the loop, and the plain form
  // only sees pages of the cached prefix.
  const AttnLds lds = (AttnLds)smem_raw;
  // byte offsets of a lane in a page: K row l / 8, V dim l / 2 (in the second half row 8 + l / 8: 1024 on, position ^ 4; dim 32 + l / 2)
  const int vk = (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 4)) << 4);
  const int vv = (lane >> 1) * 32 + (((lane & 1) ^ ((lane >> 4) & 1)) << 4);
  const int32_t *table_row = kv.block_table + static_cast<size_t>(slot) * kv.max_blocks_per_seq;
  const int last_entry = kv.max_blocks_per_seq - 1;
  // ids: lane NP j + i holds that of page wq + QS i of stage id0 + j
  int ids, id0;
  auto fetch_ids = [&](int kt) {
    id0 = kt;
    const int id = table_row[min((kt + lane / NP) * (kAttnKeys / kBlk) + wq + QS * (lane % NP), last_entry)];
    ids = (id >= 0 && id < kv.n_blocks) ? id : 0;
  };
  auto page = [&](int kt, int i) { return kv_block_offset(kv, __builtin_amdgcn_readlane(ids, (kt - id0) * NP + i), kvh); };
  // K is requested a stage ahead of V: next_k and next_v are the stages to come, k_put the K slot of the former
  int next_k = kt0, next_v = kt0, k_put = 0;
  auto issue_k = [&]() {
    if (next_k - id0 == 64 / NP) fetch_ids(next_v);   // V is behind and still needs its own
#pragma unroll
    for (int i = 0; i < NP; ++i)
      attn_load_page(static_cast<const bf16 *>(kv.k_pool) + page(next_k, i), lds + k_put * kAttnHalfStage + (wq + QS * i) * 2048, vk, (vk ^ 64) + 1024);
    ++next_k;
    k_put = k_put + 1 == kAttnKStages ? 0 : k_put + 1;
  };
  auto issue_v = [&]() {
#pragma unroll
    for (int i = 0; i < NP; ++i)
      attn_load_page(static_cast<const bf16 *>(kv.v_pool) + page(next_v, i),
                     lds + (kAttnKStages + (next_v & 1)) * kAttnHalfStage + (wq + QS * i) * 2048, vv, vv + 1024);
    ++next_v;
  };
  // Everything requested so far has landed, in every wave, and every wave is done with what it read.
  auto landed = [&]() {
    HSD_ATTN_VMCNT(0);
    __syncthreads();
  };
  fetch_ids(kt0);
  issue_k();
  issue_v();
  if (next_k < kt1) issue_k();

  // ---- query fragments (B operand of S^T): lane holds dims 16*kk + 8*half .. +7 of its query
  Frag8 qf[4];
  {
    const bf16 *qp = q + static_cast<size_t>(base + my_row) * qdim + head * kHd + half * 8;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qf[kk].u = *reinterpret_cast<const uint4 *>(qp + kk * 16);
  }
  int ka[4];   // K fragment kk of a block of 32 keys: byte offset in the block
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) ka[kk] = qj * 128 + (((2 * kk + half) ^ ((qj >> 1) & 7)) << 4);
  const int va = qj * 32 + ((half ^ ((qj >> 3) & 1)) << 4);

  // What a parity has summed (O^T and the row sum), scores and probabilities of its current group
  struct Half {
    floatx16 o[2];
    float l;
    floatx16 st[2];
    bf16x8 pf[4];
  };
  Half he, ho;
  // Reference point of the lane's query (-inf: no visible key so far); what its scores start from: -m, or 0 while there is none;
  // whether the points of the wave are set, and within the range in which a group may skip the rule (wave-uniform)
  float m = -INFINITY;
  floatx16 from = {};
  bool set = false;
  auto init = [](Half &h) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) h.o[i][v] = 0.f;
    h.l = 0.f;
#pragma unroll
    for (int pg = 0; pg < 4; ++pg)
#pragma unroll
      for (int e = 0; e < 8; ++e) h.pf[pg][e] = static_cast<__bf16>(0.0f);
  };
  init(he);
  init(ho);
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  // K and V of the 64 keys of parity `par` of a stage: of K in the given slot, of V by the stage's number
  auto k_half = [&](int slot_k, int par) { return smem_raw + slot_k * kAttnHalfStage + par * 8192; };
  auto v_half = [&](int kt, int par) { return smem_raw + (kAttnKStages + (kt & 1)) * kAttnHalfStage + par * 8192; };
  // S^T of a group, added to `start`
  auto products = [&](Half &h, const unsigned char *ks, const floatx16 &start) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      h.st[b] = start;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        h.st[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(ks + b * 4096 + ka[kk]), qf[kk].v, h.st[b], 0, 0, 0);
    }
  };
  // O^T += V^T P^T.  CHECKED: slots of positions that hold no data of this sequence must read as 0 (their probability is 0,
  // but 0 * stale-NaN would poison the product); slot order of a V page: see kv_v_slot
  auto accumulate = [&](Half &h, int kt, int par, auto checked_tag) {
    const unsigned char *vs = v_half(kt, par);
#pragma unroll
    for (int pg = 0; pg < 4; ++pg)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        Frag8 f;
        f.v = *reinterpret_cast<const bf16x8 *>(vs + pg * 2048 + i * 1024 + va);
        if constexpr (decltype(checked_tag)::value) {
          const int p0 = kt * kAttnKeys + par * 64 + pg * kBlk;
          if (p0 + kBlk > n_valid) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (p0 + (e < 4 ? 0 : 4) + 4 * half + e >= n_valid) f.h[e] = 0;
          }
        }
        h.o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.v, h.pf[pg], h.o[i], 0, 0, 0);
      }
  };
  auto mask = [&](Half &h, int kb) {
    if constexpr (TREE) {
      // packed prefix tree (tree-ancestry mask): inside the block, the key in slot S + p is visible to local
      // row r iff p is r itself or an ancestor of r, i.e. p <= r < end of p's subtree (rows are in pre-order)
      if (kb + 63 >= S) {  // the wave's keys reach into the block (wave-uniform)
        // branch-free: the subtree ends of 32 keys are fetched (index clamped into the block) before any is looked at, so
        // that 16 reads are in flight together (all 32 would not fit the registers)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          int e_sub[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int kpos = kb + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
            e_sub[v] = row_end[base + min(max(kpos - S, 0), Lq - 1)];
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int kpos = kb + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
            const bool vis = (kpos <= pos_j) & ((kpos < S) | (e_sub[v] > base + my_row));
            h.st[b][v] = vis ? h.st[b][v] : -INFINITY;
          }
        }
      }
    } else if (kb + 63 > S + row0) {  // the wave's keys reach past its first query: causal mask (wave-uniform)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int kpos = kb + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
          if (kpos > pos_j) h.st[b][v] = -INFINITY;
        }
    }
  };
  // The probabilities of a group (first key kb) by the general rule: masks (checked form), the largest score, a reference point
  // set or moved where it has to be.  Returns whether `from` has changed (wave-uniform).
  auto general = [&](Half &h, const unsigned char *ks, int kb, auto checked_tag) {
    constexpr bool CHECKED = decltype(checked_tag)::value;
    const floatx16 zero = {};
    products(h, ks, zero);
    if constexpr (CHECKED) mask(h, kb);
    float mx = fmaxf(h.st[0][0], h.st[1][0]);
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(fmaxf(mx, h.st[0][v]), h.st[1][v]);
    const float m_new = attn_reference(m, half_max(mx));
    int changed = 0;
    // when no reference point moved every factor is exactly 1 and the rescale is skipped (wave-uniform branch, same bits
    // either way)
    if (__any(m_new != m)) {
      const float corr = (m == -INFINITY) ? 0.f : ldexpf(1.0f, static_cast<int>(m - m_new));
      for (Half *x : {&he, &ho}) {
        x->l *= corr;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) x->o[i][v] *= corr;
      }
      m = m_new;
      set = __all(fabsf(m) <= kAttnShiftRange);
      const float start = m == -INFINITY ? 0.f : 0.f - m;   // no visible key yet: p = 0 without producing inf - inf
      changed = __any(start != from[0]);
#pragma unroll
      for (int v = 0; v < 16; ++v) from[v] = start;
    }
    if (__any(from[0] != 0.f)) {
      products(h, ks, from);
      if constexpr (CHECKED) mask(h, kb);
    }
    floatx4 ps[2] = {};
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
      floatx8 pv;
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(h.st[pg >> 1][8 * (pg & 1) + e]);
      h.pf[pg] = __builtin_convertvector(pv, bf16x8);
      ps[pg & 1] = attn_add_page(h.pf[pg], ps[pg & 1]);
    }
    h.l += ps[0][0] + ps[1][0];
    return changed;
  };
  // A turn: the products of half x -- V^T P^T of one group, K Q^T of the next but one -- beside the
  // exponentials of half y, whose scores are there.  Returns whether y's probabilities stand (wave-uniform), as they do unless a
  // reference point is to be set or moved; l is its row sum then.
  // The order is fixed by hand: a matrix instruction, the fragment read of one further on, two exponentials, and what follows
  // from those of the slot before, so that neither pipe waits for the other.  The V fragments of the first four slots
  // are there (pre); those of the following turn are read from vn, if it is given, before this one's result is looked at.
  bf16x8 pre[4];
  auto read_v = [&](const unsigned char *vs, int i) { return *reinterpret_cast<const bf16x8 *>(vs + (i >> 1) * 2048 + (i & 1) * 1024 + va); };
  auto read_pre = [&](const unsigned char *vs) {
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] = read_v(vs, i);
  };
  auto turn = [&](Half &x, const unsigned char *vs, const unsigned char *ks, Half &y, float &l, const unsigned char *vn) {
    constexpr int kAhead = SPLIT && (TREE || QS == 4) ? 4 : 5;   // 5 does not fit the registers there
    // slot: 0 to 7 = V fragment (page s / 2, dims 32 (s % 2) ..), 8 + = K fragment (block s % 2, k-step (s - 8) / 2)
    constexpr int kSeq[16] = {0, 1, 2, 3, 8, 9, 4, 5, 10, 11, 6, 7, 12, 13, 14, 15};
    auto read = [&](int j) {
      const int f = kSeq[j];
      return f < 8 ? read_v(vs, f) : *reinterpret_cast<const bf16x8 *>(ks + (f & 1) * 4096 + ka[(f - 8) >> 1]);
    };
    bf16x8 fr[16];
    float e0[16], e1[16];
    bf16x2 pw[16];
    floatx4 ps[2] = {};
    auto pack = [&](int j) { pw[j] = __builtin_convertvector((floatx2){e0[j], e1[j]}, bf16x2); };
    auto add = [&](int i) {   // words 2 i and 2 i + 1: half of page i / 2
      ps[(i >> 1) & 1] = attn_add_4(make_uint2(__builtin_bit_cast(uint32_t, pw[2 * i]), __builtin_bit_cast(uint32_t, pw[2 * i + 1])), ps[(i >> 1) & 1]);
    };
#pragma unroll
    for (int j = 0; j < kAhead; ++j) fr[j] = j < 4 ? pre[j] : read(j);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int f = kSeq[j], c = f & 1;
      if (f < 8) {
        x.o[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j], x.pf[f >> 1], x.o[c], 0, 0, 0);
      } else {
        x.st[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j], qf[(f - 8) >> 1].v, f < 10 ? from : x.st[c], 0, 0, 0);
      }
      if (j + kAhead < 16) fr[j + kAhead] = read(j + kAhead);
      // bare hardware exponential: results below 2^-126 may flush to zero, far beneath half a bf16 unit of any
      // probability that matters
      e0[j] = __builtin_amdgcn_exp2f(y.st[j >> 3][2 * (j & 7)]);
      e1[j] = __builtin_amdgcn_exp2f(y.st[j >> 3][2 * (j & 7) + 1]);
      asm volatile("" : "+v"(e0[j]), "+v"(e1[j]));   // computed here: pure instructions are moved across scheduling barriers
      if (j >= 1) {
        pack(j - 1);
        asm volatile("" : "+v"(pw[j - 1]));
      }
      if (j >= 3 && (j & 1)) add((j - 3) >> 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (vn != nullptr) read_pre(vn);
    pack(15);
    add(7);
    const float sum = ps[0][0] + ps[1][0];
    l = y.l + sum;
#pragma unroll
    for (int pg = 0; pg < 4; ++pg)
      y.pf[pg] = __builtin_shufflevector(__builtin_shufflevector(pw[4 * pg], pw[4 * pg + 1], 0, 1, 2, 3),
                                         __builtin_shufflevector(pw[4 * pg + 2], pw[4 * pg + 3], 0, 1, 2, 3), 0, 1, 2, 3, 4, 5, 6, 7);
    return static_cast<int>(set) & __all(sum < kAttnSumLimit);
  };
  const auto plain = std::false_type{};
  const auto checked = std::true_type{};

  // ---- plain stages.  Beside the exponentials of one parity run the products of the other: its last group's V^T P^T and its
  // next group's K Q^T.
  landed();
  int kt = kt0, k_at = 0;   // k_at: K slot of stage kt
  auto next_slot = [](int k) { return k + 1 == kAttnKStages ? 0 : k + 1; };
  if (kt < kt_plain) {
    products(he, k_half(k_at, 0), from);
    read_pre(v_half(kt, 1));
#pragma clang loop unroll(disable)   // a first iteration of its own costs code and spills
    for (; kt < kt_plain; ++kt) {
      float l;
      // first turn: o's probabilities are 0, any V will do
      const int ok_e = turn(ho, v_half(max(kt - 1, kt0), 1), k_half(k_at, 1), he, l, nullptr);
      if (ok_e) he.l = l;
      else if (general(he, k_half(k_at, 0), kt * kAttnKeys, plain)) products(ho, k_half(k_at, 1), from);
      landed();                                     // K of stage kt + 1, V of stage kt
      read_pre(v_half(kt, 0));
      if (next_k < kt1) issue_k();                  // K of stage kt + 2, over that of kt - 1
      if (next_v < kt1) issue_v();                  // V of stage kt + 1, over that of kt - 1
      const int k_next = next_slot(k_at);
      const int ok_o = turn(he, v_half(kt, 0), k_half(k_next, 0), ho, l, v_half(kt, 1));   // last turn: the scores are not used
      if (ok_o) ho.l = l;
      else if (general(ho, k_half(k_at, 1), kt * kAttnKeys + 64, plain)) products(he, k_half(k_next, 0), from);
      k_at = k_next;
    }
    accumulate(ho, kt - 1, 1, plain);
  }
#pragma clang loop unroll(disable)
  for (; kt < kt1; ++kt) {
    if (kt > kt0) landed();
    if (next_k < kt1 && next_k <= kt + 1) issue_k();
    if (next_v < kt1 && next_v <= kt + 1) issue_v();
    if (wave_active && kt * kAttnKeys < wave_keys) {
      general(he, k_half(k_at, 0), kt * kAttnKeys, checked);
      accumulate(he, kt, 0, checked);
    }
    if (wave_active && kt * kAttnKeys + 64 < wave_keys) {
      general(ho, k_half(k_at, 1), kt * kAttnKeys + 64, checked);
      accumulate(ho, kt, 1, checked);
    }
    k_at = next_slot(k_at);
  }

  // ---- fold the two parities, even first.  (A chunk of a split pass may hold no visible key for a row: m = -inf, sums 0.)
  if (!wave_active || row0 + qj >= Lq) return;
  const float l_tot = half_sum(he.l) + half_sum(ho.l);
  const float inv = SPLIT ? 1.0f : 1.0f / l_tot;
  const size_t rh = (static_cast<size_t>(blockIdx.z) * n_q_heads + head) * sp.total_q + base + row0 + qj;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      floatx4 ov;
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = he.o[i][4 * g + e] + ho.o[i][4 * g + e];
      if constexpr (SPLIT) {
        *reinterpret_cast<floatx4 *>(sp.part_o + rh * kHd + i * 32 + 8 * g + 4 * half) = ov;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] *= inv;
        *reinterpret_cast<bf16x4 *>(out + static_cast<size_t>(base + row0 + qj) * qdim + head * kHd + i * 32 + 8 * g + 4 * half) =
            __builtin_convertvector(ov, bf16x4);
      }
    }
  if constexpr (SPLIT)
    if (half == 0) sp.part_ml[rh] = make_float2(m, l_tot);
}

// Folds the key chunks of a split pass: row r (cache slot row_slot[r]) has chunks 0 .. min(kAttnMaxChunks - 1,
// slot / chunk_keys), merged in ascending order with exact power-of-two factors, then normalised.
// One thread per (head, row, 4 dims); grid ceil(n_q_heads * total_q * 16 / 256), block 256.
__global__ void __launch_bounds__(256) k_attn_merge(int n_q_heads, const int32_t *__restrict__ row_slot, AttnSplit sp,
                                                    bf16 *__restrict__ out) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int rh = idx >> 4, piece = idx & 15;            // rh = head * total_q + row
  if (rh >= n_q_heads * sp.total_q) return;
  const int head = rh / sp.total_q, row = rh - head * sp.total_q;
  const int nc = min(kAttnMaxChunks, row_slot[row] / sp.chunk_keys + 1);
  const size_t cstride = static_cast<size_t>(n_q_heads) * sp.total_q;
  float2 ml = sp.part_ml[rh];
  floatx4 o = *reinterpret_cast<const floatx4 *>(sp.part_o + static_cast<size_t>(rh) * kHd + piece * 4);
  float m_run = ml.x, l_run = ml.y;
  for (int c = 1; c < nc; ++c) {
    const float2 b = sp.part_ml[c * cstride + rh];
    const floatx4 ob = *reinterpret_cast<const floatx4 *>(sp.part_o + (c * cstride + rh) * kHd + piece * 4);
    const float m_tot = fmaxf(m_run, b.x);
    const float ca = (m_run > -INFINITY) ? ldexpf(1.0f, static_cast<int>(m_run - m_tot)) : 0.f;
    const float cb = (b.x > -INFINITY) ? ldexpf(1.0f, static_cast<int>(b.x - m_tot)) : 0.f;
    l_run = l_run * ca + b.y * cb;
    m_run = m_tot;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = o[e] * ca + ob[e] * cb;
  }
  const float inv = 1.0f / l_run;
  floatx4 ov;
#pragma unroll
  for (int e = 0; e < 4; ++e) ov[e] = o[e] * inv;
  *reinterpret_cast<bf16x4 *>(out + static_cast<size_t>(row) * n_q_heads * kHd + head * kHd + piece * 4) =
      __builtin_convertvector(ov, bf16x4);
}

}  // namespace hsd
