// Verification attention for passes with few query rows: the keys of ONE query set are spread over the waves of a
// workgroup.
//
// Why.  k_attn_mfma gives a wave 32 queries and lets it walk every second 64-key group of the sequence on its own:
// 64 keys after 64 keys.  A pass with few rows has few such
// walks (one token of one sequence: 4 workgroups on 256 compute units), so the launch lasts as long as one of them,
// most of it latency.  What truly depends on the previous group is little: the accumulation of O and of the row sum, and a
// reference point that hardly ever moves.  Here the scoring waves take one 64-key group each (S^T = K Q^T,
// probabilities) and leave their probabilities in LDS.
// Four accumulating waves -- (key parity, half of the head dimension) -- walk the groups in order and add V^T P^T and the row
// sums: a chain of four matrix instructions a group, with V straight from memory to registers (a V page is stored as the operand).
//
// Every number is formed by the same instructions on the same operands in the same order as in k_attn_mfma (groups at
// absolute positions, even and odd groups in separate sums, reference points by attn_reference group by group), so the two kernels give the same bits and the choice between them may follow the batch.
//
// Query sets.  A set is QW = 32 columns: 32 rows of one query head, or, where a sequence has few rows, the rows of several
// query heads of one kv head (16 rows of two heads, 8 rows of four), so that K and V are read once for all of them.  The
// task table says which (AttnTile::pack).  A pass whose every block fits 16 columns (4 rows of four heads: token-by-token
// decoding) takes QW = 16: half the maxima, exponentials and probabilities, products on 16x16x32 instructions (the same
// sums as on 32x32x16, see gemm_mfma_r.h).
#pragma once

#include "attn_mfma.h"

namespace hsd {

// LDS: probabilities of two steps of four groups (4 KB a group: [page][lane][8 bf16]); which waves ask for the general rule; for
// that, the groups' largest scores and the reference points that follow from them; the odd parity's (O, sum) for the final fold
constexpr int kAttnWideScorers = 4;
constexpr int kKsStride = kHd + 8;   // bf16 per K row in LDS
template <int QW>
struct AttnWideLds {
  uint4 p[2][kAttnWideScorers][QW / 8][64];
  float mx[kAttnWideScorers][QW], mg[2][kAttnWideScorers][QW];
  int moves[2][4], sets;
  union __attribute__((aligned(16))) {   // (16-byte LDS accesses: a workgroup takes 1.6 times as long if they lie elsewhere)
    uint16_t k[kAttnWideScorers][64 * kKsStride];   // a scoring wave's own 64 keys (see k_row)
    float fold[2][QW / 2 + 1][64];                  // after the last products
  };
};
// Offset of a key's row in AttnWideLds::k: rows 144 B apart, those of odd pages 16 B further, so that the fragment reads of
// 16 rows (16 keys in a row, or 8 of a page and the same 8 of the next) cover all 64 banks once.
__device__ __forceinline__ int k_row(int key) { return key * kKsStride + ((key >> 4) & 1) * 8; }

// Exchange with the lanes 16 away (the max and the sum over l and l ^ 16), as half_max and half_sum
__device__ __forceinline__ float quarter_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float quarter_sum(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// NS scoring waves and four accumulating ones; a step covers NS 64-key groups.
// grid: attn_grid_size(...) tasks, block 64 * (NS + 4), dynamic LDS sizeof(AttnWideLds).
// The walk over the steps has two forms.  The first takes every reference point for 0 and has one barrier a step, behind which
// the step's probabilities are in LDS: nothing else is waited for.  Whether the first group sets another point, and whether a
// sum shows a score that would move one, is found out beside the next step's work, and every wave alike leaves this form.  The
// walk then starts again in the general form, from the points of the first group: a step whose points stand has one barrier there
// too, but the outcome is waited for behind it; one that moves a point has three more, behind which the groups' largest scores,
// the points that follow and the probabilities are in LDS.
// us a launch, with points found and moved inside the one loop / in forms of their own: one token at 1055 keys 8.9 / 7.9, 7 blocks
// of 1 to 47 rows 13.1 / 12.3, 64 tokens 17.9 / 17.4.  Where scores are so extreme that every set ends in the general form (first
// groups beyond 64 binary orders, 44 in natural logarithms, and later scores beyond 96) one token takes 14.
// What bounds it (one token at 1055 keys, 7.9 us): 2.6 us until the first scores (descriptor, page
// ids, keys: three dependent reads), then the 270 KB of a kv head through one unit's load path (a bare read of 256 KB by a
// workgroup takes 5 us with its launch), 1 us of last accumulation, fold and store.  Tried: eight scoring waves (32 columns: 13.4
// us against 12.1); keys and values two steps ahead in registers (16 tokens a step 13.58 ms against 13.15); four more waves that
// only request the keys into a ring of three or four steps (13.66; 64 tokens 9.05 ms against 8.62, one workgroup a unit); starting
// again from the first group's points in the common form before the general one (nothing gained where points move as well).
static_assert(2 * sizeof(AttnWideLds<32>) <= 160 * 1024, "two workgroups a compute unit");
template <int QW, bool TREE>
__global__ void __launch_bounds__(64 * (kAttnWideScorers + 4), 4) k_attn_wide(int n_q_heads, int g4, const AttnTile *__restrict__ tiles,
                                                                           PagedKV kv, const bf16 *__restrict__ q,
                                                                           bf16 *__restrict__ out,
                                                                           const int32_t *__restrict__ row_end) {
  constexpr int NS = kAttnWideScorers;
  static_assert(NS % 4 == 0 && 16 % (NS / 2) == 0, "an even number of groups a step and parity, page ids of whole steps in 64 lanes");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  AttnWideLds<QW> &sm = *reinterpret_cast<AttnWideLds<QW> *>(smem_raw);

  typedef const int32_t __attribute__((address_space(4))) *ConstI32;
  const ConstI32 td = (ConstI32)(reinterpret_cast<const int32_t *>(tiles + blockIdx.x));
  if (td[0] < 0) return;  // uniform for the whole workgroup
  const int tile = td[1], slot = td[2], S = td[3], base = td[4], Lq = td[5], ty = td[6], pack = td[7];

  const int group = n_q_heads / kv.n_kv_heads, hb = (group + g4 - 1) / g4;
  const int kvh = ty / hb, hgrp = ty % hb;
  const int lhp = pack & 3, rshift = (QW == 32 ? 5 : 4) - lhp;     // 2^lhp heads of 2^rshift rows each
  // QW = 32: operand row / result column l % 32, k group l / 32.  QW = 16: l % 16 and l / 16.
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5, qj = lane & (QW - 1), kg = lane / QW;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int head = kvh * group + hgrp * g4 + ((pack >> 2) << lhp) + (qj >> rshift);
  const int row0 = tile << rshift, row = row0 + (qj & ((1 << rshift) - 1));
  const int my_row = min(row, Lq - 1);
  const int pos_j = S + my_row;
  const int n_valid = S + Lq;                                      // positions holding data of this round
  const int n_keys = S + min(row0 + (1 << rshift), Lq);            // keys any query of the set can see
  const int n_groups = (n_keys + 63) >> 6, n_steps = (n_groups + NS - 1) / NS;
  const int qdim = n_q_heads * kHd;

  const int32_t *table_row = kv.block_table + static_cast<size_t>(slot) * kv.max_blocks_per_seq;
  const int last_entry = kv.max_blocks_per_seq - 1;
  // Pages are numbered through the pool, (layer, block, kv head); a lane turns the id it fetched into such a number once.  An
  // id out of range (a page beyond the data of this round, a damaged table) becomes block 0; every position such a page
  // could stand for is masked and its V zeroed.
  auto page_number = [&](int entry) {
    const int id = table_row[min(entry, last_entry)];
    return (kv.layer * kv.n_blocks + ((id >= 0 && id < kv.n_blocks) ? id : 0)) * kv.n_kv_heads + kvh;
  };
  // element offset of the page whose number lane `src` of `pages` holds
  auto page_off = [&](int pages, int src) {
    return static_cast<size_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(pages, src))) * (kBlk * kHd);
  };
  // Whether the general form is asked for.  moves[x]: by the accumulating waves' sums of the last step with s % 2 = x; sets: by
  // the first group's scores.  Looked at beside the work between the barriers of steps t - 1 and t, when the flags
  // of step t - 2 are complete (at t = 1 the first group's); at the end those of the last two steps.
  auto asks = [&](int t) { return __any(t == 1 ? sm.sets : sm.moves[t & 1][lane & 3]); };
  auto asked_at_end = [&]() { return __any(sm.moves[(lane >> 2) & 1][lane & 3]) || (n_steps == 1 && __any(sm.sets)); };
  const auto common = std::false_type{};
  const auto general = std::true_type{};
  if (wave >= 4) {
    // ---- a scoring wave: groups w, w + NS, w + 2 NS, ...
    const int w = wave - 4;
    const bf16 *kpool = static_cast<const bf16 *>(kv.k_pool);
    constexpr int KQ = QW / 8;   // k-steps over the 64 dims: 4 of 16, or 2 of 32
    Frag8 qf[KQ];
    // pages: lane 4 s + p holds the number of page p of this wave's group in step s0 + s (16 steps at a time)
    auto fetch_pages = [&](int s0) { return page_number(((s0 + (lane >> 2)) * NS + w) * 4 + (lane & 3)); };
    int pages = fetch_pages(0);   // requested before q: the ids are on the way to the first keys
    {
      const bf16 *qp = q + static_cast<size_t>(base + my_row) * qdim + head * kHd + kg * 8;
#pragma unroll
      for (int kk = 0; kk < KQ; ++kk) qf[kk].u = *reinterpret_cast<const uint4 *>(qp + kk * (64 / KQ));
    }
    // K of a group: four pages of 2 KB, loaded as they lie (64 lanes read 1 KB in a row; a load in operand order, 32 rows of
    // 128 bytes, takes the address unit 64 cycles instead of 16), turned into operands through the wave's own LDS rows
    u32x4 rk[8];
    auto load_k = [&](int s) {
#pragma unroll
      for (int pg = 0; pg < 4; ++pg) {
        const bf16 *kp = kpool + page_off(pages, (s & 15) * 4 + pg) + lane * 8;
#pragma unroll
        for (int c = 0; c < 2; ++c) rk[2 * pg + c] = *reinterpret_cast<const u32x4 *>(kp + c * 512);
      }
    };
    uint16_t *ks = sm.k[w];
    auto store_k = [&]() {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // LDS runs a wave's accesses in order: only the compiler
      __builtin_amdgcn_wave_barrier();                         // has to be kept from reordering them
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4 *>(ks + k_row(8 * i + (lane >> 3)) + (lane & 7) * 8) = rk[i];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    constexpr int NB = QW == 32 ? 2 : 4, NV = QW == 32 ? 16 : 4;
    // Scores of 64 keys x QW queries: register v of block b is key_of(b, v) of the group.  QW = 16: blocks 2 p and 2 p + 1
    // cover pages 2 p and 2 p + 1, the keys dealt to the operand rows so that a lane's eight registers of the two are the
    // eight contraction slots that the second product takes from it.
    auto key_of = [&](int b, int v) {
      return QW == 32 ? 32 * b + 8 * (v >> 2) + 4 * half + (v & 3) : 32 * (b >> 1) + 8 * (b & 1) + 16 * (kg >> 1) + 4 * (kg & 1) + v;
    };
    float st[NB][NV];
    auto fragment = [&](int j) {   // QW = 32: block j / 4, k-step j % 4; QW = 16: j / 2, j % 2
      if constexpr (QW == 32) {
        return *reinterpret_cast<const bf16x8 *>(ks + k_row((j >> 2) * 32 + qj) + (j & 3) * 16 + half * 8);
      } else {
        const int b = j >> 1, key = 32 * (b >> 1) + 8 * (b & 1) + 16 * (qj >> 3) + 4 * ((qj >> 2) & 1) + (qj & 3);
        return *reinterpret_cast<const bf16x8 *>(ks + k_row(key) + (j & 1) * 32 + kg * 8);
      }
    };
    auto products = [&](float from) {   // the scores, added to `from`
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if constexpr (QW == 32) {
          floatx16 acc;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = from;
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fragment(4 * b + kk), qf[kk].v, acc, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < NV; ++v) st[b][v] = acc[v];
        } else {
          floatx4 acc = {from, from, from, from};
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fragment(2 * b + kk), qf[kk].v, acc, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < NV; ++v) st[b][v] = acc[v];
        }
      }
    };
    auto mask = [&](int kb, auto form_tag) {
      if constexpr (TREE) {
        if (kb + 63 >= S) {  // the group reaches into the block: tree-ancestry mask (see k_attn_mfma)
          // a block at a time, in the general form four keys: the registers of all would decide between one and two workgroups a unit
          constexpr int NC = decltype(form_tag)::value ? 4 : NV;
#pragma unroll
          for (int c = 0; c < NB * NV / NC; ++c) {
            const int b = c * NC / NV, v0 = c * NC % NV;
            int e_sub[NC];
#pragma unroll
            for (int v = 0; v < NC; ++v) e_sub[v] = row_end[base + min(max(kb + key_of(b, v0 + v) - S, 0), Lq - 1)];
#pragma unroll
            for (int v = 0; v < NC; ++v) {
              const int kpos = kb + key_of(b, v0 + v);
              const bool vis = (kpos <= pos_j) & ((kpos < S) | (e_sub[v] > base + my_row));
              st[b][v0 + v] = vis ? st[b][v0 + v] : -INFINITY;
            }
            if constexpr (NC < NV) __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else if (kb + 63 > S + row0) {  // the group reaches past the first query: causal mask
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int v = 0; v < NV; ++v)
            if (kb + key_of(b, v) > pos_j) st[b][v] = -INFINITY;
      }
    };
    auto query_max = [&]() {   // the group's largest score of the lane's query
      float mx = st[0][0];
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < NV; ++v) mx = fmaxf(mx, st[b][v]);
      mx = half_max(mx);
      return QW == 16 ? quarter_max(mx) : mx;
    };
    // The group's probabilities; WITH_SUM: returns the lane's sum of them
    auto probs = [&](int s, auto with_sum_tag) {
      floatx4 ps = {};
#pragma unroll
      for (int f = 0; f < QW / 8; ++f) {   // operand f: page f of the group, or pages 2 f and 2 f + 1
        floatx8 pv;
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(QW == 32 ? st[f >> 1][8 * (f & 1) + e] : st[2 * f + (e >> 2)][e & 3]);
        Frag8 pf;
        pf.v = __builtin_convertvector(pv, bf16x8);
        sm.p[s & 1][w][f][lane] = pf.u;
        if constexpr (decltype(with_sum_tag)::value) ps = attn_add_page(pf.v, ps);
      }
      return ps[0];
    };
    auto next_k = [&](int s) {   // K of the next step to LDS, that of the one after it requested
      if (s + 1 >= n_steps) return;
      store_k();
      if (s + 2 < n_steps) {
        if (((s + 2) & 15) == 0) pages = fetch_pages(s + 2);
        load_k(s + 2);
      }
    };
    auto first_k = [&](int s) {   // K of step s to LDS (pages: those of s & ~15), that of the next one requested
      load_k(s);
      store_k();
      if (s + 1 < n_steps) {
        if (((s + 1) & 15) == 0) pages = fetch_pages(s + 1);
        load_k(s + 1);
      }
    };
    // The common form.  Returns whether it stands.
    auto walk = [&]() {
      bool asked = false;
#pragma clang loop unroll(disable)   // a first iteration of its own doubles the code
      for (int s = 0; s < n_steps; ++s) {
        const int g = s * NS + w;
        if (s > 0) asked = asks(s);
        if (g < n_groups) products(0.f);
        next_k(s);
        if (g < n_groups) {
          mask(g * 64, common);
          probs(s, common);
          if (g == 0) {   // this group holds a visible key of every query and sets its point
            const float m = attn_reference(-INFINITY, query_max());
            if (kg == 0) sm.mg[0][0][qj] = m;
            const int sets = __any(m != 0.f);
            if (lane == 0) sm.sets = sets;
          }
        }
        if (asked) return false;
        __syncthreads();   // the step's probabilities
      }
      __syncthreads();   // the fold
      return !asked_at_end();
    };
    first_k(0);
    if (walk()) return;
    // The general form.  m: reference point of the lane's query
    __syncthreads();   // every wave has seen the outcome
    pages = fetch_pages(0);
    float m = sm.mg[0][0][qj];   // the first group's
    first_k(0);
#pragma clang loop unroll(disable)
    for (int s = 0; s < n_steps; ++s) {
      const int g = s * NS + w;
      // phase 0: with the points as they are; where they do not stand, phase 1: the largest scores, and 2: with the points that
      // follow from them
#pragma clang loop unroll(disable)
      for (int phase = 0;; ++phase) {
        float m_own = m, mx = -INFINITY;
        if (phase == 2) {
          m_own = sm.mg[s & 1][w][qj];
          m = sm.mg[s & 1][min(NS, n_groups - s * NS) - 1][qj];
        }
        bool moves = false;
        // no visible key yet: p = 0 without producing inf - inf
        if (g < n_groups) products(phase == 1 || m_own == -INFINITY ? 0.f : 0.f - m_own);
        if (phase != 1) next_k(s);
        if (g < n_groups) {
          int kb = g * 64;
          asm volatile("" : "+s"(kb));   // the masks' addresses are made here: hoisted out of the phases they would spill
          mask(kb, general);
          if (phase == 1) mx = query_max();
          else moves = !__all(probs(s, general) < kAttnSumLimit && fabsf(m) <= kAttnShiftRange);
        }
        if (phase == 1 && kg == 0) sm.mx[w][qj] = mx;
        if (phase == 0 && lane == 0) sm.moves[s & 1][w] = moves;
        __syncthreads();
        if (phase == 2) break;
        if (phase == 0) {
          int f = 0;
#pragma unroll
          for (int k = 0; k < NS; ++k) f |= sm.moves[s & 1][k];
          if (!__builtin_amdgcn_readfirstlane(f)) break;
          pages = fetch_pages(s & ~15);
          first_k(s);
        } else {
          // every scoring wave finds the point behind its own group
          float m_run = s == 0 ? -INFINITY : m;
          for (int k = 0; k <= w; ++k)
            if (s * NS + k < n_groups) m_run = attn_reference(m_run, sm.mx[k][qj]);
          if (kg == 0) sm.mg[s & 1][w][qj] = m_run;
          __syncthreads();
        }
      }
    }
    __syncthreads();   // the fold
    return;
  }

  // ---- an accumulating wave: parity par, head dims 32 i .. 32 i + 31
  constexpr int KG = NS / 2;                     // its groups a step: s * NS + 2 k + par
  constexpr int SPF = 16 / KG;                   // steps whose page ids fit 64 lanes: lane (s * KG + k) * 4 + page
  const int i = wave & 1, par = wave >> 1;
  const bf16 *vpool = static_cast<const bf16 *>(kv.v_pool);
  auto fetch_pages = [&](int s0) {
    const int x = lane >> 2;
    return page_number(((s0 + x / KG) * NS + 2 * (x % KG) + par) * 4 + (lane & 3));
  };
  // V operands of a group.  QW = 32: page f, dims 32 i + l % 32, slots 8 (l / 32) ..  QW = 16: pages 2 (f / 2) + l / 32,
  // dims 32 i + 16 (f % 2) + l % 16, slots 8 (l / 16 % 2) ..
  Frag8 vf[KG][4];
  int pages;
  auto load_v = [&](int s, int k) {
    const int l0 = ((s % SPF) * KG + k) * 4;
    if constexpr (QW == 32) {
#pragma unroll
      for (int f = 0; f < 4; ++f)
        vf[k][f].u = *reinterpret_cast<const uint4 *>(vpool + page_off(pages, l0 + f) + (i * 32 + qj) * kBlk + half * 8);
    } else {
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const size_t o0 = page_off(pages, l0 + 2 * p), o1 = page_off(pages, l0 + 2 * p + 1);
        const bf16 *vp = vpool + (half ? o1 : o0) + (i * 32 + qj) * kBlk + (kg & 1) * 8;
#pragma unroll
        for (int d = 0; d < 2; ++d) vf[k][2 * p + d].u = *reinterpret_cast<const uint4 *>(vp + d * 16 * kBlk);
      }
    }
  };
  constexpr int NO = QW / 2;       // accumulators of a lane: 32 dims x QW queries over 64 lanes
  floatx16 o32;
  floatx4 o16[2];
  float l = 0.f;
  auto accumulate = [&](int s, int k) {   // returns the lane's sum over the group
    const int w = 2 * k + par, g = s * NS + w;
    if (g >= n_groups) return 0.f;
    if (g * 64 + 64 > n_valid) {
      // slots of positions that hold no data of this sequence must read as 0 (their probability is 0, but 0 * stale-NaN
      // would poison the product); slot order of a V page: see kv_v_slot
#pragma unroll
      for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int page = QW == 32 ? f : 2 * (f >> 1) + half, hf = QW == 32 ? half : (kg & 1);
          const int tok = (e < 4 ? 0 : 4) + 4 * hf + e;
          if (g * 64 + page * kBlk + tok >= n_valid) vf[k][f].h[e] = 0;
        }
    }
    Frag8 pf[QW / 8];
#pragma unroll
    for (int f = 0; f < QW / 8; ++f) pf[f].u = sm.p[s & 1][w][f][lane];
    floatx4 ps[2] = {};
    if constexpr (QW == 32) {
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        o32 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k][f].v, pf[f].v, o32, 0, 0, 0);
        ps[f & 1] = attn_add_page(pf[f].v, ps[f & 1]);
      }
    } else {
      // the lower lane half holds the even pages, the upper the odd ones
#pragma unroll
      for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int d = 0; d < 2; ++d) o16[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[k][2 * p + d].v, pf[p].v, o16[d], 0, 0, 0);
        ps[0] = attn_add_page(pf[p].v, ps[0]);
      }
    }
    const float sum = QW == 32 ? ps[0][0] + ps[1][0] : half_sum(ps[0][0]);
    l += sum;
    return sum;
  };
  auto first_v = [&]() {
    l = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) o32[v] = 0.f;
#pragma unroll
    for (int v = 0; v < 8; ++v) o16[v >> 2][v & 3] = 0.f;
    pages = fetch_pages(0);
#pragma unroll
    for (int k = 0; k < KG; ++k) load_v(0, k);
  };
  // ---- fold the two parities (even first), as k_attn_mfma does
  float o[NO];
  auto leave_odd = [&]() {
    l = QW == 32 ? half_sum(l) : quarter_sum(l);
#pragma unroll
    for (int v = 0; v < NO; ++v) o[v] = QW == 32 ? o32[v] : o16[(v >> 2) & 1][v & 3];
    if (par == 1) {
#pragma unroll
      for (int v = 0; v < NO; ++v) sm.fold[i][v][lane] = o[v];
      sm.fold[i][NO][lane] = l;
    }
  };
  // The common form.  Returns whether it stands.
  auto walk = [&]() {
    bool asked = false, moves = false;
    auto take_in = [&](int s, int k) { moves |= !__all(accumulate(s, k) < kAttnSumLimit); };
    __syncthreads();   // the first step's probabilities
#pragma clang loop unroll(disable)
    for (int s = 0; s + 1 < n_steps; ++s) {
      asked = asks(s + 1);
      if ((s + 1) % SPF == 0) pages = fetch_pages(s + 1);
      moves = false;
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        take_in(s, k);
        load_v(s + 1, k);
      }
      if (lane == 0) sm.moves[s & 1][wave] = moves;
      if (asked) return false;
      __syncthreads();   // the next step's
    }
    moves = false;
#pragma unroll
    for (int k = 0; k < KG; ++k) take_in(n_steps - 1, k);
    if (lane == 0) sm.moves[(n_steps - 1) & 1][wave] = moves;
    if (lane == 0 && n_steps == 1) sm.moves[1][wave] = 0;
    leave_odd();
    __syncthreads();
    return !asked_at_end();
  };
  first_v();
  if (!walk()) {
    // The general form.  m: reference point of the lane's query
    __syncthreads();
    float m = sm.mg[0][0][qj];
    // every group's move, also of the other parity, so that the factors come one by one as in k_attn_mfma
    auto rescale = [&](int s, int w) {
      if (s * NS + w >= n_groups) return;
      const float m_new = sm.mg[s & 1][w][qj];
      if (__any(m_new != m)) {
        const float corr = (m == -INFINITY) ? 0.f : ldexpf(1.0f, static_cast<int>(m - m_new));
        l *= corr;
        if constexpr (QW == 32) {
#pragma unroll
          for (int v = 0; v < 16; ++v) o32[v] *= corr;
        } else {
#pragma unroll
          for (int v = 0; v < 8; ++v) o16[v >> 2][v & 3] *= corr;
        }
      }
      m = m_new;
    };
    first_v();
#pragma clang loop unroll(disable)
    for (int s = 0; s < n_steps; ++s) {
      __syncthreads();   // phase 0
      int f = 0;
#pragma unroll
      for (int k = 0; k < NS; ++k) f |= sm.moves[s & 1][k];
      const bool moved = __builtin_amdgcn_readfirstlane(f) != 0;
      if (moved) {
        __syncthreads();   // phase 1: largest scores, points
        __syncthreads();
        __syncthreads();   // phase 2
      }
      if (s + 1 < n_steps && (s + 1) % SPF == 0) pages = fetch_pages(s + 1);
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        if (moved) rescale(s, 2 * k);
        if (moved && par == 1) rescale(s, 2 * k + 1);
        accumulate(s, k);
        if (moved && par == 0) rescale(s, 2 * k + 1);
        if (s + 1 < n_steps) load_v(s + 1, k);
      }
    }
    leave_odd();
    __syncthreads();
  }
  if (par == 0 && row < Lq) {
    const float inv = 1.0f / (l + sm.fold[i][NO][lane]);
    // four dims in a row: 8 g + 4 (l / 32), or 16 g + 4 (l / 16)
    bf16 *op = out + static_cast<size_t>(base + row) * qdim + head * kHd + i * 32 + 4 * kg;
#pragma unroll
    for (int gq = 0; gq < NO / 4; ++gq) {
      floatx4 ov;
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = (o[4 * gq + e] + sm.fold[i][4 * gq + e][lane]) * inv;
      *reinterpret_cast<bf16x4 *>(op + (256 / QW) * gq) = __builtin_convertvector(ov, bf16x4);
    }
  }
}

}  // namespace hsd
