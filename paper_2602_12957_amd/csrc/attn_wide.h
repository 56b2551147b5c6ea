// Verification attention for passes with few query rows: the keys of ONE query set are spread over the waves of a
// workgroup.
//
// Why.  k_attn_mfma gives a wave 32 queries and lets it walk every second 64-key group of the sequence on its own:
// products, maximum, exponentials and products again in one dependent chain per group.  A pass with few rows has few such
// walks (one token of one sequence: 4 workgroups on 256 compute units), so the launch lasts as long as one of them:
// 15 us at 1055 keys, most of it latency.  What truly depends on the previous group is little: the running maximum (one
// number per query) and the accumulation of O and of the row sum.  Here the scoring waves take one 64-key group each
// (S^T = K Q^T, maximum, probabilities), exchange their maxima through LDS, so
// that each knows the reference point the serial walk would have had at its group, and leave their probabilities in LDS.
// Four accumulating waves -- (key parity, half of the head dimension) -- walk the groups in order and add V^T P^T: a chain
// of four matrix instructions a group, with V straight from memory to registers (a V page is stored as the operand).
//
// Every number is formed by the same instructions on the same operands in the same order as in k_attn_mfma (groups at
// absolute positions, even and odd groups in separate sums, the reference point of a group = the largest seen so far in
// its parity), so the two kernels give the same bits and the choice between them may follow the batch.
//
// Query sets.  A set is 32 columns: 32 rows of one query head, or, where a sequence has few rows, the rows of several
// query heads of one kv head (16 rows of two heads, 8 rows of four), so that K and V are read once for all of them.  The
// task table says which (AttnTile::pack).
#pragma once

#include "attn_mfma.h"

namespace hsd {

// LDS: probabilities of two steps of four groups (4 KB a group: [page][lane][8 bf16]), the groups' maxima of two steps, and
// the odd parity's (O, reference point, sum) for the final fold
constexpr int kAttnWideScorers = 4;
struct AttnWideLds {
  uint4 p[2][kAttnWideScorers][4][64];
  float mg[2][kAttnWideScorers][32];
  uint16_t k[kAttnWideScorers][64 * kKsStride];   // a scoring wave's own 64 keys
  float fold[2][18][64];
};

// NS scoring waves and four accumulating ones; a step covers NS 64-key groups.
// grid: attn_grid_size(...) tasks, block 64 * (NS + 4), dynamic LDS sizeof(AttnWideLds).
// Two barriers a step, executed by every wave: behind the first the maxima of the step's groups are in LDS, behind the
// second its probabilities.  The accumulating waves work on a step between its second barrier and that of the next step.
// What bounds it (in-kernel timestamps, one token at 1055 keys, 12 us): 2.2 us until the first scores (descriptor, page
// ids, keys: three dependent reads from HBM), five steps of 1.2 us (0.25 products, 0.35 maximum, 0.4 exponentials, the
// rest the unit's load path, which takes 64 KB a step at 64 B a cycle) and 1.1 us of last accumulation, fold and store.
// Eight scoring waves: 13.4 us (the load path again); keys and values requested two steps ahead: 13.8 us.
template <bool TREE>
__global__ void __launch_bounds__(64 * (kAttnWideScorers + 4), 4) k_attn_wide(int n_q_heads, int g4, const AttnTile *__restrict__ tiles,
                                                                           PagedKV kv, const bf16 *__restrict__ q,
                                                                           bf16 *__restrict__ out,
                                                                           const int32_t *__restrict__ row_end) {
  constexpr int NS = kAttnWideScorers;
  static_assert(NS % 4 == 0 && 16 % (NS / 2) == 0, "an even number of groups a step and parity, page ids of whole steps in 64 lanes");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  AttnWideLds &sm = *reinterpret_cast<AttnWideLds *>(smem_raw);

  typedef const int32_t __attribute__((address_space(4))) *ConstI32;
  const ConstI32 td = (ConstI32)(reinterpret_cast<const int32_t *>(tiles + blockIdx.x));
  if (td[0] < 0) return;  // uniform for the whole workgroup
  const int tile = td[1], slot = td[2], S = td[3], base = td[4], Lq = td[5], ty = td[6], pack = td[7];

  const int group = n_q_heads / kv.n_kv_heads, hb = (group + g4 - 1) / g4;
  const int kvh = ty / hb, hgrp = ty % hb;
  const int lhp = pack & 3, rshift = 5 - lhp;                      // 2^lhp heads of 2^rshift rows each
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5, qj = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int head = kvh * group + hgrp * g4 + ((pack >> 2) << lhp) + (qj >> rshift);
  const int row0 = tile << rshift, row = row0 + (qj & ((1 << rshift) - 1));
  const int my_row = min(row, Lq - 1);
  const int pos_j = S + my_row;
  const int n_valid = S + Lq;                                      // positions holding data of this round
  const int n_keys = S + min(row0 + (1 << rshift), Lq);            // keys any query of the set can see
  const int n_groups = (n_keys + 63) >> 6, n_steps = (n_groups + NS - 1) / NS;
  const int qdim = n_q_heads * kHd;
  const float sc = 0.125f * 1.4426950408889634f;

  const int32_t *table_row = kv.block_table + static_cast<size_t>(slot) * kv.max_blocks_per_seq;
  const int last_entry = kv.max_blocks_per_seq - 1;
  // Element offset of the page whose id lane `src` of `ids` holds.  An id out of range (a page beyond the data of this
  // round, a damaged table) reads block 0 instead; every position such a page could stand for is masked and its V zeroed.
  auto page_off = [&](int ids, int src) {
    const int id = __builtin_amdgcn_readlane(ids, src);
    return kv_block_offset(kv, (id >= 0 && id < kv.n_blocks) ? id : 0, kvh);
  };

  if (wave >= 4) {
    // ---- a scoring wave: groups w, w + NS, w + 2 NS, ...
    const int w = wave - 4;
    const bf16 *kpool = static_cast<const bf16 *>(kv.k_pool);
    Frag8 qf[4];
    // page ids: lane 4 s + p holds the id of page p of this wave's group in step s0 + s (16 steps at a time)
    auto fetch_ids = [&](int s0) { return table_row[min(((s0 + (lane >> 2)) * NS + w) * 4 + (lane & 3), last_entry)]; };
    int ids = fetch_ids(0);
    {
      const bf16 *qp = q + static_cast<size_t>(base + my_row) * qdim + head * kHd + half * 8;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) qf[kk].u = *reinterpret_cast<const uint4 *>(qp + kk * 16);
    }
    // K of a group: four pages of 2 KB, loaded as they lie (64 lanes read 1 KB in a row; a load in operand order, 32 rows of
    // 128 bytes, takes the address unit 64 cycles instead of 16), turned into operands through the wave's own LDS rows
    u32x4 rk[8];
    auto load_k = [&](int s) {
#pragma unroll
      for (int pg = 0; pg < 4; ++pg) {
        const bf16 *kp = kpool + page_off(ids, (s & 15) * 4 + pg) + lane * 8;
#pragma unroll
        for (int c = 0; c < 2; ++c) rk[2 * pg + c] = *reinterpret_cast<const u32x4 *>(kp + c * 512);
      }
    };
    uint16_t *ks = sm.k[w];
    auto store_k = [&]() {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // LDS runs a wave's accesses in order: only the compiler
      __builtin_amdgcn_wave_barrier();                         // has to be kept from reordering them
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4 *>(ks + (8 * i + (lane >> 3)) * kKsStride + (lane & 7) * 8) = rk[i];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    load_k(0);
    store_k();
    if (n_steps > 1) load_k(1);
    float m_run = -INFINITY;   // largest reference point of this wave's parity in the steps so far
    for (int s = 0; s < n_steps; ++s) {
      const int g = s * NS + w, kb = g * 64;
      floatx16 st[2];
      float mi = -INFINITY;
      if (g < n_groups) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
          for (int v = 0; v < 16; ++v) st[b][v] = 0.f;
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(ks + (b * 32 + qj) * kKsStride + kk * 16 + half * 8);
            st[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk].v, st[b], 0, 0, 0);
          }
        }
      }
      if (s + 1 < n_steps) {
        store_k();
        if (s + 2 < n_steps) {
          if (((s + 2) & 15) == 0) ids = fetch_ids(s + 2);
          load_k(s + 2);
        }
      }
      if (g < n_groups) {
        if constexpr (TREE) {
          if (kb + 63 >= S) {  // the group reaches into the block: tree-ancestry mask (see k_attn_mfma)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              int e_sub[16];   // half of the keys at a time: the other half's registers decide between one and two workgroups a unit
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const int kpos = kb + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
                e_sub[v] = row_end[base + min(max(kpos - S, 0), Lq - 1)];
              }
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const int kpos = kb + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
                const bool vis = (kpos <= pos_j) & ((kpos < S) | (e_sub[v] > base + my_row));
                st[b][v] = vis ? st[b][v] : -INFINITY;
              }
            }
          }
        } else if (kb + 63 > S + row0) {  // the group reaches past the first query: causal mask
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const int kpos = kb + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
              if (kpos > pos_j) st[b][v] = -INFINITY;
            }
        }
        float mx = fmaxf(st[0][0], st[1][0]);
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(fmaxf(mx, st[0][v]), st[1][v]);
        mi = ceilf(half_max(mx) * sc);   // integer reference point in the base-2 exponent domain (see k_attn_mfma)
      }
      if (half == 0) sm.mg[s & 1][w][qj] = mi;
      __syncthreads();
      // the reference point at this group: the largest of the parity's groups up to and including it
      float m_new = m_run;
#pragma unroll
      for (int k = 0; k < NS / 2; ++k) {
        const int w2 = 2 * k + (w & 1);
        const float v = sm.mg[s & 1][w2][qj];
        if (w2 <= w) m_new = fmaxf(m_new, v);
        m_run = fmaxf(m_run, v);
      }
      if (g < n_groups) {
        // a query that has seen no visible key yet: reference point 0 yields p = 0 without producing inf - inf
        const float msc = m_new == -INFINITY ? 0.f : m_new;
#pragma unroll
        for (int pg = 0; pg < 4; ++pg) {
          floatx8 pv;
#pragma unroll
          for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(fmaf(st[pg >> 1][8 * (pg & 1) + e], sc, -msc));
          Frag8 pf;
          pf.v = __builtin_convertvector(pv, bf16x8);
          sm.p[s & 1][w][pg][lane] = pf.u;
        }
      }
      __syncthreads();
    }
    __syncthreads();   // the fold below
    return;
  }

  // ---- an accumulating wave: parity par, head dims 32 i .. 32 i + 31
  constexpr int KG = NS / 2;                     // its groups a step: s * NS + 2 k + par
  constexpr int SPF = 16 / KG;                   // steps whose page ids fit 64 lanes: lane (s * KG + k) * 4 + page
  const int i = wave & 1, par = wave >> 1;
  const bf16 *vpool = static_cast<const bf16 *>(kv.v_pool);
  auto fetch_ids = [&](int s0) {
    const int x = lane >> 2;
    return table_row[min(((s0 + x / KG) * NS + 2 * (x % KG) + par) * 4 + (lane & 3), last_entry)];
  };
  Frag8 vf[KG][4];
  int ids = fetch_ids(0);
  auto load_v = [&](int s, int k) {
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
      const bf16 *vp = vpool + page_off(ids, ((s % SPF) * KG + k) * 4 + pg) + (i * 32 + qj) * kBlk + half * 8;
      vf[k][pg].u = *reinterpret_cast<const uint4 *>(vp);
    }
  };
#pragma unroll
  for (int k = 0; k < KG; ++k) load_v(0, k);
  floatx16 o;
#pragma unroll
  for (int v = 0; v < 16; ++v) o[v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};

  auto accumulate = [&](int s, int k) {
    const int w = 2 * k + par, g = s * NS + w;
    if (g >= n_groups) return;
    if (g * 64 + 64 > n_valid) {
      // slots of positions that hold no data of this sequence must read as 0 (their probability is 0, but 0 * stale-NaN
      // would poison the product); slot order of a V page: see kv_v_slot
#pragma unroll
      for (int pg = 0; pg < 4; ++pg)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int tok = (e < 4 ? 0 : 4) + 4 * half + e;
          if (g * 64 + pg * kBlk + tok >= n_valid) vf[k][pg].h[e] = 0;
        }
    }
    const float m_new = fmaxf(m_run, sm.mg[s & 1][w][qj]);
    if (__any(m_new != m_run)) {
      const float corr = (m_run == -INFINITY) ? 0.f : ldexpf(1.0f, static_cast<int>(m_run - m_new));
      l_run *= corr;
#pragma unroll
      for (int v = 0; v < 16; ++v) o[v] *= corr;
    }
    m_run = m_new;
    Frag8 pf[4];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) pf[pg].u = sm.p[s & 1][w][pg][lane];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
      o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k][pg].v, pf[pg].v, o, 0, 0, 0);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[pg].v, pf[pg].v, 0, 1), ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[pg].v, pf[pg].v, 2, 3), ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[pg].v, pf[pg].v, 4, 5), ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[pg].v, pf[pg].v, 6, 7), ones, l_run, false);
    }
  };

  __syncthreads();   // first step: maxima
  __syncthreads();   // first step: probabilities
  for (int s = 0; s + 1 < n_steps; ++s) {
    if ((s + 1) % SPF == 0) ids = fetch_ids(s + 1);
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      accumulate(s, k);
      load_v(s + 1, k);
      if (k == KG / 2 - 1) __syncthreads();   // step s + 1: maxima
    }
    __syncthreads();                          // step s + 1: probabilities
  }
#pragma unroll
  for (int k = 0; k < KG; ++k) accumulate(n_steps - 1, k);

  // ---- fold the two parities (even first), as k_attn_mfma does
  l_run = half_sum(l_run);
  if (par == 1) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sm.fold[i][v][lane] = o[v];
    sm.fold[i][16][lane] = m_run;
    sm.fold[i][17][lane] = l_run;
  }
  __syncthreads();
  if (par == 0 && row < Lq) {
    const float m_b = sm.fold[i][16][lane], l_b = sm.fold[i][17][lane];
    const float m_tot = fmaxf(m_run, m_b);
    const float ca = (m_run > -INFINITY) ? ldexpf(1.0f, static_cast<int>(m_run - m_tot)) : 0.f;
    const float cb = (m_b > -INFINITY) ? ldexpf(1.0f, static_cast<int>(m_b - m_tot)) : 0.f;
    const float inv = 1.0f / (l_run * ca + l_b * cb);
    bf16 *op = out + static_cast<size_t>(base + row) * qdim + head * kHd + i * 32 + 4 * half;
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      floatx4 ov;
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = (o[4 * gq + e] * ca + sm.fold[i][4 * gq + e][lane] * cb) * inv;
      *reinterpret_cast<bf16x4 *>(op + 8 * gq) = __builtin_convertvector(ov, bf16x4);
    }
  }
}

}  // namespace hsd
