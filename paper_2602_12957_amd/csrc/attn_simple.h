// Verification attention, plain version (fp32 debug path and cross-check of the MFMA kernel).
// Row r of sequence s at absolute position p attends to cached positions 0..p of s: the accepted prefix
// plus the draft rows before it in the same block, which the QKV epilogue has already appended to the
// pages (the chain case of the tree-ancestry mask, paper Section 3.2; with row_end given, the packed prefix tree
// itself).  Query head h reads kv head h/group.
// One wave per (row, query head): lanes own one key each for the scores and one head dimension each for
// the weighted sum of values; online softmax in fp32.
#pragma once

#include "common.h"
#include "gemm_simple.h"
#include "misc_kernels.h"

namespace hsd {

// grid: (total_q, ceil(n_q_heads/4)), block 256 = 4 waves = 4 query heads of one row.
template <typename T>
__global__ void __launch_bounds__(256) k_attn_simple(int n_q_heads, RowMeta meta, PagedKV kv,
                                                     const T *__restrict__ q, T *__restrict__ out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = blockIdx.x, head = blockIdx.y * 4 + wave;
  if (head >= n_q_heads) return;
  const int group = n_q_heads / kv.n_kv_heads, kvh = head / group;
  // keys live in cache slots 0 .. slot(r); slots before the block hold the accepted context (all visible), slot
  // S + i holds row i of the block: visible iff i is r's own row or (packed prefix tree) one of its ancestors
  const int s = meta.row_seq[r], n_keys = meta.row_slot[r] + 1;
  const int row0 = meta.row_base[r], S = meta.row_slot[r] - (r - row0);
  const T *kpool = static_cast<const T *>(kv.k_pool);
  const T *vpool = static_cast<const T *>(kv.v_pool);

  float qv[kHd];
  const T *qr = q + static_cast<size_t>(r) * (n_q_heads * kHd) + head * kHd;
#pragma unroll
  for (int d = 0; d < kHd; d += 8) load8(qr + d, qv + d);

  // 16 consecutive values of a lane's dimension as they lie in a V page (one page, slot order: kv_v_slot)
  auto load_page = [&](int id, float *v) {
    const T *p = vpool + kv_block_offset(kv, max(id, 0), kvh) + lane * kBlk;
#pragma unroll
    for (int i = 0; i < 16; i += 4) {   // (the pool needs no more than its elements' alignment)
      const floatx4 x = load4(p + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i + e] = x[e];
    }
  };
  // 1/sqrt(64); bf16 query rows carry it, with a log2(e) (EpiQKV::kQScale)
  const float scale = std::is_same<T, float>::value ? 0.125f : 0.69314718056f;
  float m = -INFINITY, l = 0.f, acc = 0.f;
  int id = lane < n_keys ? kv_lookup_block(kv, s, lane) : -1;   // block of the lane's key
  for (int j0 = 0; j0 < n_keys; j0 += kWave) {
    const int j = j0 + lane;
    // The chunk's values -- four pages, a lane's dimension of a page is 16 values in a row -- and the next chunk's block ids
    // are requested before the keys are looked at (132 rows of 4 heads over 272 to 304 keys: one value at a time 74.5 us,
    // eight in flight 47.4, this 24.5; 2048 rows over 1024 keys and more 1245 -> 385).
    float vv[4][16];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) load_page(__builtin_amdgcn_readlane(id, pg * kBlk), vv[pg]);
    bool seen = id >= 0;
    if (meta.row_end != nullptr && j >= S && j < n_keys && meta.row_end[row0 + j - S] <= r) seen = false;  // not an ancestor
    float score = -INFINITY;
    if (seen) {
      const T *kp = kpool + kv_block_offset(kv, id, kvh) + (j % kBlk) * kHd;
      float dot = 0.f;
#pragma unroll
      for (int d = 0; d < kHd; d += 8) {
        float kk[8];
        load8(kp + d, kk);
#pragma unroll
        for (int e = 0; e < 8; ++e) dot = fmaf(qv[d + e], kk[e], dot);
      }
      score = dot * scale;
    }
    id = j + kWave < n_keys ? kv_lookup_block(kv, s, j + kWave) : -1;
    float m_new = fmaxf(m, wave_max(score));
    if (m_new == -INFINITY) continue;  // no readable key in this chunk (wave-uniform)
    float pj = seen ? expf(score - m_new) : 0.f;
    float corr = (m == -INFINITY) ? 0.f : expf(m - m_new);
    l = l * corr + wave_sum(pj);
    acc *= corr;
    // a key that is not seen is left out, not multiplied by 0: its slot may hold anything
    const unsigned long long mask = __ballot(seen);
#pragma unroll
    for (int k = 0; k < kWave; ++k) {
      const float pb = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pj), k));
      const float v = vv[k / kBlk][kv_v_slot(k % kBlk)];
      acc = (mask >> k) & 1 ? fmaf(pb, v, acc) : acc;
    }
    m = m_new;
  }
  float o = (l > 0.f) ? acc / l : 0.f;
  out[static_cast<size_t>(r) * (n_q_heads * kHd) + head * kHd + lane] = from_f32<T>(o);
}

}  // namespace hsd
