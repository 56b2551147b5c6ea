// Small kernels around the GEMMs and the attention: row metadata + rotary table, embedding gather,
// RMSNorm, KV block reservation, LM-head arg-max reduction, acceptance scan, KV commit/rollback.
#pragma once

#include "common.h"

namespace hsd {

// ------------------------------------------------------------------------------------------------
// What a pass needs before its first projection, in one launch (k_pass_setup below): the pieces are independent, each is a
// few microseconds of dependent reads, and launches of their own would cost as much again each.
// ------------------------------------------------------------------------------------------------
struct AttnTile;   // attn_mfma.h
struct PassSetup {
  int n_seq, total_q, n_slots, max_blocks, n_blocks, d, vocab, n_dump;
  const int32_t *cu_q, *seq_slot, *seq_len, *tokens, *tree_end, *tree_depth, *dump_rows;
  const float *embeds, *gain;
  const void *table;
  int32_t *block_table, *free_list, *free_count, *status;
  int32_t *row_seq, *row_pos, *row_slot, *row_base, *row_end, *row_par, *row_kv, *dump_slot;
  float2 *rope_cs;
  float *want_logit, *x;
  void *h;
  float rope_theta, eps;
  // attention task table (n_wg = 0: none), see attn_tiles_block
  AttnTile *tasks;
  int q_tile, n_y, sub_tiles, n_wg, wide_g4;
};

// Last sequence whose first row is <= r
__device__ __forceinline__ int seq_of_row(const int32_t *cu_q, int n_seq, int r) {
  int lo = 0, hi = n_seq - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cu_q[mid] <= r) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Row metadata of packed row r: sequence, rotary position and (cos, sin) table, cache slot, and the packed tree it
// belongs to.  A chain block is the tree in which every row's subtree is the rest of the block.
//   row_pos  = seq_len + depth   (position on the row's own root-to-node path: what the rotary embedding sees)
//   row_slot = seq_len + local index (where its K/V are stored until commit)
//   row_end  = GLOBAL row index one past the row's subtree, clamped into (row, end of the sequence's block]
//   row_par  = GLOBAL row index of the parent (nearest earlier row whose subtree contains this one), -1 for a root
// The angle is formed in fp64 (position * theta^(-2i/64)) so that positions of many thousands lose nothing before the fp32
// rounding of cos/sin themselves.  32 adjacent lanes call it for one row, lane i with frequency index i; all of them look
// for the parent, 32 rows at a time (a walk by one lane was a read per row: 12 us for trees of 126 rows).
__device__ __forceinline__ void row_meta(const PassSetup &ps, int r, int i) {
  const int s = seq_of_row(ps.cu_q, ps.n_seq, r);
  const int base = ps.cu_q[s], stop = ps.cu_q[s + 1], local = r - base;
  const int slot = slot_of(ps.seq_slot, s, ps.n_slots), len = ps.seq_len[slot];
  int depth = local;
  if (ps.tree_depth != nullptr) {
    depth = ps.tree_depth[r];
    if (depth < 0 || depth > local || (local > 0 && depth == 0)) {
      depth = local > 0 ? 1 : 0;
      if (i == 0) atomicOr(ps.status, HSD_STATUS_BAD_TREE);
    }
  }
  const int pos = len + depth;
  int par = local > 0 ? r - 1 : -1;
  if (ps.row_par != nullptr && ps.tree_end != nullptr && local > 0) {
    // nearest earlier row whose (clamped) subtree reaches past r; row `base` (the root) always qualifies
    par = base;
    for (int hi = r - 1; hi > base; hi -= 32) {
      const int j = hi - i;
      const int ej = j > base ? base + ps.tree_end[j] : 0;
      const uint32_t hit = static_cast<uint32_t>(__ballot(j > base && ej > r && ej <= stop) >> (threadIdx.x & 32));
      if (hit != 0) {
        par = hi - (__ffs(hit) - 1);
        break;
      }
    }
  }
  if (i == 0) {
    ps.row_seq[r] = slot;
    ps.row_pos[r] = pos;
    ps.row_slot[r] = len + local;
    ps.row_base[r] = base;
    int e = stop;
    if (ps.tree_end != nullptr) {
      e = base + ps.tree_end[r];
      if (e <= r || e > stop || (local == 0 && e != stop)) {
        e = local == 0 ? stop : r + 1;
        atomicOr(ps.status, HSD_STATUS_BAD_TREE);
      }
    }
    ps.row_end[r] = e;
    if (ps.row_par != nullptr) {
      ps.row_par[r] = par;
      ps.want_logit[r] = -INFINITY;
    }
  }
  const double inv_freq = pow(static_cast<double>(ps.rope_theta), -2.0 * i / static_cast<double>(kHd));
  const double ang = static_cast<double>(pos) * inv_freq;
  double sn, cs;
  sincos(ang, &sn, &cs);
  ps.rope_cs[static_cast<size_t>(r) * 32 + i] = make_float2(static_cast<float>(cs), static_cast<float>(sn));
}

// dump_slot[r] = index into logits_dump for row r, or -1.  One block of 1024 threads.
__device__ inline void dump_slots_block(const PassSetup &ps) {
  for (int r = threadIdx.x; r < ps.total_q; r += 1024) ps.dump_slot[r] = -1;
  __threadfence_block();
  __syncthreads();
  for (int i = threadIdx.x; i < ps.n_dump; i += 1024) {
    const int r = ps.dump_rows[i];
    if (r >= 0 && r < ps.total_q) ps.dump_slot[r] = i;
  }
}

// ------------------------------------------------------------------------------------------------
// RMSNorm: h[r,:] = x[r,:] * rsqrt(mean(x^2) + eps) * gain, fp32 math, output in the GEMM operand type.
// One wave per row, 4 rows per 256-thread block; d is a multiple of 128 so every lane reads float4s.  The
// first kNormCache float4 of a lane (rows up to 2048 wide) stay in registers between the two passes.
// ------------------------------------------------------------------------------------------------
constexpr int kNormCache = 8;

__device__ __forceinline__ float sumsq4(const floatx4 &v) { return v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]; }

__device__ __forceinline__ void norm_store4(float *dst, const floatx4 &v, float rstd, const floatx4 &g) {
  floatx4 o = {v[0] * rstd * g[0], v[1] * rstd * g[1], v[2] * rstd * g[2], v[3] * rstd * g[3]};
  *reinterpret_cast<floatx4 *>(dst) = o;
}
__device__ __forceinline__ void norm_store4(bf16 *dst, const floatx4 &v, float rstd, const floatx4 &g) {
  floatx4 o = {v[0] * rstd * g[0], v[1] * rstd * g[1], v[2] * rstd * g[2], v[3] * rstd * g[3]};
  *reinterpret_cast<bf16x4 *>(dst) = __builtin_convertvector(o, bf16x4);   // round-to-nearest-even, 8-byte store
}

// second pass of both kernels: scale the row (cached part from registers, the rest re-read) and store it
template <typename T>
__device__ __forceinline__ void norm_write_row(const floatx4 *xr, const floatx4 (&cache)[kNormCache], int n4, int lane,
                                               float ss, int d, float eps, const float *gain, T *hr) {
  ss = wave_sum(ss);
  const float rstd = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
  const floatx4 *g4 = reinterpret_cast<const floatx4 *>(gain);
#pragma unroll
  for (int i = 0; i < kNormCache; ++i) {
    const int c = lane + kWave * i;
    if (c < n4) norm_store4(hr + 4 * c, cache[i], rstd, g4[c]);
  }
  for (int c = lane + kWave * kNormCache; c < n4; c += kWave) norm_store4(hr + 4 * c, xr[c], rstd, g4[c]);
}

template <typename T>
__global__ void k_rmsnorm(int n_rows, int d, float eps, const float *__restrict__ x, const float *__restrict__ gain,
                          T *__restrict__ h) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + wave;
  if (r >= n_rows) return;
  const floatx4 *xr = reinterpret_cast<const floatx4 *>(x + static_cast<size_t>(r) * d);
  const int n4 = d >> 2;
  floatx4 cache[kNormCache];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kNormCache; ++i) {
    const int c = lane + kWave * i;
    if (c < n4) {
      cache[i] = xr[c];
      ss += sumsq4(cache[i]);
    }
  }
  for (int c = lane + kWave * kNormCache; c < n4; c += kWave) ss += sumsq4(xr[c]);
  norm_write_row<T>(xr, cache, n4, lane, ss, d, eps, gain, h + static_cast<size_t>(r) * d);
}

// Residual row r and the first norm's operand: x[r,:] = table[tokens[r],:] (widened to fp32), or embeds[r,:] if tokens[r] < 0
// (zeros without embeds), and h[r,:] as k_rmsnorm makes it from x -- same lanes, same sums.  One wave.
// Table and embeddings come from the caller and need no more than their element's alignment.
__device__ __forceinline__ floatx4 load4(const float *p) {
  typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
  return *reinterpret_cast<const floatx4u *>(p);
}
__device__ __forceinline__ floatx4 load4(const bf16 *p) {
  typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));
  const u32x2u u = *reinterpret_cast<const u32x2u *>(p);
  return floatx4{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xffff0000u)};
}
template <typename T>
__device__ __forceinline__ void embed_norm_row(const PassSetup &ps, int r, int lane) {
  const int t = min(ps.tokens[r], ps.vocab - 1);   // ids are validated by the caller; clamp keeps the read in bounds
  const T *tok = static_cast<const T *>(ps.table) + static_cast<size_t>(max(t, 0)) * ps.d;
  const float *emb = ps.embeds != nullptr ? ps.embeds + static_cast<size_t>(r) * ps.d : nullptr;
  floatx4 *xr = reinterpret_cast<floatx4 *>(ps.x + static_cast<size_t>(r) * ps.d);
  const int n4 = ps.d >> 2;
  auto value = [&](int c) { return t >= 0 ? load4(tok + 4 * c) : emb != nullptr ? load4(emb + 4 * c) : floatx4{0.f, 0.f, 0.f, 0.f}; };
  floatx4 cache[kNormCache];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kNormCache; ++i) {
    const int c = lane + kWave * i;
    if (c < n4) {
      cache[i] = value(c);
      xr[c] = cache[i];
      ss += sumsq4(cache[i]);
    }
  }
  for (int c = lane + kWave * kNormCache; c < n4; c += kWave) {
    const floatx4 v = value(c);
    xr[c] = v;
    ss += sumsq4(v);
  }
  norm_write_row<T>(xr, cache, n4, lane, ss, ps.d, ps.eps, ps.gain, static_cast<T *>(ps.h) + static_cast<size_t>(r) * ps.d);
}

// ------------------------------------------------------------------------------------------------
// Block-wide exclusive scan of up to HSD_MAX_SEQ ints held in LDS (1024 threads, 4 items each), which the caller's barrier
// has made visible.
// On return s_val[i] holds the exclusive prefix and the function returns the grand total.
// ------------------------------------------------------------------------------------------------
__device__ inline int block_exclusive_scan_4096(int *s_val, int n, int *s_part /*[16]*/) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, base = t * 4;
  int v[4], sum = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = (base + j < n) ? s_val[base + j] : 0;
    sum += v[j];
  }
  int incl = sum;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int up = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += up;
  }
  if (lane == kWave - 1) s_part[wave] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int p = s_part[w];
    if (w < wave) before += p;
    total += p;
  }
  int run = before + incl - sum;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (base + j < n) s_val[base + j] = run;
    run += v[j];
  }
  __syncthreads();
  return total;
}

// ------------------------------------------------------------------------------------------------
// KV block reservation for the speculative append.  For every sequence, every block-table slot that
// covers positions seq_len .. seq_len+q_len-1 and holds no block gets one popped from the free stack.
// Deterministic: sequence s takes its blocks after all sequences < s, slots in increasing order.
// Afterwards row_kv[r] = where packed row r's key and value land in the paged pools: 16 * block id + slot within the block,
// or -1 when the table holds no valid block for the row's position (reservation failed).  Block ids are the same in every
// layer, so the projection epilogues of all layers read this one array instead of walking row -> sequence -> table
// themselves.
// One block of 1024 threads (16 waves; waves stride over sequences, lanes over slots).  `lds`: HSD_MAX_SEQ + 18 ints.
// ------------------------------------------------------------------------------------------------
__device__ inline void kv_reserve_block(const PassSetup &ps, int *lds) {
  int *s_cnt = lds, *s_part = lds + HSD_MAX_SEQ, *s_flags = s_part + 16;
  const int32_t *__restrict__ cu_q = ps.cu_q;
  const int maxb = ps.max_blocks, n_seq = ps.n_seq;
  int32_t *block_table = ps.block_table;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (threadIdx.x == 0) *s_flags = 0;
  __syncthreads();
  for (int s = wave; s < n_seq; s += 16) {
    const int sl = slot_of(ps.seq_slot, s, ps.n_slots);
    if (lane == 0 && ps.seq_slot != nullptr && ps.seq_slot[s] != sl) atomicOr(s_flags, HSD_STATUS_BAD_SLOT);
    const int S = ps.seq_len[sl], Lq = cu_q[s + 1] - cu_q[s];
    const int lo = S / kBlk;
    int hi = (S + Lq + kBlk - 1) / kBlk;
    if (hi > maxb) {
      if (lane == 0) atomicOr(s_flags, HSD_STATUS_TABLE_OVERFLOW);
      hi = maxb;
    }
    int cnt = 0;
    for (int i = lo + lane; i < hi; i += kWave) cnt += (block_table[static_cast<size_t>(sl) * maxb + i] < 0);
    cnt = wave_sum_i(cnt);
    if (lane == 0) s_cnt[s] = cnt;
  }
  __syncthreads();
  const int total = block_exclusive_scan_4096(s_cnt, n_seq, s_part);
  int avail = *ps.free_count;
  if (avail > ps.n_blocks) avail = ps.n_blocks;
  if (total > avail) {
    // nothing is taken; slots stay -1 and every later kernel skips them
    if (threadIdx.x == 0) atomicOr(ps.status, *s_flags | HSD_STATUS_POOL_EXHAUSTED);
  } else {
    for (int s = wave; s < n_seq; s += 16) {
      const int sl = slot_of(ps.seq_slot, s, ps.n_slots);
      const int S = ps.seq_len[sl], Lq = cu_q[s + 1] - cu_q[s];
      const int lo = S / kBlk;
      int hi = (S + Lq + kBlk - 1) / kBlk;
      if (hi > maxb) hi = maxb;
      int taken = s_cnt[s];  // exclusive prefix = blocks taken by earlier sequences
      for (int i0 = lo; i0 < hi; i0 += kWave) {
        const int i = i0 + lane;
        const bool need = (i < hi) && (block_table[static_cast<size_t>(sl) * maxb + i] < 0);
        const unsigned long long m = __ballot(need);
        const int rank = __popcll(m & ((1ull << lane) - 1ull));
        if (need) block_table[static_cast<size_t>(sl) * maxb + i] = ps.free_list[avail - 1 - (taken + rank)];
        taken += __popcll(m);
      }
    }
  }
  __threadfence_block();
  __syncthreads();   // the table is complete (for this block, which is all that reads it here)
  if (threadIdx.x == 0 && total <= avail) {
    *ps.free_count = avail - total;
    if (*s_flags) atomicOr(ps.status, *s_flags);
  }
  for (int r = threadIdx.x; r < ps.total_q; r += 1024) {
    const int s = seq_of_row(cu_q, n_seq, r);
    const int sl = slot_of(ps.seq_slot, s, ps.n_slots);
    const int pos = ps.seq_len[sl] + (r - cu_q[s]), bi = pos / kBlk;
    int b = -1;
    if (bi < maxb) b = block_table[static_cast<size_t>(sl) * maxb + bi];
    ps.row_kv[r] = (b >= 0 && b < ps.n_blocks) ? b * kBlk + pos % kBlk : -1;
  }
}

// ------------------------------------------------------------------------------------------------
// KV commit / rollback.  seq_len += 1 + alpha (alpha >= 0), or += q_len when commit_all (prefill);
// slots wholly beyond the new length are pushed back on the free stack in (sequence, slot) order.
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) k_kv_commit(int n_seq, const int32_t *__restrict__ cu_q,
                                                    const int32_t *__restrict__ seq_slot, int n_slots,
                                                    int32_t *__restrict__ seq_len, int32_t *__restrict__ block_table,
                                                    int maxb, int n_blocks, int32_t *__restrict__ free_list,
                                                    int32_t *__restrict__ free_count,
                                                    const int32_t *__restrict__ accept_len,
                                                    const int32_t *__restrict__ bonus, int32_t *__restrict__ pending_out,
                                                    int commit_all) {
  __shared__ int s_cnt[HSD_MAX_SEQ];
  __shared__ int s_new[HSD_MAX_SEQ];
  __shared__ int s_part[16];
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int s = wave; s < n_seq; s += 16) {
    int sl = slot_of(seq_slot, s, n_slots);
    int S = seq_len[sl], Lq = cu_q[s + 1] - cu_q[s];
    int new_len = S;
    if (commit_all) {
      new_len = S + Lq;
    } else {
      int a = accept_len[s];
      if (a > Lq - 1) a = Lq - 1;
      if (a >= 0) new_len = S + 1 + a;
    }
    int keep = (new_len + kBlk - 1) / kBlk, hi = (S + Lq + kBlk - 1) / kBlk;
    if (hi > maxb) hi = maxb;
    int cnt = 0;
    for (int i = keep + lane; i < hi; i += kWave) {
      int b = block_table[static_cast<size_t>(sl) * maxb + i];
      cnt += (b >= 0 && b < n_blocks);
    }
    cnt = wave_sum_i(cnt);
    if (lane == 0) {
      s_cnt[s] = cnt;
      s_new[s] = new_len;
    }
  }
  __syncthreads();
  int total = block_exclusive_scan_4096(s_cnt, n_seq, s_part);
  int height = *free_count;
  if (height < 0) height = 0;
  if (height + total > n_blocks) total = 0, height = -1;  // corrupted accounting: free nothing
  for (int s = wave; s < n_seq; s += 16) {
    int sl = slot_of(seq_slot, s, n_slots);
    int S = seq_len[sl], Lq = cu_q[s + 1] - cu_q[s];
    int new_len = s_new[s];
    int keep = (new_len + kBlk - 1) / kBlk, hi = (S + Lq + kBlk - 1) / kBlk;
    if (hi > maxb) hi = maxb;
    int pushed = s_cnt[s];
    if (height >= 0) {
      for (int i0 = keep; i0 < hi; i0 += kWave) {
        int i = i0 + lane;
        int b = (i < hi) ? block_table[static_cast<size_t>(sl) * maxb + i] : -1;
        bool has = (b >= 0 && b < n_blocks);
        unsigned long long m = __ballot(has);
        int rank = __popcll(m & ((1ull << lane) - 1ull));
        if (has) {
          free_list[height + pushed + rank] = b;
          block_table[static_cast<size_t>(sl) * maxb + i] = -1;
        }
        pushed += __popcll(m);
      }
    }
  }
  __syncthreads();
  for (int s = threadIdx.x; s < n_seq; s += blockDim.x) {
    bool advanced = commit_all || accept_len[s] >= 0;
    seq_len[slot_of(seq_slot, s, n_slots)] = s_new[s];
    if (!commit_all && advanced && pending_out != nullptr) pending_out[s] = bonus[s];
  }
  if (threadIdx.x == 0 && height >= 0) *free_count = height + total;
}

__global__ void k_pool_init(int n_blocks, int32_t *__restrict__ free_list, int32_t *__restrict__ free_count) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_blocks) free_list[i] = n_blocks - 1 - i;  // popping from the top hands out 0, 1, 2, ...
  if (i == 0) *free_count = n_blocks;
}

// ------------------------------------------------------------------------------------------------
// LM-head arg-max, second stage: merge the per-(row, column tile) Top2 partials of the LM-head GEMM.
// One wave per row.  Output u_hat (Eq. 10: arg-max over the vocabulary; arg-max of logits equals
// arg-max of probabilities) and the top-1/top-2 logit margin.
// ------------------------------------------------------------------------------------------------
__global__ void k_lm_reduce(int n_rows, int n_tiles, const Top2 *__restrict__ part, int32_t *__restrict__ argmax,
                            float *__restrict__ margin, float *__restrict__ row_max, int32_t *__restrict__ accept_len,
                            int32_t *__restrict__ bonus, float *__restrict__ draft_gap) {
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int r = blockIdx.x * 4 + wave;
  if (r >= n_rows) return;
  Top2 t = top2_init();
  for (int c = lane; c < n_tiles; c += kWave) t = top2_merge(t, part[static_cast<size_t>(r) * n_tiles + c]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    Top2 u;
    u.m1 = __shfl_xor(t.m1, o, kWave);
    u.i1 = __shfl_xor(t.i1, o, kWave);
    u.m2 = __shfl_xor(t.m2, o, kWave);
    t = top2_merge(t, u);
  }
  if (lane == 0) {
    argmax[r] = t.i1;
    if (margin != nullptr) margin[r] = t.m1 - t.m2;
    if (row_max != nullptr) row_max[r] = t.m1;
    if (accept_len != nullptr) {   // every block is its pending token alone: nothing to accept, the arg-max is the bonus
      accept_len[r] = 0;
      bonus[r] = t.i1;
      if (draft_gap != nullptr) draft_gap[r] = -INFINITY;
    }
  }
}

// Relaxed acceptance (Eq. 11) in logits: log p(u*) - log p(u_hat) = logit(u*) - max logit, both taken at the PARENT
// row of the candidate.  draft_gap[r] = (logit of row r's own token at its parent's row) - (parent's row maximum);
// -inf for root rows.  One thread per row.
__global__ void k_draft_gap(int n_rows, const int32_t *__restrict__ row_par, const float *__restrict__ want_logit,
                            const float *__restrict__ row_max, float *__restrict__ draft_gap) {
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rows) return;
  const int p = row_par[r];
  draft_gap[r] = p < 0 ? -INFINITY : want_logit[r] - row_max[p];
}

// ------------------------------------------------------------------------------------------------
// Draft compare + longest-prefix acceptance on chain blocks (Eq. 9, 11; Eq. 12 bonus; alpha of Eq. 15).
// One wave per sequence: lanes test 64 draft positions at a time, a ballot finds the first rejection.
// Exact rule (log_tau == 0): reject_i = (tokens[base+i] != argmax[base+i-1]) for i = 1..k.
// Relaxed rule (log_tau < 0): reject_i = !(draft_gap[base+i] >= log_tau).
// ------------------------------------------------------------------------------------------------
__global__ void k_accept(int n_seq, const int32_t *__restrict__ cu_q, const int32_t *__restrict__ tokens,
                         const int32_t *__restrict__ argmax, const float *__restrict__ draft_gap, float log_tau,
                         int32_t *__restrict__ accept_len, int32_t *__restrict__ bonus) {
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int s = blockIdx.x * 4 + wave;
  if (s >= n_seq) return;
  int base = cu_q[s], k = cu_q[s + 1] - base - 1;
  const bool relaxed = log_tau < 0.f && draft_gap != nullptr;
  int alpha = k;
  for (int i0 = 1; i0 <= k; i0 += kWave) {
    int i = i0 + lane;
    bool reject = false;
    if (i <= k) reject = relaxed ? !(draft_gap[base + i] >= log_tau) : (tokens[base + i] != argmax[base + i - 1]);
    unsigned long long m = __ballot(reject);
    if (m != 0ull) {
      alpha = i0 + (__ffsll(static_cast<long long>(m)) - 1) - 1;  // accepted = index of first rejection - 1
      break;
    }
  }
  if (lane == 0) {
    accept_len[s] = alpha;
    bonus[s] = argmax[base + alpha];
  }
}

// ------------------------------------------------------------------------------------------------
// Greedy traversal of a packed prefix tree (Eq. 9-12).  At node s the children are s+1, row_end[s+1], ... while <
// row_end[s].
// Exact rule: enter the child whose token is the row's arg-max token, if there is one (then u* = u_hat).
// Relaxed rule: u* = the child with the largest logit at row s (lowest row among equals); enter it iff
// draft_gap[u*] >= log_tau.  Outputs alpha = depth reached, the bonus token (arg-max at the stop node) and the
// stop node's local row.
// The walk is a chain of dependent reads, one record per child looked at.  One wave per sequence first brings the records
// of its rows into LDS (trees of more rows than fit walk global memory): 31 -> 17 us for trees of 126 rows and 56 levels.
// grid: n_seq blocks of 64 threads.
// ------------------------------------------------------------------------------------------------
constexpr int kTreeRowsLds = 2048;
__global__ void __launch_bounds__(64) k_accept_tree(int n_seq, const int32_t *__restrict__ cu_q, const int32_t *__restrict__ tokens,
                                                    const int32_t *__restrict__ argmax, const int32_t *__restrict__ row_end,
                                                    const float *__restrict__ want_logit, const float *__restrict__ draft_gap,
                                                    float log_tau, int32_t *__restrict__ accept_len, int32_t *__restrict__ bonus,
                                                    int32_t *__restrict__ stop_row) {
  __shared__ int4 s_rec[kTreeRowsLds];
  const int sq = blockIdx.x, lane = threadIdx.x;
  const int base = cu_q[sq], Lq = cu_q[sq + 1] - base;
  const bool relaxed = log_tau < 0.f && draft_gap != nullptr;
  // row_end, arg-max, and: the token, or the wanted logit and the gap
  auto global_rec = [&](int r) {
    return relaxed ? int4{row_end[r], argmax[r], __float_as_int(want_logit[r]), __float_as_int(draft_gap[r])}
                   : int4{row_end[r], argmax[r], tokens[r], 0};
  };
  const bool in_lds = Lq <= kTreeRowsLds;
  if (in_lds) {
    for (int i = lane; i < Lq; i += kWave) s_rec[i] = global_rec(base + i);
    __syncthreads();
  }
  // (the same for all lanes: handed on through scalar registers, so that the walk branches on the scalar unit)
  auto rec = [&](int r) {
    const int4 v = in_lds ? s_rec[r - base] : global_rec(r);
    return int4{__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y), __builtin_amdgcn_readfirstlane(v.z),
                __builtin_amdgcn_readfirstlane(v.w)};
  };
  int s = base, alpha = 0;
  int4 node = rec(s);
  for (;;) {
    int best = -1;
    float best_v = -INFINITY;
    int4 best_rec = node;
    for (int c = s + 1; c < node.x;) {
      const int4 child = rec(c);
      if (relaxed) {
        const float v = __int_as_float(child.z);
        if (best < 0 || v > best_v) best = c, best_v = v, best_rec = child;
      } else if (child.z == node.y) {
        best = c, best_rec = child;
        break;
      }
      c = child.x;
    }
    if (best < 0) break;
    if (relaxed && !(__int_as_float(best_rec.w) >= log_tau)) break;
    s = best;
    node = best_rec;
    ++alpha;
  }
  if (lane == 0) {
    accept_len[sq] = alpha;
    bonus[sq] = node.y;
    stop_row[sq] = s - base;
  }
}

// ------------------------------------------------------------------------------------------------
// Commit of a packed tree: the accepted root-to-stop path becomes ordinary context.  Its node at depth d was stored
// at cache slot S + (local row) and moves to slot S + d, d = 1..alpha.  A node's pre-order row is never smaller than its
// depth and rows grow along the path, so a target slot is never the source of a later move: moves go in batches, every
// source of a batch read before its first target is written.
// The path is found in LDS, 64 levels at a time (level d's lane looks up its two slots); found and moved node by node in
// global memory it took 40 us for 56 levels, now 31.
// grid: (n_seq, n_layers * n_kv_heads), block 64: lane = head dimension.  Runs BEFORE the length update.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(64) k_kv_compact(const int32_t *__restrict__ cu_q, const int32_t *__restrict__ seq_slot, int n_slots,
                                                   const int32_t *__restrict__ seq_len, const int32_t *__restrict__ block_table,
                                                   int maxb, int n_blocks, int n_kv_heads, const int32_t *__restrict__ tree_end,
                                                   const int32_t *__restrict__ accept_len, const int32_t *__restrict__ stop_row,
                                                   T *k_pool, T *v_pool) {
  __shared__ int s_end[kTreeRowsLds];
  const int sq = blockIdx.x, layer = blockIdx.y / n_kv_heads, kvh = blockIdx.y % n_kv_heads, dim = threadIdx.x;
  const int base = cu_q[sq], Lq = cu_q[sq + 1] - base;
  const int sl = slot_of(seq_slot, sq, n_slots);
  const int S = seq_len[sl];
  const int alpha = accept_len[sq], stop = stop_row[sq];
  if (alpha < 1 || stop < 1 || stop >= Lq) return;   // uniform for the block
  auto global_end = [&](int i) {   // same clamping as the row metadata
    const int e = tree_end[base + i];
    return (e <= i || e > Lq) ? i + 1 : e;
  };
  const bool in_lds = stop < kTreeRowsLds;   // no row past the stop node is looked at
  if (in_lds) {
    for (int i = dim; i <= stop; i += kWave) s_end[i] = global_end(i);
    __syncthreads();
  }
  auto end_of = [&](int i) { return __builtin_amdgcn_readfirstlane(in_lds ? s_end[i] : global_end(i)); };
  int s = 0;
  for (int d0 = 1; d0 <= alpha; d0 += kWave) {
    const int m = min(kWave, alpha - d0 + 1);
    int row = -1, found = 0;   // lane j: the path's node at depth d0 + j
    for (; found < m; ++found) {
      // the child of s whose subtree contains the stop node
      int c = s + 1;
      while (c <= stop) {
        const int e = end_of(c);
        if (stop < e) break;
        c = e;
      }
      if (c > stop) break;   // malformed tree: nothing sensible to move
      s = c;
      if (dim == found) row = c;
    }
    size_t os = 0, od = 0;
    bool ok = row >= 0;
    if (ok && row != d0 + dim) {   // (otherwise already in place)
      const int src = S + row, dst = S + d0 + dim;
      ok = src / kBlk < maxb;
      if (ok) {
        const int bs = block_table[static_cast<size_t>(sl) * maxb + src / kBlk];
        const int bd = block_table[static_cast<size_t>(sl) * maxb + dst / kBlk];
        ok = bs >= 0 && bs < n_blocks && bd >= 0 && bd < n_blocks;
        os = ((static_cast<size_t>(layer) * n_blocks + bs) * n_kv_heads + kvh) * (kBlk * kHd);
        od = ((static_cast<size_t>(layer) * n_blocks + bd) * n_kv_heads + kvh) * (kBlk * kHd);
      }
    }
    const unsigned long long bad = __ballot(!ok);
    const int n_move = min(found, bad != 0 ? static_cast<int>(__ffsll(static_cast<long long>(bad))) - 1 : kWave);
    constexpr int U = 8;
    for (int j0 = 0; j0 < n_move; j0 += U) {
      T kv_[U], vv[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int l = min(j0 + j, n_move - 1), r = __shfl(row, l, kWave);
        const size_t o = __shfl(os, l, kWave);
        if (j0 + j < n_move && r != d0 + l) {
          kv_[j] = k_pool[o + ((S + r) % kBlk) * kHd + dim];
          vv[j] = v_pool[o + kv_v_elem((S + r) % kBlk, dim)];
        }
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int l = min(j0 + j, n_move - 1), r = __shfl(row, l, kWave);
        const size_t o = __shfl(od, l, kWave);
        if (j0 + j < n_move && r != d0 + l) {
          k_pool[o + ((S + d0 + l) % kBlk) * kHd + dim] = kv_[j];
          v_pool[o + kv_v_elem((S + d0 + l) % kBlk, dim)] = vv[j];
        }
      }
    }
    if (found < m || n_move < found) return;
  }
}

}  // namespace hsd
