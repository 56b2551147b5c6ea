// bf16 MFMA GEMM for passes of a few rows (token-by-token decoding, the rests of drafts): 16-row tiles, operands by
// LDS-direct loads in long runs, a whole projection in flight.
//
// Why.  With a few rows a launch reads the weights once, from HBM, and little else; its time is that of one workgroup's
// bytes through its compute unit's load path, plus latencies.  Measured: a unit streams 25 to 29 B/ns of cold weights with
// 32 KB in flight and twice that when they lie in its L2; a 32x32 tile brings 32 activation rows (of which one token
// fills one) beside 32 weight rows, 512 KB a workgroup for the down projection.  Here a tile has 16 rows per multiplying wave, its weight side as few as 16 columns, so that twice the units
// stream half the bytes each, rows past the end of the activations are not fetched at all (the buffer's range check
// answers them), and up to 144 KB are in flight: both K = 1024 slices of a tile from the start.
//
// The products run on v_mfma_f32_16x16x32_bf16.  One of them adds the same products in the same order as two
// v_mfma_f32_32x32x16_bf16 on the halves of its K range, bit for bit (compared on this chip over 1.3 M sums of 32 to 4096
// products with exponents spread over 20 binades, and by tests/test_gpu_small_launches.py), so results are identical to
// every other tile configuration.
//
// Tile.  RT multiplying waves, 16 rows each, share 16 CW weight rows: 8 CW output columns and their partners -- the
// columns 32 further on (rotary pairs), or in dual mode the up rows of the same columns.  Four more waves only request.
// Stage: SK values of K per row.  A load instruction brings 1 KB of one row (SK = 512) or 512 bytes of two; the 16-byte
// piece p of tile row r lies at position p ^ (r & 15) of its LDS row, so that the fragment reads of 16 rows cover all 64
// banks once.
//
// Measured on the 24-layer model (d 1024, traces, us; before: 32x32, 64x64 and 64x128 tiles): down 13.0 -> 6.3 at one row (64
// workgroups, 1.3 TB/s), 13.2 -> 7.6 at 64, 23.5 -> 21.3 at 1008, 31.3 -> 26.7 at 1856 (128x64 tiles, 50 B/ns a unit); O 6.0 ->
// 4.1, 6.3 -> 4.9, 10.4 -> 9.1, 13.6 -> 11.6; QKV 7.1 -> 4.3 and gate/up 8.0 -> 5.7 at one row.  A launch over one row is 0.5 us
// to the first request, 1.1 to 1.5 until the first stage has landed, the chain of products, 0.5 of epilogue and 1.5 of
// launch and drain.
#pragma once

#include "gemm_mfma_d.h"

namespace hsd {

template <int RT_, int CW_, int SK_, int STAGES_>
struct GemmCfgR {
  static constexpr int RT = RT_, CW = CW_, SK = SK_, kStages = STAGES_;
  static constexpr int BP = 16 * RT_, BQ = 16 * CW_;               // activation rows, weight rows of a tile
  static constexpr int kCols = 8 * CW_;                            // output columns up to their partners
  static constexpr int kRowBytes = SK_ * 2;
  static constexpr int kStageBytes = (BP + BQ) * kRowBytes;
  static constexpr int kEpiStride = BQ + 4;                        // floats per row of a wave's epilogue staging
  static constexpr int kSmemBytes = STAGES_ * kStageBytes;         // kRowScaleBytes more follow them
  static constexpr int kLoaders = 4;
  static constexpr int kLoadsP = BP * kRowBytes / 1024 / kLoaders, kLoadsQ = BQ * kRowBytes / 1024 / kLoaders;
  static constexpr int kThreads = 64 * (RT_ + kLoaders);
  static_assert(SK_ == 128 || SK_ == 256 || SK_ == 512, "16, 32 or 64 pieces a row");
  static_assert(BP * kRowBytes % (1024 * kLoaders) == 0 && BQ * kRowBytes % (1024 * kLoaders) == 0, "requests divide evenly over the waves");
  static_assert(CW_ == 1 || CW_ == 2 || CW_ == 4, "a quarter, half or whole 64-column group");
  static_assert(STAGES_ >= 2 && STAGES_ <= 4 && (STAGES_ - 1) * (kLoadsP + kLoadsQ) < 64, "the load counter holds 63");
  static_assert(RT_ * 16 * kEpiStride * 4 <= kSmemBytes && kSmemBytes + kRowScaleBytes <= 160 * 1024, "LDS");
};

// grid: ceil((M - m_base) / BP) * (N / kCols / (dual ? 1 : 2)) workgroups of Cfg::kThreads threads, Cfg::kSmemBytes +
// kRowScaleBytes dynamic LDS; the tiles cover rows m_base .. M-1 (see k_gemm_mfma_d).  K a multiple of 32; N a multiple of 64; both matrices below 2 GiB (32-bit buffer offsets).
// band >= 0: band_grid workgroups in the order of band_tile.
// Every wave executes exactly ceil(K / SK) + 1 workgroup barriers (none in a workgroup without a tile).
// NT: the weight loads are non-temporal (weights_pass_by in hsd_api.hip says when).
template <typename Cfg, int MODE, typename Epi, bool NT>
__global__ void __launch_bounds__(Cfg::kThreads) k_gemm_mfma_r(int M, int N, int K, int m_base, int band, const bf16 *__restrict__ A,
                                                               const bf16 *__restrict__ W, Epi epi) {
  static_assert(MODE == kModeNormal || MODE == kModeDual, "normal or dual mode");
  constexpr int BP = Cfg::BP, CW = Cfg::CW, S = Cfg::kStages, RB = Cfg::kRowBytes, COLS = Cfg::kCols;
  constexpr int NLP = Cfg::kLoadsP, NLQ = Cfg::kLoadsQ, NL = NLP + NLQ;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tiles_act = (M - m_base + BP - 1) / BP;
  // (the grid is computed, not read: gridDim lies behind the kernel arguments in memory, a read on the way to the first load)
  int ta, tw;
  const int tiles_w = N / (MODE == kModeDual ? COLS : 2 * COLS);
  if (band < 0) xcd_tile(blockIdx.x, tiles_act, tiles_act * tiles_w, ta, tw);
  else if (!band_tile(blockIdx.x, tiles_act, tiles_w, band, ta, tw)) return;   // the whole workgroup
  const int m0 = m_base + ta * BP;
  constexpr int GR = 4 / CW;                           // tiles of a 64-column group
  const int n0 = (MODE == kModeDual) ? tw * COLS : tw / GR * 64 + tw % GR * COLS;
  const int nf = K / Cfg::SK, ns = (K + Cfg::SK - 1) / Cfg::SK;   // full stages; the last one may be partly filled

  if (wave >= Cfg::RT) {
    // ---- a requesting wave.  Rows from M on read as zero: the hardware checks the vector offset against the matrix's
    // size.  It does not check the scalar one, so a partly filled last stage, which reaches past the end of the last row,
    // carries its K offset in the vector part.  Of the 1 KB pieces of a stage's activation rows, and of its weight rows,
    // requesting wave lw fetches pieces 4 j + lw.
    constexpr int LPR = RB / 16;                       // lanes of a row
    const int lw = wave - Cfg::RT;
    const LdsBytePtr lds = (LdsBytePtr)smem_raw;
    const __amdgpu_buffer_rsrc_t rs_p = make_rsrc(A, static_cast<size_t>(M) * K * 2);
    const __amdgpu_buffer_rsrc_t rs_q = make_rsrc(W, static_cast<size_t>(MODE == kModeDual ? 2 * N : N) * K * 2);
    int vp[NLP], vq[NLQ];
#pragma unroll
    for (int j = 0; j < NLP; ++j) {
      const int r = (4 * j + lw) * (64 / LPR) + lane / LPR;
      vp[j] = ((m0 + r) * K + ((lane % LPR) ^ (r & 15)) * 8) * 2;
    }
#pragma unroll
    for (int j = 0; j < NLQ; ++j) {
      const int r = (4 * j + lw) * (64 / LPR) + lane / LPR;
      const int row = n0 + r % COLS + r / COLS * (MODE == kModeDual ? N : 32);   // COLS output columns, then their partners
      vq[j] = (row * K + ((lane % LPR) ^ (r & 15)) * 8) * 2;
    }
#define HSD_GR_ISSUE(slot, s)                                                                          \
  {                                                                                                    \
    const LdsBytePtr dst = lds + (slot) * Cfg::kStageBytes;                                            \
    const int kv = (s) < nf ? 0 : (s) * RB, ks = (s) < nf ? (s) * RB : 0;                              \
    _Pragma("unroll") for (int j = 0; j < NLQ; ++j)                                                    \
        lds_load16<NT>(rs_q, dst + (BP * RB + (4 * j + lw) * 1024), vq[j] + kv, ks);                   \
    _Pragma("unroll") for (int j = 0; j < NLP; ++j)                                                    \
        lds_load16(rs_p, dst + (4 * j + lw) * 1024, vp[j] + kv, ks);                                   \
  }
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
      if (s < ns) HSD_GR_ISSUE(s, s)
    int slot = S - 1;   // of stage s - 1, free once everyone is past barrier s
    for (int s = 0; s < ns; ++s) {
      // stage s has landed; stages s + 1 .. s + S - 2 (requested so far) may stay in flight
      const int ahead = min(ns - 1 - s, S - 2);
#define HSD_GR_WAIT(n) case n: HSD_VMCNT((n) * NL < 63 ? (n) * NL : 63); break;
      switch (ahead) { HSD_GR_WAIT(0) HSD_GR_WAIT(1) HSD_GR_WAIT(2) default: HSD_VMCNT(0); }
#undef HSD_GR_WAIT
      __builtin_amdgcn_s_barrier();
      if (s + S - 1 < ns) HSD_GR_ISSUE(slot, s + S - 1)
      slot = slot + 1 == S ? 0 : slot + 1;
    }
#undef HSD_GR_ISSUE
    __builtin_amdgcn_s_barrier();
    return;
  }

  // ---- a multiplying wave: rows m0 + 16 wave .. + 15
  if constexpr (Epi::kRowScale) {
    float *rsl = reinterpret_cast<float *>(smem_raw + Cfg::kSmemBytes);
    for (int r = t; r < BP; r += 64 * Cfg::RT) rsl[r] = (m0 + r < M) ? epi.rs.at(m0 + r) : 1.0f;
  }
  floatx4 acc[CW];
#pragma unroll
  for (int c = 0; c < CW; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, kg = lane >> 4;            // operand row; k group of the lane: piece 4 kk + kg of a 32-wide step
  const unsigned char *pa = smem_raw + (wave * 16 + fr) * RB, *pb = smem_raw + (BP + fr) * RB;
  // Half a stage at a time: the fragments of one half are read while the other half's products run.  A stage's products
  // are one chain, and a step of read, wait, multiply took 60 cycles of it against 25 without the reads (K = 4096).
  constexpr int HS = Cfg::SK / 64;                     // 32-wide steps of half a stage
  bf16x8 fa[2][HS], fb[2][HS][CW];
  int slot = 0;
#define HSD_GR_READ(h)                                                                                 \
  _Pragma("unroll") for (int i = 0; i < HS; ++i) {                                                     \
    const int off = slot * Cfg::kStageBytes + (((4 * ((h) * HS + i) + kg) ^ fr) << 4);                 \
    fa[h][i] = *reinterpret_cast<const bf16x8 *>(pa + off);                                            \
    _Pragma("unroll") for (int c = 0; c < CW; ++c) fb[h][i][c] = *reinterpret_cast<const bf16x8 *>(pb + c * 16 * RB + off); \
  }                                                                                                    \
  __builtin_amdgcn_sched_barrier(0);
#define HSD_GR_MMA(h)                                                                                  \
  _Pragma("unroll") for (int i = 0; i < HS; ++i) _Pragma("unroll") for (int c = 0; c < CW; ++c)        \
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][i][c], acc[c], 0, 0, 0);        \
  __builtin_amdgcn_sched_barrier(0);
  if (nf > 0) {
    __builtin_amdgcn_s_barrier();                      // barrier 0: stage 0 is complete
    __builtin_amdgcn_sched_barrier(0);
    HSD_GR_READ(0)
    for (int s = 0; s < nf; ++s) {
      HSD_GR_READ(1)
      HSD_GR_MMA(0)
      slot = slot + 1 == S ? 0 : slot + 1;
      if (s + 1 < nf) {
        __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this wave is done with stage s ...
        __builtin_amdgcn_s_barrier();                  // ... barrier s + 1: stage s + 1 is complete
        __builtin_amdgcn_sched_barrier(0);
        HSD_GR_READ(0)
      }
      HSD_GR_MMA(1)
    }
  }
  if (nf < ns) {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    for (int kk = 0; kk < (K - nf * Cfg::SK) / 32; ++kk) {
      const int off = slot * Cfg::kStageBytes + (((4 * kk + kg) ^ fr) << 4);
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(pa + off);
#pragma unroll
      for (int c = 0; c < CW; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8 *>(pb + c * 16 * RB + off), acc[c], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#undef HSD_GR_READ
#undef HSD_GR_MMA
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();                        // the epilogue stages through the operand stages

  // Result layout: lane l holds column l % 16 (of sub-tile c) and rows 4 (l / 16) + v.  Through LDS to row pieces of
  // PC = Epi::kPiece columns and their partners, as gemm_epilogue does; LPR lanes own a row.
  constexpr int ST = Cfg::kEpiStride, PC = Epi::kPiece, LPR = COLS / PC, RPI = 64 / LPR;
  float *wst = reinterpret_cast<float *>(smem_raw) + wave * 16 * ST;
  const float *rsl = reinterpret_cast<const float *>(smem_raw + Cfg::kSmemBytes) + wave * 16;
#pragma unroll
  for (int c = 0; c < CW; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) wst[(4 * kg + v) * ST + c * 16 + fr] = acc[c][v];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int it = 0; it < (16 + RPI - 1) / RPI; ++it) {
    const int r = it * RPI + lane / LPR, pc = lane % LPR;
    const int m = m0 + wave * 16 + r;
    if (r >= 16 || m >= M) continue;
    const float rsc = Epi::kRowScale ? rsl[r] : 1.0f;
    float lo[PC], hi[PC];
    const float *src = wst + r * ST + PC * pc;
#pragma unroll
    for (int e = 0; e < PC; ++e) {
      lo[e] = Epi::kRowScale ? src[e] * rsc : src[e];
      hi[e] = Epi::kRowScale ? src[COLS + e] * rsc : src[COLS + e];
    }
    if constexpr (MODE == kModeDual) epi.piece_dual(m, n0 + PC * pc, lo, hi);
    else epi.piece(m, n0 + PC * pc, lo, hi);
  }
}

}  // namespace hsd
