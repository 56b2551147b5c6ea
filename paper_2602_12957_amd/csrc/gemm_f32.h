// GEMM of the fp32 path on the matrix cores: C[m,n] = sum_k A[m,k] * W[n,k], v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// Why.  With multiply-adds on the vector unit (gemm_simple.h) every four of them wait for a quarter of their operands out of
// LDS: four blocks of 33 rows spend 23 us on the down projection (K = 1024, 36 workgroups), two thirds of it LDS reads, the
// rest a memory latency per slab of 32.  Here a lane's operand is one float per matrix instruction, so a 16-byte read feeds
// four of them; with 16-row tiles straight from memory to registers: no LDS, no barrier in the loop, and a chunk of up to 128 K
// values per row travels while the one before is multiplied.
//
// Tile: 16 RT rows by the 64 weight rows of one column group, four waves of 16 weight rows each; or by half a group (two waves,
// columns 16 h .. + 15 and their partners 32 further on), so that a launch of a few dozen tiles reads through twice the compute
// units: the bytes of a workgroup at 50 B/ns are its time.  A step covers 16 values of K:
// lane l holds the four from 4 (l / 16) on of row l % 16, and matrix instruction e takes element e of every lane.  Every output
// sums its products step by step in this order, so neither RT nor the chunk length changes a bit.
// RT = 1 or 2 for launches that leave part of the chip idle, 4 (a weight fragment serves 64 rows) for the others; see the launch.
//
// From RT = 2 on the operands come through LDS.  Straight from memory every lane of a request meets another row, so that each of
// its 64 pieces is a cache access of its own: with 64-row tiles the L1 was busy for 87 % of the launch (43 M accesses, LM head at
// 2064 rows), the matrix pipe for 35 %.  A chunk of 32 K values of all rows of the tile is requested in runs of 128 bytes, four
// lanes to an access, and stored a chunk ahead (rows 144 bytes apart: the fragment reads of 16 rows cover all 64 banks once).
#pragma once

#include "common.h"
#include "epilogues.h"

namespace hsd {

// grid: (N/(16 WV), ceil(M/(16 RT))), 64 WV threads; WV = 2 not for the LM head (its records are of whole groups).  N % 64 == 0, K % 32 == 0; rows of A and W 16-byte aligned.
// For Epi::kDual the second weight block starts N rows after the first (W is [2N, K]: gate | up).
template <typename Epi, int RT, int WV>
__global__ void __launch_bounds__(64 * WV) k_gemm_f32(int M, int N, int K, const float *__restrict__ A, const float *__restrict__ W, Epi epi) {
  constexpr int WB = Epi::kDual ? 2 : 1;                     // weight blocks
  constexpr bool STAGED = RT > 1;                            // operands through LDS
  constexpr int U = Epi::kDual ? 4 : 8;                      // not STAGED: steps of a chunk
  constexpr int PC = 8 * WV, ST = 2 * PC + 4;                // column pairs of a tile, floats per row of the result staging
  constexpr int KC = 32, SS = KC + 4, ROWS = 16 * RT + 64 * WB;   // STAGED: K values of a chunk, floats per staged row, rows of the tile
  static_assert(!STAGED || (WV == 4 && RT % 2 == 0), "32 rows a request of the workgroup");
  __shared__ __attribute__((aligned(16))) union {
    float res[WB][16 * RT][ST];
    float stage[STAGED ? 2 : 1][STAGED ? ROWS : 1][SS];   // activation rows, then weight rows
  } sm;
  auto &res = sm.res;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int m0 = blockIdx.y * 16 * RT, n0 = WV == 4 ? blockIdx.x * 64 : (blockIdx.x >> 1) * 64 + (blockIdx.x & 1) * 16;
  const int fr = lane & 15, kg = lane >> 4;
  floatx4 acc[WB][RT];
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[b][i] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](const floatx4 (&a)[RT], const floatx4 (&w)[WB]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[b][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], w[b][e], acc[b][i], 0, 0, 0);
  };
  if constexpr (STAGED) {
    constexpr int NL = ROWS / 32;                            // requests of a thread: rows t / 8 + 32 j, 16 bytes t % 8
    const float *src[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int r = 32 * j + (t >> 3), n = r - 16 * RT;      // (whole requests are of one kind: 16 RT is a multiple of 32)
      src[j] = (n < 0 ? A + static_cast<size_t>(min(m0 + r, M - 1)) * K : W + static_cast<size_t>((n >> 6) * N + n0 + (n & 63)) * K) + 4 * (t & 7);
    }
    floatx4 in[NL];
    auto request = [&](int c) {
#pragma unroll
      for (int j = 0; j < NL; ++j) in[j] = *reinterpret_cast<const floatx4 *>(src[j] + c * KC);
    };
    auto store = [&](int c) {
#pragma unroll
      for (int j = 0; j < NL; ++j) *reinterpret_cast<floatx4 *>(&sm.stage[c & 1][32 * j + (t >> 3)][4 * (t & 7)]) = in[j];
    };
    const int nc = K / KC;
    request(0);
    store(0);
    if (nc > 1) request(1);
    for (int c = 0; c < nc; ++c) {
      __syncthreads();   // chunk c is there, chunk c - 1 has been read
      if (c + 1 < nc) {
        store(c + 1);
        if (c + 2 < nc) request(c + 2);
      }
#pragma unroll
      for (int s = 0; s < KC / 16; ++s) {
        floatx4 a[RT], w[WB];
#pragma unroll
        for (int b = 0; b < WB; ++b) w[b] = *reinterpret_cast<const floatx4 *>(&sm.stage[c & 1][16 * RT + 64 * b + 16 * wave + fr][16 * s + 4 * kg]);
#pragma unroll
        for (int i = 0; i < RT; ++i) a[i] = *reinterpret_cast<const floatx4 *>(&sm.stage[c & 1][16 * i + fr][16 * s + 4 * kg]);
        step(a, w);
      }
    }
    __syncthreads();   // the results take the stages' place
  } else {
    const float *pa[RT], *pw[WB];
#pragma unroll
    for (int i = 0; i < RT; ++i) pa[i] = A + static_cast<size_t>(min(m0 + 16 * i + fr, M - 1)) * K + 4 * kg;
#pragma unroll
    for (int b = 0; b < WB; ++b)
      pw[b] = W + static_cast<size_t>(b * N + n0 + (WV == 4 ? 16 : 32) * wave + fr) * K + 4 * kg;
    floatx4 fa[2][U][RT], fw[2][U][WB];
    auto request = [&](auto set, int k0) {
#pragma unroll
      for (int s = 0; s < U; ++s) {
#pragma unroll
        for (int b = 0; b < WB; ++b) fw[set][s][b] = *reinterpret_cast<const floatx4 *>(pw[b] + k0 + 16 * s);
#pragma unroll
        for (int i = 0; i < RT; ++i) fa[set][s][i] = *reinterpret_cast<const floatx4 *>(pa[i] + k0 + 16 * s);
      }
    };
    auto multiply = [&](auto set) {
#pragma unroll
      for (int s = 0; s < U; ++s) step(fa[set][s], fw[set][s]);
    };
    constexpr auto s0 = std::integral_constant<int, 0>{};
    constexpr auto s1 = std::integral_constant<int, 1>{};
    const int nc = K / (16 * U);                               // full chunks
    if (nc > 0) request(s0, 0);
    for (int c = 0; c < nc; c += 2) {
      if (c + 1 < nc) request(s1, (c + 1) * 16 * U);
      multiply(s0);
      if (c + 1 < nc) {
        if (c + 2 < nc) request(s0, (c + 2) * 16 * U);
        multiply(s1);
      }
    }
    for (int k = nc * 16 * U; k < K; k += 16) {
      floatx4 a[RT], w[WB];
#pragma unroll
      for (int b = 0; b < WB; ++b) w[b] = *reinterpret_cast<const floatx4 *>(pw[b] + k);
#pragma unroll
      for (int i = 0; i < RT; ++i) a[i] = *reinterpret_cast<const floatx4 *>(pa[i] + k);
      step(a, w);
    }
  }

  // Result layout: lane l holds column l % 16 and rows 4 (l / 16) + v.  Through LDS, so that a thread has the column pair
  // (n, n + 32) of a row.
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) res[b][16 * i + 4 * kg + v][16 * wave + fr] = acc[b][i][v];
  __syncthreads();
  const int tx = t % PC, ty = t / PC;
#pragma unroll
  for (int i = 0; i < 2 * RT; ++i) {
    const int r = 8 * i + ty, m = m0 + r;
    const float lo = res[0][r][tx], hi = res[0][r][tx + PC];
    if constexpr (std::is_same<Epi, EpiLMHead>::value) {
      Top2 tp = top2_init();
      top2_push(tp, lo, n0 + tx);
      top2_push(tp, hi, n0 + tx + 32);
      if (m < M) epi.dump(m, n0 + tx, lo, hi);
      if (m < M && epi.want_logit != nullptr) {
        epi.capture(m, [&](int want, float &out) {
          if (want == n0 + tx) { out = lo; return true; }
          if (want == n0 + tx + 32) { out = hi; return true; }
          return false;
        });
      }
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) {  // stays inside the 32 lanes that share this row
        Top2 u;
        u.m1 = __shfl_xor(tp.m1, o, kWave);
        u.i1 = __shfl_xor(tp.i1, o, kWave);
        u.m2 = __shfl_xor(tp.m2, o, kWave);
        tp = top2_merge(tp, u);
      }
      if (tx == 0 && m < M) epi.part[static_cast<size_t>(m) * epi.n_tiles + blockIdx.x] = tp;
    } else if (m < M) {
      if constexpr (Epi::kDual) epi.pair2(m, n0 + tx, lo, hi, res[WB - 1][r][tx], res[WB - 1][r][tx + PC]);
      else epi.pair(m, n0 + tx, lo, hi);
    }
  }
}

}  // namespace hsd
