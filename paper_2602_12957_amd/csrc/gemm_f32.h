// GEMM of the fp32 path on the matrix cores: C[m,n] = sum_k A[m,k] * W[n,k], v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// Why.  With multiply-adds on the vector unit (gemm_simple.h) every four of them wait for a quarter of their operands out of
// LDS: four blocks of 33 rows spend 23 us on the down projection (K = 1024, 36 workgroups), two thirds of it LDS reads, the
// rest a memory latency per slab of 32.  Here a lane's operand is one float per matrix instruction, so a 16-byte read feeds
// four of them, straight from memory to registers: no LDS, no barrier in the loop, and a chunk of up to 128 K values per row
// travels while the one before is multiplied.
//
// Tile: 16 RT rows by the 64 weight rows of one column group, four waves of 16 weight rows each; or by half a group (two waves,
// columns 16 h .. + 15 and their partners 32 further on), so that a launch of a few dozen tiles reads through twice the compute
// units: the bytes of a workgroup at 50 B/ns are its time.  A step covers 16 values of K:
// lane l holds the four from 4 (l / 16) on of row l % 16, and matrix instruction e takes element e of every lane.  Every output
// sums its products step by step in this order, so neither RT nor the chunk length changes a bit.
// RT = 1 or 2 for launches that leave part of the chip idle, 4 (a weight fragment serves 64 rows) for the others; see the launch.
#pragma once

#include "common.h"
#include "epilogues.h"

namespace hsd {

// grid: (N/(16 WV), ceil(M/(16 RT))), 64 WV threads; WV = 2 not for the LM head (its records are of whole groups).  N % 64 == 0, K % 32 == 0; rows of A and W 16-byte aligned.
// For Epi::kDual the second weight block starts N rows after the first (W is [2N, K]: gate | up).
template <typename Epi, int RT, int WV>
__global__ void __launch_bounds__(64 * WV) k_gemm_f32(int M, int N, int K, const float *__restrict__ A, const float *__restrict__ W, Epi epi) {
  constexpr int WB = Epi::kDual ? 2 : 1;                     // weight blocks
  constexpr int U = RT == 4 ? 2 : RT == 2 ? (Epi::kDual ? 2 : 4) : Epi::kDual ? 4 : 8;         // steps of a chunk
  constexpr int PC = 8 * WV, ST = 2 * PC + 4;                // column pairs of a tile, floats per row of the result staging
  __shared__ __attribute__((aligned(16))) float res[WB][16 * RT][ST];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int m0 = blockIdx.y * 16 * RT, n0 = WV == 4 ? blockIdx.x * 64 : (blockIdx.x >> 1) * 64 + (blockIdx.x & 1) * 16;
  const int fr = lane & 15, kg = lane >> 4;
  const float *pa[RT], *pw[WB];
#pragma unroll
  for (int i = 0; i < RT; ++i) pa[i] = A + static_cast<size_t>(min(m0 + 16 * i + fr, M - 1)) * K + 4 * kg;
#pragma unroll
  for (int b = 0; b < WB; ++b)
    pw[b] = W + static_cast<size_t>(b * N + n0 + (WV == 4 ? 16 : 32) * wave + fr) * K + 4 * kg;
  floatx4 acc[WB][RT];
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[b][i] = floatx4{0.f, 0.f, 0.f, 0.f};
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
  auto step = [&](const floatx4 (&a)[RT], const floatx4 (&w)[WB]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[b][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], w[b][e], acc[b][i], 0, 0, 0);
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
