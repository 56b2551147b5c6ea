// Plain LDS-tiled GEMM with fp32 FMA accumulation: C[m,n] = sum_k A[m,k] * W[n,k].
// The cross-check for the bf16 MFMA kernels (the fp32 path has k_gemm_f32).
// Tile 64x64x32 or 16x64x32, 256 threads; thread (ty, tx) owns TR rows from ty*TR and the column pair (tx, tx+32).
#pragma once

#include "common.h"
#include "epilogues.h"

namespace hsd {

__device__ __forceinline__ void load8(const float *p, float *out) {
  float4 a = reinterpret_cast<const float4 *>(p)[0];
  float4 b = reinterpret_cast<const float4 *>(p)[1];
  out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
  out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16 *p, float *out) {
  uint4 r = reinterpret_cast<const uint4 *>(p)[0];
  uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = __uint_as_float(w[i] << 16);
    out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}

// grid: (N/64, ceil(M/(8*TR))).  Requirements checked by the host: N % 64 == 0, K % 32 == 0.
// For Epi::kDual the second weight block starts N rows after the first (W is [2N, K]: gate | up).
// TR rows per thread: 8 (64-row tiles) or 2 (16-row tiles, for launches that leave most of the chip idle; see the
// launch).  The next K slab is requested before the current one is multiplied, and operands are read from LDS four k
// at a time (rows of 36 floats: 16-byte aligned, and 16 consecutive rows spread over the banks).  Every output still
// sums its products one by one in ascending k, so neither TR nor the slab width changes a bit.
// 4 blocks of 33 rows on the two-layer d256 fp32 model, down projection (12 workgroups of 64-row tiles, 36 of 16-row
// ones) and whole pass in us, each step on top of the one before: 77.4 and 576 with exposed slab loads and one k at a
// time from LDS; the next slab requested early 73.2 and 563; four k at a time 52.8 and 493; 16-row tiles 24.2 and 359.
template <typename T, typename Epi, int TR>
__global__ void __launch_bounds__(256) k_gemm_simple(int M, int N, int K, const T *__restrict__ A,
                                                     const T *__restrict__ W, Epi epi) {
  constexpr int BK = 32, LS = BK + 4, BM = 8 * TR;
  __shared__ __attribute__((aligned(16))) float As[BM][LS];
  __shared__ __attribute__((aligned(16))) float Bs[64][LS];
  __shared__ __attribute__((aligned(16))) float Bs2[Epi::kDual ? 64 : 1][LS];
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * 64;
  const int lr = t >> 2, lk = (t & 3) * 8;
  const bool loads_a = lr < BM;   // the first BM * 4 threads bring in the activation rows

  float acc[TR][2], acc2[TR][2];
#pragma unroll
  for (int i = 0; i < TR; ++i) acc[i][0] = acc[i][1] = acc2[i][0] = acc2[i][1] = 0.f;

  float va[8], vb[8], vb2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) va[i] = 0.f;
  auto request = [&](int k0) {
    if (loads_a && m0 + lr < M) load8(A + static_cast<size_t>(m0 + lr) * K + k0 + lk, va);
    load8(W + static_cast<size_t>(n0 + lr) * K + k0 + lk, vb);
    if (Epi::kDual) load8(W + static_cast<size_t>(N + n0 + lr) * K + k0 + lk, vb2);
  };
  auto put = [&](float *dst, const float *v) {
    reinterpret_cast<floatx4 *>(dst)[0] = floatx4{v[0], v[1], v[2], v[3]};
    reinterpret_cast<floatx4 *>(dst)[1] = floatx4{v[4], v[5], v[6], v[7]};
  };
  request(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();  // previous tile fully consumed
    if (loads_a) put(&As[lr][lk], va);
    put(&Bs[lr][lk], vb);
    if (Epi::kDual) put(&Bs2[lr][lk], vb2);
    __syncthreads();
    if (k0 + BK < K) request(k0 + BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const floatx4 b0 = *reinterpret_cast<const floatx4 *>(&Bs[tx][kk]);
      const floatx4 b1 = *reinterpret_cast<const floatx4 *>(&Bs[tx + 32][kk]);
      floatx4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
      if (Epi::kDual) {
        c0 = *reinterpret_cast<const floatx4 *>(&Bs2[tx][kk]);
        c1 = *reinterpret_cast<const floatx4 *>(&Bs2[tx + 32][kk]);
      }
#pragma unroll
      for (int i = 0; i < TR; ++i) {
        const floatx4 a = *reinterpret_cast<const floatx4 *>(&As[ty * TR + i][kk]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[i][0] = fmaf(a[e], b0[e], acc[i][0]);
          acc[i][1] = fmaf(a[e], b1[e], acc[i][1]);
          if (Epi::kDual) {
            acc2[i][0] = fmaf(a[e], c0[e], acc2[i][0]);
            acc2[i][1] = fmaf(a[e], c1[e], acc2[i][1]);
          }
        }
      }
    }
  }

  if constexpr (std::is_same<Epi, EpiLMHead>::value) {
#pragma unroll
    for (int i = 0; i < TR; ++i) {
      int m = m0 + ty * TR + i;
      Top2 tp = top2_init();
      top2_push(tp, acc[i][0], n0 + tx);
      top2_push(tp, acc[i][1], n0 + tx + 32);
      if (m < M) epi.dump(m, n0 + tx, acc[i][0], acc[i][1]);
      if (m < M && epi.want_logit != nullptr) {
        const float v0 = acc[i][0], v1 = acc[i][1];
        epi.capture(m, [&](int want, float &out) {
          if (want == n0 + tx) { out = v0; return true; }
          if (want == n0 + tx + 32) { out = v1; return true; }
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
    }
  } else {
#pragma unroll
    for (int i = 0; i < TR; ++i) {
      int m = m0 + ty * TR + i;
      if (m >= M) continue;
      if constexpr (Epi::kDual) {
        epi.pair2(m, n0 + tx, acc[i][0], acc[i][1], acc2[i][0], acc2[i][1]);
      } else {
        epi.pair(m, n0 + tx, acc[i][0], acc[i][1]);
      }
    }
  }
}

}  // namespace hsd
