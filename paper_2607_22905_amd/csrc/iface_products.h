// Wave-level products with symmetric dense interface operators (the blocks
// of the nested-dissection solve and of the block-Jacobi preconditioner of
// the inexact interface solve).  Internal header.
#pragma once

#include "am_common.h"

namespace am {

typedef double nd_d4 __attribute__((ext_vector_type(4)));

// M rows of X, m0 .. m0 + M - 1 (the last row of the share again beyond it),
// for the 64 outputs r0 .. of a wave, as one batch of loads without a branch:
// NR <= 2: lane = column, a[u] = X[m0 + u][r0 + lane]; NR >= 4: the operands
// of M / 4 matrix-core steps of four rows, a[4 u + t] = X[m0 + 4 u + lane / 16]
// [r0 + 16 t + lane % 16].  Columns from rmax on repeat the last one.
template <int NR, bool NT> struct NdRows {
  static constexpr int M = NR <= 2 ? 16 : 8;
  double a[M];
  __device__ __forceinline__ void load(const double* __restrict__ X, int64_t ld, int r0, int rmax,
                                       int m0, int me) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const int m = max(0, min(NR <= 2 ? m0 + i : m0 + 4 * (i / 4) + lane / 16, me - 1));
      const int r = min(NR <= 2 ? r0 + lane : r0 + 16 * (i % 4) + lane % 16, rmax - 1);
      const double* p = X + (size_t)m * ld + r;
      a[i] = NT ? __builtin_nontemporal_load(p) : *p;
    }
  }
};

// One wave's share of out[r][k] = sum_{m in [mb, me)} X[m][r] v[m][k] for the
// 64 outputs r = r0 .. r0 + 63 of a symmetric matrix X (leading dimension
// ld; its row m stands for column m), v[m][.] in LDS at v + (m - vbase) NR.
// NR <= 2: lane = r, NR FMAs per coalesced load of 64 values.  NR >= 4: four
// 16 x 16 tiles on the FP64 matrix cores (v_mfma_f64_16x16x4f64: lane l holds
// A[l % 16][l / 16] = X[m0 + l / 16][r0 + 16 t + l % 16], B[l / 16][l % 16] =
// v[m0 + l / 16][l % 16] (zero beyond NR) and D[l / 16 + 4 q][l % 16]).  The
// first rows come in f (loaded by the caller, ahead of what v waits for), the
// next batch is requested before the products of the last.  Outputs
// r >= rmax are undefined.  acc: [4][4] (matrix cores: tile t, entry q) or
// [NR] (lane = row) in acc[0..NR-1][0].
template <int NR, bool NT>
__device__ __forceinline__ void nd_wave_product(const double* __restrict__ X, int64_t ld, int r0,
                                                int rmax, int mb, int me, const double* v,
                                                int vbase, NdRows<NR, NT>& f, nd_d4 (&acc)[4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = nd_d4{0.0, 0.0, 0.0, 0.0};
  constexpr int M = NdRows<NR, NT>::M;
  double a0[2] = {0.0, 0.0};
  for (int m0 = mb; m0 < me; m0 += M) {
    NdRows<NR, NT> g;
    if constexpr (NR <= 2) {
      g.load(X, ld, r0, rmax, m0 + M, me);
#pragma unroll
      for (int u = 0; u < M; ++u) {
        const int m = min(m0 + u, me - 1);
        const double a = m0 + u < me ? f.a[u] : 0.0;
#pragma unroll
        for (int k = 0; k < NR; ++k) a0[k] = fma(a, v[(m - vbase) * NR + k], a0[k]);
      }
    } else {
      const int li = lane % 16, lk = lane / 16;
      double bv[M / 4];  // (before the next rows: loads return in order, and v may be
                         // in memory; after them, C^{-1} of 5700 rows took 70 us, so 54)
#pragma unroll
      for (int u = 0; u < M / 4; ++u) bv[u] = v[(min(m0 + 4 * u + lk, me - 1) - vbase) * NR + min(li, NR - 1)];
      g.load(X, ld, r0, rmax, m0 + M, me);
#pragma unroll
      for (int u = 0; u < M / 4; ++u) {
        const bool ok = m0 + 4 * u + lk < me;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? f.a[4 * u + t] : 0.0,
                                                        ok && li < NR ? bv[u] : 0.0, acc[t], 0, 0, 0);
      }
    }
    f = g;
  }
  if constexpr (NR <= 2)
#pragma unroll
    for (int k = 0; k < NR; ++k) acc[k][0] = a0[k];
}

// calls f(row offset in 0 .. 63, column k, value) for the wave's results
template <int NR, typename F>
__device__ __forceinline__ void nd_wave_each(const nd_d4 (&acc)[4], F&& f) {
  const int lane = threadIdx.x & 63;
  if constexpr (NR <= 2) {
#pragma unroll
    for (int k = 0; k < NR; ++k) f(lane, k, acc[k][0]);
  } else {
    const int li = lane % 16, lk = lane / 16;
    if (li < NR)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) f(16 * t + lk + 4 * q, li, acc[t][q]);
  }
}

}  // namespace am
