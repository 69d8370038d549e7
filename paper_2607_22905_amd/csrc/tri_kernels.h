// Local solves of the subdomains whose band fits 64 rows, for gfx950.  In the
// device order the local operator A_i = A_ii - sum_j D_ij (eq. A_i) of such a
// subdomain is block tridiagonal in blocks of 64 rows: block b couples only
// to blocks b - 1 and b + 1, through entries of A itself (E_b: the few
// couplings of block b's rows to block b - 1).  It is eliminated from both
// ends towards a middle block h = NB / 2:
//   S_0 = A_00,          S_b = A_bb - E_b X_{b-1} E_b^T          (b < h)
//   S_{NB-1} = A_{NB-1,NB-1},  S_b = A_bb - E_{b+1}^T X_{b+1} E_{b+1}  (b > h)
//   S_h = A_hh - E_h X_{h-1} E_h^T - E_{h+1}^T X_{h+1} E_{h+1},  X_b = S_b^{-1}
// and the solve keeps the explicit inverses X_b (symmetric, nonnegative: S_b
// is an M-matrix) and the sparse E_b:
//   t_b = r_b - E_b w_{b-1} (above h: E_{b+1}^T w_{b+1}),  w_b = X_b t_b
//   x_h = X_h (r_h - E_h w_{h-1} - E_{h+1}^T w_{h+1})
//   x_b = w_b - X_b (E_{b+1}^T x_{b+1})   (above h: X_b E_b x_{b-1}).
// The chain of dependent 64 x 64 products is NB + 1 long (both halves run
// side by side) and every X_b is symmetric, so half of it is stored.
//
// Packed symmetric tile: off-diagonals c = 1 .. 32, element (c, l) holds
// X[l][(l + c) % 64]; the diagonals 33 .. 63 are the same entries seen from
// the other row, and c = 32 would be counted from both sides, so it is stored
// halved (exact).  With lane l holding row l of every stored diagonal,
//   y[l]         += X[l][l + c] t[l + c]     t read from LDS at l + c
//   y[(l + c)]   += X[l][l + c] t[l]         the lane's own t, moved c lanes
// and the second sum is a Horner scheme of one-lane wave rotations, so a
// wave's factor values never leave its registers.  The main diagonal is a
// separate array (arithmetic type), as are the couplings.
//
// Triangular form (FP32 and BF16 factors).  The local operator that is applied
// is congruent to diag(X_b), and rounding the entries of X_b can make it
// indefinite: where a conductive body lies inside a subdomain, X_b is nearly
// of rank one over that body, and its small eigenvalues are below the rounding
// of the large entries.  k_tri_factor therefore bounds the change in every
// block; a subdomain beyond the bound keeps X_b = K^T D K instead, K unit lower
// triangular, D > 0 diagonal, in the same storage: the pair (i, j), i > j, of
// the tile holds K[i][j], the main diagonal D.  That is definite whatever the
// rounding, and y = X_b t is two triangular products,
//   u = t + Ks t,   v = D u,   y = v + Ks^T v    (Ks: K without its diagonal).
// In the first, lane l takes its element (c, l) as an entry of its own row if
// l + c >= 64 and of the other row if not; in the second the other way round.
#pragma once
#include <type_traits>

#include "am_common.h"
#include "mf_ops.h"

#define AM_INLINE __attribute__((always_inline))

namespace am {

constexpr int kTriElems = 32 * 64;  // stored elements of a tile
template <typename FT> struct TriAcc { using T = float; };
template <> struct TriAcc<double> { using T = double; };

// element (c, l), c = 1 .. 32, of a tile: 16-byte groups of V diagonals
template <typename FT> __host__ __device__ constexpr int tri_at(int c, int l) {
  constexpr int V = 16 / (int)sizeof(FT);
  return ((c - 1) / V) * 64 * V + l * V + (c - 1) % V;
}

// value of lane l - 1 (lane 0: of lane 63)
__device__ __forceinline__ int wave_ror1(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x13C, 0xF, 0xF, false);
}
__device__ __forceinline__ float wave_ror1(float v) {
  return __builtin_bit_cast(float, wave_ror1(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double wave_ror1(double v) {
  int2 a = __builtin_bit_cast(int2, v);
  a.x = wave_ror1(a.x);
  a.y = wave_ror1(a.y);
  return __builtin_bit_cast(double, a);
}

// One wave's LDS writes before its later LDS reads of other lanes' data.
__device__ __forceinline__ void tri_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ND consecutive diagonals c0 + 1 .. c0 + ND of a tile, this lane's elements
// (c0 a multiple of ND), as loaded: 16-byte groups, or one of 8 bytes.
template <typename FT, int ND> struct TriFrag {
  static constexpr int BYTES = ND * (int)sizeof(FT);
  static constexpr int V = 16 / (int)sizeof(FT);
  static_assert(BYTES >= 8 && (BYTES % 16 == 0 || BYTES == 8), "whole groups");
  static constexpr int NQ = BYTES >= 16 ? BYTES / 16 : 1;
  using Q = typename std::conditional<(BYTES >= 16), uint4, uint2>::type;
  Q q[NQ];
  __device__ __forceinline__ void load(const FT* __restrict__ tile, int c0, int lane) {
    if constexpr (BYTES >= 16) {
      const uint4* p = reinterpret_cast<const uint4*>(tile) + (size_t)(c0 / V) * 64 + lane;
#pragma unroll
      for (int u = 0; u < NQ; ++u) q[u] = p[u * 64];
    } else {
      q[0] = *reinterpret_cast<const uint2*>(tile + tri_at<FT>(c0 + 1, lane));
    }
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int u = 0; u < NQ; ++u) q[u] = Q{};
  }
  __device__ __forceinline__ typename TriAcc<FT>::T get(int j) const {
    using AT = typename TriAcc<FT>::T;
    if constexpr (sizeof(FT) == 8) {
      const uint4& w = q[j / 2];
      return j % 2 ? __builtin_bit_cast(double, (uint64_t)w.w << 32 | w.z)
                   : __builtin_bit_cast(double, (uint64_t)w.y << 32 | w.x);
    } else if constexpr (sizeof(FT) == 4) {
      const uint4& w = q[j / 4];
      const uint32_t b = j % 4 == 0 ? w.x : j % 4 == 1 ? w.y : j % 4 == 2 ? w.z : w.w;
      return __builtin_bit_cast(AT, b);
    } else {
      uint32_t b;
      if constexpr (BYTES >= 16) {
        const uint4& w = q[j / 8];
        const int e = j % 8 / 2;
        b = e == 0 ? w.x : e == 1 ? w.y : e == 2 ? w.z : w.w;
      } else {
        b = j / 2 == 0 ? q[0].x : q[0].y;
      }
      return __builtin_bit_cast(AT, j % 2 ? b & 0xFFFF0000u : b << 16);
    }
  }
};

// Partial products of the diagonals in f with NT vectors: t (this lane's
// values), tw: the wave's LDS copy, value (k, i) at tw[128 k + i], rows
// repeated at i + 64.  On return a[k] adds to row l, h[k] to row
// (l + c0 + 1) % 64.  PART: 0 the symmetric tile, 1 its strict lower triangle
// (Ks), 2 the transpose of that.
template <typename FT, int ND, int NT, int PART = 0>
__device__ __forceinline__ void tri_partial(const TriFrag<FT, ND>& f, int c0, int lane,
                                            const typename TriAcc<FT>::T (&t)[NT],
                                            const typename TriAcc<FT>::T* tw,
                                            typename TriAcc<FT>::T (&a)[NT],
                                            typename TriAcc<FT>::T (&h)[NT]) {
  using AT = typename TriAcc<FT>::T;
  const AT* p = tw + lane + c0 + 1;
#pragma unroll
  for (int j = ND - 1; j >= 0; --j) {
    const AT d = f.get(j);
    const bool own = (lane + c0 + j + 1 >= 64) == (PART == 1);
    const AT da = PART == 0 || own ? d : (AT)0, dh = PART == 0 || !own ? d : (AT)0;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      a[k] = j == ND - 1 ? da * p[128 * k + j] : fma(da, p[128 * k + j], a[k]);
      h[k] = j == ND - 1 ? dh * t[k] : fma(dh, t[k], wave_ror1(h[k]));
    }
  }
}

// value of lane `from`
__device__ __forceinline__ float lane_value(float v, int from) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * from, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double lane_value(double v, int from) {
  int2 a = __builtin_bit_cast(int2, v);
  a.x = __builtin_amdgcn_ds_bpermute(4 * from, a.x);
  a.y = __builtin_amdgcn_ds_bpermute(4 * from, a.y);
  return __builtin_bit_cast(double, a);
}

// The whole tile (32 diagonals) in one wave: y[k] += X t without the main
// diagonal.  FP64: one Horner chain of 32 rotations, 29 cycles a link, the row
// sums beside it in two accumulators.  FP32 arithmetic: two chains of 16 (the
// second's sum moved 16 lanes at the end) and four accumulators, for shorter
// sums.
template <typename FT, int NT>
__device__ __forceinline__ void tri_full(const TriFrag<FT, 32>& f, int lane,
                                         const typename TriAcc<FT>::T (&t)[NT],
                                         const typename TriAcc<FT>::T* tw,
                                         typename TriAcc<FT>::T (&y)[NT]) {
  using AT = typename TriAcc<FT>::T;
  constexpr int CH = sizeof(AT) == 8 ? 1 : 2, L = 32 / CH, NA = 2 * CH;
  const AT* p = tw + lane + 1;
  AT h[CH][NT], a[NA][NT];
#pragma unroll
  for (int j = L - 1; j >= 0; --j)
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int jj = L * c + j;
      const AT d = f.get(jj);
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        h[c][k] = j == L - 1 ? d * t[k] : fma(d, t[k], wave_ror1(h[c][k]));
        AT& s = a[2 * c + j % 2][k];
        s = j >= L - 2 ? d * p[128 * k + jj] : fma(d, p[128 * k + jj], s);
      }
    }
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    if constexpr (CH == 2)
      y[k] += ((a[0][k] + a[1][k]) + (a[2][k] + a[3][k])) +
              (wave_ror1(h[0][k]) + lane_value(h[1][k], (lane - 17) & 63));
    else
      y[k] = (y[k] + (a[0][k] + a[1][k])) + wave_ror1(h[0][k]);
  }
}

// ---------------------------------------------------------------------------
// Couplings between neighbouring blocks, from the device-order CSR rows: for
// row i of block b, list 0 holds its entries in block b - 1, list 1 those in
// block b + 1; value (list, k, row) at cpl[(list kc + k) NP + row], the
// column's row within its block in the byte array; unused places are zero.
// (An entry beyond the neighbouring blocks was an explicit zero when the order
// of the rows was chosen.  New values may have given it one since; it is not
// part of the local operator, here as in the factors and basis functions.)
template <typename FT>
__global__ __launch_bounds__(256) void k_tri_couplings(
    const int32_t* __restrict__ subs, const int64_t* __restrict__ sub_ptr,
    const int64_t* __restrict__ roff, const int64_t* __restrict__ cpl_off,
    const int32_t* __restrict__ cpl_k, const int64_t* __restrict__ prp,
    const int32_t* __restrict__ pci, const double* __restrict__ pv,
    typename TriAcc<FT>::T* __restrict__ cpl, uint8_t* __restrict__ cidx) {
  using AT = typename TriAcc<FT>::T;
  const int s = subs[blockIdx.x];
  const int64_t base = sub_ptr[s];
  const int N = (int)(sub_ptr[s + 1] - base);
  const int NP = (int)(roff[s + 1] - roff[s]);
  const int kc = cpl_k[s];
  AT* cv = cpl + cpl_off[s];
  uint8_t* ci = cidx + cpl_off[s];
  for (int row = threadIdx.x; row < NP; row += blockDim.x) {
    int cnt[2] = {0, 0};
    if (row < N) {
      const int b = row / 64;
      for (int64_t p = prp[base + row]; p < prp[base + row + 1]; ++p) {
        const int64_t c = (int64_t)pci[p] - base;
        if (c < 0 || c >= N) continue;
        const int cb = (int)c / 64;
        if (cb == b || cb < b - 1 || cb > b + 1) continue;
        const int list = cb < b ? 0 : 1;
        const int at = (list * kc + cnt[list]) * NP + row;
        cv[at] = (AT)pv[p];
        ci[at] = (uint8_t)(c % 64);
        cnt[list] += 1;
      }
    }
    for (int list = 0; list < 2; ++list)
      for (int k = cnt[list]; k < kc; ++k) {
        cv[(list * kc + k) * NP + row] = (AT)0;
        ci[(list * kc + k) * NP + row] = 0;
      }
  }
}

// ---------------------------------------------------------------------------
// Largest change of a block inverse by the rounding of its entries that the
// symmetric form is kept for.  With X~ = X + E the stored block, S = X^{-1}
// and D = diag(S): S is an M-matrix, so D^{-1/2} S D^{-1/2} has its eigenvalues
// below 2 and X >= D^{-1} / 2; where every row sum of D^{1/2} |E| D^{1/2} is at
// most tau, -2 tau X <= E <= 2 tau X.  tau < 1/2 keeps X~ definite; the values
// lie where the symmetric form begins to need more iterations than the
// triangular one, whose products take longer (an iteration 46 -> 58 us): 8^3
// boxes with a 4^3 body in each, 64^3 cells, by contrast: row sums, iterations
// of the triangular and of the symmetric form.  BF16: 100: 0.25, 23, 23; 1e4:
// 21, 35, breakdown.  FP32: 1e4: 4e-4, 18, 18; 1e6: 0.05, 30, 34 (8 columns);
// 1e8: 5, 20, breakdown.  (Below, both are as good as their FP32 arithmetic.)
// Gaussian and layered fields stay below 0.23 (BF16; in 3-D 0.05) and 4e-6
// (FP32).
template <typename FT> struct TriTau { static constexpr double v = 1.0 / 1024; };
template <> struct TriTau<bf16_t> { static constexpr double v = 1.0 / 4; };

// v as stored in FT
template <typename FT> __device__ __forceinline__ double tri_stored(double v) {
  FT b;
  st_fac(&b, v);
  return (double)widen_lds(b);
}

// X_b of every block (set-up): one workgroup per subdomain, two groups of 256
// threads eliminating from the two ends side by side, group 0 then the middle
// block.  A thread keeps a 4 x 4 piece of its group's 64 x 64 block in
// registers (sweep_inverse_64), FP64 throughout.  A pivot that is not positive
// names the subdomain and row in fail.  FP32 and BF16: where the rounding of a
// block is beyond TriTau, the elimination is done again for the triangular
// form.  Bound by the chain of 64 barriers per
// block: 4096 boxes 2.6 ms (band Cholesky and its diagonal inverses 16 ms).
template <typename FT>
__global__ __launch_bounds__(512) void k_tri_factor(
    const int32_t* __restrict__ subs, SubDesc* __restrict__ desc,
    const int64_t* __restrict__ prp, const int32_t* __restrict__ pci,
    const double* __restrict__ pv, FT* __restrict__ fac,
    typename TriAcc<FT>::T* __restrict__ dg, int32_t* __restrict__ fail, int plain) {
  using AT = typename TriAcc<FT>::T;
  constexpr bool kRounded = sizeof(FT) < 8;
  constexpr int P = 65;
  __shared__ double M[2][64 * P];
  __shared__ double prow[2][2][64];
  // entries of each row of the group's new block in its two neighbours:
  // [group][list][row] first CSR position and count
  __shared__ int64_t e0[2][2][64];
  __shared__ int32_t en[2][2][64];
  __shared__ double dsq[2][64];  // square roots of the block's diagonal
  __shared__ int far;            // a block is beyond TriTau
  const int s = subs[blockIdx.x];
  const int64_t base = desc[s].base, ro = desc[s].ro;
  const int N = desc[s].N, NB = (N + 63) / 64;
  FT* fs = fac + desc[s].fac;
  const int g = threadIdx.x >> 8, tid = threadIdx.x & 255;
  const int i0 = 4 * (tid / 16), j0 = 4 * (tid % 16);
  const int h = NB / 2, len1 = NB - 1 - h;
  double* Mg = M[g];

  // acc += sum_{k,l} e_ik X[k][l] e_jl with X the block in src, e the rows'
  // entries in list `list` (column rows relative to block nb)
  auto reduce = [&](double (&acc)[4][4], const double* src, int list, int nb) {
    const int64_t cb = base + 64 * nb;
    int ki = 0, kj = 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      ki = max(ki, en[g][list][i0 + a]);
      kj = max(kj, en[g][list][j0 + a]);
    }
    for (int k = 0; k < ki; ++k) {
      double ei[4];
      int ri[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const bool ok = k < en[g][list][i0 + a];
        const int64_t p = e0[g][list][i0 + a] + (ok ? k : 0);
        ei[a] = ok ? pv[p] : 0.0;
        ri[a] = ok ? (int)(pci[p] - cb) : 0;
      }
      for (int l = 0; l < kj; ++l)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (l >= en[g][list][j0 + b]) continue;
          const int64_t p = e0[g][list][j0 + b] + l;
          const double ej = pv[p];
          const int rj = (int)(pci[p] - cb);
#pragma unroll
          for (int a = 0; a < 4; ++a) acc[a][b] = fma(ei[a] * ej, src[ri[a] * P + rj], acc[a][b]);
        }
    }
  };

  if (threadIdx.x == 0) far = 0;
  // the symmetric form (0), then where needed the triangular one (1)
  for (int form = 0; form < 2; ++form) {
    // blocks in elimination order: step k < h: group 0 block k, group 1 block
    // NB - 1 - k; step h: the middle block
    for (int step = 0; step <= h; ++step) {
      const bool mid = step == h;
      const bool act = mid ? g == 0 : (g == 0 || step < len1);
      const int b = mid ? h : (g == 0 ? step : NB - 1 - step);
      // CSR ranges of the block's rows in the neighbouring blocks (row c of the
      // list: couplings to the eliminated neighbour on that side)
      if (act && tid < 128) {
        const int list = tid / 64, i = tid % 64, row = 64 * b + i;
        int64_t first = 0;
        int cnt = 0;
        if (row < N) {
          const int64_t lo = base + 64 * (int64_t)(list == 0 ? b - 1 : b + 1);
          const int64_t hi = min(lo + 64, base + (int64_t)N);
          if (lo >= base && lo < base + N)
            for (int64_t p = prp[base + row]; p < prp[base + row + 1]; ++p) {
              const int64_t c = pci[p];
              if (c >= lo && c < hi) {
                if (cnt == 0) first = p;
                ++cnt;
              }
            }
        }
        e0[g][list][i] = first;
        en[g][list][i] = cnt;
      }
      __syncthreads();
      double upd[4][4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) upd[a][c] = 0.0;
      if (act) {
        if (g == 0 && step > 0) reduce(upd, M[0], 0, b - 1);
        if (g == 1 && step > 0) reduce(upd, M[1], 1, b + 1);
        if (mid && len1 > 0) reduce(upd, M[1], 1, b + 1);
      }
      __syncthreads();
      if (act)
        for (int t = tid; t < 64 * P; t += 256) Mg[t] = 0.0;
      __syncthreads();
      if (act && tid < 64) {
        const int row = 64 * b + tid;
        double dout = 0.0;
        if (row < N) {
          const int64_t lo = base + 64 * (int64_t)b;
          for (int64_t p = prp[base + row]; p < prp[base + row + 1]; ++p) {
            const int64_t c = pci[p];
            const double v = pv[p];
            if (c >= base && c < base + N) {
              if (c >= lo && c < lo + 64) Mg[tid * P + (int)(c - lo)] = v;
            } else {
              dout += v;
            }
          }
          if (!plain) Mg[tid * P + tid] -= dout;
        } else {
          Mg[tid * P + tid] = 1.0;
        }
      }
      __syncthreads();
      double x[4][4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) x[a][c] = act ? Mg[(i0 + a) * P + j0 + c] - upd[a][c] : 0.0;
      if (kRounded && act && i0 == j0)
#pragma unroll
        for (int a = 0; a < 4; ++a) dsq[g][i0 + a] = sqrt(x[a][a]);
      FT* ft = fs + (size_t)b * kTriElems;
      sweep_inverse_64(
          x, prow[g], tid, act,
          [&](int k) {
            if (atomicCAS(fail, -1, s) == -1) fail[1] = 64 * b + k;
          },
          [&](int k, const double* pr, double rd) {
            if constexpr (kRounded) {
              if (form == 0) return;
              if (tid < k) {  // K[k][tid], where the pair (k, tid) is kept
                const double v = -pr[tid];
                const int c = k - tid;
                if (c <= 32) st_fac(ft + tri_at<FT>(c, tid), c == 32 ? 0.5 * v : v);
                if (c >= 32) st_fac(ft + tri_at<FT>(64 - c, k), c == 32 ? 0.5 * v : v);
              }
              if (tid == k) dg[ro + 64 * b + k] = (AT)rd;
            }
          });
      // x = -X_b
      if (kRounded && act && form == 0) {
        bool over = false;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          double sum = 0.0;  // of the row's |E| over the sixteen threads of its row
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double v = -x[a][c];
            const double t = i0 + a == j0 + c ? (double)(AT)v : tri_stored<FT>(v);
            sum = fma(fabs(t - v), dsq[g][j0 + c], sum);
          }
          sum = add_ror<1>(add_ror<2>(add_ror<4>(add_ror<8>(sum))));
          over |= !(sum * dsq[g][i0 + a] <= TriTau<FT>::v);  // (not a number: over)
        }
        if (over) far = 1;
      }
      if (act)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int c = 0; c < 4; ++c) Mg[(i0 + a) * P + j0 + c] = -x[a][c];
      __syncthreads();
      if (act && form == 0) {
        for (int t = tid; t < kTriElems; t += 256) {
          const int c = t / 64 + 1, l = t % 64;
          const double v = Mg[l * P + ((l + c) & 63)];
          st_fac(ft + tri_at<FT>(c, l), c == 32 ? 0.5 * v : v);
        }
        if (tid < 64) dg[ro + 64 * b + tid] = (AT)Mg[tid * P + tid];
      }
    }
    if constexpr (!kRounded) return;
    __syncthreads();
    if (form == 1 || !far) {
      if (threadIdx.x == 0) desc[s].tri = form;
      return;
    }
  }
}

// ---------------------------------------------------------------------------
// One subdomain's blocks as the solve kernels see them.
template <typename FT> struct TriSub {
  using AT = typename TriAcc<FT>::T;
  int N, NP, NB, h, len1, d, kc;  // d: steps group 1 waits at the start
  bool tri;                       // the triangular form
  const FT* fac;
  const AT* dg;
  const AT* cpl;
  const uint8_t* cidx;
};
template <typename FT>
__device__ __forceinline__ TriSub<FT> tri_sub(const SubDesc& e, const FT* fac,
                                              const typename TriAcc<FT>::T* dg,
                                              const typename TriAcc<FT>::T* cpl,
                                              const uint8_t* cidx) {
  TriSub<FT> t;
  t.N = e.N;
  t.NB = (e.N + 63) / 64;
  t.NP = 64 * t.NB;
  t.h = t.NB / 2;
  t.len1 = t.NB - 1 - t.h;
  t.d = t.h - t.len1;
  t.kc = e.kc;
  t.tri = sizeof(FT) < 8 && e.tri;
  t.fac = fac + e.fac;
  t.dg = dg + e.ro;
  t.cpl = cpl + e.cpl;
  t.cidx = cidx + e.cpl;
  return t;
}

// Multiscale basis functions (set-up): one wave per (subdomain, slot), the
// right-hand side -B_s psi_n scattered from the boundary weights, then the
// block elimination one block after the other in the vector v (LDS; for a
// subdomain of more than kMbfRows rows, ONCHIP = false, memory of the set-up:
// tmp, ldt a workgroup).
// The interface matrix S is made of 1 - phat at the interfaces, which
// cancels where phat is near 1, so phat is improved once by the correction
// for its residual b - A_s phat, accumulated in twice the working precision
// (the applied z of a 100-cell chain with interfaces on every cell: error
// 4e-13 with S from unrefined values, 4e-14 so).
constexpr int kMbfRows = 4096;  // 32 KB
template <bool ONCHIP>
__global__ __launch_bounds__(64) void k_tri_mbf(
    const int32_t* __restrict__ pairs, const int32_t* __restrict__ pair_sub,
    const int32_t* __restrict__ pair_q, const SubDesc* __restrict__ desc,
    const double* __restrict__ fac, const double* __restrict__ dg,
    const double* __restrict__ cpl, const uint8_t* __restrict__ cidx,
    const int64_t* __restrict__ prp, const int32_t* __restrict__ pci,
    const double* __restrict__ pv, double* mbf, const int64_t* __restrict__ bw_ptr,
    const int32_t* __restrict__ bw_row, const double* __restrict__ bw_val, int plain,
    double* tmp, int ldt) {
  __shared__ double tw[128];
  __shared__ double yw[64];
  __shared__ double hw[64];
  extern __shared__ double dyn[];
  const int pi = pairs[blockIdx.x];
  const int s = pair_sub[pi], q = pair_q[pi];
  const SubDesc e = desc[s];
  const TriSub<double> T = tri_sub(e, fac, dg, cpl, cidx);
  double* col = mbf + e.mbf + (size_t)q * T.N;
  double* v = ONCHIP ? dyn : tmp + (size_t)blockIdx.x * ldt;
  const int lane = threadIdx.x;
  auto scatter = [&]() {
    for (int row = lane; row < T.N; row += 64) v[row] = 0.0;
    __syncthreads();
    for (int64_t t = bw_ptr[pi] + lane; t < bw_ptr[pi + 1]; t += 64) v[bw_row[t]] = bw_val[t];
    __syncthreads();
  };
  // sum of the couplings of row (b, lane) in `list` times the block vector in yw
  auto couple = [&](int b, int list) -> double {
    double x = 0.0;
    for (int k = 0; k < T.kc; ++k) {
      const int at = (list * T.kc + k) * T.NP + 64 * b + lane;
      x = fma(T.cpl[at], yw[T.cidx[at]], x);
    }
    return x;
  };
  auto put = [&](double x) {
    tri_wave_sync();
    yw[lane] = x;
    tri_wave_sync();
  };
  // X_b t
  auto product = [&](int b, double t0) -> double {
    double t[1] = {t0};
    tri_wave_sync();
    tw[lane] = t0;
    tw[lane + 64] = t0;
    tri_wave_sync();
    double y = T.dg[64 * b + lane] * t0;
    for (int c0 = 0; c0 < 32; c0 += 8) {
      TriFrag<double, 8> f;
      f.load(T.fac + (size_t)b * kTriElems, c0, lane);
      double a[1], hh[1];
      tri_partial<double, 8, 1>(f, c0, lane, t, tw, a, hh);
      tri_wave_sync();
      hw[(lane + c0 + 1) & 63] = hh[0];
      tri_wave_sync();
      y += a[0] + hw[lane];
    }
    return y;
  };
  auto ld = [&](int b) -> double {
    const int row = 64 * b + lane;
    return row < T.N ? v[row] : 0.0;
  };
  auto st = [&](int b, double x) {
    const int row = 64 * b + lane;
    if (row < T.N) v[row] = x;
  };
  auto solve = [&]() {  // v = A_s^{-1} v
    for (int b = 0; b < T.h; ++b) {
      double t = ld(b);
      if (b > 0) t -= couple(b, 0);
      const double w = product(b, t);
      st(b, w);
      put(w);
    }
    double th = ld(T.h);
    if (T.h > 0) th -= couple(T.h, 0);
    for (int b = T.NB - 1; b > T.h; --b) {
      double t = ld(b);
      if (b < T.NB - 1) t -= couple(b, 1);
      const double w = product(b, t);
      st(b, w);
      put(w);
    }
    if (T.len1 > 0) th -= couple(T.h, 1);
    const double xh = product(T.h, th);
    st(T.h, xh);
    put(xh);
    for (int b = T.h - 1; b >= 0; --b) {
      const double x = ld(b) - product(b, couple(b, 1));
      st(b, x);
      put(x);
    }
    put(xh);
    for (int b = T.h + 1; b < T.NB; ++b) {
      const double x = ld(b) - product(b, couple(b, 0));
      st(b, x);
      put(x);
    }
    __syncthreads();
  };
  scatter();
  solve();
  for (int row = lane; row < T.N; row += 64) col[row] = v[row];
  __syncthreads();
  scatter();
  for (int row = lane; row < T.N; row += 64) {
    double hi = v[row], lo = 0.0;
    auto add = [&](double a) {  // (hi, lo) += a
#pragma clang fp contract(off)
      const double u = hi + a, w = u - hi;
      lo += (hi - (u - w)) + (a - w);
      hi = u;
    };
    auto sub = [&](double a, double x) {  // (hi, lo) -= a x
#pragma clang fp contract(off)
      const double m = a * x;
      add(-m);
      lo -= fma(a, x, -m);
    };
    double dout = 0.0, diag = 0.0;
    for (int64_t p = prp[e.base + row]; p < prp[e.base + row + 1]; ++p) {
      const int64_t c = (int64_t)pci[p] - e.base;
      const double a = pv[p];
      if (c < 0 || c >= T.N)
        dout += a;
      else if (c == row)
        diag = a;
      else if (abs((int)c / 64 - row / 64) <= 1)  // (see k_tri_couplings)
        sub(a, col[c]);
    }
    sub(plain ? diag : diag - dout, col[row]);
    v[row] = hi + lo;
  }
  __syncthreads();
  solve();
  for (int row = lane; row < T.N; row += 64) col[row] += v[row];
}

// ---------------------------------------------------------------------------
// Fused interface solve: stop test and interface values of one subdomain's
// workgroup.  Wave v forms the partial dots of the subdomain's rows of S^{-1}
// with b over its share of the columns; the partials meet in etap
// ([NW][ns][NT]).  Returns true when the solve has stopped (workgroup 0 of
// this very launch may be writing the stop flag, so the decision comes from
// the stop test's own partials, the first wave's for the workgroup); else
// eta_s holds the subdomain's ns interface values, a barrier having passed.
template <int NT, int NW>
__device__ __forceinline__ bool local_prologue(int mode, int ns, int64_t i0,
                                               const int32_t* __restrict__ isub_list,
                                               const double* __restrict__ Sinv, int NL, int ldS,
                                               const double* __restrict__ bpart,
                                               const double* __restrict__ pb, int npb, int init,
                                               PcgScalars* sc, PcgShared* sh, double* etap,
                                               double* eta_s, int* stop_s) {
  constexpr int NTHR = 64 * NW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int stop = 0;
  if (mode == 2) stop = stop_test<NT>(pb, npb, init, sc, sh, threadIdx.x == 0) ? 1 : 0;
  if (threadIdx.x == 0) *stop_s = stop;
  if (!stop) {
    // rows per chunk (six: a box's faces) and columns per lane and round;
    // a round's loads are all issued before the first is used
    constexpr int EQ = NT == 1 ? 6 : NT == 2 ? 3 : NT == 4 ? 2 : 1;
    constexpr int UM = NT == 1 ? 4 : NT == 2 ? 2 : 1;
    const int per = (NL + NW - 1) / NW;
    const int mb = wave * per, me = min(NL, mb + per);
    for (int q0 = 0; q0 < ns; q0 += EQ) {
      const double* rowp[EQ];
#pragma unroll
      for (int qq = 0; qq < EQ; ++qq)
        rowp[qq] = Sinv + (size_t)isub_list[i0 + min(q0 + qq, ns - 1)] * ldS;
      double a[EQ][NT];
#pragma unroll
      for (int qq = 0; qq < EQ; ++qq)
#pragma unroll
        for (int k = 0; k < NT; ++k) a[qq][k] = 0.0;
      for (int m0 = mb; m0 < me; m0 += 64 * UM) {
        double bm[UM][2][NT], sv[UM][EQ];
#pragma unroll
        for (int u = 0; u < UM; ++u) {
          const int m = min(m0 + 64 * u + lane, NL - 1);
#pragma unroll
          for (int k = 0; k < NT; ++k) {
            bm[u][0][k] = bpart[(size_t)(2 * m) * NT + k];
            bm[u][1][k] = bpart[(size_t)(2 * m + 1) * NT + k];
          }
#pragma unroll
          for (int qq = 0; qq < EQ; ++qq) sv[u][qq] = rowp[qq][m];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < UM; ++u) {
          const bool ok = m0 + 64 * u + lane < me;
#pragma unroll
          for (int k = 0; k < NT; ++k) {
            const double bv = ok ? bm[u][0][k] + bm[u][1][k] : 0.0;
#pragma unroll
            for (int qq = 0; qq < EQ; ++qq) a[qq][k] = fma(sv[u][qq], bv, a[qq][k]);
          }
        }
      }
#pragma unroll
      for (int qq = 0; qq < EQ; ++qq)
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          const double t = wave_sum(a[qq][k]);
          if (lane == 0 && q0 + qq < ns) etap[((size_t)wave * ns + q0 + qq) * NT + k] = t;
        }
    }
  }
  __syncthreads();
  if (*stop_s) return true;
  for (int t = threadIdx.x; t < ns * NT; t += NTHR) {
    double e = 0.0;
    for (int v = 0; v < NW; ++v) e += etap[(size_t)v * ns * NT + t];
    eta_s[t] = e;
  }
  __syncthreads();  // etap is free again
  return false;
}

// ---------------------------------------------------------------------------
// The solve, 1 to 4 right-hand sides: two waves per subdomain, one for each
// half.  A wave holds all 32 stored diagonals of its half's HT blocks next to
// the middle in registers (both waves 16 of the middle block's) and uses them
// in both sweeps: with HT = 4 a subdomain of up to nine blocks (a 512-cell
// box: 135 KB of FP64 factor) is read exactly once.  A step of the chain stays inside the wave: the neighbour's values
// through lane permutes, t through the wave's own LDS copy, the transposed
// half of the product by wave rotations; the halves meet only at the middle
// block.  (More waves per half, each with a share of the diagonals, cost a
// barrier and a round of partial sums per step: 1.0 us a step with four waves
// against 0.45.)  Blocks further out than HT are read again on the way back.
// x goes to LDS, and all threads form z = x + sum eta phat and the PCG dots
// over the rows at the end.  128^3 (4096 boxes), FP64: 168 us for 0.79 GB (counters), the
// loads of one workgroup beside the chain of the other on its CU (band tiles
// read once per sweep, 32 barriers: 342 us for 2.1 GB); FP32 99 us; 64^3 21 us
// (52 us with the interface rows formed inside).
template <typename FT, int NT, int HT> constexpr int tri_waves() {
  constexpr int regs = (2 * HT + 1) * 4 * (int)sizeof(FT) + 16 * NT + 72;
  return regs <= 128 ? 4 : regs <= 256 ? 2 : 1;
}
// The arguments of k_tri_solve once more, for the body of the triangular form
// (aligned: a gap keeps the loads of both from being merged).
template <typename FT> struct alignas(64) TriArgs {
  const SubDesc* desc;
  const FT* fac;
  const typename TriAcc<FT>::T *dg, *cpl;
  const uint8_t* cidx;
  const double* rin;
  double* out;
  int mode;
  const int32_t* isub_list;
  const double *mbf, *eta, *qv;
  double* partial;
  unsigned blk_off;
  int fuse_eta;
  const double* Sinv;
  int NL, ldS;
  const double *bpart, *pb;
  int npb, init;
  PcgScalars* sc;
  PcgShared* sh;
};
template <typename FT, int NT, int HT, bool BFOP = false>
__global__ __launch_bounds__(128, (tri_waves<FT, NT, HT>())) void k_tri_solve(
    const int32_t* __restrict__ subs, const SubDesc* __restrict__ desc,
    const FT* __restrict__ fac, const typename TriAcc<FT>::T* __restrict__ dg,
    const typename TriAcc<FT>::T* __restrict__ cpl, const uint8_t* __restrict__ cidx,
    const double* rin, double* out, int mode, const int32_t* __restrict__ isub_list,
    const double* __restrict__ mbf, const double* __restrict__ eta, const double* __restrict__ qv,
    double* __restrict__ partial, unsigned blk_off, int fuse_eta, const double* __restrict__ Sinv,
    int NL, int ldS, const double* __restrict__ bpart, const double* __restrict__ pb, int npb,
    int init, PcgScalars* sc, PcgShared* sh, TriArgs<FT> again) {
  using AT = typename TriAcc<FT>::T;
  constexpr int NTHR = 128;
  constexpr int RR = (2 * HT + 1) * 64;  // rows held on chip
  __shared__ AT tw_all[2][NT * 128];
  __shared__ AT ex[2][3][NT * 64];  // what a half hands to the other at the middle
  __shared__ AT rs[RR * NT];        // r; then w, then x of the blocks already done
  __shared__ AT ds[RR];             // diagonals of the block inverses
  __shared__ double eta_s[128 * NT];
  __shared__ double etap[256];  // interface partials of the prologue
  __shared__ double dots[2][2 * NT];
  __shared__ int stop_s;

  const int s = subs ? subs[blockIdx.x] : (int)blockIdx.x;  // null: the identity list
  const SubDesc e = desc[s];
  // a solve that has stopped (with the fused interface solve workgroup 0 of
  // this launch may be writing the flag: the stop test below decides)
  if (mode == 2 && !fuse_eta && all_done(sh)) return;
  // The triangular form has a body of its own, which streams all blocks but the
  // middle one, and arguments of its own: scalar loads with a use in both
  // bodies would stay before the branch, more of them than there are registers.
  // (The FP32 kernel at 128^3: with a branch around each product 8% slower,
  // with shared arguments 6%, so as without the form.)
  auto solve = [&](auto form, const SubDesc& e, const FT* fac, const AT* dg, const AT* cpl, const uint8_t* cidx,
                   const double* rin, double* out, int mode, const int32_t* isub_list,
                   const double* mbf, const double* eta, const double* qv, double* partial,
                   unsigned blk_off, int fuse_eta, const double* Sinv, int NL, int ldS,
                   const double* bpart, const double* pb, int npb, int init, PcgScalars* sc,
                   PcgShared* sh) AM_INLINE {
    constexpr bool TRI = decltype(form)::value;
    constexpr int HE = TRI ? 0 : HT;        // blocks of a half that are held
    constexpr int RH = (2 * HE + 1) * 64;   // rows held on chip
    constexpr int NS = HE + 1;              // rows per thread of those, rounded up
    const int64_t base = e.base, i0 = e.i0;
    const TriSub<FT> T = tri_sub(e, fac, dg, cpl, cidx);
    const int lane = threadIdx.x & 63;
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ns = mode >= 1 ? e.ns : 0;
    const double* P = mbf + e.mbf;
    AT* tw = tw_all[g];

    // step k of a half (k = 0 the outermost block); off steps are streamed
    const int off = max(0, T.h - HE);
    const int r_lo = 64 * off;             // first row held on chip
    const int r_n = min(T.NP - r_lo, RH);  // rows held on chip
    auto blk = [&](int k) AM_INLINE { return g == 0 ? k : T.NB - 1 - (k - T.d); };
    auto active = [&](int k) AM_INLINE { return g == 0 || k >= T.d; };
    // list of a row's couplings to the block that comes before it on the way to
    // the middle (F) and after it (B)
    const int LF = g == 0 ? 0 : 1, LB = 1 - LF;

    // ---- loads: what goes to LDS, then the tiles (in the order of their use:
    // a wait for an early load does not wait for the later ones) ----
    AT rv[NS][NT], dv[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int t = u * NTHR + threadIdx.x, row = r_lo + t;
#pragma unroll
      for (int k = 0; k < NT; ++k)
        rv[u][k] = (t < r_n && row < T.N) ? (AT)rin[(size_t)(base + row) * NT + k] : (AT)0;
      dv[u] = t < r_n ? T.dg[row] : (AT)0;
    }
    int eid = 0;  // basis function of the thread's first interface value
    if (!fuse_eta && (int)threadIdx.x < ns * NT) eid = isub_list[i0 + threadIdx.x / NT];
    // the tiles: two steps ahead of their use (the first two here); all of
    // them at once flood the memory system, and no workgroup gets its first
    // tile before the others have got their last.  No branch around the loads:
    // waits at the joins would put them one after the other; a half with fewer
    // blocks loads its last one again.
    TriFrag<FT, 32> D[HE > 0 ? HE : 1];
    TriFrag<FT, 16> Dm;
    auto fetch_tile = [&](auto jc) AM_INLINE {
      constexpr int j = decltype(jc)::value;
      if constexpr (j < HE) {
        const int k = min(off + j, T.h - 1);
        D[j].load(T.fac + (size_t)(k >= 0 && active(k) ? blk(k) : T.h) * kTriElems, 0, lane);
      } else if constexpr (j == HE) {
        Dm.load(T.fac + (size_t)T.h * kTriElems, 16 * g, lane);
      }
    };
    fetch_tile(std::integral_constant<int, 0>{});
    fetch_tile(std::integral_constant<int, 1>{});
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int t = u * NTHR + threadIdx.x;
      if (t < r_n) {
#pragma unroll
        for (int k = 0; k < NT; ++k) rs[k * RR + t] = rv[u][k];
        ds[t] = dv[u];
      }
    }
    double ev = 0.0;
    if (!fuse_eta && (int)threadIdx.x < ns * NT) ev = eta[(size_t)eid * NT + threadIdx.x % NT];
    __syncthreads();

    // row values of block b for this lane, and v += sign * (couplings of list
    // `list`) . (the neighbour's values y)
    auto rhs = [&](int b, AT (&v)[NT]) AM_INLINE {
      const int t = 64 * b + lane - r_lo;
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        if (64 * b >= r_lo && 64 * b < r_lo + r_n)  // uniform
          v[k] = rs[k * RR + t];
        else
          v[k] = 64 * b + lane < T.N ? (AT)rin[(size_t)(base + 64 * b + lane) * NT + k] : (AT)0;
      }
    };
    // the next step's couplings (this lane's row, places 0 .. KA-1), requested
    // a product ahead and before the tile that is requested with them
    constexpr int KA = 5;  // boxes have one place, bisection parts three to five
    AT cv[KA];
    int ci[KA];
    auto ahead = [&](int b, int list) AM_INLINE {
      if (T.kc == 0) return;
      const int at = list * T.kc * T.NP + 64 * b + lane;
      cv[0] = T.cpl[at];
      ci[0] = T.cidx[at];
      if (T.kc > 1)
#pragma unroll
        for (int k = 1; k < KA; ++k) {
          const int ak = at + min(k, T.kc - 1) * T.NP;
          cv[k] = T.cpl[ak];
          ci[k] = T.cidx[ak];
        }
    };
    auto couple = [&](int b, int list, AT sign, const AT (&y)[NT], AT (&v)[NT]) AM_INLINE {
      if (T.kc == 0) return;
      if constexpr (NT > 1) {
        tri_wave_sync();
#pragma unroll
        for (int c = 0; c < NT; ++c) tw[128 * c + lane] = y[c];
        tri_wave_sync();
      }
      auto add = [&](AT w, int i) AM_INLINE {
#pragma unroll
        for (int c = 0; c < NT; ++c)
          v[c] = fma(w, NT > 1 ? tw[128 * c + i] : lane_value(y[c], i), v[c]);
      };
      add(sign * cv[0], ci[0]);
      if (T.kc > 1) {
#pragma unroll
        for (int k = 1; k < KA; ++k) add(k < T.kc ? sign * cv[k] : (AT)0, ci[k]);
        for (int k = KA; k < T.kc; ++k) {
          const int at = (list * T.kc + k) * T.NP + 64 * b + lane;
          add(sign * T.cpl[at], T.cidx[at]);
        }
      }
    };
    // a product's vector operand: rounded to BF16 on request (the stored
    // diagonals are BF16 then, so their products are exact in FP32)
    auto operand = [&](AT v) AM_INLINE -> AT {
      if constexpr (BFOP)
        return __builtin_bit_cast(float, (uint32_t)(uint16_t)am_bf16_rne(v) << 16);
      else
        return v;
    };
    auto put = [&](const AT (&v)[NT]) AM_INLINE {  // t where the product reads it, twice
      tri_wave_sync();
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        tw[128 * k + lane] = v[k];
        tw[128 * k + lane + 64] = v[k];
      }
      tri_wave_sync();
    };
    // y = X_b t, the tile in f
    auto product = [&](const TriFrag<FT, 32>& f, int b, const AT (&t)[NT], AT (&y)[NT]) AM_INLINE {
      AT tp[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) tp[k] = operand(t[k]);
      put(tp);
      const int i = 64 * b + lane - r_lo;
      const AT dgv = (64 * b >= r_lo && 64 * b < r_lo + r_n) ? ds[i] : T.dg[64 * b + lane];
#pragma unroll
      for (int k = 0; k < NT; ++k) y[k] = dgv * t[k];
      tri_full<FT, NT>(f, lane, tp, tw, y);
    };
    // the same of a streamed block, in either form
    auto product_streamed = [&](const TriFrag<FT, 32>& f, int b, const AT (&t)[NT],
                                AT (&y)[NT]) AM_INLINE {
      if constexpr (TRI) {
        AT tp[NT], v[NT], a[NT], h[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) tp[k] = operand(t[k]);
        put(tp);
        tri_partial<FT, 32, NT, 1>(f, 0, lane, tp, tw, a, h);
        const AT dgv = T.dg[64 * b + lane];
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          v[k] = dgv * (t[k] + (a[k] + wave_ror1(h[k])));
          tp[k] = operand(v[k]);
        }
        put(tp);
        tri_partial<FT, 32, NT, 2>(f, 0, lane, tp, tw, a, h);
#pragma unroll
        for (int k = 0; k < NT; ++k) y[k] = v[k] + (a[k] + wave_ror1(h[k]));
      } else {
        product(f, b, t, y);
      }
    };

    AT y[NT], t[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) y[k] = (AT)0;
    // ---- elimination towards the middle: streamed blocks, then resident ----
    const int first = g == 0 ? 0 : T.d;
    for (int k = first; k < off; ++k) {
      const int b = blk(k);
      TriFrag<FT, 32> f;
      f.load(T.fac + (size_t)b * kTriElems, 0, lane);
      rhs(b, t);
      if (k > first) couple(b, LF, (AT)-1, y, t);
      ahead(k + 1 < T.h ? blk(k + 1) : T.h, LF);
      product_streamed(f, b, t, y);
      if (64 * b + lane < T.N)
#pragma unroll
        for (int c = 0; c < NT; ++c) out[(size_t)(base + 64 * b + lane) * NT + c] = (double)y[c];
    }
    auto inward = [&](auto jc) AM_INLINE {
      constexpr int j = decltype(jc)::value;
      if constexpr (j < HE) {
        const int k = off + j;
        const bool act = k < T.h && k >= first;  // uniform
        const int b = act ? blk(k) : 0;
        if (act) {
          rhs(b, t);
          if (k > first) couple(b, LF, (AT)-1, y, t);
          ahead(k + 1 < T.h ? blk(k + 1) : T.h, LF);
        }
        fetch_tile(std::integral_constant<int, j + 2>{});
        if (act) {
          product(D[j], b, t, y);
#pragma unroll
          for (int c = 0; c < NT; ++c) rs[c * RR + 64 * b - r_lo + lane] = y[c];
        }
      }
    };
    static_assert(HE <= 6, "steps written out");
    inward(std::integral_constant<int, 0>{});
    inward(std::integral_constant<int, 1>{});
    inward(std::integral_constant<int, 2>{});
    inward(std::integral_constant<int, 3>{});
    inward(std::integral_constant<int, 4>{});
    inward(std::integral_constant<int, 5>{});
    // the fused interface solve and its stop test here: its loads would queue
    // behind the tiles at the start (64^3: 6 us before the first step)
    if (fuse_eta && local_prologue<NT, 2>(mode, ns, i0, isub_list, Sinv, NL, ldS, bpart, pb, npb, init,
                                          sc, sh, etap, eta_s, &stop_s))
      return;
    // ---- middle block: both waves ----
    {
      AT cm[NT];
#pragma unroll
      for (int c = 0; c < NT; ++c) cm[c] = (AT)0;
      if (g == 0 ? T.h > 0 : T.len1 > 0) couple(T.h, LF, (AT)1, y, cm);
#pragma unroll
      for (int c = 0; c < NT; ++c) ex[g][0][64 * c + lane] = cm[c];
      if (!fuse_eta) {
        if ((int)threadIdx.x < ns * NT) eta_s[threadIdx.x] = ev;
        for (int q = NTHR + threadIdx.x; q < ns * NT; q += NTHR)
          eta_s[q] = eta[(size_t)isub_list[i0 + q / NT] * NT + q % NT];
      }
      rhs(T.h, t);
      __syncthreads();
#pragma unroll
      for (int c = 0; c < NT; ++c)
        t[c] = (t[c] - ex[0][0][64 * c + lane]) - ex[1][0][64 * c + lane];
      AT tp[NT], a[NT], h[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) tp[k] = operand(t[k]);
      put(tp);
      if (g == 0 ? T.h > 0 : T.len1 > 0) ahead(blk(T.h - 1), LB);
      // both waves' 16 diagonals and the main one, added up
      auto meet = [&]() AM_INLINE {
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          ex[g][1][64 * k + lane] = a[k];
          ex[g][2][64 * k + ((lane + 16 * g + 1) & 63)] = h[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NT; ++k)
          y[k] = (ex[0][1][64 * k + lane] + ex[1][1][64 * k + lane]) +
                 (ex[0][2][64 * k + lane] + ex[1][2][64 * k + lane]);
      };
      if constexpr (TRI) {
        tri_partial<FT, 16, NT, 1>(Dm, 16 * g, lane, tp, tw, a, h);
        if (g == 0)
#pragma unroll
          for (int k = 0; k < NT; ++k) a[k] += t[k];
        meet();
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          t[k] = ds[64 * T.h + lane - r_lo] * y[k];
          tp[k] = operand(t[k]);
        }
        put(tp);
        tri_partial<FT, 16, NT, 2>(Dm, 16 * g, lane, tp, tw, a, h);
        if (g == 0)
#pragma unroll
          for (int k = 0; k < NT; ++k) a[k] += t[k];
        __syncthreads();  // the sums of the first product are read
      } else {
        tri_partial<FT, 16, NT>(Dm, 16 * g, lane, tp, tw, a, h);
        if (g == 0) {
          const AT dgv = ds[64 * T.h + lane - r_lo];
#pragma unroll
          for (int k = 0; k < NT; ++k) a[k] = fma(dgv, t[k], a[k]);
        }
      }
      meet();
      if (g == 0)
#pragma unroll
        for (int k = 0; k < NT; ++k) rs[k * RR + 64 * T.h - r_lo + lane] = y[k];
    }
    // ---- back outwards ----
    double rz[NT], qz[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) rz[k] = qz[k] = 0.0;
    // (q, z) enters the flexible beta only
    const int flexible = mode == 2 ? sh->flexible : 0;
    // z of a row from its x and its share of the dots; the row's basis functions
    // (six: a box's faces) and vector values are loaded before
    struct RowIn {
      double p[6], r[NT], q[NT];
    };
    auto load_in = [&](int row, RowIn& in) AM_INLINE {
#pragma unroll
      for (int u = 0; u < 6; ++u) in.p[u] = u < ns ? P[(size_t)u * T.N + row] : 0.0;
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        const size_t o = (size_t)(base + row) * NT + k;
        in.r[k] = mode == 2 ? rin[o] : 0.0;
        in.q[k] = flexible ? qv[o] : 0.0;
      }
    };
    auto finish = [&](int row, const AT (&x)[NT], const RowIn& in) AM_INLINE {
      double z[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) z[k] = (double)x[k];
#pragma unroll
      for (int u = 0; u < 6; ++u)
        if (u < ns)
#pragma unroll
          for (int k = 0; k < NT; ++k) z[k] = fma(in.p[u], eta_s[u * NT + k], z[k]);
      for (int q0 = 6; q0 < ns; q0 += 6) {
        double pq[6];
#pragma unroll
        for (int u = 0; u < 6; ++u) pq[u] = P[(size_t)min(q0 + u, ns - 1) * T.N + row];
#pragma unroll
        for (int u = 0; u < 6; ++u)
          if (q0 + u < ns)
#pragma unroll
            for (int k = 0; k < NT; ++k) z[k] = fma(pq[u], eta_s[(q0 + u) * NT + k], z[k]);
      }
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        rz[k] = fma(in.r[k], z[k], rz[k]);
        qz[k] = fma(in.q[k], z[k], qz[k]);
        out[(size_t)(base + row) * NT + k] = z[k];
      }
    };
    // the resident rows are finished RB at a time with their loads together;
    // the first ones' loads go out before the way back (after it, their round
    // trip stands alone at the end of the workgroup)
    const int rows = min(r_n, T.N - r_lo);
    constexpr int RB = NT == 1 ? 4 : NT == 2 ? 2 : 1;
    RowIn ri[RB];
    auto load_first = [&]() AM_INLINE {
#pragma unroll
      for (int u = 0; u < RB; ++u) load_in(r_lo + min((int)threadIdx.x + NTHR * u, rows - 1), ri[u]);
    };
    constexpr bool kEarly = NT == 1 && HE == 4;  // (elsewhere the registers don't allow it)
    if constexpr (kEarly) load_first();
#pragma unroll
    for (int j = HE - 1; j >= 0; --j) {
      const int k = off + j;
      if (k >= T.h || k < first) continue;  // uniform
      const int b = blk(k);
      AT wv[NT];
      rhs(b, wv);
#pragma unroll
      for (int c = 0; c < NT; ++c) t[c] = (AT)0;
      couple(b, LB, (AT)1, y, t);
      if (k > first) ahead(blk(k - 1), LB);
      product(D[j], b, t, y);
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        y[c] = wv[c] - y[c];
        rs[c * RR + 64 * b - r_lo + lane] = y[c];
      }
    }
    for (int k = off - 1; k >= first; --k) {
      const int b = blk(k);
      TriFrag<FT, 32> f;
      f.load(T.fac + (size_t)b * kTriElems, 0, lane);
      const bool in = 64 * b + lane < T.N;
      AT wv[NT];
#pragma unroll
      for (int c = 0; c < NT; ++c) wv[c] = in ? (AT)out[(size_t)(base + 64 * b + lane) * NT + c] : (AT)0;
#pragma unroll
      for (int c = 0; c < NT; ++c) t[c] = (AT)0;
      couple(b, LB, (AT)1, y, t);
      if (k > first) ahead(blk(k - 1), LB);
      product_streamed(f, b, t, y);
#pragma unroll
      for (int c = 0; c < NT; ++c) y[c] = wv[c] - y[c];
      if (in) {
        RowIn ri;
        load_in(64 * b + lane, ri);
        finish(64 * b + lane, y, ri);
      }
    }
    if constexpr (!kEarly) load_first();
    __syncthreads();
    for (int i0r = 0; i0r < rows; i0r += RB * NTHR) {
      if (i0r > 0)
#pragma unroll
        for (int u = 0; u < RB; ++u) load_in(r_lo + min(i0r + (int)threadIdx.x + NTHR * u, rows - 1), ri[u]);
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int i = i0r + threadIdx.x + NTHR * u;
        if (i < rows) {
          AT x[NT];
#pragma unroll
          for (int k = 0; k < NT; ++k) x[k] = rs[k * RR + i];
          finish(r_lo + i, x, ri[u]);
        }
      }
    }
    if (mode != 2) return;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const double a = wave_sum(rz[k]);
      const double b2 = wave_sum(qz[k]);
      if (lane == 0) {
        dots[g][k] = a;
        dots[g][NT + k] = b2;
      }
    }
    __syncthreads();
    if (threadIdx.x < 2 * NT)
      partial[(size_t)(blk_off + blockIdx.x) * 2 * NT + threadIdx.x] =
          dots[0][threadIdx.x] + dots[1][threadIdx.x];
  };
  if constexpr (sizeof(FT) < 8) {
    if (__builtin_expect(e.tri, 0)) {  // uniform over the workgroup
      const TriArgs<FT>& a = again;
      solve(std::true_type{}, a.desc[s], a.fac, a.dg, a.cpl, a.cidx, a.rin, a.out, a.mode, a.isub_list, a.mbf,
            a.eta, a.qv, a.partial, a.blk_off, a.fuse_eta, a.Sinv, a.NL, a.ldS, a.bpart, a.pb,
            a.npb, a.init, a.sc, a.sh);
      return;
    }
  }
  solve(std::false_type{}, e, fac, dg, cpl, cidx, rin, out, mode, isub_list, mbf, eta, qv, partial,
        blk_off, fuse_eta, Sinv, NL, ldS, bpart, pb, npb, init, sc, sh);
}

// Two 16-row strips of the product, sharing the vector operand (operands as in
// mf_pass; afn(u, c, m) of strip u): four operand triples read at a time, two
// chains per strip.
template <bool BFOP, typename V, typename AT, typename AF, typename BF>
__device__ __forceinline__ void tri_mf_pass(V (&acc)[2], AF&& afn, BF&& bfn) {
  if constexpr (BFOP) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      acc[u] = mf_pass<true>(V{0, 0, 0, 0}, [&](int c, int m) { return afn(u, c, m); }, bfn);
  } else {
    V c[2][2] = {{V{0, 0, 0, 0}, V{0, 0, 0, 0}}, {V{0, 0, 0, 0}, V{0, 0, 0, 0}}};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      AT a[2][4], b[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[0][t] = afn(0, 4 * (4 * h + t), 1);
        a[1][t] = afn(1, 4 * (4 * h + t), 1);
        b[t] = bfn(4 * (4 * h + t), 1);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        c[0][t % 2] = mf4(a[0][t], b[t], c[0][t % 2]);
        c[1][t % 2] = mf4(a[1][t], b[t], c[1][t % 2]);
      }
    }
    acc[0] = c[0][0] + c[0][1];
    acc[1] = c[1][0] + c[1][1];
  }
}

// ---------------------------------------------------------------------------
// The solve, 8 or 16 right-hand sides, on the matrix cores: two groups of two
// waves per subdomain, eliminating from the two ends.  A step is the 64 x 64
// by 64 x 16 product of the group's tile with its block vector, each wave 32
// output rows over all 64 columns (v_mfma_f64_16x16x4f64, FP32 and BF16
// factors on v_mfma_f32_16x16x4f32, or BF16 x BF16 products with BFOP).  The
// packed tile is fetched into registers one step ahead and stored to LDS by
// diagonals (pitch TP: the operand A[i][j], element (j - i) mod 64 of row i or
// (i - j) mod 64 of row j, then falls on distinct banks for the 16 rows of a
// strip).  The block vector t is formed by rows (two threads a row, eight
// columns each, the couplings of the row in the thread's registers) and
// written to LDS for the product; the result y goes to an LDS buffer of its
// own for the next step's couplings: two barriers a step.  w_b waits in `out`
// for the way back (a 512-row subdomain's 16 columns are 64 KB; beside the
// tiles they would leave room for one workgroup per CU instead of two).  Both
// groups form the middle block's x themselves: no exchange on the way back.
// z = x + sum eta phat is FP64 for every factor type (v_mfma_f64_16x16x4f64; x
// changes its result layout through LDS).  A subdomain in the triangular form
// takes two products and two more barriers a step.
// Bound by the LDS and memory latencies of a step (about 5 us with two
// workgroups on the CU, 0.5 of it the product): 1721 subdomains of 200-800
// cells, 16 columns, FP64: 347 us (band tiles, four products a step: 458).
// Eight waves of 128 registers spilled, and their scratch loads waited behind
// the tile loads: 885 us.
constexpr int kTriTP = 66;
template <typename AT> constexpr size_t tri_mf_lds() {  // static part
  return sizeof(AT) * (2 * 33 * kTriTP + 4 * 64 * 16) + 64;
}
template <typename FT, int NT, bool BFOP = false>
__global__ __launch_bounds__(256, 2) void k_tri_mf(
    const int32_t* __restrict__ subs, const SubDesc* __restrict__ desc,
    const FT* __restrict__ fac, const typename TriAcc<FT>::T* __restrict__ dg,
    const typename TriAcc<FT>::T* __restrict__ cpl, const uint8_t* __restrict__ cidx,
    const double* rin, double* out, int mode, const int32_t* __restrict__ isub_list,
    const double* __restrict__ mbf, const double* __restrict__ eta, const double* __restrict__ qv,
    double* __restrict__ partial, unsigned blk_off, int fuse_eta, const double* __restrict__ Sinv,
    int NL, int ldS, const double* __restrict__ bpart, const double* __restrict__ pb, int npb,
    int init, PcgScalars* sc, PcgShared* sh) {
  static_assert(NT == 8 || NT == 16, "one 16-column matrix-core tile");
  using AT = typename TriAcc<FT>::T;
  using V = typename MfAcc<AT>::V;
  constexpr int TP = kTriTP, VEC = 16 / (int)sizeof(FT);
  constexpr int NLD = kTriElems / (VEC * 128);  // 16-byte loads per thread and tile
  constexpr int NC = NT / 2;                    // columns per thread in the row layout
  __shared__ AT tile[2][33 * TP];
  __shared__ AT vb[2][64 * 16];  // t of each group
  __shared__ AT yb[2][64 * 16];  // its last w or x
  __shared__ int stop_s;
  static_assert(sizeof(tile) + sizeof(vb) + sizeof(yb) + 64 <= tri_mf_lds<AT>(),
                "the launcher sizes the dynamic part by this");
  extern __shared__ double eta_s[];  // [max_ni][NT] interface values

  const int s = subs ? subs[blockIdx.x] : (int)blockIdx.x;
  const SubDesc e = desc[s];
  if (mode == 2 && !fuse_eta && all_done(sh)) return;
  const int64_t base = e.base, i0 = e.i0;
  const TriSub<FT> T = tri_sub(e, fac, dg, cpl, cidx);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = wave / 2, w = wave % 2, tid = threadIdx.x & 127;
  const int li = lane % 16, lk = lane / 16;
  const int rrow = tid / 2, rc0 = tid % 2 * NC;  // row layout: this thread's row and columns
  const bool colok = li < NT;
  const int ns = mode >= 1 ? e.ns : 0;
  const double* P = mbf + e.mbf;
  const int LF = g == 0 ? 0 : 1, LB = 1 - LF;
  const int nstep = 2 * T.h + 1;
  // block and state of step q: forward q < h, the middle block, backward
  auto kof = [&](int q) AM_INLINE { return q <= T.h ? q : 2 * T.h - q; };
  auto active = [&](int q) AM_INLINE { return q == T.h || g == 0 || kof(q) >= T.d; };
  auto blk = [&](int q) AM_INLINE {
    const int k = kof(q);
    return q == T.h ? T.h : g == 0 ? k : T.NB - 1 - (k - T.d);
  };
  // result layout: element v of strip u
  auto drow = [&](int u, int v) AM_INLINE { return 32 * w + 16 * u + MfAcc<AT>::row(lk, v); };
  // the same of the reconstruction, FP64 for every factor type
  auto zrow = [&](int u, int v) AM_INLINE { return 32 * w + 16 * u + MfAcc<double>::row(lk, v); };
  // the subdomain's rows: uniform bases, 32-bit lane offsets; loads use a
  // clamped offset (always in bounds), the values of rows outside are zeroed
  const double* rsub = rin + (size_t)base * NT;
  double* osub = out + (size_t)base * NT;
  const double* qsub = qv + (size_t)base * NT;
  const int lic = colok ? li : NT - 1;
  auto row_off = [&](int row) AM_INLINE { return min(row, T.N - 1) * NT + lic; };

  if (fuse_eta && local_prologue<NT, 4>(mode, ns, i0, isub_list, Sinv, NL, ldS, bpart, pb, npb, init,
                                        sc, sh, reinterpret_cast<double*>(&tile[0][0]), eta_s,
                                        &stop_s))
    return;
  const int flexible = mode == 2 ? sh->flexible : 0;

  // one step ahead in registers: the row's couplings (to the block before it
  // on the way in, after it on the way out), its r, and the tile
  constexpr int KA = 5;
  AT cv[KA];
  int ci[KA];
  double prv[8];  // r by rows on the way in; on the way back w, result layout
  uint4 pre[NLD];
  AT pdg = (AT)0;
  auto fetch = [&](int q) AM_INLINE {
    const int b = blk(q);
    if (T.kc > 0) {
      const int at = (q <= T.h ? LF : LB) * T.kc * T.NP + 64 * b + rrow;
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        cv[k] = T.cpl[at + min(k, T.kc - 1) * T.NP];
        ci[k] = T.cidx[at + min(k, T.kc - 1) * T.NP];
      }
    }
    if (q <= T.h) {
      const double* src = rsub + min(64 * b + rrow, T.N - 1) * NT + rc0;
#pragma unroll
      for (int c = 0; c < NC; ++c) prv[c] = src[c];
    } else {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) prv[4 * u + v] = osub[row_off(64 * b + drow(u, v))];
    }
    const uint4* src = reinterpret_cast<const uint4*>(T.fac + (size_t)b * kTriElems);
#pragma unroll
    for (int u = 0; u < NLD; ++u) pre[u] = src[u * 128 + tid];
    pdg = T.dg[64 * b + rrow];
  };
  AT* tl = tile[g];
  auto store_tile = [&]() AM_INLINE {
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int e0 = (u * 128 + tid) * VEC;
      const int c = e0 / (64 * VEC) * VEC + 1, l = e0 % (64 * VEC) / VEC;
      FT v[VEC];
      __builtin_memcpy(v, &pre[u], 16);
#pragma unroll
      for (int t = 0; t < VEC; ++t) {
        const AT x = (AT)widen_lds(v[t]);
        tl[(c + t) * TP + l] = c + t == 32 ? x + x : x;
      }
    }
    tl[rrow] = pdg;  // (both threads of a row: the same value)
  };
  // t -= / += the couplings of the thread's row of block b times y
  auto couple = [&](int b, int list, AT sign, const AT* y, AT (&t)[NC]) AM_INLINE {
    if (T.kc == 0) return;
#pragma unroll
    for (int k = 0; k < KA; ++k) {
      const AT f = k < T.kc ? sign * cv[k] : (AT)0;
#pragma unroll
      for (int c = 0; c < NC; ++c) t[c] = fma(f, y[ci[k] * 16 + rc0 + c], t[c]);
    }
    for (int k = KA; k < T.kc; ++k) {
      const int at = (list * T.kc + k) * T.NP + 64 * b + rrow;
      const AT f = sign * T.cpl[at];
      const int i = T.cidx[at];
#pragma unroll
      for (int c = 0; c < NC; ++c) t[c] = fma(f, y[i * 16 + rc0 + c], t[c]);
    }
  };

  fetch(active(0) ? 0 : 1);  // (a group that waits at first: its second step)
  if (!fuse_eta)
    for (int t = threadIdx.x; t < ns * NT; t += 256)
      eta_s[t] = eta[(size_t)isub_list[i0 + t / NT] * NT + t % NT];
  // columns NT .. 15 of the vectors stay zero
  if (NT < 16)
    for (int t = threadIdx.x; t < 2 * 64 * 16; t += 256) {
      (&vb[0][0])[t] = (AT)0;
      (&yb[0][0])[t] = (AT)0;
    }
  __syncthreads();
  double rz = 0.0, qz = 0.0;  // column li of this lane's rows

  for (int q = 0; q < nstep; ++q) {
    const bool act = active(q);
    const int b = blk(q);
    const bool mid = q == T.h;
    const int k = kof(q);
    AT t[NC];
    double w8[8];
#pragma unroll
    for (int c = 0; c < NC; ++c) t[c] = (AT)0;
    if (mid && T.h > 0) {  // what each half takes off the middle block's r
      if (g == 0 || T.len1 > 0) couple(b, LF, (AT)-1, yb[g], t);
#pragma unroll
      for (int c = 0; c < NC; ++c) vb[g][rrow * 16 + rc0 + c] = t[c];
      __syncthreads();
#pragma unroll
      for (int c = 0; c < NC; ++c)
        t[c] = vb[0][rrow * 16 + rc0 + c] + vb[1][rrow * 16 + rc0 + c];
      __syncthreads();
    }
    if (act) {
      if (q <= T.h) {
        const bool in = 64 * b + rrow < T.N;
#pragma unroll
        for (int c = 0; c < NC; ++c) t[c] += in ? (AT)prv[c] : (AT)0;
        if (!mid && k > (g == 0 ? 0 : T.d)) couple(b, LF, (AT)-1, yb[g], t);
      } else {
        couple(b, LB, (AT)1, yb[g], t);
#pragma unroll
        for (int v = 0; v < 8; ++v) w8[v] = prv[v];
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) vb[g][rrow * 16 + rc0 + c] = t[c];
      store_tile();
    }
    __syncthreads();
    const bool post = act && (q > T.h || (mid && g == 0));  // z of this block
    // r for the dots and the first 16 slots' basis functions, in flight
    // during the product: A[row][slot 4 c + lk] of z += phat eta
    double rp[8], pa[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        rp[4 * u + v] = 0.0;
        pa[u][v] = 0.0;
      }
    if (post) {  // uniform
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (mode == 2) rp[4 * u + v] = rsub[row_off(64 * b + zrow(u, v))];
          if (4 * v < ns)
            pa[u][v] = P[min(4 * v + lk, ns - 1) * T.N + min(64 * b + 32 * w + 16 * u + li, T.N - 1)];
        }
    }
    if (q + 1 < nstep && active(q + 1) && (act || q > 0)) fetch(q + 1);
    // entry (i, j) of the tile (its pair of rows), and the product with vb
    auto entry = [&](int u, int c, int m) AM_INLINE {
      const int i = 32 * w + 16 * u + li, j = c + m * lk, o = (j - i) & 63;
      return o <= 32 ? tl[o * TP + i] : tl[(64 - o) * TP + j];
    };
    auto operand = [&](int c, int m) AM_INLINE { return vb[g][(c + m * lk) * 16 + li]; };
    V acc[2];
    if constexpr (sizeof(FT) < 8) {
      if (T.tri) {  // uniform over the workgroup: u = t + Ks t, v = D u
        if (act) {
          tri_mf_pass<BFOP, V, AT>(
              acc,
              [&](int u, int c, int m) {
                return c + m * lk < 32 * w + 16 * u + li ? entry(u, c, m) : (AT)0;
              },
              operand);
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              acc[u][v] = tl[drow(u, v)] * (vb[g][drow(u, v) * 16 + li] + acc[u][v]);
        }
        __syncthreads();
        if (act)
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) vb[g][drow(u, v) * 16 + li] = acc[u][v];
        __syncthreads();
      }
    }
    if (act) {
      if (sizeof(FT) < 8 && T.tri) {  // v + Ks^T v
        const V add[2] = {acc[0], acc[1]};
        tri_mf_pass<BFOP, V, AT>(
            acc,
            [&](int u, int c, int m) {
              return c + m * lk > 32 * w + 16 * u + li ? entry(u, c, m) : (AT)0;
            },
            operand);
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u] += add[u];
      } else if constexpr (BFOP) {  // the main diagonal in FP32, on unrounded values
        tri_mf_pass<BFOP, V, AT>(
            acc,
            [&](int u, int c, int m) {
              return c + m * lk != 32 * w + 16 * u + li ? entry(u, c, m) : (AT)0;
            },
            operand);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            acc[u][v] = fma(tl[drow(u, v)], vb[g][drow(u, v) * 16 + li], acc[u][v]);
      } else {
        tri_mf_pass<BFOP, V, AT>(acc, entry, operand);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (q > T.h) acc[u][v] = (64 * b + drow(u, v) < T.N ? (AT)w8[4 * u + v] : (AT)0) - acc[u][v];
          yb[g][drow(u, v) * 16 + li] = colok ? acc[u][v] : (AT)0;
          const int row = 64 * b + drow(u, v);
          if (q < T.h && row < T.N && colok) osub[row * NT + li] = (double)acc[u][v];
        }
      if (post) {
        tri_wave_sync();  // x of the wave's own rows, in the layout of z
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          am_mf_d4 z;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if constexpr (sizeof(AT) == 8)
              z[v] = acc[u][v];
            else
              z[v] = (double)yb[g][zrow(u, v) * 16 + li];
          }
          const int ra = min(64 * b + 32 * w + 16 * u + li, T.N - 1);
          for (int c0 = 0; c0 < ns; c0 += 16) {  // slots in chunks of 4 x 4
            if (c0 > 0)
#pragma unroll
              for (int c = 0; c < 4; ++c) pa[u][c] = P[min(c0 + 4 * c + lk, ns - 1) * T.N + ra];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              if (c0 + 4 * c >= ns) break;  // uniform
              const int qq = c0 + 4 * c + lk;
              const double ev = (qq < ns && colok) ? eta_s[qq * NT + li] : 0.0;
              z = mf4(qq < ns ? pa[u][c] : 0.0, ev, z);
            }
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = 64 * b + zrow(u, v);
            if (row < T.N && colok) {
              const int o = row * NT + li;
              osub[o] = z[v];
              rz = fma(rp[4 * u + v], z[v], rz);
              if (flexible) qz = fma(qsub[o], z[v], qz);
            }
          }
        }
      }
    }
    __syncthreads();  // y complete; tile and vector are free
  }

  if (mode != 2) return;
  // lanes l, l ^ 16, l ^ 32, l ^ 48 hold the same column
  rz = add_xor32(add_xor16(rz));
  qz = add_xor32(add_xor16(qz));
  double* dots = reinterpret_cast<double*>(&tile[0][0]);  // [4][2 NT]
  if (lane < NT) {
    dots[wave * 2 * NT + lane] = rz;
    dots[wave * 2 * NT + NT + lane] = qz;
  }
  __syncthreads();
  if (threadIdx.x < 2 * NT) {
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) a += dots[u * 2 * NT + threadIdx.x];
    partial[(size_t)(blk_off + blockIdx.x) * 2 * NT + threadIdx.x] = a;
  }
}

}  // namespace am
