// Interface kernels for gfx950: assembly of the interface matrix
//   S[n, m] = -delta_nm sum_{e in E_n} a_e + sum_{e in E_n} a_e (phat^(m)_k + phat^(m)_l)/2
// (eq. interface-problem-alg with the sign of Corollary eq. k-schur), its
// symmetrisation, explicit inverses by a tiled symmetric sweep, and the
// per-apply interface solve
// eta = S^{-1} b as a dense GEMV/GEMM (Algorithm 2).
//
// Dense tiles are 64 x 64, row-major with leading dimension ldS (a multiple
// of 64); rows/columns beyond N_Lambda hold the identity.
#include <algorithm>

#include "am_common.h"

namespace am {

// ---------------------------------------------------------------------------
// One wave per interface row n.  Every write to row n comes from lane 0 of
// that wave, in a fixed order.  The diagonal's -sum a_e is folded into the
// basis function's values, a_e (phat - 1) / 2 per side (exact differences
// where phat is near 1, instead of sums that cancel).
__global__ __launch_bounds__(256) void k_assemble_S(
    int NL, int ldS, const int64_t* __restrict__ iface_ptr, const int32_t* __restrict__ iface_ij,
    const int32_t* __restrict__ e_kloc, const int32_t* __restrict__ e_lloc,
    const double* __restrict__ e_a, const int64_t* __restrict__ sub_ptr,
    const int64_t* __restrict__ isub_ptr, const int32_t* __restrict__ isub_list,
    const int64_t* __restrict__ mbf_off, const double* __restrict__ mbf, double* S) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= NL) return;
  const int i = iface_ij[2 * n], j = iface_ij[2 * n + 1];
  const int64_t e0 = iface_ptr[n], e1 = iface_ptr[n + 1];
  double* Srow = S + (size_t)n * ldS;
  for (int side = 0; side < 2; ++side) {
    const int sd = side == 0 ? i : j;
    const int Ns = (int)(sub_ptr[sd + 1] - sub_ptr[sd]);
    const double* P = mbf + mbf_off[sd];
    const int32_t* loc = side == 0 ? e_kloc : e_lloc;
    const int64_t q0 = isub_ptr[sd];
    const int nq = (int)(isub_ptr[sd + 1] - q0);
    for (int q = 0; q < nq; ++q) {
      const int m = isub_list[q0 + q];
      double v = 0.0;
      const double one = m == n ? 1.0 : 0.0;
      for (int64_t e = e0 + lane; e < e1; e += 64)
        v = fma(e_a[e], P[(size_t)q * Ns + loc[e]] - one, v);
      v = wave_sum(v);
      if (lane == 0) Srow[m] += 0.5 * v;
    }
  }
}

// (S + S^T)/2, identity on the padding.  S couples a basis function n to those
// of its two subdomains only: wave n takes its couplings m < n, and writes
// both entries.  (Over the whole square: 2.5 ms at 128^3, NL = 11904.)
__global__ __launch_bounds__(256) void k_symmetrize(int NL, int ldS,
                                                    const int32_t* __restrict__ iface_ij,
                                                    const int64_t* __restrict__ isub_ptr,
                                                    const int32_t* __restrict__ isub_list,
                                                    double* S) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= ldS) return;
  if (n >= NL) {
    if (lane == 0) S[(size_t)n * ldS + n] = 1.0;
    return;
  }
  const int i = iface_ij[2 * n], j = iface_ij[2 * n + 1];
  for (int side = 0; side < 2; ++side) {
    const int sd = side == 0 ? i : j;
    for (int64_t t = isub_ptr[sd] + lane; t < isub_ptr[sd + 1]; t += 64) {
      const int m = isub_list[t];
      if (m >= n) continue;
      // basis functions between the same two subdomains are in both lists
      if (side == 1 && iface_ij[2 * m] == i && iface_ij[2 * m + 1] == j) continue;
      const double v = 0.5 * (S[(size_t)n * ldS + m] + S[(size_t)m * ldS + n]);
      S[(size_t)n * ldS + m] = v;
      S[(size_t)m * ldS + n] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// dense tile helpers (64 x 64, 256 threads, 4 x 4 outputs per thread)
typedef double Tile[64][65];

// A tile through registers, for 256-thread workgroups: tile_fetch issues all
// 16 loads of the thread before any is used (one memory round trip per tile
// instead of one per row of threads), tile_put stores them to LDS.
struct TileRegs {
  double v[16];
};

__device__ __forceinline__ void tile_fetch(TileRegs& R, const double* p, int ld) {
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = (threadIdx.x >> 6) + 4 * u, c = threadIdx.x & 63;
    R.v[u] = p[(size_t)r * ld + c];
  }
}

__device__ __forceinline__ void tile_put(Tile& T, const TileRegs& R, bool trans) {
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = (threadIdx.x >> 6) + 4 * u, c = threadIdx.x & 63;
    if (trans)
      T[c][r] = R.v[u];
    else
      T[r][c] = R.v[u];
  }
}

// acc += A * B for two 64 x 64 tiles on the FP64 matrix cores: wave w owns
// rows 16 w .. 16 w + 15 and keeps four 16 x 16 accumulators (columns 16 t ..);
// v_mfma_f64_16x16x4_f64 lane l holds A[l % 16][l / 16], B[l / 16][l % 16]
// and D[l / 16 + 4 v][l % 16], v < 4.
typedef double am_d4 __attribute__((ext_vector_type(4)));
struct MfAcc {
  am_d4 t[4];
};

__device__ __forceinline__ void mf_zero(MfAcc& acc) {
#pragma unroll
  for (int t = 0; t < 4; ++t) acc.t[t] = am_d4{0.0, 0.0, 0.0, 0.0};
}

// 256 threads = 4 waves
__device__ __forceinline__ void mf_mac(MfAcc& acc, const Tile& A, const Tile& B) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane % 16, lk = lane / 16;
#pragma unroll 4
  for (int ks = 0; ks < 16; ++ks) {
    const double a = A[16 * w + li][4 * ks + lk];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc.t[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[4 * ks + lk][16 * t + li], acc.t[t], 0, 0, 0);
  }
}

// calls f(row, col, value) for the thread's 16 entries of the tile
template <typename F>
__device__ __forceinline__ void mf_each(const MfAcc& acc, F&& f) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane % 16, lk = lane / 16;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) f(16 * w + lk + 4 * v, 16 * t + li, acc.t[t][v]);
}

// Explicit inverse of symmetric positive definite matrices in 64 x 64 tiles,
// by the symmetric sweep over tile pivots: with D = A_kk^{-1}, step k is
//   A_ij <- A_ij - (A_ik D) A_jk^T,   A_ik <- A_ik D,   A_kk <- -D
// for i, j != k, and after the last step the matrix is -A^{-1}.  Lower tiles
// only (i >= j), read from src and written to dst, which change places from
// step to step (no tile is read after it was overwritten); A_ik with i < k is
// tile (k, i) transposed.  The workgroup of tile (k + 1, k + 1) inverts it at
// the end of its step, beside the others' products, so a step is one launch
// and the chain one tile inverse (25 us) and two tile products a step.  (A
// tiled Cholesky, triangular inverse and L^{-T} L^{-1} took five launches and
// 115 us a step for half the products.)  blockIdx.z: matrix, at moff[z] with
// T[z] tiles a side (batch of one: moff null, T0); its row r is rowbase[z] + r
// in fail, which keeps the smallest row (-1, the largest unsigned, for none).
__global__ __launch_bounds__(256) void k_sweep_first(const double* src, const int64_t* moff,
                                                     const int32_t* T, int T0, double* Dbuf,
                                                     const int64_t* rowbase, int64_t rowbase0,
                                                     int32_t* fail) {
  const int z = blockIdx.x, ld = 64 * (moff ? T[z] : T0), tid = threadIdx.x;
  const double* A = src + (moff ? moff[z] : 0);
  const int64_t rb = rowbase ? rowbase[z] : rowbase0;
  __shared__ double prow[2][64];
  const int i0 = 4 * (tid / 16), j0 = 4 * (tid % 16);
  double x[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) x[a][c] = A[(size_t)(i0 + a) * ld + j0 + c];
  sweep_inverse_64(x, prow, tid, true, [&](int k) {
    atomicMin((unsigned*)fail, (unsigned)(rb + k));
  });
  double* D = Dbuf + (size_t)z * 2 * 4096;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) D[(i0 + a) * 64 + j0 + c] = -x[a][c];
}

__global__ __launch_bounds__(256) void k_sweep_step(const double* __restrict__ src,
                                                    double* __restrict__ dst, const int64_t* moff,
                                                    const int32_t* Tz, int T0, int k, double* Dbuf,
                                                    const int64_t* rowbase, int64_t rowbase0,
                                                    int32_t* fail) {
  const int z = blockIdx.z, T = moff ? Tz[z] : T0, ld = 64 * T;
  const int j = blockIdx.x, i = blockIdx.y;
  if (k >= T || i >= T || j > i) return;
  const double* A = src + (moff ? moff[z] : 0);
  double* B = dst + (moff ? moff[z] : 0);
  const double* D = Dbuf + ((size_t)z * 2 + (k & 1)) * 4096;
  double* out = B + (size_t)i * 64 * ld + (size_t)j * 64;
  if (i == k && j == k) {
    for (int t = threadIdx.x; t < 4096; t += 256) out[(size_t)(t >> 6) * ld + (t & 63)] = -D[t];
    return;
  }
  __shared__ Tile As;
  __shared__ Tile Bs;
  TileRegs ra, rb;
  MfAcc acc;
  mf_zero(acc);
  // tile (r, k) of the symmetric matrix: stored at (k, r), transposed, above
  auto fetch = [&](TileRegs& R, int r) {
    if (r > k)
      tile_fetch(R, A + (size_t)r * 64 * ld + (size_t)k * 64, ld);
    else
      tile_fetch(R, A + (size_t)k * 64 * ld + (size_t)r * 64, ld);
  };
  if (i == k) {  // row k: D A_kj
    tile_fetch(ra, D, 64);
    tile_fetch(rb, A + (size_t)k * 64 * ld + (size_t)j * 64, ld);
    tile_put(As, ra, false);
    tile_put(Bs, rb, false);
    __syncthreads();
    mf_mac(acc, As, Bs);
    mf_each(acc, [&](int r, int c, double v) { out[(size_t)r * ld + c] = v; });
    return;
  }
  fetch(ra, i);
  tile_fetch(rb, D, 64);
  tile_put(As, ra, i < k);
  tile_put(Bs, rb, false);
  __syncthreads();
  if (j != k) fetch(rb, j);  // in flight during the first product
  mf_mac(acc, As, Bs);       // A_ik D
  if (j == k) {
    mf_each(acc, [&](int r, int c, double v) { out[(size_t)r * ld + c] = v; });
    return;
  }
  __syncthreads();
  mf_each(acc, [&](int r, int c, double v) { As[r][c] = v; });
  tile_put(Bs, rb, j > k);  // A_jk^T
  tile_fetch(ra, A + (size_t)i * 64 * ld + (size_t)j * 64, ld);
  __syncthreads();
  mf_zero(acc);
  mf_mac(acc, As, Bs);
  __syncthreads();
  mf_each(acc, [&](int r, int c, double v) { As[r][c] = v; });
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = (threadIdx.x >> 6) + 4 * u, c = threadIdx.x & 63;
    const double v = ra.v[u] - As[r][c];
    out[(size_t)r * ld + c] = v;
    Bs[r][c] = v;
  }
  if (i != k + 1 || j != k + 1) return;
  // the next pivot
  __syncthreads();
  const int tid = threadIdx.x, i0 = 4 * (tid / 16), j0 = 4 * (tid % 16);
  double x[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // the lower half defines both halves
      const int r = i0 + a, q = j0 + c;
      x[a][c] = r >= q ? Bs[r][q] : Bs[q][r];
    }
  const int64_t base = (rowbase ? rowbase[z] : rowbase0) + 64 * (k + 1);
  __syncthreads();
  sweep_inverse_64(x, reinterpret_cast<double(*)[64]>(&As[0][0]), tid, true, [&](int q) {
    atomicMin((unsigned*)fail, (unsigned)(base + q));
  });
  double* Dn = Dbuf + ((size_t)z * 2 + ((k + 1) & 1)) * 4096;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) Dn[(i0 + a) * 64 + j0 + c] = -x[a][c];
}

// out = the symmetric inverse from a finished sweep (sign changed, the lower
// half mirrored): nrow x ldo, row-major, columns from ncol on zero.
// Workgroups over 64 x 64 tiles (blockIdx.x, y); blockIdx.z: matrix.
__global__ __launch_bounds__(256) void k_sweep_out(const double* m0, const double* m1,
                                                   const int64_t* moff, const int32_t* Tz, int T0,
                                                   double* out, const int64_t* ooff,
                                                   const int64_t* nrow_off, int nrow0, int ldo0) {
  const int z = blockIdx.z, T = moff ? Tz[z] : T0, ld = 64 * T;
  if ((int)blockIdx.x >= T || (int)blockIdx.y >= T) return;
  const double* M = (T & 1 ? m1 : m0) + (moff ? moff[z] : 0);
  const int nr = nrow_off ? (int)(nrow_off[z + 1] - nrow_off[z]) : nrow0;
  const int ldo = nrow_off ? nr : ldo0;
  double* o = out + (ooff ? ooff[z] : 0);
  __shared__ Tile S;
  const int bi = max((int)blockIdx.x, (int)blockIdx.y), bj = min((int)blockIdx.x, (int)blockIdx.y);
  TileRegs r;
  tile_fetch(r, M + (size_t)bi * 64 * ld + (size_t)bj * 64, ld);
  tile_put(S, r, false);
  __syncthreads();
  const bool up = blockIdx.x > blockIdx.y;  // column tile beyond the row tile
  for (int t = threadIdx.x; t < 4096; t += 256) {
    const int a = t >> 6, c = t & 63;
    const int gr = blockIdx.y * 64 + a, gc = blockIdx.x * 64 + c;
    if (gr >= nr || gc >= ldo) continue;
    const double v = up || (bi == bj && c > a) ? S[c][a] : S[a][c];
    o[(size_t)gr * ldo + gc] = gc < nr ? -v : 0.0;
  }
}

// One correction step of the explicit inverse where it is small (applied
// inside the local kernel): X <- X + X (I - S X).  S has the few entries of
// the basis functions that share a subdomain, so the residual is sparse rows
// times X, accumulated in twice the working precision; the product with X is
// one more dense tile product.  The factorization alone leaves an error of
// the order of cond(S) eps in z (1e-12 on a 100-cell chain, cond(S) 1.5e5;
// 5e-14 after the step).  Wave: row n, 64 columns.
__global__ __launch_bounds__(256) void k_sinv_residual(
    int NL, int ldS, const int32_t* __restrict__ iface_ij, const int64_t* __restrict__ isub_ptr,
    const int32_t* __restrict__ isub_list, const double* __restrict__ S,
    const double* __restrict__ X, double* __restrict__ R) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.y * 4 + (threadIdx.x >> 6), c = blockIdx.x * 64 + lane;
  if (n >= ldS) return;
  double hi = (n < NL && n == c) ? 1.0 : 0.0, lo = 0.0;
  if (n < NL) {
    const int i = iface_ij[2 * n], j = iface_ij[2 * n + 1];
    for (int side = 0; side < 2; ++side) {
      const int sd = side == 0 ? i : j;
      for (int64_t t = isub_ptr[sd]; t < isub_ptr[sd + 1]; ++t) {
        const int m = isub_list[t];
        // basis functions between the same two subdomains are in both lists
        if (side == 1 && iface_ij[2 * m] == i && iface_ij[2 * m + 1] == j) continue;
        const double a = S[(size_t)n * ldS + m], x = X[(size_t)m * ldS + c];
        const double pr = a * x, u = hi - pr, w = u - hi;
        lo += (hi - (u - w)) - (pr + w);
        lo -= fma(a, x, -pr);
        hi = u;
      }
    }
  }
  R[(size_t)n * ldS + c] = hi + lo;
}

// out = X + X R (lower tile half, mirrored)
__global__ __launch_bounds__(256) void k_sinv_correct(const double* X, const double* R,
                                                      double* __restrict__ out, int ld, int T) {
  const int j = blockIdx.x, i = blockIdx.y;
  if (j > i) return;
  __shared__ Tile As;
  __shared__ Tile Bs;
  MfAcc acc;
  mf_zero(acc);
  TileRegs ra, rb;
  tile_fetch(ra, X + (size_t)i * 64 * ld, ld);
  tile_fetch(rb, R + (size_t)j * 64, ld);
  for (int k = 0; k < T; ++k) {
    tile_put(As, ra, false);
    tile_put(Bs, rb, false);
    __syncthreads();
    if (k + 1 < T) {
      tile_fetch(ra, X + (size_t)i * 64 * ld + (size_t)(k + 1) * 64, ld);
      tile_fetch(rb, R + (size_t)(k + 1) * 64 * ld + (size_t)j * 64, ld);
    }
    mf_mac(acc, As, Bs);
    __syncthreads();
  }
  mf_each(acc, [&](int r, int c, double v) {
    const size_t gr = (size_t)i * 64 + r, gc = (size_t)j * 64 + c;
    if (gr < gc) return;
    const double x = X[gr * ld + gc] + v;
    out[gr * ld + gc] = x;
    out[gc * ld + gr] = x;
  });
}

// ---------------------------------------------------------------------------
// eta = S^{-1} b with a small dense S^{-1} (at most 64 MB, resident in the
// caches), in one launch: a workgroup forms RW rows, its four waves a quarter
// of the columns each, with a round's loads all issued before the first is
// used (and before the stop flag is looked at).  In a solve one more workgroup
// takes the stop decision.  Bound by the round trips: 64^3 (NL = 1344) one
// round, 5.5 us (two rows a wave over all columns, four rounds: 5.8 us); the
// same rows formed in the local kernel, by its two waves per subdomain, held
// every subdomain up for 5.6 us, and the four columns of a bisection part's 23
// rows for over 100.
template <int NR>
constexpr int eta_rows() { return NR == 1 ? 8 : 4; }
template <int NR>
__global__ __launch_bounds__(256) void k_eta_dense(int NL, int ldS, const double* __restrict__ Sinv,
                                                   const double* __restrict__ bpart,
                                                   double* __restrict__ eta, int pcg, int init,
                                                   const double* __restrict__ pb, int npb,
                                                   PcgScalars* sc, PcgShared* sh) {
  constexpr int RW = eta_rows<NR>();
  constexpr int UM = NR == 1 ? 6 : NR <= 4 ? 2 : 1;
  __shared__ double lds[4 * RW * NR];
  // a solve that stopped earlier (this launch's last workgroup may be writing
  // the flag: threads that read it late leave with the same outcome, as a
  // stopped solve reads no eta)
  const int stopped = pcg && !init ? (int)all_done(sh) : 0;
  if (pcg && blockIdx.x == gridDim.x - 1) {
    if (!stopped) stop_test_wg<NR>(pb, npb, init, sc, sh, lds);
    return;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = blockIdx.x * RW;
  const int per = (NL + 3) / 4, me = min(NL, (w + 1) * per);
  const double* row[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) row[r] = Sinv + (size_t)min(r0 + r, NL - 1) * ldS;
  double a[RW * NR];
#pragma unroll
  for (int r = 0; r < RW * NR; ++r) a[r] = 0.0;
  for (int m0 = w * per + lane; m0 < me + lane; m0 += 64 * UM) {
    double bm[UM][2][NR], sv[UM][RW];
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const int m = min(m0 + 64 * u, NL - 1);
#pragma unroll
      for (int r = 0; r < RW; ++r) sv[u][r] = row[r][m];
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        bm[u][0][k] = bpart[(size_t)(2 * m) * NR + k];
        bm[u][1][k] = bpart[(size_t)(2 * m + 1) * NR + k];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (stopped) break;
#pragma unroll
    for (int u = 0; u < UM; ++u) {
      const bool ok = m0 + 64 * u < me;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const double b = ok ? bm[u][0][k] + bm[u][1][k] : 0.0;
#pragma unroll
        for (int r = 0; r < RW; ++r) a[r * NR + k] = fma(sv[u][r], b, a[r * NR + k]);
      }
    }
  }
  const double t = block_sum_spread<RW * NR>(a, lds);
  const int r = r0 + (int)threadIdx.x / NR;
  if ((int)threadIdx.x < RW * NR && r < NL && !stopped) eta[(size_t)r * NR + threadIdx.x % NR] = t;
}

// ---------------------------------------------------------------------------
// eta = S^{-1} b, b_m = bpart[2m] + bpart[2m+1], as a sum of outer products
// over the rows of the symmetric S^{-1}: eta[r] = sum_m S^{-1}[m][r] b_m.
// Wave (rb, p) takes the 64 entries r = 64 rb + lane and the rows m of part
// p: each row is one coalesced 64-value load and NR FMAs with b_m, a uniform
// (scalar) load, so S^{-1} is read exactly once per product.  The loads are
// non-temporal: S^{-1} is streamed once per product and would otherwise evict
// the vectors and the SpMV arrays from L2 and the Infinity Cache.  The part
// sums go to ypart[p][r][k]; k_iface_reduce adds them in part order.
template <int NR>
__global__ __launch_bounds__(256) void k_iface_op(int NL, int ldS, const double* __restrict__ Sinv,
                                                  const double* __restrict__ bpart,
                                                  double* __restrict__ ypart, int P, int pcg,
                                                  int init, const PcgShared* sh) {
  if (pcg && !init && all_done(sh)) return;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int nrb = (NL + 63) / 64;
  if (wv >= nrb * P) return;
  const int rb = wv % nrb, p = wv / nrb;
  const int per = (NL + P - 1) / P;
  const int mb = p * per, me = min(NL, mb + per);
  const int r = rb * 64 + lane;  // < ldS (padded to 64)
  const double* col = Sinv + r;
  double acc[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) acc[k] = 0.0;
#pragma unroll 8
  for (int m = mb; m < me; ++m) {
    const double sv = __builtin_nontemporal_load(col + (size_t)m * ldS);
#pragma unroll
    for (int k = 0; k < NR; ++k)
      acc[k] = fma(sv, bpart[(size_t)(2 * m) * NR + k] + bpart[(size_t)(2 * m + 1) * NR + k], acc[k]);
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) ypart[((size_t)p * ldS + r) * NR + k] = acc[k];
}

// The same product for 4 to 16 right-hand sides on the FP64 matrix cores:
// wave (rb, p) accumulates the 64 x NR block ypart[p][64 rb ..][.] as four
// 16 x 16 tiles, D += A B with A = S^{-1}[m0 .. m0+3][16 rows] (symmetric,
// so the rows m of S^{-1} stand for its columns) and B = b[m0 .. m0+3][NR
// columns, zero-padded to 16].  v_mfma_f64_16x16x4_f64 lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and D[l / 16 + 4 v][l % 16], v < 4.
// S^{-1} is read once (four coalesced 128-byte rows per load, non-temporal
// as in k_iface_op); the FMAs run on the matrix cores, so 16 right-hand sides
// cost no more issue slots than 4.
template <int NR>
__global__ __launch_bounds__(256) void k_iface_op_mfma(int NL, int ldS, const double* __restrict__ Sinv,
                                                       const double* __restrict__ bpart,
                                                       double* __restrict__ ypart, int P, int pcg,
                                                       int init, const PcgShared* sh) {
  static_assert(NR >= 1 && NR <= 16, "one 16-column tile");
  if (pcg && !init && all_done(sh)) return;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int nrb = (NL + 63) / 64;
  if (wv >= nrb * P) return;
  const int rb = wv % nrb, p = wv / nrb;
  const int per = (NL + P - 1) / P;
  const int mb = p * per, me = min(NL, mb + per);
  const int li = lane % 16, lk = lane / 16;
  const double* col = Sinv + 64 * rb + li;  // column 64 rb + 16 sub + li of row m
  am_d4 acc[4];
#pragma unroll
  for (int sub = 0; sub < 4; ++sub) acc[sub] = am_d4{0.0, 0.0, 0.0, 0.0};
  // U chunks of 4 rows per step, every load of the step issued before its
  // products.  U = 2 leaves room for five waves per SIMD: the loads wait on
  // memory far longer than the products take, and more waves hide more of
  // it than more loads per wave (at 16 RHS on 14,616 rows: 396 us against
  // 435 with U = 4 and 419 with U = 1)
  constexpr int U = 2;
  for (int m0 = mb; m0 < me; m0 += 4 * U) {
    double av[U][4], bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + 4 * u + lk;
      const bool ok = m < me;
      bv[u] = (ok && li < NR)
                  ? bpart[(size_t)(2 * m) * NR + li] + bpart[(size_t)(2 * m + 1) * NR + li]
                  : 0.0;
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) av[u][sub] = ok ? __builtin_nontemporal_load(col + (size_t)m * ldS + 16 * sub) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
        acc[sub] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u][sub], bv[u], acc[sub], 0, 0, 0);
  }
  if (li < NR)
#pragma unroll
    for (int sub = 0; sub < 4; ++sub)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 64 * rb + 16 * sub + lk + 4 * v;
        ypart[((size_t)p * ldS + r) * NR + li] = acc[sub][v];
      }
}

// eta[r][k] = sum_p ypart[p][r][k] in part order.  In PCG mode workgroup 0
// first folds the ||r||^2 partials of the update launch and applies the stop
// test ||r|| <= tol ||b|| (the next launches read its outcome).
template <int NR>
__global__ __launch_bounds__(256) void k_iface_reduce(int NL, int ldS, const double* __restrict__ ypart,
                                                      int P, double* __restrict__ eta, int pcg,
                                                      int init, const double* __restrict__ pb,
                                                      int npb, PcgScalars* sc, PcgShared* sh) {
  __shared__ double lds[4 * NR];
  if (pcg && !init && all_done(sh)) return;
  if (pcg && blockIdx.x == 0) {
    const int nrhs = sh->nrhs, maxit = sh->maxit;
    double rr[NR];
    reduce_partials<NR>(rr, pb, (unsigned)npb, lds);
    int alld = 1;
    for (int k = 0; k < nrhs; ++k) {
      const PcgScalars S = sc[k];
      int done = S.done, conv = S.conv, status = S.status;
      double bb = S.bb;
      if (!done) {
        if (init) {
          bb = rr[k];
          if (bb == 0.0) done = conv = 1;
        } else if (rr[k] <= S.tol2 * S.bb) {
          done = conv = 1;
        } else if (S.it >= maxit) {
          done = 1;
          status = AM_ERR_NO_CONVERGENCE;
        }
      }
      alld &= done;
      if (threadIdx.x == 0) {
        sc[k].rr = rr[k];
        sc[k].bb = bb;
        sc[k].done = done;
        sc[k].conv = conv;
        sc[k].status = status;
      }
    }
    if (threadIdx.x == 0) sh->all_done = alld;
  }
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)NL * NR) return;
  const int64_t r = t / NR;
  const int k = (int)(t % NR);
  double e = 0.0;
  for (int p = 0; p < P; ++p) e += ypart[((size_t)p * ldS + r) * NR + k];
  eta[r * NR + k] = e;
}

// ---------------------------------------------------------------------------
hipError_t launch_assemble_S(DeviceState& d, hipStream_t st) {
  if (d.NL == 0) return hipSuccess;
  hipError_t e = hipMemsetAsync(d.S, 0, sizeof(double) * (size_t)d.ldS * d.ldS, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_assemble_S, dim3((unsigned)((d.NL + 3) / 4)), dim3(256), 0, st, (int)d.NL,
                     d.ldS, d.iface_ptr, d.iface_ij, d.e_kloc, d.e_lloc, d.e_a, d.sub_ptr,
                     d.isub_ptr, d.isub_list, d.mbf_off, d.mbf, d.S);
  hipLaunchKernelGGL(k_symmetrize, dim3((unsigned)((d.ldS + 3) / 4)), dim3(256), 0, st,
                     (int)d.NL, d.ldS, d.iface_ij, d.isub_ptr, d.isub_list, d.S);
  return hipGetLastError();
}

hipError_t sweep_inverse(double* m0, double* m1, const int64_t* moff, const int32_t* T, int nmat,
                         int Tmax, double* Dbuf, const int64_t* rowbase, int64_t rowbase0,
                         int32_t* fail, hipStream_t st) {
  if (nmat < 1 || Tmax < 1) return hipSuccess;
  hipLaunchKernelGGL(k_sweep_first, dim3(nmat), dim3(256), 0, st, m0, moff, T, Tmax, Dbuf, rowbase,
                     rowbase0, fail);
  for (int k = 0; k < Tmax; ++k)
    hipLaunchKernelGGL(k_sweep_step, dim3(Tmax, Tmax, nmat), dim3(256), 0, st, k & 1 ? m1 : m0,
                       k & 1 ? m0 : m1, moff, T, Tmax, k, Dbuf, rowbase, rowbase0, fail);
  return hipGetLastError();
}

hipError_t sweep_output(const double* m0, const double* m1, const int64_t* moff, const int32_t* T,
                        int nmat, int Tmax, double* out, const int64_t* ooff,
                        const int64_t* nrow_off, int nrow0, int ldo0, hipStream_t st) {
  if (nmat < 1 || Tmax < 1) return hipSuccess;
  hipLaunchKernelGGL(k_sweep_out, dim3(Tmax, Tmax, nmat), dim3(256), 0, st, m0, m1, moff, T, Tmax,
                     out, ooff, nrow_off, nrow0, ldo0);
  return hipGetLastError();
}

hipError_t dense_inverse(DeviceState& d, const double* S, double* m0, double* m1, double* Dbuf,
                         double* out, hipStream_t st) {
  const int ld = d.ldS, T = ld / 64;
  if (T == 0) return hipSuccess;
  const size_t bytes = sizeof(double) * (size_t)ld * ld;
  hipError_t e = hipMemcpyAsync(m0, S, bytes, hipMemcpyDeviceToDevice, st);
  if (e == hipSuccess)
    e = sweep_inverse(m0, m1, nullptr, nullptr, 1, T, Dbuf, nullptr, 0, d.fail + 2, st);
  if (e == hipSuccess)
    e = sweep_output(m0, m1, nullptr, nullptr, 1, T, out, nullptr, nullptr, ld, ld, st);
  if (e != hipSuccess || !d.fuse_eta) return e;
  hipLaunchKernelGGL(k_sinv_residual, dim3(T, ld / 4), dim3(256), 0, st, (int)d.NL, ld, d.iface_ij,
                     d.isub_ptr, d.isub_list, d.S, out, m0);
  hipLaunchKernelGGL(k_sinv_correct, dim3(T, T), dim3(256), 0, st, out, m0, m1, ld, T);
  e = hipMemcpyAsync(out, m1, bytes, hipMemcpyDeviceToDevice, st);
  return e != hipSuccess ? e : hipGetLastError();
}

template <int NR>
static void gemv_t(DeviceState& d, hipStream_t st, int pcg, int init) {
  const int nrb = (int)((d.NL + 63) / 64);
  const unsigned nw = (unsigned)std::max(1, nrb * d.op_parts);
  if constexpr (NR >= 4)
    am_launch(d, true, false, k_iface_op_mfma<NR>, dim3((nw + 3) / 4), dim3(256), st, (int)d.NL,
              d.ldS, d.Sinv, d.bpart, d.ypart, d.op_parts, pcg, init, d.shared);
  else
    am_launch(d, true, false, k_iface_op<NR>, dim3((nw + 3) / 4), dim3(256), st, (int)d.NL, d.ldS,
              d.Sinv, d.bpart, d.ypart, d.op_parts, pcg, init, d.shared);
  const unsigned nb = (unsigned)std::max<int64_t>(1, (d.NL * NR + 255) / 256);
  am_launch(d, false, true, k_iface_reduce<NR>, dim3(nb), dim3(256), st, (int)d.NL, d.ldS, d.ypart,
            d.op_parts, d.eta, pcg, init, d.red.pb, d.m, d.sc, d.shared);
}

template <int NR>
static void eta_dense_t(DeviceState& d, hipStream_t st, int pcg, int init) {
  const unsigned nb = (unsigned)((d.NL + eta_rows<NR>() - 1) / eta_rows<NR>()) + (pcg ? 1 : 0);
  am_launch(d, true, true, k_eta_dense<NR>, dim3(nb), dim3(256), st, (int)d.NL, d.ldS, d.Sinv,
            d.bpart, d.eta, pcg, init, d.red.pb, d.m, d.sc, d.shared);
}

hipError_t launch_iface_gemv(DeviceState& d, int nr, int pcg, int init, hipStream_t st) {
  if (d.fuse_eta) {
    switch (nr) {
      case 1: eta_dense_t<1>(d, st, pcg, init); break;
      case 2: eta_dense_t<2>(d, st, pcg, init); break;
      case 4: eta_dense_t<4>(d, st, pcg, init); break;
      case 8: eta_dense_t<8>(d, st, pcg, init); break;
      case 16: eta_dense_t<16>(d, st, pcg, init); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  if (d.NL == 0 && !pcg) return hipSuccess;
  if (d.nd.on) return launch_nd_solve(d, nr, pcg, init, st);
  if (d.ix.on) return launch_ix_solve(d, nr, pcg, init, st);
  // the part sums exist only on handles whose interface solve is not fused
  // into the local kernel (with no interface, the launches only take the
  // stop decision and touch no part sums)
  if (d.NL > 0 && (d.ypart == nullptr || d.op_parts < 1 || nr > d.max_nrhs))
    return hipErrorInvalidValue;
  switch (nr) {
    case 1: gemv_t<1>(d, st, pcg, init); break;
    case 2: gemv_t<2>(d, st, pcg, init); break;
    case 4: gemv_t<4>(d, st, pcg, init); break;
    case 8: gemv_t<8>(d, st, pcg, init); break;
    case 16: gemv_t<16>(d, st, pcg, init); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace am
