// Nested-dissection interface solve eta = S^{-1} b for gfx950 (the interface
// solve of Algorithm 2; S is SPD, Corollary cor-schur-eta).
//
// The host layout (iface_nd.cpp) orders the basis functions so that the
// first rows form mutually uncoupled diagonal blocks B of S and the last ones
// are the separators T above them.  Block elimination then gives
//   y_B   = S_BB^{-1} b_B                          k_nd_blocks, pass 0
//   eta_T = C^{-1} (b_T - S_TB y_B)                 k_nd_top (row parts), k_nd_fold
//   eta_B = S_BB^{-1} (b_B - S_BT eta_T)            k_nd_blocks, pass 1
// where C = S_TT - S_TB S_BB^{-1} S_BT.  Every S_bb^{-1} and C^{-1} is held
// explicitly (dense, exactly symmetric), so each step is a set of matrix
// products with no dependent chain inside a launch.  Set-up inverts the blocks
// together, forms C from the sparse couplings and inverts it, with the tiled
// sweep of kernels_iface.hip on matrices padded to 64-row tiles.
//
// Right-hand sides b = bpart[2p] + bpart[2p+1] at ND position p (the slots are
// numbered by it in this form, see DeviceState::bdst); eta is written in the original basis-function order, [n][NR].
#include <algorithm>

#include "am_common.h"
#include "iface_products.h"

namespace am {

// rows of a block (and of a part of the top rows) whose right-hand side a
// workgroup keeps in LDS: at most 64 KB
template <int NR> struct NdCap {
  static constexpr int rows = (7936 / NR) < 4096 ? 7936 / NR : 4096;
};

int64_t nd_max_rows(int nr_max) {
  switch (nr_max) {
    case 1: return NdCap<1>::rows;
    case 2: return NdCap<2>::rows;
    case 4: return NdCap<4>::rows;
    case 8: return NdCap<8>::rows;
    default: return NdCap<16>::rows;
  }
}

// Workgroup (block b, rows row0 .. row0 + 63 of it): the block's right-hand
// side goes to LDS, then out = Sbb^{-1} rhs for those 64 rows, the eight
// waves taking an eighth of the block's columns each (nd_wave_product); their
// partial sums are added in wave order.  Pass 0 writes y_B (ND order), pass 1
// subtracts S_BT eta_T from the right-hand side first (or, with from_y1,
// takes that right-hand side from y1, where k_nd_rb formed it) and writes
// eta_B in the original order.  Dynamic LDS: max(rows of the largest block,
// 512) NR doubles.
template <int NR> struct NdWaves { static constexpr int v = 8; };

// x - sum_{q in [qb, qe)} val[q] vec[pos[q] NR + k], the terms subtracted in
// q order; the positions, values and gathers of four couplings are issued
// before their products, so a row's chain waits once per four couplings.
template <int NR>
__device__ __forceinline__ double nd_sub_couplings(double x, int64_t qb, int64_t qe,
                                                   const int32_t* __restrict__ pos,
                                                   const double* __restrict__ val,
                                                   const double* __restrict__ vec, int k) {
  int64_t q = qb;
  for (; q + 4 <= qe; q += 4) {
    int32_t c[4];
    double a[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      c[u] = pos[q + u];
      a[u] = val[q + u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = vec[(size_t)c[u] * NR + k];
#pragma unroll
    for (int u = 0; u < 4; ++u) x = fma(-a[u], y[u], x);
  }
  for (; q < qe; ++q) x = fma(-val[q], vec[(size_t)pos[q] * NR + k], x);
  return x;
}

template <int NR>
__global__ __launch_bounds__(64 * NdWaves<NR>::v) void k_nd_blocks(
    int pass, int from_y1, int nwg, const NdWg* __restrict__ wg, const double* __restrict__ binv,
    const int32_t* __restrict__ ord, const double* __restrict__ bpart,
    const int64_t* __restrict__ b_ptr, const int32_t* __restrict__ b_top,
    const double* __restrict__ b_val, const double* __restrict__ eta2, double* __restrict__ y1,
    double* __restrict__ eta, int pcg, int init, const double* __restrict__ opb, int npb,
    PcgScalars* sc, PcgShared* sh) {
  constexpr int NW = NdWaves<NR>::v;
  extern __shared__ double rhs[];
  __shared__ int skip;
  __shared__ double red[NW * NR];
  const NdWg W = (int)blockIdx.x < nwg ? wg[blockIdx.x] : NdWg{};  // with the stop flag
  if (threadIdx.x == 0) skip = (pcg && !init && all_done(sh)) ? 1 : 0;
  __syncthreads();
  if (skip) return;  // uniform: one read for the whole workgroup
  if ((int)blockIdx.x == nwg) {
    // the extra workgroup of the first launch of the solve: the PCG stop
    // decision, beside the products (the later launches read its outcome;
    // the other workgroups of this launch may see it or not, which changes
    // nothing but work that the stop makes unneeded)
    stop_test_wg<NR>(opb, npb, init, sc, sh, red);
    return;
  }
  const int64_t o = W.o;
  const int s = W.s, row0 = W.row0;
  const int w = threadIdx.x >> 6;
  const int per = (s + NW - 1) / NW;
  const int jb = min(s, w * per), je = min(s, jb + per);
  // the first rows of the inverse, on their way while the right-hand side is
  // formed
  NdRows<NR, false> f;
  f.load(binv + W.inv, s, row0, s, jb, je);
  if (from_y1) {  // pass 1: b_B - S_BT eta_T, formed by k_nd_rb
    for (int t = threadIdx.x; t < s * NR; t += blockDim.x) rhs[t] = y1[(size_t)o * NR + t];
  } else {
    for (int t = threadIdx.x; t < s * NR; t += blockDim.x) {
      const int j = t / NR, k = t % NR;
      double v = bpart[(size_t)(2 * (o + j)) * NR + k] + bpart[(size_t)(2 * (o + j) + 1) * NR + k];
      if (pass)
        v = nd_sub_couplings<NR>(v, b_ptr[o + j], b_ptr[o + j + 1], b_top, b_val, eta2, k);
      rhs[t] = v;
    }
  }
  __syncthreads();
  nd_d4 acc[4];
  nd_wave_product<NR, false>(binv + W.inv, s, row0, s, jb, je, rhs, 0, f, acc);
  __syncthreads();  // every wave is done with rhs
  double* part = rhs;  // [NW][64][NR]
  nd_wave_each<NR>(acc, [&](int l, int k, double v) { part[(w * 64 + l) * NR + k] = v; });
  __syncthreads();
  for (int t = threadIdx.x; t < 64 * NR; t += blockDim.x) {
    const int l = t / NR, k = t % NR;
    const int r = row0 + l;
    if (r >= s) continue;
    double v = part[l * NR + k];
#pragma unroll
    for (int u = 1; u < NW; ++u) v += part[(64 * u + l) * NR + k];
    if (pass == 0)
      y1[(size_t)(o + r) * NR + k] = v;
    else
      eta[(size_t)ord[o + r] * NR + k] = v;
  }
}

// Row parts of eta_T = C^{-1} r_T, r_T = b_T - S_TB y_B.  Workgroup
// (part p, group g): the part's rows j of r_T are formed in LDS (each from its
// couplings to block rows), then wave w of the group takes the 64 outputs
// 64 (4 g + w) .. and sums over the part's j (nd_wave_product; C^{-1} is
// streamed once, non-temporal).  The part sums go to ypart[p][row][k].
// Dynamic LDS: rows per part times NR doubles.
template <int NR, bool PRE>
__global__ __launch_bounds__(256) void k_nd_top(
    int R, int ldC, const double* __restrict__ cinv, int P, int per, int nrb,
    const double* __restrict__ btop, const int64_t* __restrict__ t_ptr,
    const int32_t* __restrict__ t_pos, const double* __restrict__ t_val,
    const double* __restrict__ y1, const double* __restrict__ eta2, double* __restrict__ ypart,
    int pcg, int init,
    const PcgShared* sh) {
  extern __shared__ double r2[];
  __shared__ int skip;
  if (threadIdx.x == 0) skip = (pcg && !init && all_done(sh)) ? 1 : 0;
  __syncthreads();
  if (skip) return;
  const int p = blockIdx.x % P, g = blockIdx.x / P;
  const int jb = min(R, p * per), je = min(R, jb + per);
  const int w = threadIdx.x >> 6;
  const int rb = 4 * g + w;
  NdRows<NR, true> f;  // the first rows of C^{-1}, as in k_nd_blocks
  f.load(cinv, ldC, 64 * min(rb, nrb - 1), ldC, jb, je);
  const double* v = r2;  // the part's rows of r_T
  int vbase = jb;
  if (PRE) {  // formed by k_nd_rt (held in eta2 until k_nd_fold)
    v = eta2;
    vbase = 0;
  } else {
    for (int t = threadIdx.x; t < (je - jb) * NR; t += blockDim.x) {
      const int j = jb + t / NR, k = t % NR;
      double x = btop[(size_t)(2 * j) * NR + k] + btop[(size_t)(2 * j + 1) * NR + k];
      r2[t] = nd_sub_couplings<NR>(x, t_ptr[j], t_ptr[j + 1], t_pos, t_val, y1, k);
    }
    __syncthreads();
  }
  if (rb >= nrb) return;
  nd_d4 acc[4];
  nd_wave_product<NR, true>(cinv, ldC, 64 * rb, ldC, jb, je, v, vbase, f, acc);
  double* out = ypart + (size_t)p * ldC * NR;
  nd_wave_each<NR>(acc, [&](int l, int k, double v) { out[(size_t)(64 * rb + l) * NR + k] = v; });
}

// eta_T = sum of the part sums, to eta2 (ND order, for pass 1) and to eta
// (original order).  Eight neighbouring lanes share an output: lane u sums
// the parts u, u + 8, ... in order (their loads all in flight), then the
// eight lane sums are added pairwise by shuffles (every lane ends with the
// same bits, as a + b = b + a exactly).  The order is fixed, so the result
// is the same on every run.
constexpr int kNdFoldLanes = 8;
template <int NR>
__global__ __launch_bounds__(256) void k_nd_fold(int R, int ldC, int P,
                                                 const double* __restrict__ ypart,
                                                 const int32_t* __restrict__ ord_top,
                                                 double* __restrict__ eta2, double* __restrict__ eta,
                                                 int pcg, int init, const PcgShared* sh) {
  if (pcg && !init && all_done(sh)) return;
  const int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kNdFoldLanes;
  const int u = threadIdx.x % kNdFoldLanes;
  const bool ok = t < (int64_t)R * NR;  // the lanes of an output agree
  const int64_t tc = ok ? t : 0;
  const int64_t r = tc / NR;
  const int k = (int)(tc % NR);
  double v = 0.0;
#pragma unroll 8
  for (int p = u; p < P; p += kNdFoldLanes) v += ypart[((size_t)p * ldC + r) * NR + k];
  static_assert(kNdFoldLanes == 8, "three steps");
  v = add_mirror(add_xor2(add_xor1(v)));
  if (ok && u == 0) {
    eta2[r * NR + k] = v;
    eta[(size_t)ord_top[r] * NR + k] = v;
  }
}

// r_T = b_T - S_TB y_B, one thread per (top row, column), into eta2 (which
// holds eta_T only from k_nd_fold on)
template <int NR>
__global__ __launch_bounds__(256) void k_nd_rt(int R, const double* __restrict__ btop,
                                               const int64_t* __restrict__ t_ptr,
                                               const int32_t* __restrict__ t_pos,
                                               const double* __restrict__ t_val,
                                               const double* __restrict__ y1,
                                               double* __restrict__ rt, int pcg, int init,
                                               const PcgShared* sh) {
  if (pcg && !init && all_done(sh)) return;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)R * NR) return;
  const int64_t j = t / NR;
  const int k = (int)(t % NR);
  double x = btop[(size_t)(2 * j) * NR + k] + btop[(size_t)(2 * j + 1) * NR + k];
  rt[t] = nd_sub_couplings<NR>(x, t_ptr[j], t_ptr[j + 1], t_pos, t_val, y1, k);
}

// b_B - S_BT eta_T, one thread per (block row, column), into y1 (y_B is no
// longer needed once r_T is formed)
template <int NR>
__global__ __launch_bounds__(256) void k_nd_rb(int64_t nrows, const double* __restrict__ bpart,
                                               const int64_t* __restrict__ b_ptr,
                                               const int32_t* __restrict__ b_top,
                                               const double* __restrict__ b_val,
                                               const double* __restrict__ eta2,
                                               double* __restrict__ rb, int pcg, int init,
                                               const PcgShared* sh) {
  if (pcg && !init && all_done(sh)) return;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nrows * NR) return;
  const int64_t j = t / NR;
  const int k = (int)(t % NR);
  double x = bpart[(size_t)(2 * j) * NR + k] + bpart[(size_t)(2 * j + 1) * NR + k];
  rb[t] = nd_sub_couplings<NR>(x, b_ptr[j], b_ptr[j + 1], b_top, b_val, eta2, k);
}

// Launch sequence.  1-2 columns: four launches, the coupling terms formed in
// the prologues of the top product and of the second block pass (few
// couplings per row there, and no launch boundary to pay).  4-16 columns:
// r_T and b_B - S_BT eta_T get launches of their own, so that the products
// read them instead of each workgroup forming its share again.
template <int NR>
static void nd_solve_t(DeviceState& d, hipStream_t st, int pcg, int init) {
  constexpr bool PRE = NR >= 4;
  constexpr int NW = NdWaves<NR>::v;
  const NdDevice& nd = d.nd;
  const size_t shb = (size_t)std::max<int64_t>(nd.smax, 64 * NW) * NR * sizeof(double);
  // the PCG stop test rides in one extra workgroup of the first launch
  const unsigned extra = pcg ? 1u : 0u;
  const double* btop = d.bpart + (size_t)2 * nd.nrows * NR;  // the top rows' slots
  if (nd.R > 0) {
    am_launch_shm(d, true, false, k_nd_blocks<NR>, dim3(nd.nwg + extra), dim3(64 * NW), shb, st,
                  0, 0, nd.nwg, nd.wg, nd.binv, nd.ord, d.bpart,
                  nd.b_ptr, nd.b_top, nd.b_val, nd.eta2, nd.y1, d.eta, pcg, init,
                  d.red.pb, d.m, d.sc, d.shared);
    if (PRE)
      am_launch(d, false, false, k_nd_rt<NR>, dim3((unsigned)((nd.R * NR + 255) / 256)),
                dim3(256), st, nd.R, btop, nd.t_ptr, nd.t_pos, nd.t_val,
                nd.y1, nd.eta2, pcg, init, d.shared);
    const int nrb = (nd.ldC + 63) / 64;
    am_launch_shm(d, false, false, k_nd_top<NR, PRE>, dim3(nd.P * ((nrb + 3) / 4)), dim3(256),
                  PRE ? 0 : (size_t)nd.per * NR * sizeof(double), st, nd.R, nd.ldC, nd.cinv, nd.P,
                  nd.per, nrb, btop, nd.t_ptr, nd.t_pos, nd.t_val, nd.y1,
                  nd.eta2, nd.ypart, pcg, init, d.shared);
  }
  const unsigned nb =
      (unsigned)std::max<int64_t>(1, ((int64_t)nd.R * NR * kNdFoldLanes + 255) / 256);
  if (nd.R > 0)
    am_launch(d, false, false, k_nd_fold<NR>, dim3(nb), dim3(256), st, nd.R, nd.ldC, nd.P,
              nd.ypart, nd.ord + nd.nrows, nd.eta2, d.eta, pcg, init, d.shared);
  if (PRE && nd.R > 0)
    am_launch(d, false, false, k_nd_rb<NR>, dim3((unsigned)((nd.nrows * NR + 255) / 256)),
              dim3(256), st, nd.nrows, d.bpart, nd.b_ptr, nd.b_top, nd.b_val, nd.eta2,
              nd.y1, pcg, init, d.shared);
  // with no top rows this is the only launch (it then carries the stop test)
  const unsigned extra1 = nd.R > 0 ? 0u : extra;
  am_launch_shm(d, nd.R == 0, true, k_nd_blocks<NR>, dim3(nd.nwg + extra1), dim3(64 * NW), shb,
                st, 1, (PRE && nd.R > 0) ? 1 : 0, nd.nwg, nd.wg, nd.binv, nd.ord, d.bpart, nd.b_ptr, nd.b_top, nd.b_val, nd.eta2, nd.y1,
                d.eta, pcg, init, d.red.pb, d.m, d.sc, d.shared);
}

hipError_t launch_nd_solve(DeviceState& d, int nr, int pcg, int init, hipStream_t st) {
  if (nr > d.max_nrhs) return hipErrorInvalidValue;
  switch (nr) {
    case 1: nd_solve_t<1>(d, st, pcg, init); break;
    case 2: nd_solve_t<2>(d, st, pcg, init); break;
    case 4: nd_solve_t<4>(d, st, pcg, init); break;
    case 8: nd_solve_t<8>(d, st, pcg, init); break;
    case 16: nd_solve_t<16>(d, st, pcg, init); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---- the operator that the solve applies, for export -------------------------

// unit right-hand sides: column k is 1 at ND position p0 + k
__global__ __launch_bounds__(256) void k_nd_units(int64_t count, int nr, int64_t p0,
                                                  double* __restrict__ bpart) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) bpart[t] = t / nr == 2 * (p0 + t % nr) ? 1.0 : 0.0;
}

// row ord[p0 + k] of X from column k of eta
__global__ __launch_bounds__(256) void k_nd_take(int64_t NL, int nr, int64_t p0,
                                                 const int32_t* __restrict__ ord,
                                                 const double* __restrict__ eta,
                                                 double* __restrict__ X) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t k = t / NL, r = t % NL;
  if (k < nr && p0 + k < NL) X[(size_t)ord[p0 + k] * NL + r] = eta[r * nr + k];
}

// X = S^{-1} (NL x NL) as the interface solve applies it, a batch of unit
// right-hand sides at a time, on vectors of its own (applications of the
// handle may be running).  Synchronizes st.
hipError_t nd_operator(const DeviceState& d0, double* X, hipStream_t st) {
  DeviceState d = d0;
  const int nr = d.max_nrhs;
  const int64_t n_b = 2 * d.NL * nr, n_e = (int64_t)d.ldS * nr,
                n_y = std::max<int64_t>(d.nd.nrows, 1) * nr,
                n_t = (int64_t)std::max<int32_t>(d.nd.R, 1) * nr,
                n_p = (int64_t)d.nd.P * std::max<int32_t>(d.nd.ldC, 1) * nr;
  double* t = nullptr;
  hipError_t e = hipMalloc((void**)&t, sizeof(double) * (size_t)(n_b + n_e + n_y + n_t + n_p));
  if (e != hipSuccess) return e;
  d.bpart = t;
  d.eta = d.bpart + n_b;
  d.nd.y1 = d.eta + n_e;
  d.nd.eta2 = d.nd.y1 + n_y;
  d.nd.ypart = d.nd.eta2 + n_t;
  for (int64_t p0 = 0; p0 < d.NL && e == hipSuccess; p0 += nr) {
    hipLaunchKernelGGL(k_nd_units, dim3((unsigned)((n_b + 255) / 256)), dim3(256), 0, st, n_b, nr,
                       p0, d.bpart);
    e = launch_nd_solve(d, nr, 0, 0, st);
    if (e == hipSuccess)
      hipLaunchKernelGGL(k_nd_take, dim3((unsigned)((d.NL * nr + 255) / 256)), dim3(256), 0, st,
                         d.NL, nr, p0, d.nd.ord, d.eta, X);
  }
  if (e == hipSuccess) e = hipGetLastError();
  const hipError_t e2 = hipStreamSynchronize(st);
  (void)hipFree(t);
  return e != hipSuccess ? e : e2;
}

// ---- set-up ----------------------------------------------------------------

// block z of S, padded with the identity to T[z] tiles a side
__global__ __launch_bounds__(256) void k_nd_gather(const double* __restrict__ S, int ldS,
                                                   const int32_t* __restrict__ ord,
                                                   const int64_t* __restrict__ blk_off,
                                                   const int64_t* __restrict__ moff,
                                                   const int32_t* __restrict__ T,
                                                   double* __restrict__ M) {
  const int z = blockIdx.y, ld = 64 * T[z];
  const int64_t o = blk_off[z];
  const int s = (int)(blk_off[z + 1] - o);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < ld * ld; t += gridDim.x * blockDim.x) {
    const int a = t / ld, c = t % ld;
    M[moff[z] + t] = a < s && c < s ? S[(size_t)ord[o + a] * ldS + ord[o + c]] : (a == c ? 1.0 : 0.0);
  }
}

// Schur complement C = S_TT - sum_b S_Tb S_bb^{-1} S_bT over the top rows, in
// 64 x 64 tiles (identity beyond R; only the lower tiles are needed).  Row by
// row from the sparse couplings: the workgroup of row t forms S_tb S_bb^{-1}
// over the blocks it couples to (y, one row of scratch per workgroup, zero
// elsewhere) and takes its product with the couplings of every row t2 up to
// the end of t's tile.  The values of S_TT are gathered; the whole pass moves
// little.
__global__ __launch_bounds__(256) void k_nd_schur(
    const double* __restrict__ S, int ldS, int64_t nrows, int R, int ldC,
    const int32_t* __restrict__ ord, const int64_t* __restrict__ blk_off,
    const int64_t* __restrict__ inv_off, const double* __restrict__ binv,
    const int64_t* __restrict__ t_ptr, const int32_t* __restrict__ t_pos,
    const int32_t* __restrict__ t_blk, const double* __restrict__ t_val, double* yrows,
    double* __restrict__ C) {
  double* y = yrows + (size_t)blockIdx.x * nrows;
  for (int t = blockIdx.x; t < ldC; t += gridDim.x) {
    double* Ct = C + (size_t)t * ldC;
    const int end = (t & ~63) + 64;
    if (t >= R) {
      for (int c = threadIdx.x; c < end; c += 256) Ct[c] = c == t ? 1.0 : 0.0;
      continue;
    }
    for (int64_t p = threadIdx.x; p < nrows; p += 256) y[p] = 0.0;
    __syncthreads();
    for (int64_t q = t_ptr[t]; q < t_ptr[t + 1]; ++q) {  // one thread per entry of y throughout
      const int b = t_blk[q];
      const int64_t o = blk_off[b];
      const int s = (int)(blk_off[b + 1] - o);
      const double* row = binv + inv_off[b] + (t_pos[q] - o) * s;
      const double v = t_val[q];
      for (int p = threadIdx.x; p < s; p += 256) y[o + p] = fma(v, row[p], y[o + p]);
    }
    __syncthreads();
    const double* St = S + (size_t)ord[nrows + t] * ldS;
    for (int c = threadIdx.x; c < end; c += 256) {
      double v = 0.0;
      if (c < R) {
        for (int64_t q = t_ptr[c]; q < t_ptr[c + 1]; ++q) v = fma(t_val[q], y[t_pos[q]], v);
        v = St[ord[nrows + c]] - v;
      }
      Ct[c] = v;
    }
    __syncthreads();  // y is rewritten
  }
}

// out[q] = S[ri[q]][ci[q]]
__global__ __launch_bounds__(256) void k_nd_pairs(const double* __restrict__ S, int ldS,
                                                  const int32_t* __restrict__ ri,
                                                  const int32_t* __restrict__ ci, int64_t cnt,
                                                  double* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < cnt) out[t] = S[(size_t)ri[t] * ldS + ci[t]];
}

static int64_t nd_schur_groups(const NdDevice& nd) { return std::min(nd.ldC, 1024); }

int64_t nd_scratch(const NdDevice& nd) {
  return 2 * nd.mrows + (int64_t)nd.nblk * 8192 + 2 * (int64_t)nd.ldC * nd.ldC + 8192 +
         nd_schur_groups(nd) * nd.nrows;
}

// The numeric part of the set-up, on the S of the handle (original order).
// The blocks are not coupled to one another, so all are inverted together and
// the dense work beyond them is C alone; the chain is the tiles of the largest
// block and of C.  Time with a Cholesky factorization and triangular inverse
// of the whole reordered S, and in this form: 96^3 in 8^3 boxes
// (80 tiles) 14.6 and 0.9 ms, 128^3 (186 tiles) 71.9 and 1.8 ms.
hipError_t nd_numeric(DeviceState& d, double* scratch, hipStream_t st) {
  NdDevice& nd = d.nd;
  double* m0 = scratch;
  double* m1 = m0 + nd.mrows;
  double* db = m1 + nd.mrows;
  double* c0 = db + (int64_t)nd.nblk * 8192;
  double* c1 = c0 + (int64_t)nd.ldC * nd.ldC;
  double* dc = c1 + (int64_t)nd.ldC * nd.ldC;
  double* yrows = dc + 8192;
  hipError_t e = hipSuccess;
  if (nd.nblk > 0) {
    const unsigned gx = (unsigned)std::max(1, nd.tmax * nd.tmax * 4);
    hipLaunchKernelGGL(k_nd_gather, dim3(gx, nd.nblk), dim3(256), 0, st, d.S, d.ldS, nd.ord,
                       nd.blk_off, nd.moff, nd.tiles, m0);
    e = sweep_inverse(m0, m1, nd.moff, nd.tiles, nd.nblk, nd.tmax, db, nd.pad_off, 0, d.fail + 2, st);
    if (e == hipSuccess)
      e = sweep_output(m0, m1, nd.moff, nd.tiles, nd.nblk, nd.tmax, nd.binv, nd.inv_off, nd.blk_off,
                       0, 0, st);
    if (e != hipSuccess) return e;
  }
  if (nd.nt_pairs > 0)
    hipLaunchKernelGGL(k_nd_pairs, dim3((unsigned)((nd.nt_pairs + 255) / 256)), dim3(256), 0, st,
                       d.S, d.ldS, nd.t_ri, nd.t_ci, nd.nt_pairs, nd.t_val);
  if (nd.nb_pairs > 0)
    hipLaunchKernelGGL(k_nd_pairs, dim3((unsigned)((nd.nb_pairs + 255) / 256)), dim3(256), 0, st,
                       d.S, d.ldS, nd.b_ri, nd.b_ci, nd.nb_pairs, nd.b_val);
  if (nd.R > 0) {
    hipLaunchKernelGGL(k_nd_schur, dim3((unsigned)nd_schur_groups(nd)), dim3(256), 0, st, d.S,
                       d.ldS, nd.nrows, nd.R, nd.ldC, nd.ord, nd.blk_off, nd.inv_off, nd.binv,
                       nd.t_ptr, nd.t_pos, nd.t_blk, nd.t_val, yrows, c0);
    e = sweep_inverse(c0, c1, nullptr, nullptr, 1, nd.ldC / 64, dc, nullptr, nd.h_pad_off[nd.nblk],
                      d.fail + 2, st);
    if (e == hipSuccess)
      e = sweep_output(c0, c1, nullptr, nullptr, 1, nd.ldC / 64, nd.cinv, nullptr, nullptr, nd.R,
                       nd.ldC, st);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace am
