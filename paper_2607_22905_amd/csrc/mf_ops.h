// 16 x 16 matrix-core products for the local solves with many right-hand
// sides: operand and result layouts, and the 64-column strip product.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace am {

typedef double am_mf_d4 __attribute__((ext_vector_type(4)));
typedef float am_mf_f4 __attribute__((ext_vector_type(4)));
constexpr int kMfVP = 17;  // LDS pitch of a block-vector row (16 values + 1)
template <typename AT> struct MfAcc;
template <> struct MfAcc<double> {
  using V = am_mf_d4;
  // row of the 16 x 16 result held in element v of a lane with l / 16 = lk
  static __device__ __forceinline__ int row(int lk, int v) { return lk + 4 * v; }
};
template <> struct MfAcc<float> {
  using V = am_mf_f4;
  static __device__ __forceinline__ int row(int lk, int v) { return 4 * lk + v; }
};
__device__ __forceinline__ am_mf_d4 mf4(double a, double b, am_mf_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ am_mf_f4 mf4(float a, float b, am_mf_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}


// acc += sum over the 64 columns jj of A[rows][jj] B[jj][.] for a 16-row
// strip, afn(c, m) and bfn(c, m) giving this lane's operands at column
// jj = c + m lk (lk = lane / 16, held by the caller), c and m constants of
// the unrolled loop.  FP64 / FP32 (16x16x4 products): lane holds column 4 kk + lk of
// step kk; the 16 operand pairs are read from LDS first, then four
// independent chains of four products (kk = c mod 4 in chain c) are added in
// chain order.  BF16 (BFOP, FP32 arithmetic type only): four 16x16x16
// products, lane holding columns 16 c + 4 lk .. 16 c + 4 lk + 3 of step c,
// both operands rounded to BF16 (the factor values are BF16 already), two
// chains added in order.
__device__ __forceinline__ short am_bf16_rne(float x) {
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}
typedef short am_mf_s4 __attribute__((ext_vector_type(4)));
template <bool BFOP, typename V, typename AF, typename BF>
__device__ __forceinline__ V mf_pass(V acc, AF&& afn, BF&& bfn) {
  using AT = decltype(afn(0, 0));
  if constexpr (BFOP) {
    static_assert(sizeof(AT) == 4, "BF16 products: FP32 arithmetic type");
    V c[2];
    c[0] = acc;
    c[1] = V{0, 0, 0, 0};
    am_mf_s4 a[4], b[4];
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[st][t] = am_bf16_rne(afn(16 * st + t, 4));
        b[st][t] = am_bf16_rne(bfn(16 * st + t, 4));
      }
#pragma unroll
    for (int st = 0; st < 4; ++st)
      c[st % 2] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[st], b[st], c[st % 2], 0, 0, 0);
    return c[0] + c[1];
  } else {
    V c[4];
    c[0] = acc;
#pragma unroll
    for (int t = 1; t < 4; ++t) c[t] = V{0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // two halves of 8 operand pairs (registers)
      AT a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        a[u] = afn(4 * (8 * h + u), 1);
        b[u] = bfn(4 * (8 * h + u), 1);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u % 4] = mf4(a[u], b[u], c[u % 4]);
    }
    return (c[0] + c[1]) + (c[2] + c[3]);
  }
}

}  // namespace am
