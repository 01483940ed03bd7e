// Activation formulas shared by the elementwise kernels and the GEMM epilogues that apply them
// in place of a separate pass: one definition, so both roads give the same bits.
#pragma once
#include <hip/hip_runtime.h>

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}
__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + expf(-z)); }
// SwiGLU: silu(gate) * up
__device__ __forceinline__ float swiglu_f(float gate, float up) { return gate * sigmoid_f(gate) * up; }
__device__ __forceinline__ void swiglu_grad_f(float gate, float up, float d, float* dgate, float* dup) {
  const float s = sigmoid_f(gate);
  *dgate = d * up * (s * (1.0f + gate * (1.0f - s)));
  *dup = d * (gate * s);
}

// GELU of bf16 numbers from a table in LDS that the workgroup fills with erff itself: the bits of gelu_f.
// erff is odd and takes 1665 values over the bf16 numbers from 2^-10 to 8.  Below, the factor
// 1 + erf is so near 1 that z / 2, a bf16 number, is what the product rounds to (entry 0; where z / 2
// is none, because it is denormal, the factor is 1 in fp32); from 8 on erff is 1 in fp32.  The
// limits at +-infinity and NaN are those of the formula.
struct ErfTable {
  static constexpr int kLow = (117 << 7) - 1, kHigh = 130 << 7;   // bf16 bits: the last number below 2^-10, and 8
  static constexpr int kEntries = kHigh - kLow + 1;
  static __device__ __forceinline__ void fill(float* t, int first, int step) {
    for (int i = first; i < kEntries; i += step) t[i] = i == 0 ? 0.f : erff(__uint_as_float((unsigned)(kLow + i) << 16) * 0.70710678118654752f);
  }
  // z: a bf16 number
  static __device__ __forceinline__ float erf_of(const float* t, float z) {
    const int u = (int)(__float_as_uint(z) >> 16) & 0x7fff;
    return copysignf(t[min(max(u, kLow), kHigh) - kLow], z);
  }
  static __device__ __forceinline__ float gelu(const float* t, float z) { return 0.5f * z * (1.0f + erf_of(t, z)); }
  // The gradient meets its factor in fp32, where small z count: two terms of the series of
  // erf(z / sqrt 2).  1 + that is the fp32 number 1 + erff for every bf16 number below 2^-10 (compared
  // one by one; between 2^-10 and 2^-9 one differs).  A select, not a branch: the reads of a whole
  // vector are in flight together.
  static __device__ __forceinline__ float gelu_grad(const float* t, float z) {
    const float series = z * fmaf(z * z, -0.13298076013381091f, 0.79788456080286536f);
    float e = erf_of(t, z);
    e = fabsf(z) < 0x1p-10f ? series : e;
    return 0.5f * (1.0f + e) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
  }
};
