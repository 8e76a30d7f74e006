// Device-side helpers shared by the routed-FFN kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Inclusive sum over a workgroup of whole wavefronts (at most 16): wavefront prefix by shuffles, wavefront
// totals through `wtot` (16 words of LDS).  Two barriers; `total` is the sum over the workgroup.
__device__ __forceinline__ int block_inclusive_sum(int v, int32_t* wtot, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  __syncthreads();   // (wtot may still be read from the call before)
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int w = 0; w < nw; ++w) {
    const int x = wtot[w];
    before += w < wave ? x : 0;
    total += x;
  }
  return before + incl;
}

// Between a wavefront's LDS writes and its own reads of what OTHER lanes wrote (and before it
// overwrites what they read): LDS executes one wavefront's accesses in order, so no wait is
// needed; this keeps the compiler from moving the accesses across each other.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Round-to-nearest-even float -> bf16 bit pattern (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
// Two floats -> packed bf16 pair, round-to-nearest-even: one v_cvt_pk_bf16_f32 on gfx950.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Upper tail of the standard normal, Q(|z|) = erfc(|z| / sqrt 2) / 2, and gauss = exp(-z^2 / 2), branch-free.
// Q(a) exp(a^2 / 2) is smooth and bounded, so it is a polynomial in t = 1 / (1 + 0.285 a) without constant term,
// degree 6, fitted here by iteratively reweighted least squares to weigh the absolute error near 0 and the
// relative one in the tail: 3.4e-8 absolute, 4e-4 relative (up to a = 14).  As evaluated in fp32 z Phi(z) is within
// 2.4e-7 and its derivative within 3e-7 of the exact value, far under the bf16 rounding of everything they
// feed.  A lone wavefront per SIMD pays 4 cycles for each of these instructions and 16 for the reciprocal and
// the exponential, so there are 14 of them: the hardware reciprocal (1 ulp) instead of a division, base 2, no selects.
__device__ __forceinline__ float normal_tail(float z, float& a, float& gauss) {
  // (med3: one instruction, where fminf brings a canonicalisation along.  An infinite z gives tail 0, a * tail = 0;
  // a NaN reaches the result through u.)
  a = __builtin_amdgcn_fmed3f(fabsf(z), 0.f, 1e30f);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.285f, a, 1.0f));
  const float u = 0.84932180028801904f * z;   // sqrt(log2(e) / 2)
  gauss = __builtin_amdgcn_exp2f(-(u * u));
  float poly = fmaf(t, -0.09568991512060165f, 0.32859522104263306f);
  poly = fmaf(t, poly, -0.1490938514471054f);
  poly = fmaf(t, poly, 0.21077582240104675f);
  poly = fmaf(t, poly, 0.08959521353244781f);
  poly = fmaf(t, poly, 0.11581752449274063f);
  return t * poly * gauss;
}

// Activation of Eq. 4 (ReLU) or the erf-form GELU z Phi(z) = max(z, 0) - |z| Q(|z|), and its derivative
// Phi(z) + z phi(z).
template <int ACT>
__device__ __forceinline__ float act_fn(float z) {
  if (ACT == 1) return z > 0.f ? z : 0.f;
  float a, g;
  const float tail = normal_tail(z, a, g);
  return fmaf(-a, tail, __builtin_amdgcn_fmed3f(z, 0.f, __builtin_inff()));
}
template <int ACT>
__device__ __forceinline__ float act_grad(float z) {
  if (ACT == 1) return z > 0.f ? 1.f : 0.f;
  float a, g;
  const float tail = normal_tail(z, a, g);
  return fmaf(z * 0.39894228040143268f, g, z >= 0.f ? 1.0f - tail : tail);
}

}  // namespace spt
