// Small device helpers shared by the kernels: bf16 <-> fp32 (round to nearest even) and the
// activation functions with their derivatives.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tp {

__device__ __forceinline__ float bf16_to_float(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ uint16_t float_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float floatx2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const floatx2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ float to_float(float v) { return v; }
__device__ __forceinline__ float to_float(uint16_t v) { return bf16_to_float(v); }

template <typename T>
__device__ __forceinline__ T from_float(float v);
template <>
__device__ __forceinline__ float from_float<float>(float v) { return v; }
template <>
__device__ __forceinline__ uint16_t from_float<uint16_t>(float v) { return float_to_bf16(v); }

// act: 0 none, 1 ReLU, 2 GELU (exact erf form)
__device__ __forceinline__ float act_forward(float z, int act) {
  if (act == 1) return fmaxf(z, 0.f);
  if (act == 2) return 0.5f * z * (1.f + erff(z * 0.70710678118654752f));
  return z;
}

__device__ __forceinline__ float act_derivative(float z, int act) {
  if (act == 1) return z > 0.f ? 1.f : 0.f;
  if (act == 2)
    return 0.5f * (1.f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * __expf(-0.5f * z * z);
  return 1.f;
}

// GELU (erf form) and its derivative with one exponential and one reciprocal:
//   erf(x) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-x^2),  t = 1/(1 + p x),  x >= 0
// (Abramowitz & Stegun 7.1.26, |error| <= 1.5e-7), evaluated at x = |z|/sqrt(2), where
// exp(-x^2) = exp(-z^2/2) is also the Gaussian factor of the derivative.
struct GeluParts {
  float cdf;  // Phi(z) = 0.5 (1 + erf(z/sqrt 2))
  float pdf;  // phi(z) = exp(-z^2/2)/sqrt(2 pi)
};
// 1/2 and log2(e) are folded into the coefficients.  t is the hardware's reciprocal after one Newton step, for which x must
// be finite (from 64 on exp(-z^2/2) is zero anyway): 21 vector instructions, 31 with a division, and as far off fp64 (z in
// -9 .. 9: act 9.29e-8, act' 4.19e-8 rms).  With one branch for
// eight values instead of one each, 1600 x 2048 over 512 forward 15.4 -> 13.0 us.
__device__ __forceinline__ GeluParts gelu_parts(float z) {
  const float q = fmaf(0.3275911f, fminf(fabsf(z), 64.f) * 0.70710678118654752f, 1.0f);
  const float r = __builtin_amdgcn_rcpf(q), t = fmaf(fmaf(-q, r, 1.0f), r, r);
  const float e = __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);
  float poly = fmaf(0.5307027145f, t, -0.7265760135f);
  poly = fmaf(poly, t, 0.7107068705f);
  poly = fmaf(poly, t, -0.142248368f);
  poly = fmaf(poly, t, 0.127414796f);
  const float half_erfc = poly * t * e;               // 0.5 * (1 - erf(x))
  GeluParts g;
  g.cdf = z >= 0.f ? 1.0f - half_erfc : half_erfc;
  g.pdf = 0.39894228040143268f * e;
  return g;
}
// act(z) and act'(z) together (they share the exponential and the reciprocal)
struct ActPair {
  float a, d;
};
__device__ __forceinline__ ActPair act_pair_fast(float z, int act) {
  ActPair p;
  if (act == 2) {
    const GeluParts g = gelu_parts(z);
    p.a = z * g.cdf;
    p.d = fmaf(z, g.pdf, g.cdf);
  } else if (act == 1) {
    p.a = fmaxf(z, 0.f);
    p.d = z > 0.f ? 1.f : 0.f;
  } else {
    p.a = z;
    p.d = 1.f;
  }
  return p;
}
// N values at once: one branch on the activation for all of them, so that their exponentials and reciprocals overlap.
template <int N>
__device__ __forceinline__ void act_pairs_fast(const float (&z)[N], int act, float (&a)[N], float (&d)[N]) {
  auto each = [&](int kind) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const ActPair p = act_pair_fast(z[j], kind);
      a[j] = p.a;
      d[j] = p.d;
    }
  };
  if (act == 2) each(2);
  else if (act == 1) each(1);
  else each(0);
}

// Handing values from the workgroups of a launch to the one of them that finishes last.  A device-wide fence writes back and
// invalidates a whole L2, once per wave; what is handed over here goes past the L2s instead (relaxed atomics of device scope), and
// a workgroup counts itself in once its own values have arrived.
__device__ __forceinline__ void publish(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float published(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// By one thread, behind the publish() calls of its wave alone.  True for the last of `arrivals` calls, which leaves the counter at
// zero, as it has to be before the first.
__device__ __forceinline__ bool last_to_arrive(uint32_t* counter, uint32_t arrivals) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != arrivals - 1) return false;
  __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// Column sums of what the 256 threads of a block have added up, N neighbouring columns per thread, thread t those of unit
// t % units (units divides 256): out[N * units], in a fixed order.  `sm` holds N * 256 floats.
template <int N>
__device__ __forceinline__ void block_column_sums(const float (&s)[N], int units, float* sm, float* out) {
#pragma unroll
  for (int j = 0; j < N; ++j) sm[j * 256 + threadIdx.x] = s[j];
  __syncthreads();
  for (int o = threadIdx.x; o < N * units; o += 256) {
    const float* at = sm + (o % N) * 256 + o / N;
    float a = 0.f;
    for (int k = 0; k < 256; k += units) a += at[k];
    out[o] = a;
  }
}

}  // namespace tp
