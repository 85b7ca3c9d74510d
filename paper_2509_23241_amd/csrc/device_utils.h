// Small device helpers shared by the kernels: bf16 <-> fp32 (round to nearest even) and the
// activation functions with their derivatives.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

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

// Butterflies over the lanes of a wave in vector instructions.  __shfl_xor goes through LDS, some 120 cycles for each of the six
// dependent steps; a rotation within a row of 16 lanes is an operand of the addition itself, and rows and halves swap in one
// instruction.  A rotation by O stands for lane ^ O where the lanes that differ in 2 O, 4 O, .. below 16 already agree, so the
// result is that of `for (o = FROM; o > 0; o /= 2) v = op(v, __shfl_xor(v, o, 64))` bit for bit.  All lanes of a wave (FROM 16, 32)
// or of a row of 16 lanes (8) take part; for fewer a rotation would bring in lanes of other groups.  The slab normalisations, where one workgroup waits
// for such sums alone, take 8.6 -> 7.5 us (kernels_batchnorm.hip); a decoder on 200 tokens 0.6 % less.
template <int O>
__device__ __forceinline__ float rotated(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + O, 0xf, 0xf, true));  // row_ror
}
template <class Op>
__device__ __forceinline__ float over_halves(float v, const Op& op) {  // the step of lane ^ 32
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float over_rows(float v, const Op& op) {  // the step of lane ^ 16
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// The same over a row of 16 lanes from the nearest lane to the farthest: pairs and pairs of pairs swap within four lanes, and the
// mirrored half row or row holds what lane ^ 4 or lane ^ 8 does, since the lanes of four or eight agree by then.
__device__ __forceinline__ float row_sum_ascending(float v) {
  auto moved = [](float x, auto control) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(control)::value, 0xf, 0xf, true));
  };
  v += moved(v, std::integral_constant<int, 0xb1>{});   // quad_perm 1 0 3 2
  v += moved(v, std::integral_constant<int, 0x4e>{});   // quad_perm 2 3 0 1
  v += moved(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
  return v + moved(v, std::integral_constant<int, 0x140>{});  // row_mirror
}
struct Add {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct Max {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
template <int FROM, class Op>
__device__ __forceinline__ float over_lanes(float v, const Op& op) {
  static_assert(FROM == 32 || FROM == 16 || FROM == 8, "lanes that differ in 8 have to meet before those that differ in less");
  if constexpr (FROM >= 32) v = over_halves(v, op);
  if constexpr (FROM >= 16) v = over_rows(v, op);
  v = op(v, rotated<8>(v));
  v = op(v, rotated<4>(v));
  v = op(v, rotated<2>(v));
  return op(v, rotated<1>(v));
}
template <int FROM = 32>
__device__ __forceinline__ float sum_over_lanes(float v) {
  return over_lanes<FROM>(v, Add());
}
template <int FROM = 32>
__device__ __forceinline__ float max_over_lanes(float v) {
  return over_lanes<FROM>(v, Max());
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
