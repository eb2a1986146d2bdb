// Gate nonlinearities of the recurrence launches whose cell math is on the step's serial chain, in
// straight-line code on the hardware's exp2 and reciprocal, where expf, tanhf and a division cost
// twice the instructions and a branch.
//
// sigm_f32, tanh_f32: no less exact than 1 / (1 + expf(-a)) and tanhf(a), which the launches per step use.
// Largest error on the hardware, every third float of [1e-6, 80] and its negative, in units of the last place:
//                    |a| < 0.55    |a| >= 0.55
//   sigm_f32             1.19          1.75        1 / (1 + expf(-a))   2.12   2.62
//   tanh_f32             0.76          1.14        tanhf(a)             0.77   1.40
#pragma once
#include <hip/hip_runtime.h>

namespace hpsgd {

// 1 / (1 + e^x), -100 <= x <= 88 (an infinite product would leave inf - inf as its remainder).
// x log2(e) is a rounded product plus its remainder r (fused multiply-adds), so e^x = p + p r ln 2 with
// p = 2^(rounded product); what 1 + p drops and the term of r go, as d, into the one Newton step behind the
// hardware's reciprocal: neither is rounded into e^x or into the sum.  GE1: x >= 0.
template <bool GE1>
__device__ __forceinline__ float recip_1p_exp(float x) {
  constexpr float L = 1.44269504088896341f, Llo = 1.92596299112661746e-8f, LN2 = 0.693147180559945309f;
  const float t = x * L;
  const float r = __builtin_fmaf(x, Llo, __builtin_fmaf(x, L, -t));
  const float p = __builtin_amdgcn_exp2f(t);
  const float s = 1.0f + p;
  const float hi = GE1 ? p : fmaxf(p, 1.0f), lo = GE1 ? 1.0f : fminf(p, 1.0f);
  const float d = __builtin_fmaf(p, r * LN2, lo - (s - hi));
  const float y = __builtin_amdgcn_rcpf(s);
  return __builtin_fmaf(__builtin_fmaf(-d, y, __builtin_fmaf(-s, y, 1.0f)), y, y);
}
// (0 and 1 at the infinities; the clamp would turn a NaN into a number)
__device__ __forceinline__ float sigm_f32(float a) {
  const float y = recip_1p_exp<false>(__builtin_amdgcn_fmed3f(-a, -100.0f, 88.0f));
  return a == a ? y : a;
}
// |a| < 0.55: a + a^3 q(a^2), q the polynomial of degree 4 whose largest error against (tanh(a)/a - 1)/a^2
// on that range, weighted as it enters the result, is least (1e-9 of the result); else 1 - 2 / (1 + e^(2|a|)),
// which is 0.5 or more where the quotient is at most 0.5: its error counts half.  A NaN takes the
// polynomial, which keeps it.
__device__ __forceinline__ float tanh_f32(float a) {
  const float s = a * a;
  float q = __builtin_fmaf(s, -0.006273165f, 0.02107096f);
  q = __builtin_fmaf(s, q, -0.053852145f);
  q = __builtin_fmaf(s, q, 0.13332585f);
  q = __builtin_fmaf(s, q, -0.33333316f);
  const float small = __builtin_fmaf(a * s, q, a);
  const float b = fabsf(a);
  const float big = __builtin_copysignf(__builtin_fmaf(-2.0f, recip_1p_exp<true>(fminf(2.0f * b, 88.0f)), 1.0f), a);
  return b >= 0.55f ? big : small;
}

// The gates of the bf16 launches, whose cell math is a fifth of a step: the hardware's
// exp2 and reciprocal (1 ulp each) as they are.  Absolute
// error about 1e-7 (tanh near 0 included: 1 - 2 / (e^2a + 1) loses relative, not absolute, accuracy),
// against gate values that are then rounded to bf16 (4e-3 relative) as operands.
__device__ __forceinline__ float sigm_fast(float a) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * a));
}
__device__ __forceinline__ float tanh_fast(float a) {
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(2.88539008f * a));
}

// EX: a launch's choice between the two
template <bool EX>
__device__ __forceinline__ float sigm_of(float a) { return EX ? sigm_f32(a) : sigm_fast(a); }
template <bool EX>
__device__ __forceinline__ float tanh_of(float a) { return EX ? tanh_f32(a) : tanh_fast(a); }

}  // namespace hpsgd
