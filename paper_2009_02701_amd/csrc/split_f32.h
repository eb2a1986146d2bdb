// fp32 products on the bf16 matrix cores.
//
// An fp32 value is exactly the sum of three bf16 values: h0 = bf16(x), h1 = bf16(x - h0), h2 = x - h0 - h1 (24 bits of
// significand in 8 + 8 + 8; both differences are exact).  A product of two such sums is nine products of bf16 values, each
// exact in fp32; the six largest are kept,
//     a0 b0   |   a1 b0 + a0 b1 + a1 b1 + a2 b0 + a0 b2,
// and what is dropped (a1 b2, a2 b1, a2 b2) is below 2^-23 of the product, mostly below 2^-25, of either sign.  The bf16 instruction does sixteen
// times the multiply-adds of the fp32 one per cycle, so six of them are 2.7 times as fast.  Two sums are kept, one of a0 b0
// and one of the rest: the instruction adds 16 products at a time to its accumulator, so the large sum is rounded an eighth as
// often as with v_mfma_f32_32x32x2_f32, and the small sum's roundings are 2^-8 smaller.  Error against 64 bits
// (2-norm, N(0,1) operands), fp32 instruction / six bf16 products in one sum / in two sums:
//     contraction 16  7.4e-8 / 3.4e-8 / 3.2e-8,  128  2.0e-7 / 1.6e-7 / 6.6e-8,  1024  5.7e-7 / 4.9e-7 / 1.8e-7,  2240  8.5e-7 / 7.4e-7 / 2.9e-7.
//
// (Three-part splits of this kind: G. Henry, P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", 26th IEEE Symposium on Computer Arithmetic, 2019.)
//
// Where the 24 bits end.  An infinity, a NaN and a value that rounds to a bf16 infinity (above 3.39e38) make a NaN of what they reach
// (h1 = inf - inf), so a caller computes the outputs that are not finite again with the fp32 instruction, or splits with FINITE.
// Values below 2^-110 = 7.7e-34 lose low bits of h1 and h2 to the end of bf16's range.  Weight gradients over a batch of 16 with
// inputs N(0,1) times 1e-33 / 1e-34 / 1e-35 / 1e-36 have errors of 2.1e-7 / 5.5e-7 / 5.2e-6 / 5.0e-5, with the fp32 instruction 2.9e-7 /
// 2.9e-7 / 2.9e-7 / 4.1e-7; a resident recurrence (H = 300, 8 steps) with head weights of up to 0.06 times 1e-28 / 1e-32 /
// 1e-34 has 1.5e-7 / 5.0e-6 / 4.9e-4 in dW_hh, with the fp32 instruction 2.0e-7 / 2.1e-7 / 2.1e-7.
// The product between two narrow layers in one launch and, beyond H = 512, the projection in a resident launch, which have the fp32
// instruction as launches of their own, look for such values and keep it there.
// Of one term the fp32 instruction gives the rounded product, the six bf16 ones do not: callers keep it for contractions of up to
// three (the share of dW_hh that a recurrence accumulates takes the six of any batch).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hpsgd {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8s __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t split_round2(float x, float y) {
  bf16x2 v;
  v[0] = (__bf16)x;
  v[1] = (__bf16)y;
  uint32_t p = __builtin_bit_cast(uint32_t, v);
  asm("" : "+v"(p));  // (or x is rounded once more by itself where its half is widened)
  return p;
}
// (The differences as v_dot2_f32_bf16 would save the two instructions that widen a pair, but that instruction waits for the matrix
// unit, which the ones below run beside: a 32-cycle MFMA with four of them 56 cycles, with four of these 34.)
__device__ __forceinline__ float split_lo(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float split_hi(uint32_t p) { return __builtin_bit_cast(float, p & 0xffff0000u); }
// the three parts of x (low halves) and y (high halves).  FINITE: a value that would round to an infinity has the largest bf16
// for its first part (the difference is a bf16 value's worth of bits still); an infinity or a NaN makes a NaN as without.
template <bool FINITE = false>
__device__ __forceinline__ void split2(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  constexpr float most = 0x1.fep127f;
  p0 = FINITE ? split_round2(__builtin_amdgcn_fmed3f(x, -most, most), __builtin_amdgcn_fmed3f(y, -most, most)) : split_round2(x, y);
  const float rx = x - split_lo(p0), ry = y - split_hi(p0);
  p1 = split_round2(rx, ry);
  p2 = split_round2(rx - split_lo(p1), ry - split_hi(p1));
}
// ... of eight values, as the operands of a matrix instruction
__device__ __forceinline__ void split8(const float (&v)[8], uint4& p0, uint4& p1, uint4& p2) {
  split2(v[0], v[1], p0.x, p1.x, p2.x);
  split2(v[2], v[3], p0.y, p1.y, p2.y);
  split2(v[4], v[5], p0.z, p1.z, p2.z);
  split2(v[6], v[7], p0.w, p1.w, p2.w);
}

// ---- products of 16 x 16 blocks (v_mfma_f32_16x16x32_bf16): lane group lg = l / 16 takes the words 4 lg .. + 3 of a chunk of 32
// along the contraction and those 16 further on
typedef float floatx4 __attribute__((ext_vector_type(4)));

// A fragment of eight fp32 values per lane as three bf16 ones
struct SplitFrag { bf16x8s p[3]; };
__device__ __forceinline__ SplitFrag split_frag(const float4& lo, const float4& hi) {
  uint4 p0, p1, p2;
  split8({lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}, p0, p1, p2);
  return {{__builtin_bit_cast(bf16x8s, p0), __builtin_bit_cast(bf16x8s, p1), __builtin_bit_cast(bf16x8s, p2)}};
}
// big[q] += a0 w0, small[q] += the other five products, for NQ blocks of 16 columns (consecutive instructions
// update different accumulators)
template <int NQ>
__device__ __forceinline__ void split_mfmas(const SplitFrag& a, const SplitFrag (&w)[NQ], floatx4 (&big)[NQ], floatx4 (&small)[NQ]) {
  auto mul = [&](int pa, int pw, floatx4 (&to)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) to[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[pa], w[q].p[pw], to[q], 0, 0, 0);
  };
  mul(0, 0, big);
  mul(1, 0, small);
  mul(2, 0, small);
  mul(0, 1, small);
  mul(1, 1, small);
  mul(0, 2, small);
}
// acc += the products of one fragment's fp32 values with the fp32 instruction (W: the fragment of 16 columns): where the split
// gives no number
__device__ __forceinline__ void plain_mfmas(const float4 (&a)[2], const float4 (&w)[2], bool second, floatx4& acc) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && !second) continue;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h].x, w[h].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h].y, w[h].y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h].z, w[h].z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h].w, w[h].w, acc, 0, 0, 0);
  }
}
// whether one of a fragment's values (zero is none) is below 2^-110, where the parts lose low bits
__device__ __forceinline__ bool split_below(const float4& lo, const float4& hi) {
  auto size = [](float v) { return (__builtin_bit_cast(uint32_t, v) & 0x7fffffffu) - 1u; };
  const uint32_t l = min(min(size(lo.x), size(lo.y)), min(size(lo.z), size(lo.w))), h = min(min(size(hi.x), size(hi.y)), min(size(hi.z), size(hi.w)));
  return min(l, h) < 0x08800000u - 1u;
}
__device__ __forceinline__ bool any_beyond(const floatx4& v) {
  const float s = __builtin_fmaf(v[0], 0.f, __builtin_fmaf(v[1], 0.f, __builtin_fmaf(v[2], 0.f, v[3] * 0.f)));
  return __any(!(s == 0.f)) != 0;
}

// A copy of a value that the compiler computes with only here: what a rare path derives from it is not hoisted out of the time loop,
// where it would hold registers
template <typename V>
__device__ __forceinline__ V rarely(V v) {
  asm volatile("" : "+s"(v));
  return v;
}

}  // namespace hpsgd
