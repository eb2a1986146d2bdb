// Helpers of the bf16 training path that are not contractions: rounded / transposed operand
// copies, the embedding rows in that form, and the softmax-CE that emits bf16 logit gradients.
// Every time-batched GEMM of that path takes contraction-contiguous bf16 operands; these
// kernels produce the ones that no other kernel's epilogue writes.
#include "kernels.h"

namespace hpsgd {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// (the copy kernels read their input once and write what later launches read: non-temporal)
typedef float f4nt_a __attribute__((ext_vector_type(4)));
typedef unsigned u4nt_a __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x4 load4_as_bf16(const float* p) {
  const f4nt_a v = __builtin_nontemporal_load(reinterpret_cast<const f4nt_a*>(p));
  bf16x4 r;
  r[0] = (__bf16)v.x; r[1] = (__bf16)v.y; r[2] = (__bf16)v.z; r[3] = (__bf16)v.w;
  return r;
}
__device__ __forceinline__ bf16x4 load4_as_bf16(const __bf16* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const bf16x4*>(p));
}

// in: R x C (fp32 or bf16, row pitch ld_in).  out_p (nullable): the bf16 rounding, row pitch
// ld_p.  out_t (nullable): its transpose, out_t[c][r], row pitch ld_t.  One 64 x 64 tile per
// workgroup, read once: 16-byte (fp32) or 8-byte (bf16) loads, 8-byte plain stores, and the
// transposed tile goes through LDS and leaves as 16-byte pieces of 8 consecutive input rows.
// Needs C % 4 == 0, R % 8 == 0 and the alignments cvt2_supported checks.
template <typename TIN>
__device__ __forceinline__ void cvt2_tile(const TIN* __restrict__ src, long ld_in, __bf16* __restrict__ dst_p, long ld_p,
                                          __bf16* __restrict__ dst_t, long ld_t, int R, int C, int c0, int r0,
                                          __bf16 (&tile)[64][72]) {
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  // All four loads are issued before anything waits for one (clamped addresses instead of
  // branches: behind a branch each load would be waited for, and stored, before the next is issued).
  const int c = c0 + 4 * tx;
  const bool c_ok = c < C;
  const int cl = c_ok ? c : C - 4;
  bf16x4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = load4_as_bf16(src + (long)min(r0 + ty + 16 * i, R - 1) * ld_in + cl);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = ty + 16 * i, r = r0 + rl;
    if (r < R && c_ok) {
      if (dst_p) __builtin_nontemporal_store(v[i], reinterpret_cast<bf16x4*>(dst_p + (long)r * ld_p + c));
    } else {
      v[i][0] = v[i][1] = v[i][2] = v[i][3] = (__bf16)0.f;
    }
    if (dst_t) {
#pragma unroll
      for (int e = 0; e < 4; ++e) tile[4 * tx + e][rl] = v[i][e];
    }
  }
  if (!dst_t) return;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = threadIdx.x + 256 * q, col = idx >> 3, part = idx & 7;
    const int c = c0 + col, r = r0 + 8 * part;
    if (c < C && r < R)
      __builtin_nontemporal_store(*reinterpret_cast<const u4nt_a*>(&tile[col][8 * part]),
                                  reinterpret_cast<u4nt_a*>(dst_t + (long)c * ld_t + r));
  }
}

// The same for a source of any alignment whose rows come in blocks of gh (gp in the copies) and whose Cs
// columns are padded to C (C % 4 == 0): zeros where the source has nothing.  16-byte loads at 4-byte boundaries, the last
// of a row from its last four values, shifted into place.  (H = 650, K = 4, the layers' weights and the head's: 49 and
// 53 us in 4-byte loads and 2-byte stores, 38 and 37 now, 31 and 36 at the rate of a large copy.)
__device__ __forceinline__ void cvt2_tile_padded(const float* __restrict__ src, long ld_in, __bf16* __restrict__ dst_p, long ld_p,
                                                 __bf16* __restrict__ dst_t, long ld_t, int R, int C, int gp, int gh, int Cs,
                                                 int c0, int r0, __bf16 (&tile)[64][72]) {
  typedef float f4u_a __attribute__((ext_vector_type(4), aligned(4)));
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int c = c0 + 4 * tx, cl = max(min(c, Cs - 4), 0), sh = c - cl;
  const float* p[4];
  bool rok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + ty + 16 * i, q = r / gp, j = r - q * gp;
    rok[i] = r < R && j < gh;
    p[i] = src + (rok[i] ? (long)(q * gh + j) * ld_in : 0) + cl;
  }
  float v[4][4];
  if (Cs >= 4) {  // (uniform)
    f4u_a w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = __builtin_nontemporal_load(reinterpret_cast<const f4u_a*>(p[i]));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i][0] = sh == 0 ? w[i].x : sh == 1 ? w[i].y : sh == 2 ? w[i].z : w[i].w;
      v[i][1] = sh == 0 ? w[i].y : sh == 1 ? w[i].z : w[i].w;
      v[i][2] = sh == 0 ? w[i].z : w[i].w;
      v[i][3] = w[i].w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = p[i][min(c + e, Cs - 1) - cl];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = ty + 16 * i, r = r0 + rl;
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (__bf16)(rok[i] && c + e < Cs ? v[i][e] : 0.f);
    if (dst_p && r < R && c < C) __builtin_nontemporal_store(o, reinterpret_cast<bf16x4*>(dst_p + (long)r * ld_p + c));
    if (dst_t) {
#pragma unroll
      for (int e = 0; e < 4; ++e) tile[4 * tx + e][rl] = o[e];
    }
  }
  if (!dst_t) return;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = threadIdx.x + 256 * q, col = idx >> 3, part = idx & 7;
    const int c = c0 + col, r = r0 + 8 * part;
    if (c < C && r < R)
      __builtin_nontemporal_store(*reinterpret_cast<const u4nt_a*>(&tile[col][8 * part]),
                                  reinterpret_cast<u4nt_a*>(dst_t + (long)c * ld_t + r));
  }
}

template <typename TIN>
__global__ void __launch_bounds__(256)
cvt2_kernel(const TIN* __restrict__ in, long ld_in, long s_in, __bf16* __restrict__ out_p, long ld_p,
            long s_p, __bf16* __restrict__ out_t, long ld_t, long s_t, int R, int C) {
  __shared__ __attribute__((aligned(16))) __bf16 tile[64][72];  // [column][row]
  const int g = blockIdx.z;
  cvt2_tile<TIN>(in + g * s_in, ld_in, out_p ? out_p + g * s_p : nullptr, ld_p, out_t ? out_t + g * s_t : nullptr, ld_t,
                 R, C, blockIdx.x * 64, blockIdx.y * 64, tile);
}

// Several fp32 matrices in one launch (the weight matrices of a model: each is a few hundred
// tiles, and a launch of its own costs more than its copies).  blockIdx.x runs over the tiles of
// all jobs, job j owning [tile0[j], tile0[j+1]).
__global__ void __launch_bounds__(256) cvt2_pack_kernel(Cvt2Pack p) {
  __shared__ __attribute__((aligned(16))) __bf16 tile[64][72];
  int j = 0;
  while (j + 1 < p.n && (int)blockIdx.x >= p.tile0[j + 1]) ++j;  // (uniform)
  const Cvt2Job& q = p.job[j];
  const int t = blockIdx.x - p.tile0[j], g = blockIdx.z;
  __bf16* op = reinterpret_cast<__bf16*>(q.out_p);
  __bf16* ot = reinterpret_cast<__bf16*>(q.out_t);
  if (q.gp) {
    cvt2_tile_padded(q.in + g * q.s_in, q.ld_in, op ? op + g * q.s_p : nullptr, q.ld_p, ot ? ot + g * q.s_t : nullptr, q.ld_t,
                     q.R, q.C, q.gp, q.gh, q.Cs, (t % q.tiles_x) * 64, (t / q.tiles_x) * 64, tile);
    return;
  }
  cvt2_tile<float>(q.in + g * q.s_in, q.ld_in, op ? op + g * q.s_p : nullptr, q.ld_p, ot ? ot + g * q.s_t : nullptr,
                   q.ld_t, q.R, q.C, (t % q.tiles_x) * 64, (t / q.tiles_x) * 64, tile);
}

bool cvt2_supported(const void* in, int in_bf16, long ld_in, long s_in, const void* out_p, long ld_p,
                    long s_p, const void* out_t, long ld_t, long s_t, int R, int C) {
  const uintptr_t in_mask = in_bf16 ? 7 : 15;
  if (((uintptr_t)in & in_mask) != 0 || ld_in % 4 != 0 || s_in % 4 != 0 || C % 4 != 0 || R % 8 != 0) return false;
  if (out_p && (((uintptr_t)out_p & 7) != 0 || ld_p % 4 != 0 || s_p % 4 != 0)) return false;
  if (out_t && (((uintptr_t)out_t & 15) != 0 || ld_t % 8 != 0 || s_t % 8 != 0)) return false;
  return R > 0 && C > 0;
}

hipError_t launch_cvt2(const void* in, int in_bf16, long ld_in, long s_in, void* out_p, long ld_p, long s_p,
                       void* out_t, long ld_t, long s_t, int R, int C, int groups, hipStream_t s) {
  if (!cvt2_supported(in, in_bf16, ld_in, s_in, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C))
    return hipErrorInvalidValue;
  dim3 grid((C + 63) / 64, (R + 63) / 64, groups);
  // bytes: one read of the input, one write of each copy
  KernelTimer kt(KID_CVT2, (double)R * C * groups * ((in_bf16 ? 2 : 4) + (out_p ? 2 : 0) + (out_t ? 2 : 0)), s);
  if (in_bf16)
    hipLaunchKernelGGL(cvt2_kernel<__bf16>, grid, dim3(256), 0, s, (const __bf16*)in, ld_in, s_in,
                       (__bf16*)out_p, ld_p, s_p, (__bf16*)out_t, ld_t, s_t, R, C);
  else
    hipLaunchKernelGGL(cvt2_kernel<float>, grid, dim3(256), 0, s, (const float*)in, ld_in, s_in,
                       (__bf16*)out_p, ld_p, s_p, (__bf16*)out_t, ld_t, s_t, R, C);
  return hipGetLastError();
}

bool cvt2_pack_push(Cvt2Pack& p, const float* in, long ld_in, long s_in, void* out_p, long ld_p, long s_p,
                    void* out_t, long ld_t, long s_t, int R, int C) {
  if (!cvt2_supported(in, 0, ld_in, s_in, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C)) return false;
  return cvt2_pack_push_padded(p, in, ld_in, s_in, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C, 0, 0, C);
}

bool cvt2_pack_push_padded(Cvt2Pack& p, const float* in, long ld_in, long s_in, void* out_p, long ld_p, long s_p,
                           void* out_t, long ld_t, long s_t, int R, int C, int gp, int gh, int Cs) {
  if (p.n >= Cvt2Pack::MAX || R <= 0 || C <= 0) return false;
  if (gp && (gh < 1 || gh > gp || Cs < 1 || Cs > C || R % 8 != 0 || C % 4 != 0 ||
             (out_p && (((uintptr_t)out_p & 7) != 0 || ld_p % 4 != 0 || s_p % 4 != 0)) ||
             (out_t && (((uintptr_t)out_t & 15) != 0 || ld_t % 8 != 0 || s_t % 8 != 0))))
    return false;
  Cvt2Job& q = p.job[p.n];
  q.gp = gp; q.gh = gh; q.Cs = Cs;
  q.in = in; q.ld_in = ld_in; q.s_in = s_in;
  q.out_p = out_p; q.ld_p = ld_p; q.s_p = s_p;
  q.out_t = out_t; q.ld_t = ld_t; q.s_t = s_t;
  q.R = R; q.C = C;
  q.tiles_x = (C + 63) / 64;
  const long tiles = (long)q.tiles_x * ((R + 63) / 64);
  if (tiles + p.tile0[p.n] > (1L << 30)) return false;
  p.tile0[p.n + 1] = p.tile0[p.n] + (int)tiles;
  p.bytes += (double)R * C * (4 + (out_p ? 2 : 0) + (out_t ? 2 : 0));
  ++p.n;
  return true;
}

hipError_t launch_cvt2_pack(const Cvt2Pack& p, int groups, hipStream_t s) {
  if (p.n == 0 || groups <= 0) return hipSuccess;
  KernelTimer kt(KID_CVT2_PACK, p.bytes * groups, s);
  hipLaunchKernelGGL(cvt2_pack_kernel, dim3(p.tile0[p.n], 1, groups), dim3(256), 0, s, p);
  return hipGetLastError();
}

// Gate gradients r | z | n | q (row-major, R x 4H) -> (r | z | n)^T and (r | z | q)^T: a workgroup reads a
// 64 x 64 tile once and writes it to the one or two places it belongs to.  H % 32 == 0, R % 8 == 0.
__global__ void __launch_bounds__(256)
transpose_dg4_kernel(const __bf16* __restrict__ dg4, long s_dg4, __bf16* __restrict__ dgxT, __bf16* __restrict__ dghT, long ld_T,
                     long s_T, int R, int H) {
  __shared__ __attribute__((aligned(16))) __bf16 tile[64][72];  // [column][row]
  const int g = blockIdx.z, c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 7, ty = threadIdx.x >> 3;
  typedef __bf16 bf16x8t __attribute__((ext_vector_type(8)));
  bf16x8t v[2];
  const int c = min(c0 + 8 * tx, 4 * H - 8);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    v[i] = *reinterpret_cast<const bf16x8t*>(dg4 + g * s_dg4 + (long)min(r0 + ty + 32 * i, R - 1) * 4 * H + c);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[8 * tx + e][ty + 32 * i] = v[i][e];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = threadIdx.x + 256 * q, col = c0 + (idx >> 3), r = r0 + 8 * (idx & 7);
    if (col >= 4 * H || r >= R) continue;
    const u4nt_a w = *reinterpret_cast<const u4nt_a*>(&tile[idx >> 3][8 * (idx & 7)]);
    if (col < 3 * H) *reinterpret_cast<u4nt_a*>(dgxT + g * s_T + (long)col * ld_T + r) = w;
    if (col < 2 * H) *reinterpret_cast<u4nt_a*>(dghT + g * s_T + (long)col * ld_T + r) = w;
    if (col >= 3 * H) *reinterpret_cast<u4nt_a*>(dghT + g * s_T + (long)(col - H) * ld_T + r) = w;
  }
}

hipError_t launch_transpose_dg4(const void* dg4, long s_dg4, void* dgxT, void* dghT, long ld_T, long s_T, int R, int H, int groups,
                                hipStream_t s) {
  if (H % 32 != 0 || R % 8 != 0 || ld_T % 8 != 0 || s_T % 8 != 0 || s_dg4 % 8 != 0 ||
      (((uintptr_t)dg4 | (uintptr_t)dgxT | (uintptr_t)dghT) & 15) != 0)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(transpose_dg4_kernel, dim3((4 * H + 63) / 64, (R + 63) / 64, groups), dim3(256), 0, s, (const __bf16*)dg4, s_dg4,
                     (__bf16*)dgxT, (__bf16*)dghT, ld_T, s_T, R, H);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- embedding rows, rounded
// Lookup, rounding and transpose in one pass (they were three passes over the rows): a workgroup makes a
// 64 x 64 tile of the copies.  Row r = t Bp + b takes the table row of tok[t B + b].  VEC: 16-byte loads of
// table rows that allow them, else one element per load, zero beyond Ew.
template <bool VEC>
__global__ void __launch_bounds__(256)
embed_bf16_kernel(const float* __restrict__ E, long s_E, const int32_t* __restrict__ tok, long s_tok, __bf16* __restrict__ xb,
                  long s_xb, __bf16* __restrict__ xT, long ld_T, long s_xT, int R, int B, int Bp, int Ew, int Ep) {
  __shared__ __attribute__((aligned(16))) __bf16 tile[64][72];  // [column][row]
  const int g = blockIdx.z, c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const float* src[4];
  bool rok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = min(r0 + ty + 16 * i, R - 1), t = r / Bp, b = r - t * Bp;
    rok[i] = r0 + ty + 16 * i < R && b < B;
    src[i] = E + g * s_E + (long)tok[g * s_tok + (long)t * B + min(b, B - 1)] * Ew;
  }
  const int c = c0 + 4 * tx;
  bf16x4 v[4];
  if (VEC) {
    const int cl = min(c, Ew - 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = load4_as_bf16(src[i] + cl);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = (__bf16)src[i][min(c + e, Ew - 1)];
  }
  __bf16* xg = xb + g * s_xb;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = ty + 16 * i, r = r0 + rl;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!rok[i] || c + e >= Ew) v[i][e] = (__bf16)0.f;
    if (r < R && c < Ep) __builtin_nontemporal_store(v[i], reinterpret_cast<bf16x4*>(xg + (long)r * Ep + c));
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[4 * tx + e][rl] = v[i][e];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = threadIdx.x + 256 * q, col = idx >> 3, part = idx & 7;
    if (c0 + col < Ep && r0 + 8 * part < R)
      __builtin_nontemporal_store(*reinterpret_cast<const u4nt_a*>(&tile[col][8 * part]),
                                  reinterpret_cast<u4nt_a*>(xT + g * s_xT + (long)(c0 + col) * ld_T + r0 + 8 * part));
  }
}

hipError_t launch_embed_bf16(const float* E, long s_E, const int32_t* tok, long s_tok, void* xb, long s_xb, void* xT,
                             long ld_T, long s_xT, int T, int B, int Bp, int Ew, int Ep, int groups, hipStream_t s) {
  if (Bp % 8 != 0 || Bp < B || Ep % 8 != 0 || Ep < Ew || ((uintptr_t)xb & 7) != 0 || s_xb % 4 != 0 ||
      ((uintptr_t)xT & 15) != 0 || ld_T % 8 != 0 || s_xT % 8 != 0)
    return hipErrorInvalidValue;
  const int R = T * Bp;
  dim3 grid((Ep + 63) / 64, (R + 63) / 64, groups);
  // (a copy and a transposed copy like cvt2_kernel's, and counted with them) bytes: one read of a row, one write of each
  KernelTimer kt(KID_CVT2, 8.0 * R * Ew * groups, s);
  const bool vec = Ew % 4 == 0 && ((uintptr_t)E & 15) == 0 && s_E % 4 == 0;
#define HPSGD_EMB(V)                                                                                                 hipLaunchKernelGGL(embed_bf16_kernel<V>, grid, dim3(256), 0, s, E, s_E, tok, s_tok, (__bf16*)xb, s_xb, (__bf16*)xT, ld_T,                      s_xT, R, B, Bp, Ew, Ep)
  if (vec) HPSGD_EMB(true);
  else HPSGD_EMB(false);
#undef HPSGD_EMB
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- softmax-CE, bf16 gradient
// A workgroup takes rpb consecutive rows; a row (C <= 1024 * V4 logits) is read once into registers.
// Writes dlogits = (softmax - onehot)/N rounded to bf16 (row pitch ld_d) and the row's loss
// -log softmax[y]; the logits stay as they are.  It also sums the unrounded gradient of its
// rows per column (a thread owns the same columns in every row): colpart[g][block][c], the
// partial sums of the head's bias gradient, added up by a second small kernel.  The next row's
// loads are issued before the current row is reduced.  Columns from C up to Cw (C rounded up to 8) are
// written as zeros; rows of the batch's padding (b >= B in row t Bp + b) have a zero gradient.
constexpr int SMR = 2;  // the fewest rows per workgroup (a row is a chain of 3 us: 72 rows x 6 workers of 6736 words 27 us in blocks of 8)

template <int V4, int NT>
__global__ void __launch_bounds__(NT)
softmax_ce_bf16_rows_kernel(const float* __restrict__ logits, long ld_l, long s_logits, const int32_t* __restrict__ y,
                            long s_y, __bf16* __restrict__ dlog, long ld_d, long s_d,
                            float* __restrict__ rowloss, long s_rowloss, float* __restrict__ colpart, long s_colpart, int N,
                            int B, int Bp, int C, int Cw, int rpb) {
  // partial results of the NW waves, one set per reduction and row parity: a set is written
  // again two rows later, with two barriers in between, so one barrier per reduction is enough
  constexpr int NW = NT / 64;
  static_assert(NW == 4 || NW == 8, "four or eight waves");
  __shared__ float red_m[2][NW], red_s[2][NW];
  const int g = blockIdx.y, row0 = blockIdx.x * rpb;
  const int nr = min(rpb, N - row0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float inv_n = 1.0f / (float)(N / Bp * B);
  float4 acc[V4], nx[V4];
#pragma unroll
  for (int i = 0; i < V4; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  auto load_row = [&](int row) {
    const float* lr = logits + g * s_logits + (long)row * ld_l;
#pragma unroll
    for (int i = 0; i < V4; ++i) {
      const int c = 4 * (tid + NT * i);
      typedef float f4nt __attribute__((ext_vector_type(4)));
      const f4nt t4 = __builtin_nontemporal_load(reinterpret_cast<const f4nt*>(lr + (c < C ? c : 0)));
      nx[i] = make_float4(t4.x, t4.y, t4.z, t4.w);
    }
  };
  load_row(row0);
  for (int r = 0; r < nr; ++r) {
    const int row = row0 + r;
    const int t = row / Bp, b = row - t * Bp;
    const bool real = b < B;  // (uniform)
    const int label = y[g * s_y + (long)t * B + min(b, B - 1)];
    float4 v[V4];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < V4; ++i) {
      v[i] = nx[i];
      if (C & 3) {  // (uniform) the last vector of a row may reach beyond it
        const int c = 4 * (tid + NT * i);
        if (c + 1 >= C) v[i].y = -INFINITY;
        if (c + 2 >= C) v[i].z = -INFINITY;
        if (c + 3 >= C) v[i].w = -INFINITY;
      }
      if (4 * (tid + NT * i) < C) m = fmaxf(fmaxf(m, fmaxf(v[i].x, v[i].y)), fmaxf(v[i].z, v[i].w));
    }
    if (r + 1 < nr) load_row(row + 1);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (lane == 0) red_m[r & 1][wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red_m[r & 1][0], red_m[r & 1][1]), fmaxf(red_m[r & 1][2], red_m[r & 1][3]));
    if (NW == 8)
      m = fmaxf(m, fmaxf(fmaxf(red_m[r & 1][NW - 4], red_m[r & 1][NW - 3]), fmaxf(red_m[r & 1][NW - 2], red_m[r & 1][NW - 1])));
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < V4; ++i)
      if (4 * (tid + NT * i) < C) {
        v[i].x = expf(v[i].x - m); v[i].y = expf(v[i].y - m);
        v[i].z = expf(v[i].z - m); v[i].w = expf(v[i].w - m);
        sum += (v[i].x + v[i].y) + (v[i].z + v[i].w);
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (lane == 0) red_s[r & 1][wave] = sum;
    __syncthreads();
    sum = (red_s[r & 1][0] + red_s[r & 1][1]) + (red_s[r & 1][2] + red_s[r & 1][3]);
    if (NW == 8)
      sum += (red_s[r & 1][NW - 4] + red_s[r & 1][NW - 3]) + (red_s[r & 1][NW - 2] + red_s[r & 1][NW - 1]);
    const float inv_sum = 1.0f / sum;
    if (tid == 0)
      rowloss[g * s_rowloss + row] = real ? -((logits[g * s_logits + (long)row * ld_l + label] - m) - logf(sum)) : 0.f;
    __bf16* dr = dlog + g * s_d + (long)row * ld_d;
#pragma unroll
    for (int i = 0; i < V4; ++i) {
      const int c = 4 * (tid + NT * i);
      if (c < C) {
        float4 d4 = make_float4((v[i].x * inv_sum - (c + 0 == label ? 1.0f : 0.0f)) * inv_n,
                                (v[i].y * inv_sum - (c + 1 == label ? 1.0f : 0.0f)) * inv_n,
                                (v[i].z * inv_sum - (c + 2 == label ? 1.0f : 0.0f)) * inv_n,
                                (v[i].w * inv_sum - (c + 3 == label ? 1.0f : 0.0f)) * inv_n);
        // (selected: a padding row's logits are NaN where a weight is infinite)
        if (!real) d4 = make_float4(0.f, 0.f, 0.f, 0.f);
        acc[i].x += d4.x; acc[i].y += d4.y; acc[i].z += d4.z; acc[i].w += d4.w;
        bf16x4 o;
        o[0] = (__bf16)d4.x; o[1] = (__bf16)d4.y; o[2] = (__bf16)d4.z; o[3] = (__bf16)d4.w;
        __builtin_nontemporal_store(o, reinterpret_cast<bf16x4*>(dr + c));
      } else if (c < Cw) {
        const bf16x4 z = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
        __builtin_nontemporal_store(z, reinterpret_cast<bf16x4*>(dr + c));
      }
    }
  }
  float* cp = colpart + g * s_colpart + (long)blockIdx.x * Cw;
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    const int c = 4 * (tid + NT * i);
    if (c < C) *reinterpret_cast<float4*>(cp + c) = acc[i];
  }
}

// Rows per workgroup.  The kernel holds three workgroups of four waves per CU (168 registers; two of
// eight waves for long rows), and a launch
// whose workgroups outnumber those places leaves the chip half empty at its end: 1120 x 8 rows in
// blocks of 8 are 1120 workgroups for 768 places, i.e. 16 rows' time where blocks of 12 take 12.
// So: as many rows per workgroup as fill every place once, at least SMR, at most 64.
// sizing_groups: the number of workers the launch is sized for (0: the upper bound on the number
// of blocks, for allocations).
static bool softmax_rows_wide(int C) { return (C + 7) / 8 * 8 > 4096; }  // eight waves, five vectors per thread

int softmax_ce_bf16_rows_per_block(int N, int sizing_groups, int C) {
  if (sizing_groups <= 0) return SMR;
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else
      return SMR;
  }
  const int places = (softmax_rows_wide(C) ? 2 : 3) * cus;
  const long rows = (long)N * sizing_groups;
  long rpb = (rows + places - 1) / places;
  if (rpb < SMR) rpb = SMR;
  if (rpb > 64) rpb = 64;
  return (int)rpb;
}
int softmax_ce_bf16_row_blocks(int N, int sizing_groups, int C) {
  const int rpb = softmax_ce_bf16_rows_per_block(N, sizing_groups, C);
  return (N + rpb - 1) / rpb;
}

bool softmax_ce_bf16_supported(const float* logits, long ld_l, long s_logits, const void* dlog, long ld_d, long s_d,
                               int C) {
  const int Cw = (C + 7) / 8 * 8;
  return C >= 4 && C <= 1024 * 10 && ((uintptr_t)logits & 15) == 0 && s_logits % 4 == 0 && ld_l % 4 == 0 && ld_l >= Cw &&
         ((uintptr_t)dlog & 7) == 0 && ld_d % 4 == 0 && ld_d >= Cw && s_d % 4 == 0;
}

hipError_t launch_softmax_ce_bf16(const float* logits, long ld_l, long s_logits, const int32_t* y, long s_y, void* dlog,
                                  long ld_d, long s_d, float* rowloss, long s_rowloss, int N, int B, int Bp, int C,
                                  int groups, hipStream_t s, float* colpart, long s_colpart, int sizing_groups) {
  if (!softmax_ce_bf16_supported(logits, ld_l, s_logits, dlog, ld_d, s_d, C) || !colpart || ((uintptr_t)colpart & 15) != 0 ||
      s_colpart % 4 != 0 || B < 1 || Bp < B || N % Bp != 0)
    return hipErrorInvalidValue;
  // bytes: the logits read once (fp32), the logit gradient written in bf16
  KernelTimer kt(KID_SOFTMAX_CE_BF16, 6.0 * N * C * groups, s);
  const int Cw = (C + 7) / 8 * 8;
  const int rpb = softmax_ce_bf16_rows_per_block(N, sizing_groups, C);
  dim3 grid((N + rpb - 1) / rpb, groups);
#define HPSGD_SMR(V4, NT)                                                                                            hipLaunchKernelGGL((softmax_ce_bf16_rows_kernel<V4, NT>), grid, dim3(NT), 0, s, logits, ld_l, s_logits, y, s_y,                       (__bf16*)dlog, ld_d, s_d, rowloss, s_rowloss, colpart, s_colpart, N, B, Bp, C, Cw, rpb)
  if (Cw <= 1024) HPSGD_SMR(1, 256);
  else if (!softmax_rows_wide(Cw)) HPSGD_SMR(4, 256);
  else HPSGD_SMR(5, 512);
#undef HPSGD_SMR
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- matrix-core rate probe
// 16 independent 32x32 accumulator tiles per wave (256 accumulator registers: one wave per
// SIMD), operands fixed in registers: nothing but MFMA issue.  256 workgroups of 4 waves: one
// wave on every SIMD of the chip.  Records the shader-clock and the 100 MHz wall-clock ticks of workgroup 0.
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8p __attribute__((ext_vector_type(8)));

template <bool BF16>
__global__ void __launch_bounds__(256)
mfma_probe_kernel(const unsigned char* __restrict__ operands, int iters, double* __restrict__ result,
                  float* __restrict__ sink) {
  const int tid = threadIdx.x;
  uint4 ra[4], rb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ra[i] = *reinterpret_cast<const uint4*>(operands + ((tid * 4 + i) * 16) % 8192);
    rb[i] = *reinterpret_cast<const uint4*>(operands + 8192 + ((tid * 4 + i) * 16) % 8192);
  }
  floatx16 acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  const long long c0 = clock64(), w0 = wall_clock64();
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (BF16)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8p, ra[i & 3]),
                                                         __builtin_bit_cast(bf16x8p, rb[(i >> 2) & 3]), acc[i], 0, 0, 0);
      else
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, ra[i & 3].x),
                                                      __builtin_bit_cast(float, rb[(i >> 2) & 3].x), acc[i], 0, 0, 0);
    }
  }
  const long long c1 = clock64(), w1 = wall_clock64();
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum += acc[i][v];
  sink[blockIdx.x * 256 + tid] = sum;
  if (blockIdx.x == 0 && tid == 0) {
    result[0] = (double)(c1 - c0);
    result[1] = (double)(w1 - w0);
    result[2] = 16.0 * iters;
    result[3] = BF16 ? 32768.0 : 4096.0;
  }
}

hipError_t launch_mfma_probe(bool bf16, const void* operands, int iterations, double* result, float* sink,
                             hipStream_t s) {
  if (bf16)
    hipLaunchKernelGGL(mfma_probe_kernel<true>, dim3(256), dim3(256), 0, s, (const unsigned char*)operands,
                       iterations, result, sink);
  else
    hipLaunchKernelGGL(mfma_probe_kernel<false>, dim3(256), dim3(256), 0, s, (const unsigned char*)operands,
                       iterations, result, sink);
  return hipGetLastError();
}

}  // namespace hpsgd
