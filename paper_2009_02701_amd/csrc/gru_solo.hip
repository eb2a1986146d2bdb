// The recurrence of a narrow GRU layer with no exchange between workgroups (fp32, H <= 128).
//
// A resident-weight launch (gru_persist.hip) cuts a layer's hidden units over H/16 workgroups, which
// then hand each other h_t (backward: the gate gradients) through memory at every step: 4 to 9 us per
// step, whatever the width.  A layer of up to 128 units needs none of that: W_hh (196 KB at H = 128)
// fits the registers of ONE compute unit, and batch rows are independent of each other.  So here a
// workgroup owns 4 batch rows of one worker (or 8: solo_two_tiles; of very many rows 16, in a form of its own: solo_16_rows)
// and ALL hidden units, and runs all T steps by itself.  There is no flag, no residency requirement and no ordering against other streams:
// any number of workgroups may be launched.  (Two layers that share a launch, below, do have flags: a workgroup waits, a bounded time, for
// such as have drawn a ticket before it, so no residency is required of them either.)
//
// The products are v_mfma_f32_4x4x1_16b_f32 with the first operand broadcast: one instruction of 8 cycles
// multiplies 4 batch rows x 1 step of the contraction with 64 columns of weights, at the full fp32 matrix
// rate and with no row unused, where a 16 x 16 x 4 instruction has 16 rows whatever the batch.  Lane l of a
// weight register holds column l; block b = k % 16 of an operand register is lanes 4b .. 4b+3, one row
// each (row l % 4); accumulator register v of lane l is row v of column l.
//
// The contraction is cut into 4 parts, one per wave (H > 64: the columns into 2 groups too, 8 waves).  A step:
// operands from LDS, products, partial sums to LDS, barrier, cell math of one output per thread and tile
// (a wave has one row and up to 64 neighbouring units: its accesses to memory are whole lines), results to
// LDS, barrier.  Of a forward step of 1.05 us at H = 100, 0.43 us are the matrix instructions (65 per wave, two
// waves per SIMD) and 0.1 the gates; the rest is four trips through LDS and two barriers.
//
// Measured per step, forward / backward, against the form before it (16 x 16 x 4 instructions, 16 rows per
// workgroup): H = 100 batch 20, K = 4: 3.5 / 3.3 -> 1.05 / 1.05 us (two layers of 50 steps 764 -> 308 us a round);
// H = 64, batch 16, K = 1: 2.0 / 1.5 -> 0.8 / 0.6 us.  A local step of 20 time steps at H = 128, K = 16: batch 64
// 290 -> 172 us, batch 128 356 -> 276 us.
//
// Any H from 1 to 128: contraction steps beyond H have zero weights and finite operands, columns beyond
// 3H are not read.  Accesses outside the batch or beyond H carry an out-of-range buffer offset: loads
// give zero, stores are dropped, and the step has no branch around a memory access.
#include <utility>

#include "cell_math.h"
#include "kernels.h"
#include "split_f32.h"

namespace hpsgd {

namespace {

constexpr int kSoloMaxH = 128;
constexpr unsigned kOut = 0x7ffffff0u;  // beyond every buffer's length

inline int solo_tiles(int B) { return (B + 3) / 4; }

// H8 = ceil(H / 8): extents of the launches for a width
template <int H8>
struct Solo {
  static constexpr int CG = H8 > 8 ? 2 : 1;                          // column groups
  static constexpr int NT = 256 * CG;                                // threads: a wave per column group and part
  static constexpr int UP = 64 * CG;                                 // units, padded
  // forward: contraction of a part; column blocks, all of them and those of the first group (its waves and the
  // second group's of the same part share a SIMD, so an odd number is no loss)
  static constexpr int KF = 2 * H8, NF = (24 * H8 + 63) / 64, CF = (NF + CG - 1) / CG;
  static constexpr int KB = 6 * H8;                                  // backward: contraction of a part (one column block per wave)
  // LDS words of a row of h, of gate gradients: the last part's operand chunk ends inside, 16 (mod 64), so that the
  // four rows of a chunk are in different banks
  static constexpr int pitch(int k) { return (3 * k + (k + 15) / 16 * 16 + 47) / 64 * 64 + 16; }
  static constexpr int LF = pitch(KF) > UP ? pitch(KF) : UP + 16, LB = pitch(KB);
  static constexpr int PF = 64 * NF, PB = UP;                        // words of a row of a part's sums
};

template <class F, int... I>
__device__ __forceinline__ void unroll_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(0) .. f(N - 1) with the index a constant expression (the matrix instruction's block index is one)
template <int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
  unroll_seq(f, std::make_integer_sequence<int, N>{});
}

// Every load so far has landed: the compiler then puts no wait for them into the loop behind, where it would
// also wait for the step's own loads and stores.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0), the other counts at their most

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const float* base, long words) {
  const long bytes = words * 4;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)(bytes < 0x7fffffe0L ? bytes : 0x7fffffe0L),
                                           0x00020000);
}
// (DEV: at device scope, for what another workgroup of the launch writes or reads)
template <bool DEV = false>
__device__ __forceinline__ float ld_b32(__amdgpu_buffer_rsrc_t rs, unsigned off, int soff = 0) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, soff, DEV ? 16 : 0));
}
template <bool DEV = false>
__device__ __forceinline__ void st_b32(__amdgpu_buffer_rsrc_t rs, unsigned off, float v, int soff = 0) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, (int)off, soff, DEV ? 16 : 0);
}
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2s __attribute__((ext_vector_type(2)));
typedef unsigned u32x4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ floatx2 ld_b64(__amdgpu_buffer_rsrc_t rs, unsigned off) {
  return __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0));
}
__device__ __forceinline__ floatx4 ld_b128(__amdgpu_buffer_rsrc_t rs, unsigned off) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
}
__device__ __forceinline__ void st_b128(__amdgpu_buffer_rsrc_t rs, unsigned off, floatx4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4s, v), rs, (int)off, 0, 0);
}

// Two layers in one launch (gru_stack_*_kernel, below): the workgroups that pass a tile's values on.
constexpr int kChunk = 4;  // steps that are passed on together
// out: this workgroup's words, one per wave, which its waves set to the number of steps they have written (nullptr: nobody waits
// for it); in: the words of the workgroups that it waits for, those of even chunks, then those of odd ones.
struct SoloLink {
  unsigned *out, *in, *abort_w;
  unsigned limit;
  int n_in;
};
// A wave waits until the `n` words at w have reached `target`.  false: given up (limit polls, or another workgroup has given up);
// the abort word is then set.  limit == 0: every wait is.
// (NAP: 64 cycles each between two looks; looks of hundreds of waves are traffic that the values have to get through)
template <int NAP>
__device__ __forceinline__ bool link_wait(unsigned* w, int n, unsigned target, unsigned* abort_w, unsigned limit) {
  const int l = threadIdx.x & 63;
  bool ok = limit != 0;
  for (unsigned i = 0; ok; ++i) {
    const unsigned v = __hip_atomic_load(w + (l < n ? l : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__all(v >= target)) break;
    if (i >= limit || (i % 16 == 15 && __hip_atomic_load(abort_w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)) ok = false;
    else __builtin_amdgcn_s_sleep(NAP);
  }
  if (!ok && l == 0) __hip_atomic_store(abort_w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" ::: "memory");  // (what is waited for is loaded behind the wait)
  return ok;
}
// This wave's stores so far, all at device scope, are where the others see them (vmcnt(0): a write-through store is counted out
// when the level that all XCDs share has acknowledged it); then its word.
__device__ __forceinline__ void link_publish(unsigned* w, unsigned steps) {
  __builtin_amdgcn_s_waitcnt(0x0f70);
  asm volatile("" ::: "memory");
  if ((threadIdx.x & 63) == 0) __hip_atomic_store(w, steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the chunk of step index `it` (its first) is there
__device__ __forceinline__ bool link_chunk(const SoloLink& k, int it, int T) {
  const int c = it / kChunk;
  return link_wait<2>(k.in + (c & 1) * 8, k.n_in, (unsigned)min(it + kChunk, T), k.abort_w, k.limit);
}

// gx: input projections, b_ih included.  hs: h_0 .. h_T ((T+1) blocks of B x H; h_0 = 0 is written here).
// sv: (r, z, n, q) of one output as one 16-byte word, [step][tile][row][unit].
// R tiles of 4 rows, from tile ty of worker g.  LINKED: in a launch of two layers; k.in: gx is written by this launch.
template <int H8, int R, bool LINKED>
__device__ __forceinline__ void solo_fwd_body(const float* __restrict__ W_hh, const float* __restrict__ b_hh, long s_rep,
                                              const float* __restrict__ gx, long s_gx, float* __restrict__ hs, long s_hs,
                                              float* __restrict__ sv, long s_sv, int B, int H, int T, int RT, int g, int ty,
                                              const SoloLink& k) {
  using S = Solo<H8>;
  constexpr int KW = S::KF, CB = S::CF, NC = (KW + 15) / 16;
  __shared__ float hl[R * 4 * S::LF];
  __shared__ float part[R * 16 * S::PF];  // [tile][part][row][column]
  // (the wave's number in a scalar register: buffer descriptors derived from it stay scalar)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = w & 3, cg = w >> 2;  // part of the contraction, column group
  // column c = q * H + unit of the products is row c of W_hh
  float wt[CB][KW];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_of(W_hh + g * s_rep, 3L * H * H);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int col = (cg * CB + cb) * 64 + lane;
      if ((H & 1) == 0) {  // (whole 8-byte pieces of a row)
#pragma unroll
        for (int i = 0; i < KW; i += 2) {
          const int k = s * KW + i;
          const floatx2 v = ld_b64(rw, col < 3 * H && k < H ? (unsigned)(col * H + k) * 4u : kOut);
          wt[cb][i] = v[0];
          wt[cb][i + 1] = v[1];
        }
      } else {
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          const int k = s * KW + i;
          wt[cb][i] = ld_b32(rw, col < 3 * H && k < H ? (unsigned)(col * H + k) * 4u : kOut);
        }
      }
    }
  }
  const int j = cg * 64 + lane, m = w & 3;  // this thread's unit and its row of a tile
  const bool act = j < H;
  float bias[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) bias[q] = act ? (b_hh + g * s_rep)[q * H + j] : 0.f;
  // byte offsets of this thread's outputs inside a step's block of gx, of hs and of the saved gates
  unsigned ox[R], oh[R], ov[R];
  float hp[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = 4 * (ty + r) + m;
    const bool ok = act && row < B;
    ox[r] = ok ? (unsigned)(row * 3 * H + j) * 4u : kOut;
    oh[r] = ok ? (unsigned)(row * H + j) * 4u : kOut;
    ov[r] = ok ? (unsigned)((4 * r + m) * H + j) * 16u : kOut;
    hp[r] = 0.f;
  }
  const float* gxg = gx + g * s_gx;
  float* hsg = hs + g * s_hs;
  float* svg = sv + g * s_sv + (long)ty * 16 * H;
  const long sv_step = (long)RT * 16 * H, BH = (long)B * H;
  {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(hsg, BH);
#pragma unroll
    for (int r = 0; r < R; ++r) st_b32(rs, oh[r], 0.f);
  }
  for (int i = tid; i < R * 4 * S::LF; i += S::NT) hl[i] = 0.f;
  struct In { float x[R][3]; };
  auto load_gx = [&](int t, In& I) {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(gxg + (long)min(t, T - 1) * 3 * BH, 3 * BH);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 3; ++q) I.x[r][q] = ld_b32<LINKED>(rs, ox[r], q * H * 4);
  };
  // (a wait that was given up: every output from there on is NaN)
  auto wait_gx = [&](int it) {
    if (LINKED && k.in && it < T && it % kChunk == 0 && !link_chunk(k, it, T)) bias[0] = bias[1] = bias[2] = __builtin_nanf("");
  };
  In ia, ib;
  wait_gx(0);
  load_gx(0, ia);
  load_gx(1, ib);
  wait_loads();
  __syncthreads();
  // one step; I holds its input projection and receives the one of step t + 2
  auto step = [&](int t, In& I) {
    float a[R][NC];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) a[r][c] = hl[(4 * r + (lane & 3)) * S::LF + s * KW + 16 * c + (lane >> 2)];
    auto products = [&](auto n) {
      constexpr int N = n;
      floatx4 acc[R][N];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int cb = 0; cb < N; ++cb) acc[r][cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
      unroll<KW>([&](auto k) {
#pragma unroll
        for (int cb = 0; cb < N; ++cb)
#pragma unroll
          for (int r = 0; r < R; ++r)
            acc[r][cb] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[r][k / 16], wt[cb][k], acc[r][cb], 4, k % 16, 0);
      });
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int cb = 0; cb < N; ++cb)
#pragma unroll
          for (int v = 0; v < 4; ++v) part[((4 * r + s) * 4 + v) * S::PF + (cg * CB + cb) * 64 + lane] = acc[r][cb][v];
    };
    if (cg == 0) products(std::integral_constant<int, CB>{});
    else products(std::integral_constant<int, S::NF - CB>{});
    __syncthreads();
    if (LINKED && k.out && t > 0 && t % kChunk == 0) link_publish(k.out + w, t);  // (the stores of step t - 1 are a while ago)
    const __amdgpu_buffer_rsrc_t ro = rsrc_of(hsg + (long)(t + 1) * BH, BH), rv = rsrc_of(svg + (long)t * sv_step, R * 16L * H);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float y[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float* p = &part[(16 * r + m) * S::PF + min(q * H + j, S::PF - 1)];
        y[q] = (p[0] + p[4 * S::PF]) + (p[8 * S::PF] + p[12 * S::PF]) + bias[q];
      }
      const float rr = sigm_f32(I.x[r][0] + y[0]), zz = sigm_f32(I.x[r][1] + y[1]), nn = tanh_f32(I.x[r][2] + rr * y[2]);
      hp[r] = (1.0f - zz) * nn + zz * hp[r];
      hl[(4 * r + m) * S::LF + j] = act ? hp[r] : 0.f;
      st_b32<LINKED>(ro, oh[r], hp[r]);
      st_b128(rv, ov[r], (floatx4){rr, zz, nn, y[2]});
    }
    wait_gx(t + 2);
    load_gx(t + 2, I);
    __syncthreads();
  };
  int t = 0;
  for (; t + 1 < T; t += 2) {
    step(t, ia);
    step(t + 1, ib);
  }
  if (t < T) step(t, ia);
  if (LINKED && k.out) link_publish(k.out + w, T);
}

// BPTT of all steps.  dgx / dgh: gate gradients (blocks of B x 3H).  D: the gradient carried into the
// last step (nullptr: zero); above: per-step gradient from the layer above (blocks of B x H) or
// nullptr.  dbp[(g * RT + tile)][6H]: partial sums of the bias gradients (b_ih: r z n, b_hh: r z q).
// (LINKED: k.in: `above` is written by this launch.)
template <int H8, int R, bool LINKED>
__device__ __forceinline__ void solo_bwd_body(const float* __restrict__ W_hh, long s_rep, float* __restrict__ dgx,
                                              float* __restrict__ dgh, long s_dg, const float* __restrict__ D, long s_D,
                                              const float* __restrict__ above, long s_above, const float* __restrict__ sv,
                                              long s_sv, const float* __restrict__ hs, long s_hs, float* __restrict__ dbp,
                                              int B, int H, int T, int RT, int g, int ty, const SoloLink& k) {
  using S = Solo<H8>;
  constexpr int KW = S::KB, NC = (KW + 15) / 16;
  __shared__ float dl[R * 4 * S::LB];
  __shared__ float part[R * 16 * S::PB];  // [tile][part][row][unit]
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = w & 3, cg = w >> 2;
  // the contraction runs over the rows of W_hh, q * H + unit; column j is its column j
  float wt[KW];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_of(W_hh + g * s_rep, 3L * H * H);
    const int col = cg * 64 + lane;
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const int k = s * KW + i;
      wt[i] = ld_b32(rw, col < H && k < 3 * H ? (unsigned)(k * H + col) * 4u : kOut);
    }
  }
  const int j = cg * 64 + lane, m = w & 3;
  const bool act = j < H;
  unsigned ox[R], oh[R], ov[R];
  float dc[R], bs[R][4];
  const long BH = (long)B * H;
  const __amdgpu_buffer_rsrc_t rD = rsrc_of(D ? D + g * s_D : hs, D ? BH : 0);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = 4 * (ty + r) + m;
    const bool ok = act && row < B;
    ox[r] = ok ? (unsigned)(row * 3 * H + j) * 4u : kOut;
    oh[r] = ok ? (unsigned)(row * H + j) * 4u : kOut;
    ov[r] = ok ? (unsigned)((4 * r + m) * H + j) * 16u : kOut;
    dc[r] = ld_b32(rD, oh[r]);
#pragma unroll
    for (int i = 0; i < 4; ++i) bs[r][i] = 0.f;
  }
  const float* hsg = hs + g * s_hs;
  const float* abg = above ? above + g * s_above : hs;
  const float* svg = sv + g * s_sv + (long)ty * 16 * H;
  const long sv_step = (long)RT * 16 * H;
  struct In { floatx4 s[R]; float hp[R], ab[R]; };
  auto load_in = [&](int t, In& I) {
    const int tc = max(t, 0);
    const __amdgpu_buffer_rsrc_t rv = rsrc_of(svg + (long)tc * sv_step, R * 16L * H), rh = rsrc_of(hsg + (long)tc * BH, BH),
                                 ra = rsrc_of(abg + (long)tc * BH, above ? BH : 0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      I.s[r] = ld_b128(rv, ov[r]);
      I.hp[r] = ld_b32(rh, oh[r]);
      I.ab[r] = ld_b32<LINKED>(ra, oh[r]);
    }
  };
  auto wait_above = [&](int t) {
    if (LINKED && k.in && t >= 0 && (T - 1 - t) % kChunk == 0 && !link_chunk(k, T - 1 - t, T)) {
#pragma unroll
      for (int r = 0; r < R; ++r) dc[r] = __builtin_nanf("");
    }
  };
  In ia, ib;
  wait_above(T - 1);
  load_in(T - 1, ia);
  load_in(T - 2, ib);
  for (int i = tid; i < R * 4 * S::LB; i += S::NT) dl[i] = 0.f;
  static_assert(S::LB > 24 * H8, "a word beyond the gate gradients of a row");
  // where this thread's gate gradients go, r, z and q (a thread without an output: that word)
  const int od = act ? j : S::LB - 1, oq = act ? H : 0;
  wait_loads();
  __syncthreads();
  auto step = [&](int t, In& I) {
    float a[R][NC];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) a[r][c] = dl[(4 * r + (lane & 3)) * S::LB + s * KW + 16 * c + (lane >> 2)];
    floatx4 acc[R][2];  // (two chains: an instruction does not wait for the one before it)
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r][0] = acc[r][1] = (floatx4){0.f, 0.f, 0.f, 0.f};
    unroll<KW>([&](auto k) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        acc[r][k & 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[r][k / 16], wt[k], acc[r][k & 1], 4, k % 16, 0);
    });
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[((4 * r + s) * 4 + v) * S::PB + cg * 64 + lane] = acc[r][0][v] + acc[r][1][v];
    __syncthreads();
    if (LINKED && k.out && t < T - 1 && (T - 1 - t) % kChunk == 0) link_publish(k.out + w, T - 1 - t);
    const __amdgpu_buffer_rsrc_t rx = rsrc_of(dgx + g * s_dg + (long)t * 3 * BH, 3 * BH),
                                 rh = rsrc_of(dgh + g * s_dg + (long)t * 3 * BH, 3 * BH);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // (outside the batch every input is zero, and so is every gradient)
      const float* p = &part[(16 * r + m) * S::PB + j];
      const float rr = I.s[r][0], z = I.s[r][1], n = I.s[r][2], q = I.s[r][3];
      const float dh = (dc[r] + I.ab[r]) + ((p[0] + p[4 * S::PB]) + (p[8 * S::PB] + p[12 * S::PB]));
      const float dn = dh * (1.0f - z);
      const float dz = dh * (I.hp[r] - n);
      const float da_n = dn * (1.0f - n * n);
      const float dq = da_n * rr;
      const float da_r = da_n * q * rr * (1.0f - rr);
      const float da_z = dz * z * (1.0f - z);
      dc[r] = dh * z;
      float* o = &dl[(4 * r + m) * S::LB + od];
      o[0] = act ? da_r : 0.f;
      o[oq] = act ? da_z : 0.f;
      o[2 * oq] = act ? dq : 0.f;
      bs[r][0] += da_r;
      bs[r][1] += da_z;
      bs[r][2] += da_n;
      bs[r][3] += dq;
      st_b32<LINKED>(rx, ox[r], da_r);
      st_b32<LINKED>(rx, ox[r], da_z, H * 4);
      st_b32<LINKED>(rx, ox[r], da_n, H * 8);
      st_b32(rh, ox[r], da_r);
      st_b32(rh, ox[r], da_z, H * 4);
      st_b32(rh, ox[r], dq, H * 8);
    }
    wait_above(t - 2);
    load_in(t - 2, I);
    __syncthreads();
  };
  int t = T - 1;
  for (; t >= 1; t -= 2) {
    step(t, ia);
    step(t - 1, ib);
  }
  if (t >= 0) step(t, ia);
  if (LINKED && k.out) link_publish(k.out + w, T);
  // bias gradients: a tile's sums over its four rows are its own, whatever R is
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[((4 * r + i) * 4 + m) * S::PB + j] = bs[r][i];
  __syncthreads();
  if (m != 0 || !act) return;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (ty + r >= RT) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* p = &part[(4 * r + i) * 4 * S::PB + j];
      bs[r][i] = (p[0] + p[S::PB]) + (p[2 * S::PB] + p[3 * S::PB]);
    }
    float* out = dbp + (long)(g * RT + ty + r) * 6 * H;
    out[j] = out[3 * H + j] = bs[r][0];
    out[H + j] = out[4 * H + j] = bs[r][1];
    out[2 * H + j] = bs[r][2];
    out[5 * H + j] = bs[r][3];
  }
}

}  // namespace

// grid: groups * ceil(RT / R) workgroups; RT = ceil(B / 4) tiles of 4 rows, R of them per workgroup.
template <int H8, int R>
__global__ void __launch_bounds__(Solo<H8>::NT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_solo_fwd_kernel(const float* __restrict__ W_hh, const float* __restrict__ b_hh, long s_rep,
                    const float* __restrict__ gx, long s_gx, float* __restrict__ hs, long s_hs, float* __restrict__ sv,
                    long s_sv, int B, int H, int T, int RT) {
  const int n_wg = (RT + R - 1) / R, g = blockIdx.x / n_wg, ty = (blockIdx.x - g * n_wg) * R;
  solo_fwd_body<H8, R, false>(W_hh, b_hh, s_rep, gx, s_gx, hs, s_hs, sv, s_sv, B, H, T, RT, g, ty, SoloLink{});
}
template <int H8, int R>
__global__ void __launch_bounds__(Solo<H8>::NT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_solo_bwd_kernel(const float* __restrict__ W_hh, long s_rep, float* __restrict__ dgx, float* __restrict__ dgh, long s_dg,
                    const float* __restrict__ D, long s_D, const float* __restrict__ above, long s_above,
                    const float* __restrict__ sv, long s_sv, const float* __restrict__ hs, long s_hs, float* __restrict__ dbp,
                    int B, int H, int T, int RT) {
  const int n_wg = (RT + R - 1) / R, g = blockIdx.x / n_wg, ty = (blockIdx.x - g * n_wg) * R;
  solo_bwd_body<H8, R, false>(W_hh, s_rep, dgx, dgh, s_dg, D, s_D, above, s_above, sv, s_sv, hs, s_hs, dbp, B, H, T, RT, g, ty,
                              SoloLink{});
}

// ---------------------------------------------------------------------------- two layers in one launch
// Two layers one after the other are twice the chain of steps, on as few workgroups as a batch has tiles: 20 of 256 CUs at
// batch 20 and 4 workers.  But a layer's step t needs no more of the layer below than its step t (backward: of the one above), for
// the same rows.  So one launch has a workgroup per tile of 4 rows and layer, and between them two that multiply
// what the first passes on - the steps' h with the upper layer's W_ih, backward its gate gradients with W_ih^T - four steps at a time, the
// even chunks and the odd ones: the upper layer runs about ten steps behind, and the product that stood between
// the layers' launches goes too.  What is passed on goes through memory at device scope; a wave counts the steps that it has written in
// a word of its own (link_publish), once every four, half a step after the last one's stores; the reader polls the
// words of all of a workgroup's waves.
// A workgroup takes its part by ticket, in the order in which workgroups start, and waits only for those of lower tickets, which
// run or have run: whatever else is on the chip, nothing waits for a place.  Every wait is bounded all the same: a given-up one
// sets the abort word and makes NaN of everything behind it in the chain.  What a caller sees of it, NaN in the losses and the replicas' first
// parameters, is written behind the step where the abort word is set (launch_poison_on_abort).
namespace {

// Extents of the product between the layers: W_ih split into bf16 parts in registers, NB blocks of 16 columns per wave, KC chunks of 32.
template <int H8, bool BWD>
struct LinkShape {
  static constexpr int W = Solo<H8>::NT / 64;
  static constexpr int NB = ((BWD ? 8 * H8 : 24 * H8) / 16 + ((BWD ? 8 * H8 : 24 * H8) % 16 ? 1 : 0) + W - 1) / W;
  static constexpr int KC = ((BWD ? 24 * H8 : 8 * H8) + 31) / 32;
};

// The chunks c = odd, odd + 2, .. of a tile.  Forward: out[t] = in[t] W^T + bias, backward out[t] = in[t] W, over t from the end.
// W: 3H x H, row-major.  in: blocks of B x KD, out: blocks of B x ND.  Row m = 4 s + r of a product is row r of the tile at the chunk's step s.
// A product of a launch of its own has the fp32 instruction at these sizes.  The split is as exact for operands of at least 2^-110; a chunk with a
// smaller one (zero is none), and every chunk of a wave with such a weight, takes that instruction too.
template <int H8, bool BWD>
__device__ __forceinline__ void link_body(const float* __restrict__ W, const float* __restrict__ bias, const float* in, float* out, int B,
                                          int H, int T, int ty, int odd, unsigned* in_words, unsigned* out_words, unsigned* abort_w,
                                          unsigned limit) {
  using L = LinkShape<H8, BWD>;
  constexpr int NB = L::NB, KC = L::KC;
  __shared__ u32x4s al[KC * 3 * 64];  // the chunk's operands, split: [chunk of 32][part][lane]
  __shared__ int go, low[L::W];       // low: a wave has split an operand below 2^-110
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lg = lane >> 4;
  const int KD = BWD ? 3 * H : H, ND = BWD ? H : 3 * H;
  // (a piece of four at the end of `in` may reach three words beyond it)
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(W, 3L * H * H), ri = rsrc_of(in, (long)T * B * KD + 3), ro = rsrc_of(out, (long)T * B * ND);
  auto col = [&](int b) { return (w * NB + b) * 16 + lr; };
  auto w_frag = [&](int b, int c, int H, float4 (&v)[2]) {
    const int n = col(b);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 32 * c + 16 * h + 4 * lg + i;
        e[i] = ld_b32(rw, n < (BWD ? H : 3 * H) && k < (BWD ? 3 * H : H) ? (unsigned)(BWD ? k * H + n : n * H + k) * 4u : kOut);
      }
      v[h] = make_float4(e[0], e[1], e[2], e[3]);
    }
  };
  SplitFrag wf[KC][NB];
  bool low_w = false;
#pragma unroll
  for (int c = 0; c < KC; ++c)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float4 v[2];
      w_frag(b, c, H, v);
      low_w = low_w || split_below(v[0], v[1]);
      wf[c][b] = split_frag(v[0], v[1]);
      __builtin_amdgcn_sched_barrier(0);  // (or the pieces of all chunks take registers at once)
    }
  low_w = __any(low_w) != 0;
  float bv[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) bv[b] = !BWD && col(b) < 3 * H ? bias[col(b)] : 0.f;
  bool ok = true;
  for (int i0 = odd * kChunk; i0 < T; i0 += 2 * kChunk) {
    if (w == 0) {
      ok = ok && link_wait<8>(in_words, L::W, (unsigned)min(i0 + kChunk, T), abort_w, limit);
      if (lane == 0) go = ok;
    }
    __syncthreads();  // (and everyone has read the operands of the chunk before)
    ok = go != 0;
    // this lane's operand row, and its first output row
    const int ia = i0 + (lr >> 2), ra = 4 * ty + (lr & 3), io = i0 + lg;
    const unsigned off_a = ia < T && ra < B ? (unsigned)(((BWD ? T - 1 - ia : ia) * B + ra) * KD) * 4u : kOut;
    auto a_frag = [&](int c, int KD, float4 (&v)[2]) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = 32 * c + 16 * h + 4 * lg;
        v[h] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(ri, (int)(off_a != kOut && k < KD ? off_a + 4u * k : kOut), 0, 16));
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // (the next row's values)
        const int k = 32 * c + 16 * h + 4 * lg;
        v[h].y = k + 1 < KD ? v[h].y : 0.f;
        v[h].z = k + 2 < KD ? v[h].z : 0.f;
        v[h].w = k + 3 < KD ? v[h].w : 0.f;
      }
    };
    bool low_a = false;
#pragma unroll
    for (int i = 0; i < (KC + L::W - 1) / L::W; ++i) {
      const int c = w + i * L::W;
      if (c < KC) {  // (uniform)
        float4 v[2];
        a_frag(c, KD, v);
        low_a = low_a || split_below(v[0], v[1]);
        const SplitFrag f = split_frag(v[0], v[1]);
#pragma unroll
        for (int p = 0; p < 3; ++p) al[(c * 3 + p) * 64 + lane] = __builtin_bit_cast(u32x4s, f.p[p]);
      }
    }
    low_a = __any(low_a) != 0;
    if (lane == 0) low[w] = low_a;
    __syncthreads();
    const bool again = low_w || __any(low[lane & (L::W - 1)]);
    floatx4 big[NB], small[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) big[b] = small[b] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      SplitFrag f;
#pragma unroll
      for (int p = 0; p < 3; ++p) f.p[p] = __builtin_bit_cast(bf16x8s, al[(c * 3 + p) * 64 + lane]);
      split_mfmas(f, wf[c], big, small);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      big[b] += small[b];
      if (__builtin_expect(again || any_beyond(big[b]), 0)) {  // with the fp32 instruction
        const int Hr = rarely(H);
        big[b] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int c = 0; c < KC; ++c) {
          float4 v[2], x[2];
          a_frag(c, BWD ? 3 * Hr : Hr, x);
          w_frag(b, c, Hr, v);
          plain_mfmas(x, v, true, big[b]);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 4 * ty + v, n = col(b);
        st_b32<true>(ro, io < T && row < B && n < ND ? (unsigned)(((BWD ? T - 1 - io : io) * B + row) * ND + n) * 4u : kOut,
                     ok ? big[b][v] + bv[b] : __builtin_nanf(""));
      }
    }
    link_publish(out_words + w, (unsigned)min(i0 + kChunk, T));
  }
}

// A tile's words: its lower workgroup's waves' (8), then those of the two that multiply (8 each); the backward launch's in the second half
// of its 64.  (Word 32, which may be the first of a worker's slice, is nobody's.)
constexpr int kLinkWords = 64, kLinkBase = 32 * 9;
// A workgroup's part: ticket i of class blockIdx.x % 8 (often an XCD) is role i / m of the class's tile i % m, m = ceil(n / 8), n = groups * RT:
// the layer that goes first, the products of even and of odd chunks, the other layer.  (One counter for all: its 500 additions one after the other
// were 13 us.)  which: 0 forward, 1 backward.  false: the class has one tile less.
__device__ __forceinline__ bool link_part(unsigned* sync, int which, int n, int& role, int& tile) {
  __shared__ int mine;
  const int cls = blockIdx.x & 7, m = (n + 7) / 8;
  if (threadIdx.x == 0)
    mine = (int)__hip_atomic_fetch_add(sync + 32 * (1 + cls) + 8 + which, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane(mine);
  role = ticket / m;
  tile = cls + 8 * (ticket - role * m);
  return tile < n;
}

}  // namespace

// grid: 32 ceil(n / 8).  sync: the abort word; the counters of tickets, in lines of their own; the tiles' words from kLinkBase on.
template <int H8>
__global__ void __launch_bounds__(Solo<H8>::NT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_stack_fwd_kernel(GruStackLayer lo, GruStackLayer up, const float* W_ih, const float* b_ih, long s_rep, long s_gx, long s_hs,
                     long s_sv, int B, int H, int T, int RT, int n, unsigned* sync, unsigned limit) {
  constexpr int W = Solo<H8>::NT / 64;
  int role, tile;
  if (!link_part(sync, 0, n, role, tile)) return;
  const int g = tile / RT, ty = tile - g * RT;
  unsigned* words = sync + kLinkBase + (long)tile * kLinkWords;
  if (role == 0) {
    solo_fwd_body<H8, 1, true>(lo.W_hh, lo.b_hh, s_rep, lo.gx, s_gx, lo.hs, s_hs, lo.sv, s_sv, B, H, T, RT, g, ty,
                               SoloLink{words, nullptr, sync, limit, 0});
  } else if (role < 3) {
    link_body<H8, false>(W_ih + g * s_rep, b_ih + g * s_rep, lo.hs + g * s_hs + (long)B * H, up.gx + g * s_gx, B, H, T, ty, role - 1,
                         words, words + 8 * role, sync, limit);
  } else {
    solo_fwd_body<H8, 1, true>(up.W_hh, up.b_hh, s_rep, up.gx, s_gx, up.hs, s_hs, up.sv, s_sv, B, H, T, RT, g, ty,
                               SoloLink{nullptr, words + 8, sync, limit, W});
  }
}

// D, above: of the upper layer; dx: the gradient that it passes on (T blocks of B x H)
template <int H8>
__global__ void __launch_bounds__(Solo<H8>::NT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_stack_bwd_kernel(GruStackLayer lo, GruStackLayer up, const float* W_ih, long s_rep, const float* D, long s_D, const float* above,
                     long s_above, float* dx, long s_dx, long s_gx, long s_hs, long s_sv, int B, int H, int T, int RT, int n,
                     unsigned* sync, unsigned limit) {
  constexpr int W = Solo<H8>::NT / 64;
  int role, tile;
  if (!link_part(sync, 1, n, role, tile)) return;
  const int g = tile / RT, ty = tile - g * RT;
  unsigned* words = sync + kLinkBase + (long)tile * kLinkWords + 36;
  if (role == 0) {
    solo_bwd_body<H8, 1, true>(up.W_hh, s_rep, up.gx, up.dgh, s_gx, D, s_D, above, s_above, up.sv, s_sv, up.hs, s_hs, up.dbp, B, H, T, RT,
                               g, ty, SoloLink{words, nullptr, sync, limit, 0});
  } else if (role < 3) {
    link_body<H8, true>(W_ih + g * s_rep, nullptr, up.gx + g * s_gx, dx + g * s_dx, B, H, T, ty, role - 1, words, words + 8 * role, sync, limit);
  } else {
    solo_bwd_body<H8, 1, true>(lo.W_hh, s_rep, lo.gx, lo.dgh, s_gx, nullptr, 0, dx, s_dx, lo.sv, s_sv, lo.hs, s_hs, lo.dbp, B, H, T, RT,
                               g, ty, SoloLink{nullptr, words + 8, sync, limit, W});
  }
}

// ---------------------------------------------------------------------------- many rows: 16 per workgroup
// Where every CU has several tiles of 4 rows anyway, the extra waves and partial sums of the form above are no help:
// here a workgroup owns up to 16 rows and wave w the weights of units 16w .. 16w+15 (3 gates x H, at most 96 registers per
// lane), all of the contraction, so that a step is one trip through LDS and one barrier, and a SIMD's second wave
// multiplies while the first has its cell math.
//
// v_mfma_f32_16x16x4_f32 lane layout: A lane l holds A[m = l%16][k = l/16], B lane l holds
// B[k = l/16][n = l%16], accumulator register v holds C[4*(l/16) + v][l%16].  The contraction index is
// taken in the order k = 16c + 4*(l/16) + e (c-th chunk, e-th instruction), so that a lane reads its
// A values of four instructions as one 16-byte LDS word.  All three gates of a unit are accumulated by
// the same lane: the cell math needs nothing of another lane.  Matrix row m = 4*lg + v is batch row
// r0 + 4*v + lg: a tile of n rows fills ceil(n/4) of the four registers in every lane group, and
// the cell math of the others is skipped.
namespace {

inline int solo16_tiles(int B) { return (B + 15) / 16; }

// Saved gates: (r, z, n, q) of one output as one 16-byte word, in the order the backward launch's lanes
// read them: [step][row tile][unit block][register v][lane].
template <int HB>
__device__ __forceinline__ long sv_block() { return (long)HB * 4 * 64 * 4; }

}  // namespace

// grid: groups * RT workgroups of HB waves (HB = ceil(H / 16)).  gx: input projections, b_ih included.
// hs: h_0 .. h_T ((T+1) blocks of B x H; h_0 = 0 is written here).
template <int HB>
__global__ void __launch_bounds__(64 * HB) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_solo16_fwd_kernel(const float* __restrict__ W_hh, const float* __restrict__ b_hh, long s_rep,
                    const float* __restrict__ gx, long s_gx, float* __restrict__ hs, long s_hs, float* __restrict__ sv,
                    long s_sv, int B, int H, int T, int RT) {
  constexpr int HP = 16 * HB, LP = HP + 4;  // LDS pitch: an odd number of 16-byte words, no bank conflicts
  __shared__ __attribute__((aligned(16))) float hb[2][16 * LP];
  // (the wave's number in a scalar register: buffer descriptors derived from it stay scalar)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int g = blockIdx.x / RT, ty = blockIdx.x - g * RT;
  const int r0 = 16 * ty, nrow = min(16, B - r0), nv = (nrow + 3) >> 2;
  const int j = 16 * w + lr;
  const bool jok = j < H;
  float wt[3][4 * HB];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_of(W_hh + g * s_rep, 3L * H * H);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int c = 0; c < HB; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 16 * c + 4 * lg + e;
          wt[q][4 * c + e] = ld_b32(rw, jok && k < H ? (unsigned)((q * H + j) * H + k) * 4u : kOut);
        }
  }
  float bias[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) bias[q] = jok ? (b_hh + g * s_rep)[q * H + j] : 0.f;
  // byte offsets of this lane's four outputs inside a step's block of gx and of hs
  unsigned ox[4], oh[4];
  float hp[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = r0 + 4 * v + lg;
    const bool ok = jok && 4 * v + lg < nrow;
    ox[v] = ok ? (unsigned)(row * 3 * H + j) * 4u : kOut;
    oh[v] = ok ? (unsigned)(row * H + j) * 4u : kOut;
    hp[v] = 0.f;
  }
  const float* gxg = gx + g * s_gx;
  float* hsg = hs + g * s_hs;
  float* svg = sv + g * s_sv + ((long)ty * HB + w) * 1024 + lane * 4;
  const long sv_step = (long)RT * sv_block<HB>();
  const long BH = (long)B * H;
  {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(hsg, BH);
#pragma unroll
    for (int v = 0; v < 4; ++v) st_b32(rs, oh[v], 0.f);
  }
  for (int i = tid; i < 16 * LP; i += 64 * HB) hb[0][i] = 0.f;
  auto load_gx = [&](int t, float (&G)[3][4]) {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(gxg + (long)min(t, T - 1) * 3 * BH, 3 * BH);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) G[q][v] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)ox[v], q * H * 4, 0));
  };
  float ga[3][4], gb[3][4];
  load_gx(0, ga);
  load_gx(1, gb);
  __syncthreads();
  // one step; G holds its input projection and receives the one of step t + 2
  auto step = [&](int t, const float* hin, float* hout, float (&G)[3][4]) {
    floatx4 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) acc[q] = (floatx4){bias[q], bias[q], bias[q], bias[q]};
    floatx4 a[HB];
#pragma unroll
    for (int c = 0; c < HB; ++c) a[c] = *reinterpret_cast<const floatx4*>(&hin[lr * LP + 16 * c + 4 * lg]);
    __builtin_amdgcn_sched_barrier(0);  // every LDS read is issued before the first product waits for one
#pragma unroll
    for (int c = 0; c < HB; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][e], wt[q][4 * c + e], acc[q], 0, 0, 0);
    float rr[4], zz[4], nn[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      rr[v] = zz[v] = nn[v] = 0.f;
      if (v < nv) {  // uniform
        rr[v] = sigm_f32(G[0][v] + acc[0][v]);
        zz[v] = sigm_f32(G[1][v] + acc[1][v]);
        nn[v] = tanh_f32(G[2][v] + rr[v] * acc[2][v]);
        hp[v] = (1.0f - zz[v]) * nn[v] + zz[v] * hp[v];
        hout[(4 * lg + v) * LP + j] = hp[v];
      }
    }
    load_gx(t + 2, G);
    const __amdgpu_buffer_rsrc_t ro = rsrc_of(hsg + (long)(t + 1) * BH, BH);
#pragma unroll
    for (int v = 0; v < 4; ++v) st_b32(ro, oh[v], hp[v]);
    const __amdgpu_buffer_rsrc_t rv = rsrc_of(svg + (long)t * sv_step - lane * 4, 1024);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      st_b128(rv, v < nv ? (unsigned)(v * 64 + lane) * 16u : kOut, (floatx4){rr[v], zz[v], nn[v], acc[2][v]});
    __syncthreads();
  };
  // (rows of hb[1] that no output lane writes are multiplied into outputs nobody stores; they must
  // only be finite)
  for (int i = tid; i < 16 * LP; i += 64 * HB) hb[1][i] = 0.f;
  __syncthreads();
  // the first of a SIMD's two waves goes ahead: its cell math then runs under the other's products
  if (HB > 4 && w < 4) __builtin_amdgcn_s_setprio(2);
  int t = 0;
  for (; t + 1 < T; t += 2) {
    step(t, hb[0], hb[1], ga);
    step(t + 1, hb[1], hb[0], gb);
  }
  if (t < T) step(t, hb[0], hb[1], ga);
}

// (arguments as of the 4-row launch)
template <int HB>
__global__ void __launch_bounds__(64 * HB) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_solo16_bwd_kernel(const float* __restrict__ W_hh, long s_rep, float* __restrict__ dgx, float* __restrict__ dgh, long s_dg,
                    const float* __restrict__ D, long s_D, const float* __restrict__ above, long s_above,
                    const float* __restrict__ sv, long s_sv, const float* __restrict__ hs, long s_hs, float* __restrict__ dbp,
                    int B, int H, int T, int RT) {
  constexpr int HP = 16 * HB, LP = 3 * HP + 4;
  __shared__ __attribute__((aligned(16))) float db[2][16 * LP];
  // (the wave's number in a scalar register: buffer descriptors derived from it stay scalar)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int g = blockIdx.x / RT, ty = blockIdx.x - g * RT;
  const int r0 = 16 * ty, nrow = min(16, B - r0);
  const int j = 16 * w + lr;
  const bool jok = j < H;
  // B[k][n] = W_hh[q*H + k][j]: the transposed weights, 64-byte pieces of rows
  float wt[3][4 * HB];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_of(W_hh + g * s_rep, 3L * H * H);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int c = 0; c < HB; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 16 * c + 4 * lg + e;
          wt[q][4 * c + e] = ld_b32(rw, jok && k < H ? (unsigned)((q * H + k) * H + j) * 4u : kOut);
        }
  }
  unsigned ox[4], oh[4], ov[4];
  float dc[4], bs[4] = {0.f, 0.f, 0.f, 0.f};
  const long BH = (long)B * H;
  const __amdgpu_buffer_rsrc_t rD = rsrc_of(D ? D + g * s_D : hs, D ? BH : 0);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = r0 + 4 * v + lg;
    const bool ok = jok && 4 * v + lg < nrow;
    ox[v] = ok ? (unsigned)(row * 3 * H + j) * 4u : kOut;
    oh[v] = ok ? (unsigned)(row * H + j) * 4u : kOut;
    ov[v] = ok ? (unsigned)(v * 64 + lane) * 16u : kOut;
    dc[v] = ld_b32(rD, oh[v]);
  }
  const float* hsg = hs + g * s_hs;
  const float* abg = above ? above + g * s_above : hs;
  const float* svg = sv + g * s_sv + ((long)ty * HB + w) * 1024;
  const long sv_step = (long)RT * sv_block<HB>();
  struct In { floatx4 s[4]; float hp[4], ab[4]; };
  auto load_in = [&](int t, In& I) {
    const int tc = max(t, 0);
    const __amdgpu_buffer_rsrc_t rv = rsrc_of(svg + (long)tc * sv_step, 1024), rh = rsrc_of(hsg + (long)tc * BH, BH),
                                 ra = rsrc_of(abg + (long)tc * BH, above ? BH : 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      I.s[v] = ld_b128(rv, ov[v]);
      I.hp[v] = ld_b32(rh, oh[v]);
      I.ab[v] = ld_b32(ra, oh[v]);
    }
  };
  In ia, ib;
  load_in(T - 1, ia);
  load_in(T - 2, ib);
  for (int i = tid; i < 2 * 16 * LP; i += 64 * HB) db[0][i] = 0.f;  // (both buffers)
  __syncthreads();
  auto step = [&](int t, const float* din, float* dout, In& I) {
    floatx4 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) acc[q] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < HB; ++c) {
      floatx4 a[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const floatx4*>(&din[lr * LP + q * HP + 16 * c + 4 * lg]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][e], wt[q][4 * c + e], acc[q], 0, 0, 0);
    }
    const __amdgpu_buffer_rsrc_t rx = rsrc_of(dgx + g * s_dg + (long)t * 3 * BH, 3 * BH),
                                 rh = rsrc_of(dgh + g * s_dg + (long)t * 3 * BH, 3 * BH);
    float da_r[4], da_z[4], da_n[4], dq[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      // (outside the batch or beyond H every input is zero, and so is every gradient)
      const float r = I.s[v][0], z = I.s[v][1], n = I.s[v][2], q = I.s[v][3];
      const float dh = (dc[v] + I.ab[v]) + (acc[0][v] + acc[1][v] + acc[2][v]);
      const float dn = dh * (1.0f - z);
      const float dz = dh * (I.hp[v] - n);
      da_n[v] = dn * (1.0f - n * n);
      dq[v] = da_n[v] * r;
      da_r[v] = da_n[v] * q * r * (1.0f - r);
      da_z[v] = dz * z * (1.0f - z);
      dc[v] = dh * z;
      float* o = &dout[(4 * lg + v) * LP + j];
      o[0] = da_r[v];
      o[HP] = da_z[v];
      o[2 * HP] = dq[v];
      bs[0] += da_r[v];
      bs[1] += da_z[v];
      bs[2] += da_n[v];
      bs[3] += dq[v];
    }
    load_in(t - 2, I);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      st_b32(rx, ox[v], da_r[v]);
      st_b32(rx, ox[v], da_z[v], H * 4);
      st_b32(rx, ox[v], da_n[v], H * 8);
      st_b32(rh, ox[v], da_r[v]);
      st_b32(rh, ox[v], da_z[v], H * 4);
      st_b32(rh, ox[v], dq[v], H * 8);
    }
    __syncthreads();
  };
  if (HB > 4 && w < 4) __builtin_amdgcn_s_setprio(2);
  int t = T - 1;
  for (; t >= 1; t -= 2) {
    step(t, db[0], db[1], ia);
    step(t - 1, db[1], db[0], ib);
  }
  if (t >= 0) step(t, db[0], db[1], ia);
  // bias gradients: the four lane groups hold disjoint rows
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bs[i] += __shfl_xor(bs[i], 16);
    bs[i] += __shfl_xor(bs[i], 32);
  }
  if (lg == 0 && jok) {
    float* out = dbp + (long)(g * RT + ty) * 6 * H;
    out[j] = out[3 * H + j] = bs[0];
    out[H + j] = out[4 * H + j] = bs[1];
    out[2 * H + j] = bs[2];
    out[5 * H + j] = bs[3];
  }
}

bool gru_solo_supported(int B, int H) {
  // (one step's block of gate gradients is addressed with 31-bit byte offsets)
  return H >= 1 && H <= kSoloMaxH && (long)B * 3 * H * 4 < 0x7fffffe0L;
}
// 16 rows per workgroup in place of 4: where the chip is busy for more than one round either way.  `rounds`: of its workgroups
// over the CUs (a workgroup of more than 64 units has a CU to itself).  By the context's workers, not by how many are stepped:
// the sums have another order, and the bias gradients a quarter of the parts to add up, which is what decides for a few workers of very many rows.
// Local steps of 12 time steps, 4 / 16 rows, us (B rows on K workers):
//   H                      16          32          48          64          72          96          104         128
//   B = 128,  K = 16    58 / 62     64 / 72     78 / 91     87 / 102    113 / 140   139 / 167   143 / 186   162 / 208
//   B = 192,  K = 16    83 / 79     100 / 96    124 / 121   129 / 129   164 / 175   232 / 210   236 / 230   270 / 251
//   B = 256,  K = 16    85 / 79     108 / 105   134 / 131   138 / 137   200 / 196   261 / 237   265 / 258   321 / 307
//   B = 384,  K = 16    117 / 96    148 / 137   185 / 181   190 / 191   279 / 312   388 / 405   394 / 446   463 / 495
//   B = 512,  K = 16    135 / 107   173 / 155   220 / 207   253 / 238   373 / 381   502 / 475   510 / 523   605 / 582
//   B = 1024, K = 4     90 / 81     105 / 97    131 / 123   145 / 137   202 / 194   256 / 229   260 / 249   333 / 309
//   B = 2048, K = 1     88 / 80     94 / 91     105 / 104   119 / 122   136 / 151   162 / 179   179 / 208   199 / 230
//   B = 4096, K = 1     137 / 106   152 / 123   170 / 139   196 / 167   228 / 195   288 / 239   317 / 282   382 / 329
static bool solo_16_rows(int B, int H, int workers) {
  const long n = (long)workers * solo_tiles(B), rounds = ((long)workers * solo16_tiles(B) + 255) / 256;
  if (n <= 512) return H <= 32 && B >= 2048;
  if (H <= 32) return true;
  if (H <= 64) return n > 1536 || B >= 1024;
  if (H <= 80) return rounds == 1 && (n > 768 || B >= 2048);
  // (4 rows: two tiles per workgroup; 97 to 104 units are 7 blocks of 16, but 13 steps of 8)
  return 9 * rounds < 5 * ((n + 511) / 512) && (rounds == 1 || H <= 96 || H > 104);
}
int gru_solo_row_tiles(int B, int H, int workers) { return solo_16_rows(B, H, workers) ? solo16_tiles(B) : solo_tiles(B); }
size_t gru_solo_saved_words(int B, int H, int T, int workers) {
  return solo_16_rows(B, H, workers) ? (size_t)T * solo16_tiles(B) * ((H + 15) / 16) * 1024 : (size_t)T * solo_tiles(B) * 16 * H;
}

#define HPSGD_SOLO_CASES(LAUNCH) \
  switch ((H + 7) / 8) {         \
    case 1: LAUNCH(1); break;    \
    case 2: LAUNCH(2); break;    \
    case 3: LAUNCH(3); break;    \
    case 4: LAUNCH(4); break;    \
    case 5: LAUNCH(5); break;    \
    case 6: LAUNCH(6); break;    \
    case 7: LAUNCH(7); break;    \
    case 8: LAUNCH(8); break;    \
    case 9: LAUNCH(9); break;    \
    case 10: LAUNCH(10); break;  \
    case 11: LAUNCH(11); break;  \
    case 12: LAUNCH(12); break;  \
    case 13: LAUNCH(13); break;  \
    case 14: LAUNCH(14); break;  \
    case 15: LAUNCH(15); break;  \
    case 16: LAUNCH(16); break;  \
    default: return hipErrorInvalidValue; \
  }
#define HPSGD_SOLO16_CASES(LAUNCH) \
  switch ((H + 15) / 16) {         \
    case 1: LAUNCH(1); break;      \
    case 2: LAUNCH(2); break;      \
    case 3: LAUNCH(3); break;      \
    case 4: LAUNCH(4); break;      \
    case 5: LAUNCH(5); break;      \
    case 6: LAUNCH(6); break;      \
    case 7: LAUNCH(7); break;      \
    case 8: LAUNCH(8); break;      \
    default: return hipErrorInvalidValue; \
  }

// Two tiles per workgroup where single ones are more than run at once: two share a step's LDS round trips and
// barriers.  Up to 80 units a CU holds two workgroups or more, whose steps cover each other's waits, and up to 32 so many tiles
// go to workgroups of 16 rows.  A local step of 20 time steps with 512 tiles, one / two per workgroup: H = 128 294 / 276 us,
// H = 100 246 / 236, H = 64 153 / 160; 384 tiles: H = 80 172 / 180, H = 40 114 / 122; 1024 tiles: H = 80 339 / 348, H = 64 225 / 218.
constexpr bool solo_pairs(int H8) { return (H8 > 4 && H8 <= 8) || H8 > 10; }
static bool solo_two_tiles(int B, int H, int groups) {
  const long n = (long)groups * solo_tiles(B);
  return H <= 64 ? n > 512 : H > 80 && n > 256;
}

hipError_t launch_gru_solo_fwd(const float* W_hh, const float* b_hh, long s_rep, const float* gx, long s_gx, float* hs,
                               long s_hs, float* sv, long s_sv, int B, int H, int T, int groups, int workers, hipStream_t s) {
  if (!gru_solo_supported(B, H) || T < 1) return hipErrorInvalidValue;
  if (groups <= 0) return hipSuccess;
  const int RT = solo_tiles(B);
  KernelTimer kt(KID_GRU_FWD_PERSIST, 2.0 * B * 3 * H * (double)H * T * groups, s);
  if (solo_16_rows(B, H, workers)) {
    const int tiles = solo16_tiles(B);
#define HPSGD_SOLO16_FWD(HB)                                                                                            \
  hipLaunchKernelGGL(gru_solo16_fwd_kernel<HB>, dim3(groups * tiles), dim3(64 * HB), 0, s, W_hh, b_hh, s_rep, gx, s_gx, hs, \
                     s_hs, sv, s_sv, B, H, T, tiles)
    HPSGD_SOLO16_CASES(HPSGD_SOLO16_FWD)
#undef HPSGD_SOLO16_FWD
    return hipGetLastError();
  }
#define HPSGD_SOLO_FWD(H8)                                                                                                  \
  if (solo_pairs(H8) && solo_two_tiles(B, H, groups))                                                                        \
    hipLaunchKernelGGL((gru_solo_fwd_kernel<H8, solo_pairs(H8) ? 2 : 1>), dim3(groups * ((RT + 1) / 2)), dim3(Solo<H8>::NT), 0, s, W_hh, \
                       b_hh, s_rep, gx, s_gx, hs, s_hs, sv, s_sv, B, H, T, RT);                                              \
  else                                                                                                                      \
    hipLaunchKernelGGL((gru_solo_fwd_kernel<H8, 1>), dim3(groups * RT), dim3(Solo<H8>::NT), 0, s, W_hh, b_hh, s_rep, gx, s_gx, hs, \
                       s_hs, sv, s_sv, B, H, T, RT)
  HPSGD_SOLO_CASES(HPSGD_SOLO_FWD)
#undef HPSGD_SOLO_FWD
  return hipGetLastError();
}

hipError_t launch_gru_solo_bwd(const float* W_hh, long s_rep, float* dgx, float* dgh, long s_dg, const float* D, long s_D,
                               const float* above, long s_above, const float* sv, long s_sv, const float* hs, long s_hs,
                               float* dbp, int B, int H, int T, int groups, int workers, hipStream_t s) {
  if (!gru_solo_supported(B, H) || T < 1) return hipErrorInvalidValue;
  if (groups <= 0) return hipSuccess;
  const int RT = solo_tiles(B);
  KernelTimer kt(KID_GRU_BWD_PERSIST, 2.0 * B * 3 * H * (double)H * T * groups, s);
  if (solo_16_rows(B, H, workers)) {
    const int tiles = solo16_tiles(B);
#define HPSGD_SOLO16_BWD(HB)                                                                                                   \
  hipLaunchKernelGGL(gru_solo16_bwd_kernel<HB>, dim3(groups * tiles), dim3(64 * HB), 0, s, W_hh, s_rep, dgx, dgh, s_dg, D, s_D, \
                     above, s_above, sv, s_sv, hs, s_hs, dbp, B, H, T, tiles)
    HPSGD_SOLO16_CASES(HPSGD_SOLO16_BWD)
#undef HPSGD_SOLO16_BWD
    return hipGetLastError();
  }
#define HPSGD_SOLO_BWD(H8)                                                                                                     \
  if (solo_pairs(H8) && solo_two_tiles(B, H, groups))                                                                           \
    hipLaunchKernelGGL((gru_solo_bwd_kernel<H8, solo_pairs(H8) ? 2 : 1>), dim3(groups * ((RT + 1) / 2)), dim3(Solo<H8>::NT), 0, s, W_hh, \
                       s_rep, dgx, dgh, s_dg, D, s_D, above, s_above, sv, s_sv, hs, s_hs, dbp, B, H, T, RT);                   \
  else                                                                                                                         \
    hipLaunchKernelGGL((gru_solo_bwd_kernel<H8, 1>), dim3(groups * RT), dim3(Solo<H8>::NT), 0, s, W_hh, s_rep, dgx, dgh, s_dg, D,  \
                       s_D, above, s_above, sv, s_sv, hs, s_hs, dbp, B, H, T, RT)
  HPSGD_SOLO_CASES(HPSGD_SOLO_BWD)
#undef HPSGD_SOLO_BWD
  return hipGetLastError();
}

// Both layers in one launch, each way: where the chip has room for the four workgroups of every worker's tiles at once - one per CU beyond
// 64 units, two up to there.  Up to there a classifier's may be half as many again, of which the last start as the first end:
// the upper layer has nothing but the recurrence to do, and the launches between the layers are gone.  (A language model's step has products enough beside
// its recurrences, and gains nothing.)  Local steps, layer by layer / this, us (H, batch, workers, steps):
//   (100, 20, 4, 50) 298 / 195 a round   (128, 16, 4, 35) 266 / 181   (64, 20, 2, 35) 146 / 107   (32, 8, 4, 20) 88 / 65   (30, 60, 1, 60) 187 / 130
//   few steps  (100, 20, 4, 10) 110 / 88   (100, 20, 4, 5) 87 / 75       the chip full  (110, 32, 8, 30) 261 / 180   (64, 64, 8, 30) 180 / 143
//   768 workgroups, classifiers  (24, 96, 8, 8) 77 / 70   (48, 96, 8, 30) 183 / 170   (64, 96, 8, 6) 89 / 87, with an input of 256 97 / 98   (64, 96, 8, 30) 196 / 191
//   language models  (64, 64, 8, 6) 129 / 128   (64, 64, 8, 20) of 500 words 266 / 257   (32, 64, 8, 4) 96 / 93   (128, 32, 8, 12) 221 / 192
//     beyond 512 (not taken)  (24, 72, 8, 4) 95 / 97   (64, 96, 8, 5) 133 / 140   (64, 96, 8, 40) 577 / 590   (48, 96, 8, 20) 328 / 318   (16, 96, 8, 10) 161 / 161
bool gru_stack_supported(int B, int H, int T, int layers, int workers, bool lm) {
  return layers == 2 && H >= 4 && gru_solo_supported(B, H) && !solo_16_rows(B, H, workers) &&
         (long)workers * solo_tiles(B) * 4 <= (H > 64 ? 256 : lm ? 512 : 768) &&
         (long)(T + 1) * B * 3 * H * 4 < 0x7fffffe0L;
}
size_t gru_stack_sync_words(int B, int groups) { return kLinkBase + (size_t)groups * solo_tiles(B) * kLinkWords; }

hipError_t launch_gru_stack_fwd(const GruStackLayer& lo, const GruStackLayer& up, const float* W_ih, const float* b_ih, long s_rep, long s_gx,
                                long s_hs, long s_sv, int B, int H, int T, int groups, unsigned* sync, unsigned limit, hipStream_t s) {
  if (!gru_stack_supported(B, H, T, 2, groups, false)) return hipErrorInvalidValue;
  const int RT = solo_tiles(B), n = groups * RT;
  KernelTimer kt(KID_GRU_FWD_PERSIST, 2.0 * B * 3 * H * (double)H * T * groups * 2, s, 2);
#define HPSGD_STACK_FWD(H8)                                                                                                  \
  hipLaunchKernelGGL(gru_stack_fwd_kernel<H8>, dim3(32 * ((n + 7) / 8)), dim3(Solo<H8>::NT), 0, s, lo, up, W_ih, b_ih, s_rep, s_gx, s_hs, s_sv, \
                     B, H, T, RT, n, sync, limit)
  HPSGD_SOLO_CASES(HPSGD_STACK_FWD)
#undef HPSGD_STACK_FWD
  return hipGetLastError();
}

hipError_t launch_gru_stack_bwd(const GruStackLayer& lo, const GruStackLayer& up, const float* W_ih, long s_rep, const float* D, long s_D,
                                const float* above, long s_above, float* dx, long s_dx, long s_gx, long s_hs, long s_sv,
                                int B, int H, int T, int groups, unsigned* sync, unsigned limit, hipStream_t s) {
  if (!gru_stack_supported(B, H, T, 2, groups, false)) return hipErrorInvalidValue;
  const int RT = solo_tiles(B), n = groups * RT;
  KernelTimer kt(KID_GRU_BWD_PERSIST, 2.0 * B * 3 * H * (double)H * T * groups * 2, s, 2);
#define HPSGD_STACK_BWD(H8)                                                                                                       \
  hipLaunchKernelGGL(gru_stack_bwd_kernel<H8>, dim3(32 * ((n + 7) / 8)), dim3(Solo<H8>::NT), 0, s, lo, up, W_ih, s_rep, D, s_D, above, s_above, dx, s_dx, \
                     s_gx, s_hs, s_sv, B, H, T, RT, n, sync, limit)
  HPSGD_SOLO_CASES(HPSGD_STACK_BWD)
#undef HPSGD_STACK_BWD
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- bf16 operands, H <= 256
// The same idea on bf16 copies of W_hh and h (fp32 accumulation, cell math and saved values): a workgroup owns
// 4 or 8 batch rows and all units (HP = 16 HB, a multiple of 32), v_mfma_f32_16x16x32_bf16.  W_hh of 256 units is
// 393 KB: a wave holds UB = 1 (HP <= 128) or 2 blocks of 16 units, and for two blocks the third gate
// (backward: the last chunks) lives in LDS, each wave reading back only its own fragments.  Most of an
// instruction's 16 rows are unused: the matrix work of a step is 0.6 us at 256 units all the same, while the cell
// math, which is longer, goes by the rows (V = 1 or 2 outputs per lane and block).
// Row 4*lg + v of a product, v < V, is batch row r0 + V*lg + v: a lane's two values of 8 rows are neighbours in the
// transposed copies and leave as one 4-byte store.  Rows with v >= V repeat another and are ignored.
// The forward launch writes h in bf16, row-major and transposed, h_0 = 0 included; saved gates and h_{t-1} are
// kept in lane order.  The backward launch writes the gate gradients row-major only, through the LDS tile of the
// next step's operand: 16 bytes per (unit, step) of a transposed copy is a cache line per lane group, and six of
// those per output made the launch 2.5 times as long as its chain (H = 224: 4.5 us per step); a launch
// behind it transposes all steps at once.
// Bound by the chain of a step: product, cell math, barrier.  Per step of 40, launch included, B = 32 and four workers:
//   H                   64    96   128   160   192   224   256
//   forward   8 rows  0.71  0.81  1.15  1.71  2.00  2.36  2.67 us
//             4 rows  0.65  0.68  0.86  1.20  1.50  1.61  1.91 us
//   backward  8 rows  0.58  0.99  1.05  1.34  1.79  2.10  2.53 us
//             4 rows  0.52  0.58  0.88  0.96  1.16  1.66  2.03 us
// (gates of the hardware's exp2 and reciprocal; a forward step with those of the fp32 launches, EX, takes 0.2 us
// more at 224 units)
// against 3.3 and 3.5 us of the resident-weight launches, whose workgroups exchange h through L2, at all of
// these widths; 256 is as far as one CU's registers and LDS hold the weights.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
namespace {
constexpr int kSoloBMaxH = 256;
__device__ __forceinline__ unsigned pack2(float a, float b) {
  const __bf16 x = (__bf16)a, y = (__bf16)b;
  return (unsigned)__builtin_bit_cast(unsigned short, x) | ((unsigned)__builtin_bit_cast(unsigned short, y) << 16);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_b(const void* base, long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes < 0x7fffffe0L ? bytes : 0x7fffffe0L),
                                           0x00020000);
}
}  // namespace

// V: outputs per lane and block, 4 V rows per workgroup
template <int HB, int UB, int V>
struct SoloB {
  static constexpr int RO = 4 * V, NW = HB / UB, NT = 64 * NW, HP = 16 * HB, NC = HB / 2;
  static constexpr bool WL = UB == 2;                     // the n gate's weights in LDS (forward)
  static constexpr int LP = HP + 8;                       // pitch (bf16) of a row of h
  static constexpr size_t FWD_LDS = (size_t)2 * RO * LP * 2 + (WL ? (size_t)HB * NC * 1024 : 0);
  static constexpr int NC3 = 3 * NC, NCR = NC3 < 18 ? NC3 : 18, NCL = NC3 - NCR;  // chunks in registers / in LDS (backward)
  static constexpr int LP4 = 4 * HP + 8;                  // a row of gate gradients: r | z | q | n
  static constexpr size_t BWD_LDS = (size_t)2 * RO * LP4 * 2 + (size_t)HB * NCL * 1024;
};

namespace {

// (tile ty of worker g; LINKED: in a launch of two layers, as solo_fwd_body)
template <int HB, int UB, int V, bool EX, bool LINKED>
__device__ __forceinline__ void solo_fwd_bf16_body(const __bf16* __restrict__ Wb, long s_wb, const float* __restrict__ b_ih,
                                                   const float* __restrict__ b_hh, long s_rep, int Hc, const float* __restrict__ gx,
                                                   long s_gx, __bf16* __restrict__ hb, long s_hb, float* __restrict__ hs, long s_hs,
                                                   float* __restrict__ sv, long s_sv, __bf16* __restrict__ hT, long ld_hT, long s_hT,
                                                   int Bc, int B, int T, int RT, int g, int ty, const SoloLink& k) {
  static_assert(!LINKED || 4 * V * kChunk == 16, "a product of the layers' link has the rows of a chunk");
  using S = SoloB<HB, UB, V>;
  constexpr int HP = S::HP, LP = S::LP, NC = S::NC;
  extern __shared__ __attribute__((aligned(16))) unsigned char solo_lds[];
  __bf16* hl = reinterpret_cast<__bf16*>(solo_lds);                       // [2][RO][LP]
  u32x4s* wl = reinterpret_cast<u32x4s*>(solo_lds + 2 * S::RO * LP * 2);      // [HB][NC][64]: the n gate
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int r0 = ty * S::RO;
  bf16x8 wf[S::WL ? 2 : 3][UB][NC];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_b(Wb + g * s_wb, 3L * HP * HP * 2);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const u32x4s v = __builtin_amdgcn_raw_buffer_load_b128(rw, ((q * HP + (w * UB + u) * 16 + lr) * HP + 32 * c + 8 * lg) * 2, 0, 0);
          if (q < (S::WL ? 2 : 3)) wf[q < (S::WL ? 2 : 3) ? q : 0][u][c] = __builtin_bit_cast(bf16x8, v);
          else wl[((w * UB + u) * NC + c) * 64 + lane] = v;
        }
  }
  float bias[UB][3], bx[UB];  // b_hh (+ b_ih for r and z); the n gate keeps its two parts apart
#pragma unroll
  for (int u = 0; u < UB; ++u) {
    const int j = (w * UB + u) * 16 + lr;
    const bool ok = j < Hc;
    const float* bi = b_ih + g * s_rep;
    const float* bh = b_hh + g * s_rep;
    const int jc = min(j, Hc - 1);
#pragma unroll
    for (int q = 0; q < 3; ++q) bias[u][q] = ok ? bh[q * Hc + jc] : 0.f;
    bx[u] = ok ? bi[2 * Hc + jc] : 0.f;
    if (ok) {
      bias[u][0] += bi[jc];
      bias[u][1] += bi[Hc + jc];
    }
  }
  const float* gxg = gx + g * s_gx;
  const unsigned ox = (unsigned)(((r0 + V * lg) * 3 * HP + w * UB * 16 + lr) * 4);
  __bf16* hbg = hb + g * s_hb;
  __bf16* hTg = hT + g * s_hT;
  const unsigned oT = (unsigned)((w * UB * 16 + lr) * ld_hT + r0 + V * lg) * 2u;
  const long blk = (long)HB * V * 64;  // outputs of a tile and step, in lane order
  float* svg = sv + g * s_sv + (long)ty * blk * 4;
  float* hsg = hs + g * s_hs + (long)ty * blk;
  const long step_out = (long)RT * blk;
  for (int i = tid; i < S::RO * LP; i += S::NT) reinterpret_cast<unsigned*>(hl)[i] = 0u;
  // h_0 = 0: the first B rows of hb, the first B columns of hT
  for (int i = tid; i < S::RO * HP / 8; i += S::NT)
    *reinterpret_cast<u32x4s*>(hbg + (long)(r0 + i / (HP / 8)) * HP + (i % (HP / 8)) * 8) = (u32x4s){0u, 0u, 0u, 0u};
#pragma unroll
  for (int u = 0; u < UB; ++u)
    for (int v = 0; v < V; ++v) hTg[(long)((w * UB + u) * 16 + lr) * ld_hT + r0 + V * lg + v] = (__bf16)0.f;
  auto load_gx = [&](int t, float (&G)[UB][3][V]) {
    const __amdgpu_buffer_rsrc_t rs = rsrc_b(gxg + (long)min(t, T - 1) * B * 3 * HP, 12L * B * HP);
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int v = 0; v < V; ++v)
          G[u][q][v] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)ox, ((v * 3 + q) * HP + u * 16) * 4, LINKED ? 16 : 0));
  };
  // (two blocks per wave: the input projections are requested one step ahead instead of two, the registers of
  // the second set being the ones that would spill)
  constexpr int PD = UB == 2 ? 1 : 2;
  float ga[UB][3][V], gb[PD == 2 ? UB : 1][3][V], hp[UB][V];
#pragma unroll
  for (int u = 0; u < UB; ++u) for (int v = 0; v < V; ++v) hp[u][v] = 0.f;
  auto wait_gx = [&](int it) {
    if (LINKED && k.in && it < T && it % kChunk == 0 && !link_chunk(k, it, T)) {
#pragma unroll
      for (int u = 0; u < UB; ++u) bias[u][0] = bias[u][1] = bias[u][2] = __builtin_nanf("");
    }
  };
  wait_gx(0);
  load_gx(0, ga);
  if constexpr (PD == 2) load_gx(1, gb);
  __syncthreads();
  const int arow = V == 2 ? 2 * (lr >> 2) + ((lr & 3) ? 1 : 0) : lr >> 2;  // the batch row of product row lr (see above)
  auto step = [&](int t, const __bf16* hin, __bf16* hout, float (&G)[UB][3][V]) {
    bf16x8 a[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) a[c] = *reinterpret_cast<const bf16x8*>(hin + arow * LP + 32 * c + 8 * lg);
    if (UB == 1) __builtin_amdgcn_sched_barrier(0);
    floatx4 acc[UB][3];
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) acc[u][q] = (floatx4){bias[u][q], bias[u][q], bias[u][q], bias[u][q]};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        acc[u][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], wf[0][u][c], acc[u][0], 0, 0, 0);
        acc[u][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], wf[1][u][c], acc[u][1], 0, 0, 0);
        const bf16x8 wn = S::WL ? __builtin_bit_cast(bf16x8, wl[((w * UB + u) * NC + c) * 64 + lane]) : wf[S::WL ? 0 : 2][u][c];
        acc[u][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], wn, acc[u][2], 0, 0, 0);
      }
    if (LINKED && k.out && t > 0 && t % kChunk == 0) link_publish(k.out + w, t);
    float rr[UB][V], zz[UB][V], nn[UB][V];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        rr[u][v] = sigm_of<EX>(G[u][0][v] + acc[u][0][v]);
        zz[u][v] = sigm_of<EX>(G[u][1][v] + acc[u][1][v]);
        nn[u][v] = tanh_of<EX>((G[u][2][v] + bx[u]) + rr[u][v] * acc[u][2][v]);
        // Rows and units of the padding leave zeros, selected and not multiplied: an infinite value of the model
        // times their zero operands is NaN, which their h and gate gradients would hand to everyone.
        if (r0 + V * lg + v >= Bc || (w * UB + u) * 16 + lr >= Hc) rr[u][v] = zz[u][v] = nn[u][v] = acc[u][2][v] = 0.f;
      }
    }
    const __amdgpu_buffer_rsrc_t rh = rsrc_b(hsg + (long)t * step_out, blk * 4), rv = rsrc_b(svg + (long)t * step_out * 4, blk * 16);
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) {  // what the backward launch wants of this step: h_{t-1} and the gates
        const int o = ((w * UB + u) * V + v) * 64 + lane;
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, hp[u][v]), rh, o * 4, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4s, (floatx4){rr[u][v], zz[u][v], nn[u][v], acc[u][2][v]}), rv,
                                               o * 16, 0, 0);
        hp[u][v] = (1.0f - zz[u][v]) * nn[u][v] + zz[u][v] * hp[u][v];
        hout[(V * lg + v) * LP + (w * UB + u) * 16 + lr] = (__bf16)hp[u][v];
      }
    wait_gx(t + PD);
    load_gx(t + PD, G);
    const __amdgpu_buffer_rsrc_t rT = rsrc_b(hTg + (long)(t + 1) * B, ((long)HP * ld_hT - (long)(t + 1) * B) * 2);
#pragma unroll
    for (int u = 0; u < UB; ++u)
      if constexpr (V == 2)
        __builtin_amdgcn_raw_buffer_store_b32(pack2(hp[u][0], hp[u][1]), rT, (int)oT, (int)(u * 16 * ld_hT * 2), 0);
      else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, (__bf16)hp[u][0]), rT, (int)oT, (int)(u * 16 * ld_hT * 2), 0);
    __syncthreads();
    // the row-major copy of h, 16 bytes per piece, from the tile the next step multiplies
    const __amdgpu_buffer_rsrc_t rb = rsrc_b(hbg + (long)(t + 1) * B * HP, 2L * B * HP);
#pragma unroll
    for (int i = 0; i < (V * HP / 2 + S::NT - 1) / S::NT; ++i)
      if (tid + i * S::NT < V * HP / 2)
        __builtin_amdgcn_raw_buffer_store_b128(
            *reinterpret_cast<const u32x4s*>(hout + ((tid + i * S::NT) / (HP / 8)) * LP + ((tid + i * S::NT) % (HP / 8)) * 8), rb,
            (r0 * HP + (tid + i * S::NT) * 8) * 2, 0, LINKED ? 16 : 0);
  };
  __bf16* h0 = hl;
  __bf16* h1 = hl + S::RO * LP;
  int t = 0;
  for (; t + 1 < T; t += 2) {
    step(t, h0, h1, ga);
    if constexpr (PD == 2) step(t + 1, h1, h0, gb);
    else step(t + 1, h1, h0, ga);
  }
  if (t < T) step(t, h0, h1, ga);
  if (LINKED && k.out) link_publish(k.out + w, T);
}

template <int HB, int UB, int V, bool LINKED>
__device__ __forceinline__ void solo_bwd_bf16_body(const __bf16* __restrict__ WT, long s_wt, const float* __restrict__ above,
                                                   long s_above, const float* __restrict__ sv, long s_sv, const float* __restrict__ hs,
                                                   long s_hs, __bf16* __restrict__ dg4, long s_dg4, float* __restrict__ dbp, int Hc,
                                                   int B, int T, int RT, int g, int ty, const SoloLink& k) {
  using S = SoloB<HB, UB, V>;
  constexpr int HP = S::HP, LP = S::LP4, NC3 = S::NC3, NCR = S::NCR, NCL = S::NCL;
  extern __shared__ __attribute__((aligned(16))) unsigned char solo_lds[];
  __bf16* dl = reinterpret_cast<__bf16*>(solo_lds);                       // [2][RO][LP]: r | z | q | n
  u32x4s* wl = reinterpret_cast<u32x4s*>(solo_lds + 2 * S::RO * LP * 2);      // [HB][NCL][64]
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int r0 = ty * S::RO;
  // W_hh^T rows of this wave's units: [unit][3 HP]
  bf16x8 wf[UB][NCR];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_b(WT + g * s_wt, 3L * HP * HP * 2);
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int c = 0; c < NC3; ++c) {
        const u32x4s v = __builtin_amdgcn_raw_buffer_load_b128(rw, (((w * UB + u) * 16 + lr) * 3 * HP + 32 * c + 8 * lg) * 2, 0, 0);
        if (c < NCR) wf[u][c < NCR ? c : 0] = __builtin_bit_cast(bf16x8, v);
        else wl[((w * UB + u) * NCL + (c - NCR)) * 64 + lane] = v;
      }
  }
  const long blk = (long)HB * V * 64;
  const float* svg = sv + g * s_sv + (long)ty * blk * 4;
  const float* hsg = hs + g * s_hs + (long)ty * blk;
  const long step_out = (long)RT * blk;
  const float* abg = above + g * s_above;
  const unsigned oa = (unsigned)(((r0 + V * lg) * HP + w * UB * 16 + lr) * 4);
  struct In { floatx4 s[UB][V]; float hp[UB][V], ab[UB][V]; };
  auto load_in = [&](int t, In& I) {
    const int tc = max(t, 0);
    const __amdgpu_buffer_rsrc_t rv = rsrc_b(svg + (long)tc * step_out * 4, blk * 16), rh = rsrc_b(hsg + (long)tc * step_out, blk * 4),
                                 ra = rsrc_b(abg + (long)tc * B * HP, 4L * B * HP);
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int o = ((w * UB + u) * V + v) * 64 + lane;
        I.s[u][v] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rv, o * 16, 0, 0));
        I.hp[u][v] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rh, o * 4, 0, 0));
        I.ab[u][v] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ra, (int)oa, (v * HP + u * 16) * 4, LINKED ? 16 : 0));
      }
  };
  In ia;
  float dc[UB][V], bs[UB][4];
#pragma unroll
  for (int u = 0; u < UB; ++u) {
#pragma unroll
    for (int v = 0; v < V; ++v) dc[u][v] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) bs[u][i] = 0.f;
  }
  auto wait_above = [&](int t) {
    if (LINKED && k.in && t >= 0 && (T - 1 - t) % kChunk == 0 && !link_chunk(k, T - 1 - t, T)) {
#pragma unroll
      for (int u = 0; u < UB; ++u)
        for (int v = 0; v < V; ++v) dc[u][v] = __builtin_nanf("");
    }
  };
  wait_above(T - 1);
  load_in(T - 1, ia);
  for (int i = tid; i < S::RO * LP; i += S::NT) reinterpret_cast<unsigned*>(dl)[i] = 0u;
  __syncthreads();
  __bf16* dgb = dg4 + g * s_dg4;
  const int arow = V == 2 ? 2 * (lr >> 2) + ((lr & 3) ? 1 : 0) : lr >> 2;
  auto step = [&](int t, const __bf16* din, __bf16* dout) {
    floatx4 acc[UB][2];
#pragma unroll
    for (int u = 0; u < UB; ++u) acc[u][0] = acc[u][1] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC3; ++c) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(din + arow * LP + 32 * c + 8 * lg);
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const bf16x8 wv = c < NCR ? wf[u][c < NCR ? c : 0]
                                  : __builtin_bit_cast(bf16x8, wl[((w * UB + u) * NCL + (c < NCR ? 0 : c - NCR)) * 64 + lane]);
        acc[u][c & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wv, acc[u][c & 1], 0, 0, 0);
      }
    }
    if (LINKED && k.out && t < T - 1 && (T - 1 - t) % kChunk == 0) link_publish(k.out + w, T - 1 - t);
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      float da_r[V], da_z[V], da_n[V], dq[V];
      const int j = (w * UB + u) * 16 + lr;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float r = ia.s[u][v][0], z = ia.s[u][v][1], n = ia.s[u][v][2], q = ia.s[u][v][3];
        const float dh = (dc[u][v] + ia.ab[u][v]) + (acc[u][0][v] + acc[u][1][v]);
        const float dn = dh * (1.0f - z);
        const float dz = dh * (ia.hp[u][v] - n);
        da_n[v] = dn * (1.0f - n * n);
        dq[v] = da_n[v] * r;
        da_r[v] = da_n[v] * q * r * (1.0f - r);
        da_z[v] = dz * z * (1.0f - z);
        dc[u][v] = dh * z;
        __bf16* o = dout + (V * lg + v) * LP + j;
        o[0] = (__bf16)da_r[v];
        o[HP] = (__bf16)da_z[v];
        o[2 * HP] = (__bf16)dq[v];
        o[3 * HP] = (__bf16)da_n[v];
        bs[u][0] += da_r[v];
        bs[u][1] += da_z[v];
        bs[u][2] += da_n[v];
        bs[u][3] += dq[v];
      }
    }
    wait_above(t - 1);
    load_in(t - 1, ia);
    __syncthreads();
    // the gate gradients row-major (r | z | n | q), 16 bytes per piece
    const __amdgpu_buffer_rsrc_t rb = rsrc_b(dgb + (long)t * B * 4 * HP, 8L * B * HP);
#pragma unroll
    for (int i = 0; i < (2 * V * HP + S::NT - 1) / S::NT; ++i) {
      const int p = tid + i * S::NT, row = p / (HP / 2), c = (p % (HP / 2)) * 8;
      const int src = c < 2 * HP ? c : c < 3 * HP ? c + HP : c - HP;  // (in LDS q comes before n)
      if (p < 2 * V * HP)
        __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4s*>(dout + row * LP + src), rb,
                                               ((r0 + row) * 4 * HP + c) * 2, 0, LINKED ? 16 : 0);
    }
  };
  __bf16* d0 = dl;
  __bf16* d1 = dl + S::RO * LP;
  int t = T - 1;
  for (; t >= 1; t -= 2) {
    step(t, d0, d1);
    step(t - 1, d1, d0);
  }
  if (t >= 0) step(t, d0, d1);
  if (LINKED && k.out) link_publish(k.out + w, T);
#pragma unroll
  for (int u = 0; u < UB; ++u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bs[u][i] += __shfl_xor(bs[u][i], 16);
      bs[u][i] += __shfl_xor(bs[u][i], 32);
    }
    const int j = (w * UB + u) * 16 + lr;
    if (lg == 0 && j < Hc) {
      float* out = dbp + (long)(g * RT + ty) * 6 * Hc;
      out[j] = out[3 * Hc + j] = bs[u][0];
      out[Hc + j] = out[4 * Hc + j] = bs[u][1];
      out[2 * Hc + j] = bs[u][2];
      out[5 * Hc + j] = bs[u][3];
    }
  }
}

}  // namespace

template <int HB, int UB, int V, bool EX>
__global__ void __launch_bounds__(64 * HB / UB) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_solo_fwd_bf16_kernel(const __bf16* __restrict__ Wb, long s_wb, const float* __restrict__ b_ih, const float* __restrict__ b_hh,
                         long s_rep, int Hc, const float* __restrict__ gx, long s_gx, __bf16* __restrict__ hb, long s_hb,
                         float* __restrict__ hs, long s_hs, float* __restrict__ sv, long s_sv, __bf16* __restrict__ hT, long ld_hT,
                         long s_hT, int Bc, int B, int T, int RT) {
  const int g = blockIdx.x / RT;
  solo_fwd_bf16_body<HB, UB, V, EX, false>(Wb, s_wb, b_ih, b_hh, s_rep, Hc, gx, s_gx, hb, s_hb, hs, s_hs, sv, s_sv, hT, ld_hT, s_hT, Bc, B, T,
                                           RT, g, blockIdx.x - g * RT, SoloLink{});
}
template <int HB, int UB, int V>
__global__ void __launch_bounds__(64 * HB / UB) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_solo_bwd_bf16_kernel(const __bf16* __restrict__ WT, long s_wt, const float* __restrict__ above, long s_above,
                         const float* __restrict__ sv, long s_sv, const float* __restrict__ hs, long s_hs, __bf16* __restrict__ dg4,
                         long s_dg4, float* __restrict__ dbp, int Hc, int B, int T, int RT) {
  const int g = blockIdx.x / RT;
  solo_bwd_bf16_body<HB, UB, V, false>(WT, s_wt, above, s_above, sv, s_sv, hs, s_hs, dg4, s_dg4, dbp, Hc, B, T, RT, g, blockIdx.x - g * RT,
                                       SoloLink{});
}

// ---------------------------------------------------------------------------- two bf16 layers in one launch
// As the launches of two fp32 layers above, 4 rows a tile; what is passed on are the row-major bf16 copies of h and of the gate gradients.
// The product between the layers holds its weights as the recurrences hold theirs: forward W_ih [3 HP][HP] in the place of W_hh,
// backward W_ih^T [HP][3 HP] in that of W_hh^T; a chunk's operands go through LDS behind them.
namespace {

template <int HB, int UB, bool BWD>
__device__ __forceinline__ void link_bf16_body(const __bf16* __restrict__ W, const __bf16* in, float* out, int B, int T, int ty, int odd,
                                               unsigned* in_words, unsigned* out_words, unsigned* abort_w, unsigned limit) {
  using S = SoloB<HB, UB, 1>;
  constexpr int HP = S::HP, NC = BWD ? S::NC3 : S::NC, NQ = BWD ? 1 : 3;
  constexpr int QR = BWD ? 1 : S::WL ? 2 : 3, CR = BWD ? S::NCR : NC;  // gates and chunks in registers
  constexpr int IP = BWD ? 4 * HP : HP, ND = BWD ? HP : 3 * HP;        // words of a row of `in` and `out`
  extern __shared__ __attribute__((aligned(16))) unsigned char solo_lds[];
  u32x4s* wl = reinterpret_cast<u32x4s*>(solo_lds + 2 * S::RO * (BWD ? S::LP4 : S::LP) * 2);  // [HB][NC - CR, or NC of the n gate][64]
  u32x4s* al = reinterpret_cast<u32x4s*>(solo_lds + (BWD ? S::BWD_LDS : S::FWD_LDS));         // [NC][64]
  __shared__ int go;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lg = lane >> 4;
  bf16x8 wf[QR][UB][CR];
  {
    const __amdgpu_buffer_rsrc_t rw = rsrc_b(W, 3L * HP * HP * 2);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const u32x4s v = __builtin_amdgcn_raw_buffer_load_b128(rw, ((q * HP + (w * UB + u) * 16 + lr) * (BWD ? 3 * HP : HP) + 32 * c + 8 * lg) * 2, 0, 0);
          if (q < QR && c < CR) wf[q < QR ? q : 0][u][c < CR ? c : 0] = __builtin_bit_cast(bf16x8, v);
          else wl[((w * UB + u) * (BWD ? NC - CR : NC) + (BWD ? c - CR : c)) * 64 + lane] = v;
        }
  }
  const __amdgpu_buffer_rsrc_t ri = rsrc_b(in, 2L * T * B * IP), ro = rsrc_b(out, 4L * T * B * ND);
  bool ok = true;
  for (int i0 = odd * kChunk; i0 < T; i0 += 2 * kChunk) {
    if (w == 0) {
      ok = ok && link_wait<8>(in_words, S::NW, (unsigned)min(i0 + kChunk, T), abort_w, limit);
      if (lane == 0) go = ok;
    }
    __syncthreads();  // (and everyone has read the operands of the chunk before)
    ok = go != 0;
    const int ia = i0 + (lr >> 2), io = i0 + lg;
    const unsigned off_a = ia < T ? (unsigned)(((BWD ? T - 1 - ia : ia) * B + 4 * ty + (lr & 3)) * IP + 8 * lg) * 2u : kOut;
#pragma unroll
    for (int i = 0; i < (NC + S::NW - 1) / S::NW; ++i) {
      const int c = w + i * S::NW;
      if (c < NC) al[c * 64 + lane] = __builtin_amdgcn_raw_buffer_load_b128(ri, (int)off_a, c * 64, 16);  // (uniform)
    }
    __syncthreads();
    floatx4 acc[NQ][UB];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int u = 0; u < UB; ++u) acc[q][u] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, al[c * 64 + lane]);
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const bf16x8 wv = q < QR && c < CR ? wf[q < QR ? q : 0][u][c < CR ? c : 0]
                                             : __builtin_bit_cast(bf16x8, wl[((w * UB + u) * (BWD ? NC - CR : NC) + (BWD ? (c < CR ? 0 : c - CR) : c)) * 64 + lane]);
          acc[q][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wv, acc[q][u], 0, 0, 0);
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          st_b32<true>(ro, io < T ? (unsigned)(((BWD ? T - 1 - io : io) * B + 4 * ty + v) * ND + q * HP + (w * UB + u) * 16 + lr) * 4u : kOut,
                       ok ? acc[q][u][v] : __builtin_nanf(""));
    link_publish(out_words + w, (unsigned)min(i0 + kChunk, T));
  }
}

}  // namespace

// (grid, sync: as gru_stack_fwd_kernel)
template <int HB, int UB, bool EX>
__global__ void __launch_bounds__(64 * HB / UB) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_stack_fwd_bf16_kernel(GruStackLayerB lo, GruStackLayerB up, const __bf16* W_ih, long s_wih, long s_wb, long s_rep, int Hc, long s_gx,
                          long s_hb, long s_hs, long s_sv, long ld_hT, long s_hT, int Bc, int B, int T, int RT, int n, unsigned* sync,
                          unsigned limit) {
  constexpr int HP = 16 * HB, NW = HB / UB;
  int role, tile;
  if (!link_part(sync, 0, n, role, tile)) return;
  const int g = tile / RT, ty = tile - g * RT;
  unsigned* words = sync + kLinkBase + (long)tile * kLinkWords;
  if (role == 1 || role == 2) {
    link_bf16_body<HB, UB, false>(W_ih + g * s_wih, (const __bf16*)lo.hb + g * s_hb + (long)B * HP, up.gx + g * s_gx, B, T, ty, role - 1, words,
                                  words + 8 * role, sync, limit);
  } else {
    const bool first = role == 0;
    const GruStackLayerB& l = first ? lo : up;
    solo_fwd_bf16_body<HB, UB, 1, EX, true>((const __bf16*)l.W, s_wb, l.b_ih, l.b_hh, s_rep, Hc, l.gx, s_gx, (__bf16*)l.hb, s_hb, l.hs, s_hs,
                                            l.sv, s_sv, (__bf16*)l.hT, ld_hT, s_hT, Bc, B, T, RT, g, ty,
                                            SoloLink{first ? words : nullptr, first ? nullptr : words + 8, sync, limit, NW});
  }
}

template <int HB, int UB>
__global__ void __launch_bounds__(64 * HB / UB) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_stack_bwd_bf16_kernel(GruStackLayerB lo, GruStackLayerB up, const __bf16* WT_ih, long s_wih, long s_wt, const float* above, long s_above,
                          float* dx, long s_dx, long s_hs, long s_sv, long s_dg4, int Hc, int B, int T, int RT, int n,
                          unsigned* sync, unsigned limit) {
  constexpr int NW = HB / UB;
  int role, tile;
  if (!link_part(sync, 1, n, role, tile)) return;
  const int g = tile / RT, ty = tile - g * RT;
  unsigned* words = sync + kLinkBase + (long)tile * kLinkWords + 36;
  if (role == 1 || role == 2) {
    link_bf16_body<HB, UB, true>(WT_ih + g * s_wih, (const __bf16*)up.dg4 + g * s_dg4, dx + g * s_dx, B, T, ty, role - 1, words,
                                 words + 8 * role, sync, limit);
  } else {
    const bool first = role == 0;
    const GruStackLayerB& l = first ? up : lo;
    solo_bwd_bf16_body<HB, UB, 1, true>((const __bf16*)l.WT, s_wt, first ? above : dx, first ? s_above : s_dx, l.sv, s_sv, l.hs, s_hs,
                                        (__bf16*)l.dg4, s_dg4, l.dbp, Hc, B, T, RT, g, ty,
                                        SoloLink{first ? words : nullptr, first ? nullptr : words + 8, sync, limit, NW});
  }
}

bool gru_solo_bf16_supported(int B, int H) {
  return H % 32 == 0 && H >= 32 && H <= kSoloBMaxH && B % 8 == 0 && B >= 8 && 12L * B * H < 0x7fffffe0L;
}
// Rows of a workgroup: 4 up to a workgroup per CU, 8 beyond (a local step of 20 time steps, 4 / 8 rows: H = 256, 256 tiles
// of 4 rows 406 / 427 us, 512 tiles 737 / 688; H = 128, 384 tiles 412 / 400).  By the context's workers, not by how many are
// stepped: the sums of the bias gradients are the same then.
static int solo_b_rows(int B, int workers) { return (long)workers * (B / 4) <= 256 ? 4 : 8; }
int gru_solo_bf16_row_tiles(int B, int workers) { return B / solo_b_rows(B, workers); }

#define HPSGD_SOLOB_CASES(LAUNCH)         \
  switch (H / 32) {                       \
    case 1: LAUNCH(2, 1); break;          \
    case 2: LAUNCH(4, 1); break;          \
    case 3: LAUNCH(6, 1); break;          \
    case 4: LAUNCH(8, 1); break;          \
    case 5: LAUNCH(10, 2); break;         \
    case 6: LAUNCH(12, 2); break;         \
    case 7: LAUNCH(14, 2); break;         \
    case 8: LAUNCH(16, 2); break;         \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_gru_solo_fwd_bf16(const void* Wb, long s_wb, const float* b_ih, const float* b_hh, long s_rep, int Hc,
                                    const float* gx, long s_gx, void* hb, long s_hb, float* hs, long s_hs, float* sv, long s_sv,
                                    void* hT, long ld_hT, long s_hT, int Bc, int B, int H, int T, int groups, int workers,
                                    bool exact, hipStream_t s) {
  if (!gru_solo_bf16_supported(B, H) || T < 1 || Hc < 1 || Hc > H || Bc < 1 || Bc > B || (ld_hT & 1) != 0 || (s_hT & 1) != 0 ||
      (long)H * ld_hT * 2 >= 0x7fffffe0L)
    return hipErrorInvalidValue;
  if (groups <= 0) return hipSuccess;
  const int RT = gru_solo_bf16_row_tiles(B, workers);
  const bool four = B / RT == 4;
  KernelTimer kt(KID_GRU_FWD_PERSIST_BF16, 2.0 * B * 3 * H * (double)H * T * groups, s);
#define HPSGD_SOLOB_FWD_EX(HB, UB, V, EX)                                                                               \
  do {                                                                                                                \
    using S = SoloB<HB, UB, V>;                                                                                       \
    static std::atomic<size_t> allowed{0};                                                                            \
    if (const hipError_t e = allow_lds((const void*)gru_solo_fwd_bf16_kernel<HB, UB, V, EX>, S::FWD_LDS, allowed)) return e;\
    hipLaunchKernelGGL((gru_solo_fwd_bf16_kernel<HB, UB, V, EX>), dim3(groups * RT), dim3(S::NT), S::FWD_LDS, s,         \
                       (const __bf16*)Wb, s_wb, b_ih, b_hh, s_rep, Hc, gx, s_gx, (__bf16*)hb, s_hb, hs, s_hs, sv, s_sv, \
                       (__bf16*)hT, ld_hT, s_hT, Bc, B, T, RT);                                                       \
  } while (0)
#define HPSGD_SOLOB_FWD(HB, UB)                    \
  do {                                             \
    if (exact && four) HPSGD_SOLOB_FWD_EX(HB, UB, 1, true);   \
    else if (exact) HPSGD_SOLOB_FWD_EX(HB, UB, 2, true);      \
    else if (four) HPSGD_SOLOB_FWD_EX(HB, UB, 1, false);      \
    else HPSGD_SOLOB_FWD_EX(HB, UB, 2, false);                \
  } while (0)
  HPSGD_SOLOB_CASES(HPSGD_SOLOB_FWD)
#undef HPSGD_SOLOB_FWD_EX
#undef HPSGD_SOLOB_FWD
  return hipGetLastError();
}

hipError_t launch_gru_solo_bwd_bf16(const void* WT, long s_wt, const float* above, long s_above, const float* sv, long s_sv,
                                    const float* hs, long s_hs, void* dg4, long s_dg4, float* dbp, int Hc, int B, int H, int T,
                                    int groups, int workers, hipStream_t s) {
  if (!gru_solo_bf16_supported(B, H) || T < 1 || Hc < 1 || Hc > H || !above || ((uintptr_t)dg4 & 15) != 0 || (s_dg4 & 7) != 0)
    return hipErrorInvalidValue;
  if (groups <= 0) return hipSuccess;
  const int RT = gru_solo_bf16_row_tiles(B, workers);
  const bool four = B / RT == 4;
  KernelTimer kt(KID_GRU_BWD_PERSIST_BF16, 2.0 * B * 3 * H * (double)H * T * groups, s);
#define HPSGD_SOLOB_BWD1(HB, UB, V)                                                                                   \
  do {                                                                                                                \
    using S = SoloB<HB, UB, V>;                                                                                       \
    static std::atomic<size_t> allowed{0};                                                                            \
    if (const hipError_t e = allow_lds((const void*)gru_solo_bwd_bf16_kernel<HB, UB, V>, S::BWD_LDS, allowed)) return e; \
    hipLaunchKernelGGL((gru_solo_bwd_bf16_kernel<HB, UB, V>), dim3(groups * RT), dim3(S::NT), S::BWD_LDS, s, (const __bf16*)WT, \
                       s_wt, above, s_above, sv, s_sv, hs, s_hs, (__bf16*)dg4, s_dg4, dbp, Hc, B, T, RT);             \
  } while (0)
#define HPSGD_SOLOB_BWD(HB, UB)            \
  do {                                     \
    if (four) HPSGD_SOLOB_BWD1(HB, UB, 1); \
    else HPSGD_SOLOB_BWD1(HB, UB, 2);      \
  } while (0)
  HPSGD_SOLOB_CASES(HPSGD_SOLOB_BWD)
#undef HPSGD_SOLOB_BWD
#undef HPSGD_SOLOB_BWD1
  return hipGetLastError();
}

// As gru_stack_supported: one workgroup per CU beyond 64 units, two up to there, where tiles have 4 rows (solo_b_rows).  Local steps, layer by layer /
// this, us (H, batch, workers, steps; 1000 to 3000 words):
//   (256, 16, 4, 30) 386 / 284   (128, 16, 4, 35) 246 / 210   (64, 20, 4, 35) 226 / 203   (100, 10, 2, 20) 193 / 175 a round   (150, 20, 4, 6) 165 / 158
//   (220, 32, 8, 20), the chip full  361 / 309   (60, 64, 8, 20) 286 / 282       9999 words, (200, 20, 4, 20) 396 / 337 a round
bool gru_stack_bf16_supported(int B, int H, int T, int layers, int workers) {
  return layers == 2 && gru_solo_bf16_supported(B, H) && (long)workers * (B / 4) * 4 <= (H <= 64 ? 512 : 256) && 16L * T * B * H < 0x7fffffe0L;
}
size_t gru_stack_bf16_sync_words(int B, int groups) { return kLinkBase + (size_t)groups * (B / 4) * kLinkWords; }

hipError_t launch_gru_stack_fwd_bf16(const GruStackLayerB& lo, const GruStackLayerB& up, const void* W_ih, long s_wih, long s_wb, long s_rep,
                                     int Hc, long s_gx, long s_hb, long s_hs, long s_sv, long ld_hT, long s_hT, int Bc, int B, int H, int T,
                                     int groups, bool exact, unsigned* sync, unsigned limit, hipStream_t s) {
  if (!gru_stack_bf16_supported(B, H, T, 2, groups) || Hc < 1 || Hc > H || Bc < 1 || Bc > B || (ld_hT & 1) != 0 || (s_hT & 1) != 0 ||
      (long)H * ld_hT * 2 >= 0x7fffffe0L)
    return hipErrorInvalidValue;
  const int RT = B / 4, n = groups * RT;
  KernelTimer kt(KID_GRU_FWD_PERSIST_BF16, 2.0 * B * 3 * H * (double)H * T * groups * 2, s, 2);
#define HPSGD_STACKB_FWD_EX(HB, UB, EX)                                                                                      \
  do {                                                                                                                       \
    using S = SoloB<HB, UB, 1>;                                                                                              \
    constexpr size_t lds = S::FWD_LDS + (size_t)S::NC * 1024;                                                                \
    static std::atomic<size_t> allowed{0};                                                                                   \
    if (const hipError_t e = allow_lds((const void*)gru_stack_fwd_bf16_kernel<HB, UB, EX>, lds, allowed)) return e;          \
    hipLaunchKernelGGL((gru_stack_fwd_bf16_kernel<HB, UB, EX>), dim3(32 * ((n + 7) / 8)), dim3(S::NT), lds, s, lo, up,       \
                       (const __bf16*)W_ih, s_wih, s_wb, s_rep, Hc, s_gx, s_hb, s_hs, s_sv, ld_hT, s_hT, Bc, B, T, RT, n, sync, limit); \
  } while (0)
#define HPSGD_STACKB_FWD(HB, UB)                      \
  do {                                                \
    if (exact) HPSGD_STACKB_FWD_EX(HB, UB, true);     \
    else HPSGD_STACKB_FWD_EX(HB, UB, false);          \
  } while (0)
  HPSGD_SOLOB_CASES(HPSGD_STACKB_FWD)
#undef HPSGD_STACKB_FWD_EX
#undef HPSGD_STACKB_FWD
  return hipGetLastError();
}

hipError_t launch_gru_stack_bwd_bf16(const GruStackLayerB& lo, const GruStackLayerB& up, const void* WT_ih, long s_wih, long s_wt,
                                     const float* above, long s_above, float* dx, long s_dx, long s_hs, long s_sv, long s_dg4,
                                     int Hc, int B, int H, int T, int groups, unsigned* sync, unsigned limit, hipStream_t s) {
  if (!gru_stack_bf16_supported(B, H, T, 2, groups) || Hc < 1 || Hc > H || !above || (s_dg4 & 7) != 0) return hipErrorInvalidValue;
  const int RT = B / 4, n = groups * RT;
  KernelTimer kt(KID_GRU_BWD_PERSIST_BF16, 2.0 * B * 3 * H * (double)H * T * groups * 2, s, 2);
#define HPSGD_STACKB_BWD(HB, UB)                                                                                             \
  do {                                                                                                                       \
    using S = SoloB<HB, UB, 1>;                                                                                              \
    constexpr size_t lds = S::BWD_LDS + (size_t)S::NC3 * 1024;                                                               \
    static std::atomic<size_t> allowed{0};                                                                                   \
    if (const hipError_t e = allow_lds((const void*)gru_stack_bwd_bf16_kernel<HB, UB>, lds, allowed)) return e;              \
    hipLaunchKernelGGL((gru_stack_bwd_bf16_kernel<HB, UB>), dim3(32 * ((n + 7) / 8)), dim3(S::NT), lds, s, lo, up,           \
                       (const __bf16*)WT_ih, s_wih, s_wt, above, s_above, dx, s_dx, s_hs, s_sv, s_dg4, Hc, B, T, RT, n, sync, limit); \
  } while (0)
  HPSGD_SOLOB_CASES(HPSGD_STACKB_BWD)
#undef HPSGD_STACKB_BWD
  return hipGetLastError();
}

}  // namespace hpsgd
