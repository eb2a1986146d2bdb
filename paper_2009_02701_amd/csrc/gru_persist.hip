// Recurrence kernels that stay on the chip for a whole run of time steps (fp32).
//
// One launch per time step pays, at every step, a launch gap, a cold L2 and the transfer of
// the workgroup's slice of W_hh (the larger part of what a step reads).  Here a workgroup
// keeps its slice of W_hh (forward: the 3 x 16 gate rows of its 16 hidden units; backward:
// 16 rows of W_hh^T) in registers for all the steps of the launch, split into bf16 parts; the activations of the step
// (h_{t-1}, or the gate gradients of step t+1) go from memory straight into MFMA operand
// registers, every wave fetching and splitting exactly the fragments it multiplies, so that the matrix
// work of a step needs no barrier until the partial sums are combined.
//
// The steps of one launch depend on each other across workgroups: h_t of a 32-row batch tile
// is produced by the NJ = H/16 workgroups that own its hidden units, and every one of them
// needs all of it for step t+1.  Those NJ workgroups form a synchronisation group with one
// flag word per member in device memory.  Protocol (no cache-wide write-back or invalidate,
// which cost several microseconds per step when 32 workgroups of an XCD each ask for one):
//   producer: the exchanged values are stored with device-scope write-through stores (sc1);
//             the workgroup barrier waits until every wave's stores have completed; then
//             thread 0 stores the number of steps done into the member's flag (device scope);
//   consumer: wave 0 polls the group's flags (device-scope loads, one lane per member) until
//             all NJ producers have completed the step; workgroup barrier; the operand loads that follow are
//             device-scope loads (sc1), which are served from the level of the memory
//             hierarchy that all XCDs share, never from a stale line of this XCD's caches.
// Values nobody reads before the launch ends (the saved gates, dgx) take ordinary stores.
//
// Scope of the exchange.  A synchronisation group whose members all run on one XCD shares that
// XCD's L2, and the exchanged values and the counts need to get no further than that: ordinary
// stores (the CU's vector cache writes through to L2), the same sc1 loads on the consuming side
// (they bypass the vector cache, which is all that is needed of them there).  A hand-off among 32
// workgroups then takes 0.73 us instead of 1.92 us (measured).  Where a workgroup lands is the
// dispatcher's business (workgroup i of a launch is not always on XCD i % 8 when other launches
// are in flight), so a launch that wants this does not tie a workgroup's tile to its index: when
// the launch fills the chip with one workgroup per CU, every XCD necessarily receives as many
// workgroups as it has CUs, and a workgroup takes its place from where it runs - it draws a
// ticket from the counter of its XCD (HW_REG_XCC_ID) and is member `ticket` there, of the groups
// that the tile order gives to that XCD.  A ticket beyond the XCD's share (it cannot happen while
// one workgroup fills a CU) sets the abort word: the launch fails loudly.  Otherwise the tile is
// that of the workgroup index and the exchange is at device scope as described above.
//
// Waiting needs every workgroup of the grid resident at the same time: the launcher's grids have at most one
// workgroup for every compute unit of the device (a launch that places its workgroups by ticket asks for more than half of a
// CU's LDS each, so that there is one on every CU), and launches of these kernels from different streams are
// ordered against each other by the caller.  Every wait is bounded: when the spin limit runs
// out, or another workgroup has given up, the workgroup sets the abort word and the whole
// workgroup leaves the kernel, so every wave reaches its end whatever happens.
//
// Matrix work: 8 waves, 16 or 32 batch rows x 16 hidden units per workgroup.  The fp32 instruction (v_mfma_f32_16x16x4_f32)
// with the weights in LDS took 40 to 50 % of a step; the products are those of split_f32.h instead, a 2.7th of its cycles,
// the conversions beside them.  Where registers run out the smallest parts of the weights lie in LDS (persist_fwd_lw,
// persist_bwd_nl: a launch that spills is slower than the fp32 instruction, its reloads queue up with the operands; the one
// that still does, by 21 registers, 32 rows beyond H = 512 with the inputs projected, is faster than without the projection and
// with a product of its own for it, see gru_persist_xproj_supported).
// us per launch, before / now (forward, backward with its share of dW_hh):
//   35 steps, H = 512, 4 workers of 64 rows, input of 128     239 / 197    392 / 338   (168, 280 since two blocks take turns, below)
//   35 steps, H = 256, 4 workers of 16 rows, input of 128     146 /  89    182 / 134   ( 84, 114)
//    9 steps, H = 320, 4 workers of 40 rows, input of 32       48 /  38     57 /  50
// The contraction is cut into 32-wide chunks, chunk c belongs to the waves with wave % KW == c % KW; partial sums are combined
// through LDS.
// MFMA 16x16x32 lane layout: A lane l holds A[m = l%16][8 values of k], B lane l the same of B[..][n = l%16],
// accumulator register v holds C[4*(l/16) + v][l%16].  The order of the contraction index is free as long as both
// operands agree: lane group lg = l/16 takes k = 32c + 4 lg .. + 3 and 16 further on, i.e. two 16-byte pieces
// of its row per chunk, and one load instruction reads 64 contiguous bytes of each of 16 rows.
#include <type_traits>

#include "cell_math.h"
#include "kernels.h"
#include "split_f32.h"

namespace hpsgd {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int PNT = 512;     // threads per workgroup
constexpr int PJ = 16;       // hidden units per workgroup
constexpr int PC = 32;       // contraction chunk

// A synchronisation group owns PF flag words, one per member: a member stores the number of
// steps it has completed into its own word (plain device-scope stores to distinct words: no
// read-modify-write that the group's members would queue up for), and the waiting side reads
// all of them with one load instruction of wave 0, lane l looking at member l.
constexpr int PF = 64;  // flag words per group (a group has H/16 or H/32 <= 42 members)

// Wave 0 polls the group's flags until every member has reached `target` (wrap-safe), then the
// whole workgroup passes a barrier.  Returns false, for every thread alike, if the wait was
// given up; the abort word is then set.  limit == 0 makes every wait fail (the host-forced
// way to exercise the abort path).
__device__ __forceinline__ bool group_wait(unsigned* flags, int members, unsigned target, unsigned* abort_w,
                                           unsigned limit, int* lds_flag) {
  if (threadIdx.x < 64) {
    const int l = threadIdx.x;
    int ok = limit != 0;
    unsigned n = 0;
    while (ok) {
      const unsigned v = __hip_atomic_load(flags + (l < members ? l : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__all((int)(v - target) >= 0)) break;
      if (++n > limit || __hip_atomic_load(abort_w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) ok = 0;
      else __builtin_amdgcn_s_sleep(1);
    }
    if (l == 0) {
      if (!ok) __hip_atomic_store(abort_w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *lds_flag = ok;
    }
  }
  __syncthreads();
  return *lds_flag != 0;
}

// Publishes the number of steps this member has completed, after the step's exchanged values.
// Order of data and count, by construction:
//   1. every wave waits until the vector-memory counter of its own accesses is zero
//      (s_waitcnt vmcnt(0): on this target stores count in vmcnt too, and a device-scope
//      write-through store is counted out only when the level of the memory hierarchy that all
//      XCDs share has acknowledged it);
//   2. the workgroup barrier: every wave of the workgroup has passed step 1;
//   3. thread 0 stores the count (device scope).
// A consumer that reads the count (device-scope load) and then issues its operand loads
// (device-scope, behind a barrier of its own workgroup) therefore reads the data of the step.
// The wait is written out: a workgroup-scope fence would only have to order LDS traffic here,
// and an agent-scope release would write back the XCD's whole L2.
// (l2x: the group shares one L2 and an ordinary store, acknowledged by that L2, takes the place of
// the write-through store in steps 1 and 3.)
__device__ __forceinline__ void group_signal(unsigned* my_flag, unsigned steps_done, bool l2x) {
  // vmcnt = 0 (bits 3:0 and 15:14), expcnt and lgkmcnt left at their maxima (no wait)
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (l2x) __hip_atomic_store(my_flag, steps_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(my_flag, steps_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The XCD this wave runs on (HW_REG_XCC_ID, bits 3:0)
__device__ __forceinline__ unsigned xcc_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u; }

// Which tile this workgroup takes - synchronisation group sg (of the launch's n_sg, before sg0), member
// tx - and whether its group exchanges through one L2.
// tickets == nullptr: by the workgroup index, device scope.  Else (8 counters behind the flag words,
// zero at the start of the step; this launch is the one whose tickets start at ticket_base; one workgroup
// per CU of the device, per_xcd of them per XCD): ticket t of XCD x is member t % NJ of the x-th group of
// round t / NJ, so that a group's members share an XCD.  A workgroup whose ticket names no group of the
// launch waits until every ticket of the launch has been drawn (bounded) and leaves: gone earlier, it would
// make room on its XCD for a workgroup that another XCD is counting on.  A ticket beyond the XCD's share
// (it cannot happen while one workgroup fills a CU) sets the abort word.  Returns false, for every thread
// alike, if the workgroup has nothing to do.  Contains a barrier.
__device__ __forceinline__ bool persist_place(unsigned* tickets, unsigned ticket_base, unsigned per_xcd, unsigned* abort_w,
                                              unsigned limit, int* lds_word, int NJ, int n_sg, int& tx, int& sg, bool& l2x) {
  l2x = tickets != nullptr;
  if (!l2x) {
    // a group's workgroups are kept 8 apart when the number of groups allows it (workgroup i often runs on
    // XCD i % 8)
    const int i = blockIdx.x;
    if (n_sg % 8 == 0) {
      sg = (i & 7) + 8 * ((i >> 3) / NJ);
      tx = (i >> 3) % NJ;
    } else {
      sg = i / NJ;
      tx = i % NJ;
    }
    return true;
  }
  if (threadIdx.x == 0) {
    const unsigned x = xcc_id();
    unsigned t = per_xcd;
    if (x < 8u) t = __hip_atomic_fetch_add(tickets + x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - ticket_base;
    const bool ok = t < per_xcd;
    if (!ok) __hip_atomic_store(abort_w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int round = ok ? (int)t / NJ : 0, s = 8 * round + (int)x;
    lds_word[0] = ok && round < (int)per_xcd / NJ && s < n_sg ? s : -1;
    lds_word[1] = (int)t - round * NJ;
    if (ok && lds_word[0] < 0) {
      for (unsigned n = 0; n < limit; ++n) {
        unsigned left = 0;
        for (int c = 0; c < 8; ++c)
          left |= __hip_atomic_load(tickets + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - ticket_base < per_xcd ? 1u : 0u;
        if (!left) break;
        __builtin_amdgcn_s_sleep(8);
      }
    }
  }
  __syncthreads();
  // (uniform, and known as such: addresses then take scalar registers)
  sg = __builtin_amdgcn_readfirstlane(lds_word[0]);
  tx = __builtin_amdgcn_readfirstlane(lds_word[1]);
  __syncthreads();  // (the words are used again by the first wait)
  return sg >= 0;
}

// The block of the exchange buffer that holds h_t, and that of the gate gradients of step t.  Where the group shares one L2
// two blocks take turns (block 0 keeps h_0): a workgroup that writes h_t has seen every member finish step t - 1, which
// is behind the member's reads of h_{t-2}; likewise backward.  Their lines then stay in the L2, where a block per step
// would be written into new lines that push others out: the operands of a backward step of 32 rows x 1024 units (bf16)
// arrive in 4100 cycles instead of 6100 to 6900, and its launch of 35 steps takes 180 us instead of 216 (forward 128, before 152).  At device scope every step has its own block: another XCD's L2 must not
// hold its lines from an earlier step.
__device__ __forceinline__ long fwd_block(int t, bool l2x) { return l2x && t > 0 ? 2 - (t & 1) : t; }
__device__ __forceinline__ long bwd_block(int t, bool l2x) { return l2x ? t & 1 : t; }

// 16 bytes at byte offset `off` (the lane's) + `from` (uniform) of the buffer, as a device-scope load
__device__ __forceinline__ float4 ld16_dev(__amdgpu_buffer_rsrc_t rs, int off, int from) {
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, off, from, 16 /* sc1 */);
  return __builtin_bit_cast(float4, v);
}
// store of an exchanged value: device-scope (write-through), or ordinary when the group shares one L2
__device__ __forceinline__ void st_dev(float* p, float v, bool l2x) {
  if (l2x) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// not finite, or rounded to an infinity by the split
__device__ __forceinline__ bool split_beyond(float v) { return !(fabsf(v) < 3.38e38f); }
__device__ __forceinline__ bool split_beyond(const float4& v) {
  return split_beyond(v.x) || split_beyond(v.y) || split_beyond(v.z) || split_beyond(v.w);
}

// The fragment of 32-chunk c of a weight row (KD words at src, at any alignment; ok: the row exists) in the order in which
// the activations come: words 32c + 4 lg .. + 3 and 16 further on; zeros beyond KD and for a row that does not exist.
__device__ __forceinline__ void weight_row_frag(const float* __restrict__ src, bool ok, int KD, int c, float4 (&v)[2]) {
  const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int k = PC * c + 16 * h + 4 * lg;
    v[h] = make_float4(ok && k < KD ? src[k] : 0.f, ok && k + 1 < KD ? src[k + 1] : 0.f, ok && k + 2 < KD ? src[k + 2] : 0.f,
                       ok && k + 3 < KD ? src[k + 3] : 0.f);
  }
}
// The same, row `row` of the matrix rs of at least 4 words a row, for a launch's start: no branch stands between the loads, all of
// which are in flight at once.  What does not exist is read beyond the matrix, which the buffer's range check answers with zeros; a
// piece that the row ends in is the row's last four words, which weight_row_tail moves up.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_rsrc(const float* W, int rows, int KD) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W), 0, rows * KD * 4, 0x00020000);
}
__device__ __forceinline__ void weight_row_load(__amdgpu_buffer_rsrc_t rs, int row, bool ok, int KD, int c, float4 (&v)[2]) {
  constexpr int beyond = 0x7ffffff0;
  const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int k = PC * c + 16 * h + 4 * lg;
    v[h] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, ok && k < KD ? (row * KD + min(k, KD - 4)) * 4 : beyond, 0, 0));
  }
}
__device__ __forceinline__ void weight_row_tail(int KD, int c, float4 (&v)[2]) {
  if (PC * c + PC <= KD || (KD & 3) == 0) return;  // (uniform)
  const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int up = PC * c + 16 * h + 4 * lg + 4 - KD;  // (beyond 3: zeros already; below 1: all of it in the row)
    if (up == 1) v[h] = make_float4(v[h].y, v[h].z, v[h].w, 0.f);
    if (up == 2) v[h] = make_float4(v[h].z, v[h].w, 0.f, 0.f);
    if (up == 3) v[h] = make_float4(v[h].w, 0.f, 0.f, 0.f);
  }
}

// The two pieces of this lane's fragment of chunk c of a row-major tile of the layer input (row pitch KD words, a multiple
// of 16: each piece is all in or all out): rows >= rows_valid are read from row 0 (their results are never stored), columns beyond
// KD are zeros (they meet a zero weight, which an infinite input of another column would turn into NaN).
__device__ __forceinline__ void input_frag(__amdgpu_buffer_rsrc_t rs, int KD, int rows_valid, int row, int c, float4 (&a)[2]) {
  const int off = ((row < rows_valid ? row : 0) * KD + 4 * (int)((threadIdx.x & 63) >> 4)) * 4;
  a[0] = ld16_dev(rs, off, PC * 4 * c);
  a[1] = PC * c + 16 < KD ? ld16_dev(rs, off, PC * 4 * c + 64) : make_float4(0.f, 0.f, 0.f, 0.f);  // (uniform)
}

// The exchanged operands (h_t, the gate gradients) are not read from a row-major matrix: there a
// load instruction fetches 64 bytes of each of 16 rows, half a cache line per row, which a CU
// does 2.8 times slower than whole lines (see the bf16 part below).  They are kept
// fragment-major: per step a block of ceil(B/16) row blocks x ceil(KD/32) chunks x 2 halves,
// each the 1 KB one load instruction reads, lane l's 16 bytes at byte 16 l (lane l: row l % 16,
// contraction indices 16 half + 4 (l / 16) .. + 3 of the chunk): row r's index k lies at word
// (((r / 16) chunks + k / 32) 2 + (k / 16) % 2) 256 + (16 ((k % 16) / 4) + r % 16) 4 + k % 4.  Halves beyond KD are never written and never read.  KD is HP = 16 ceil(H / 16)
// for h_t and 3 HP for the gate gradients (gate q's unit j at index q HP + j): whole halves for every H.
// words of a step's block
__host__ __device__ __forceinline__ long xblock_words(int B, int KD) {
  return (long)((B + 15) / 16) * 16 * ((KD + PC - 1) / PC) * PC;
}
// the two pieces of chunk c of row block rbx of a step's block (rs); a half beyond KD: zeros
__device__ __forceinline__ void exchange_frag(__amdgpu_buffer_rsrc_t rs, int nch, int KD, int rbx, int c, float4 (&a)[2]) {
  const int off = (int)(threadIdx.x & 63) * 16, from = (rbx * nch + c) * 2048;
  a[0] = ld16_dev(rs, off, from);
  a[1] = PC * c + 16 < KD ? ld16_dev(rs, off, from + 1024) : make_float4(0.f, 0.f, 0.f, 0.f);  // (uniform)
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const float* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0x7fffffe0, 0x00020000);
}

// The KW partial sums of an output, in a fixed order (PL words apart)
template <int KW>
__device__ __forceinline__ float sum_planes(const float* red, int o, int PL) {
  float v = (red[o] + red[o + PL]) + (red[o + 2 * PL] + red[o + 3 * PL]);
  if (KW == 8) v += (red[o + 4 * PL] + red[o + 5 * PL]) + (red[o + 6 * PL] + red[o + 7 * PL]);
  return v;
}

// Whether the forward kernel keeps the smallest parts of its slice of W_hh in LDS: with them in registers it would spill.
__host__ __device__ constexpr bool persist_fwd_lw(int ncw, int xnb, int rbw) { return ncw >= 4 || rbw == 2 || (ncw == 3 && xnb == 2); }

// Forward: steps t = 0 .. T-1.  hs holds h_0 .. h_T ((T+1) blocks of B x H per worker, h_0
// given), gx the input projections of all steps, sv receives r|z|n|q of every step.
// sync: the abort word, then 64 flag words per synchronisation group; `base` is what the
// flags read when the kernel starts.
// XNB > 0: the kernel computes the input projection itself, gx_t = x_t W_ih^T + b_ih, from the
// layer input xin (blocks of B x width per step) with its 48 rows of W_ih resident in LDS;
// that part of a step does not depend on the other workgroups and is done before the wait.
// The r and z gates then take one sum over both contractions; gx is not used.
// PRT batch rows per workgroup.  KW waves share the contraction, NCW chunks each (H <= 32 KW NCW; the layer input's width
// <= 32 KW XNB); with KW = 4 the other four have the second 16 rows, with KW = 8 a wave has all rows.
template <int NCW, int XNB, int PRT, int KW>
__global__ void __launch_bounds__(PNT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_fwd_persist_kernel(const float* __restrict__ W_hh, const float* __restrict__ b_hh, long s_rep,
                       const float* __restrict__ gx, long s_gx, float* __restrict__ hs, long s_hs, float* hx, long s_hx,
                       float* __restrict__ sv, long s_sv, int B, int H, int T, int sg0, int n_sg, unsigned* sync, unsigned base,
                       unsigned spin_limit, unsigned* tickets, unsigned ticket_base, unsigned per_xcd,
                       const float* __restrict__ xin, long s_x, int width,
                       const float* __restrict__ W_ih, const float* __restrict__ b_ih) {
  extern __shared__ __attribute__((aligned(16))) float persist_lds[];
  constexpr int RB = PRT / 16, RBW = RB * KW / 8;  // row blocks of the tile, of a wave
  static_assert(RBW >= 1, "8 waves");
  constexpr bool XP = XNB > 0;
  constexpr int XB = XP ? XNB : 1;
  constexpr bool LW = persist_fwd_lw(NCW, XNB, RBW);  // the smallest parts of W_hh lie in LDS
  // The split is as exact as the fp32 instruction, which a projection by a product of few tiles has, for operands of at least 2^-110.  Beyond
  // H = 512, where every projection of a width that fits is made here, a step's input with a smaller one (zero is none), and every step
  // of a workgroup with such a weight, takes that instruction.
  constexpr bool LOW = XP && KW == 8 && NCW > 2;
  constexpr int NP = XP ? 4 : 3;             // planes of partial sums: r, z, q (+ the x part of n)
  const int NJ = (H + PJ - 1) / PJ, HP = NJ * PJ, RT = (B + PRT - 1) / PRT;
  const int nch = (HP + PC - 1) / PC, nchw = XP ? (width + PC - 1) / PC : 0;
  float* red = persist_lds;                                       // [KW][RB][NP][4][64] partial sums
  u32x4_t* wx = reinterpret_cast<u32x4_t*>(red + KW * RB * NP * 256);   // [nchw][3 gates][3 parts][64 lanes]: W_ih
  u32x4_t* wl = wx + nchw * 9 * 64;                               // [KW][NCW][3][64]
  int* lds_flag = reinterpret_cast<int*>(wl + (LW ? KW * NCW * 3 * 64 : 0));
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = wave & (KW - 1), rsel = RBW == RB ? 0 : wave / KW;   // first row block of this wave
  const int lr = lane & 15, lg = lane >> 4;
  unsigned* abort_w = sync;
  int tx, sg;
  bool l2x;
  if (!persist_place(tickets, ticket_base, per_xcd, abort_w, spin_limit, lds_flag, NJ, n_sg, tx, sg, l2x)) return;
  sg += sg0;
  const int g = sg / RT, ty = sg - g * RT;
  const int j0 = tx * PJ, r0 = ty * PRT;
  unsigned* flags = sync + 1 + sg * PF;
  __builtin_amdgcn_s_setprio(3);
  const int j = j0 + lr, jc = min(j, H - 1);
  const bool jok = j < H;
  // the resident slices: gate q's fragment of chunk c holds W_hh[q H + j][32 c ..], this wave's chunks kw + KW i
  // Everything that a launch reads before its first step is requested before anything waits for it (a piece at a time, each loaded and
  // split, was a serial chain of up to 12 trips to memory).  us per launch of one step, a piece at a time / so: H = 512, 4 workers of 64
  // rows 23.3 / 21.0,  H = 320, 4 of 40 13.3 / 11.1,  H = 256, 4 of 16 10.8 / 10.2; of 10 steps, H = 450 (rows not aligned), 6 of 40 55.6 / 48.2.
  // (In the backward kernel the same costs more registers, and its steps more than its start gains: 20 steps of H = 500, 8 of 64 rows 165.5 / 171.2.)
  const __amdgpu_buffer_rsrc_t rw = weight_rsrc(W_hh + g * s_rep, 3 * H, H);
  float4 wv[NCW][3][2];
#pragma unroll
  for (int i = 0; i < NCW; ++i)
#pragma unroll
    for (int q = 0; q < 3; ++q) weight_row_load(rw, q * H + jc, jok && kw + KW * i < nch, H, kw + KW * i, wv[i][q]);
  float4 xv[2];  // fragment u = 3 chunk + gate of the slice of W_ih, by wave u % 8
  auto load_wx = [&](int u) {
    if (u < 3 * nchw) weight_row_load(weight_rsrc(W_ih + g * s_rep, 3 * H, width), (u % 3) * H + jc, jok, width, u / 3, xv);
  };
  if (XP) load_wx(wave);
  const bool act = RB == 2 || wave < 4;             // this wave has outputs (uniform)
  const int qv = wave & 3, rbo = RB == 2 ? wave >> 2 : 0;
  const int row = r0 + rbo * 16 + 4 * lg + qv;      // this thread's element of the tile
  const int rowc = min(row, B - 1);                 // loads are clamped, stores guarded
  const bool ok = row < B && jok;
  const float* bh = b_hh + g * s_rep;
  float bias[3], biasx[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 3; ++q) bias[q] = jok ? bh[q * H + jc] : 0.f;
  if (XP) {
#pragma unroll
    for (int q = 0; q < 3; ++q) biasx[q] = jok ? (b_ih + g * s_rep)[q * H + jc] : 0.f;
  }
  float* hsg = hs + g * s_hs;
  float* hxg = hx + g * s_hx;                 // h_0 .. h_T as the workgroups exchange them
  const long xblk = xblock_words(B, HP);
  int rbx[RBW];  // this wave's row blocks (one beyond the batch: the tile's first)
#pragma unroll
  for (int rb = 0; rb < RBW; ++rb) rbx[rb] = (r0 + (rsel + rb) * 16 < B ? r0 + (rsel + rb) * 16 : r0) >> 4;
  float hpv = jok ? hsg[(long)rowc * H + jc] : 0.f;
  float4 xa[RBW][XB][2];  // this step's fragments of the layer input, loaded one step ahead
  float gxn[3] = {0.f, 0.f, 0.f};  // ... or its input projection
  // (uniform addresses and 32-bit offsets of the lane)
  const unsigned ogx = rowc * 3 * H + jc, osv = row * 4 * H + j, oh = row * H + j;
  // where the lane's unit goes in a step's block 
  const unsigned xb = ((r0 / 16 + rbo) * nch * 2 + j0 / 16) * 256, xl = (((lr >> 2) << 4) + (row & 15)) * 4 + (lr & 3);
  auto load_x = [&](int t) {
    if (XP) {
      const __amdgpu_buffer_rsrc_t rs = tile_rsrc(xin + g * s_x + ((long)t * B + r0) * width);
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
        for (int i = 0; i < XB; ++i)
          if (kw + KW * i < nchw) input_frag(rs, width, B - r0, (rsel + rb) * 16 + lr, kw + KW * i, xa[rb][i]);
    } else if (act) {
      const float* gxt = gx + g * s_gx + (long)t * B * 3 * H;
#pragma unroll
      for (int q = 0; q < 3; ++q) gxn[q] = (gxt + q * H)[ogx];
    }
  };
  load_x(0);
  __builtin_amdgcn_sched_barrier(0);
  bf16x8s w[NCW][3][LW ? 2 : 3];
  bool beyond = false;
  const int Ht = rarely(H);
#pragma unroll
  for (int i = 0; i < NCW; ++i)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      weight_row_tail(Ht, kw + KW * i, wv[i][q]);
      beyond = beyond || split_beyond(wv[i][q][0]) || split_beyond(wv[i][q][1]);
      const SplitFrag f = split_frag(wv[i][q][0], wv[i][q][1]);
      w[i][q][0] = f.p[0];
      w[i][q][1] = f.p[1];
      if (LW) wl[((kw * NCW + i) * 3 + q) * 64 + lane] = __builtin_bit_cast(u32x4_t, f.p[2]);  // (KW = 4: by two waves, the same)
      else w[i][q][LW ? 0 : 2] = f.p[2];
      __builtin_amdgcn_sched_barrier(0);  // (in the order of the loads: each piece frees the registers it came in)
    }
  beyond = __any(beyond);
  bool low_w = false;
  if (XP) {
    for (int u = wave; u < 3 * nchw; u += 8) {
      if (LOW) low_w = low_w || split_below(xv[0], xv[1]);
      const SplitFrag f = split_frag(xv[0], xv[1]);
      load_wx(u + 8);
#pragma unroll
      for (int p = 0; p < 3; ++p) wx[(u * 3 + p) * 64 + lane] = __builtin_bit_cast(u32x4_t, f.p[p]);
    }
    low_w = __any(low_w) != 0;
    if (LOW && lane == 0) reinterpret_cast<unsigned char*>(lds_flag + 2)[wave] = low_w;
  }
  __syncthreads();
  if (LOW) low_w = (lds_flag[2] | lds_flag[3]) != 0;
  for (int t = 0; t < T; ++t) {
    // what does not depend on the recurrence is computed in front of the wait
    const float gxv[3] = {gxn[0], gxn[1], gxn[2]};
    floatx4 big[RBW][3], small[RBW][3], accx[RBW];
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) {
#pragma unroll
      for (int q = 0; q < 3; ++q) big[rb][q] = small[rb][q] = (floatx4){0.f, 0.f, 0.f, 0.f};
      accx[rb] = (floatx4){0.f, 0.f, 0.f, 0.f};
    }
    if (XP) {
      bool low[RBW];
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) low[rb] = low_w;
#pragma unroll
      for (int i = 0; i < XB; ++i) {
        const int c = kw + KW * i;
        if (c >= nchw) continue;  // (uniform)
        SplitFrag wq[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int p = 0; p < 3; ++p) wq[q].p[p] = __builtin_bit_cast(bf16x8s, wx[((c * 3 + q) * 3 + p) * 64 + lane]);
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb) {
          if (LOW) low[rb] = low[rb] || split_below(xa[rb][i][0], xa[rb][i][1]);
          split_mfmas(split_frag(xa[rb][i][0], xa[rb][i][1]), wq, big[rb], small[rb]);
        }
      }
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        bool redo = LOW && __any(low[rb]) != 0;
#pragma unroll
        for (int q = 0; q < 3; ++q) redo = any_beyond(big[rb][q] + small[rb][q]) || redo;
        if (__builtin_expect(redo, 0)) {
          const int wd = rarely(width);
          const __amdgpu_buffer_rsrc_t rs = tile_rsrc(xin + g * s_x + ((long)t * B + r0) * wd);
          const float* Xr = rarely(W_ih) + g * s_rep + (long)jc * wd;
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            big[rb][q] = small[rb][q] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int c = kw; c < nchw; c += KW) {
              float4 v[2], x[2];
              input_frag(rs, wd, B - r0, (rsel + rb) * 16 + lr, c, x);
              weight_row_frag(Xr + (long)q * H * wd, jok, wd, c, v);
              plain_mfmas(x, v, PC * c + 16 < wd, big[rb][q]);
            }
          }
        }
        // n keeps its two parts apart: n = tanh(x part + r * (h part))
        accx[rb] = big[rb][2] + small[rb][2];
        big[rb][2] = small[rb][2] = (floatx4){0.f, 0.f, 0.f, 0.f};
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (t > 0 && !group_wait(flags, NJ, base + (unsigned)t, abort_w, spin_limit, lds_flag)) return;
    {
      const __amdgpu_buffer_rsrc_t rs = tile_rsrc(hxg + fwd_block(t, l2x) * xblk);
      float4 a[RBW][NCW][2];
#pragma unroll
      for (int i = 0; i < NCW; ++i)
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb)
          if (kw + KW * i < nch) exchange_frag(rs, nch, HP, rbx[rb], kw + KW * i, a[rb][i]);  // (uniform)
      __builtin_amdgcn_sched_barrier(0);  // every load is issued before anything waits for one
      if (__builtin_expect(beyond, 0)) {
        const int Hr = rarely(H);
        const float* Wr = rarely(W_hh) + g * s_rep + (long)jc * Hr;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int rb = 0; rb < RBW; ++rb) {
#pragma unroll 1
            for (int c = kw; c < nch; c += KW) {
              float4 v[2], x[2];
              exchange_frag(rs, nch, HP, rbx[rb], c, x);
              weight_row_frag(Wr + (long)q * Hr * Hr, jok, Hr, c, v);
              plain_mfmas(x, v, PC * c + 16 < HP, big[rb][q]);
            }
          }
      } else {
#pragma unroll
        for (int i = 0; i < NCW; ++i) {
          if (kw + KW * i >= nch) continue;
          SplitFrag wi[3];
#pragma unroll
          for (int q = 0; q < 3; ++q)
            wi[q] = {{w[i][q][0], w[i][q][1], LW ? __builtin_bit_cast(bf16x8s, wl[((kw * NCW + i) * 3 + q) * 64 + lane]) : w[i][q][LW ? 0 : 2]}};
#pragma unroll
          for (int rb = 0; rb < RBW; ++rb) split_mfmas(split_frag(a[rb][i][0], a[rb][i][1]), wi, big[rb], small[rb]);
        }
      }
      // Step t+1's layer input (or input projection).  Not in front of the products: a CU's loads return in the order of their
      // issue, whichever wave's they are, and the second four waves' operands would wait for these to come from memory.
      __builtin_amdgcn_sched_barrier(0);
      load_x(min(t + 1, T - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int q = 0; q < 3; ++q) red[(((kw * RB + rsel + rb) * NP + q) * 4 + v) * 64 + lane] = big[rb][q][v] + small[rb][q][v];
        if (XP) red[(((kw * RB + rsel + rb) * NP + 3) * 4 + v) * 64 + lane] = accx[rb][v];
      }
    __syncthreads();
    if (act) {
      float gh[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q)
        gh[q] = sum_planes<KW>(red, ((rbo * NP + q) * 4 + qv) * 64 + lane, RB * NP * 256);
      const float r = sigm_f32(gxv[0] + biasx[0] + (gh[0] + bias[0]));
      const float z = sigm_f32(gxv[1] + biasx[1] + (gh[1] + bias[1]));
      const float q2 = gh[2] + bias[2];
      const float n = tanh_f32((XP ? gh[NP - 1] + biasx[2] : gxv[2]) + r * q2);
      // (the lanes beyond H compute with unit H-1's projection, or an infinite input times a zero weight: whatever
      // that is - a NaN too, which a zero factor would keep - the h that the others multiply is zero)
      const float hn = jok ? (1.0f - z) * n + z * hpv : 0.f;
      if (row < B) st_dev(hxg + fwd_block(t + 1, l2x) * xblk + xb + xl, hn, l2x);
      if (ok) {
        (hsg + (long)(t + 1) * B * H)[oh] = hn;
        float* svt = sv + g * s_sv + (long)t * B * 4 * H;
        svt[osv] = r;
        (svt + H)[osv] = z;
        (svt + 2 * H)[osv] = n;
        (svt + 3 * H)[osv] = q2;
      }
      hpv = hn;
    }
    group_signal(flags + tx, base + (unsigned)t + 1u, l2x);  // (its barrier also separates the reads of red from the next step's writes)
    // Through memory the first look is not issued before this workgroup's flag is out.  Issued at once it comes back as late, behind the flag, and too
    // early to show the others'; the next look, with the abort word's before it, is 2 us further on.  us per local step of 60 steps, 16 rows, 4 workers,
    // without this / with it: H = 520, input 20  755 / 735,  576, 16  733 / 706,  640, 256  800 / 778,  704, 20  879 / 857.  (Tiles of 32 rows have more to do
    // in front of the wait: H = 640, input 64  1108 / 1125.)
    if (PRT == 16 && !l2x) __builtin_amdgcn_s_waitcnt(0x0F70);
  }
}

// Backward: steps t = T-1 down to 0.  The workgroup's resident slice is 16 columns of
// W_hh (3H x H).  dgh and
// dgx hold the gate gradients of all steps (blocks of B x 3H); block t+1 of the exchanged copy is the
// contraction operand of step t (none at t = T-1).  D holds the gradient carried into the last step (the
// head's; d_zero: it is zero and D is not read).
// above: per-step gradient from the layer above (blocks of B x H) or nullptr.
//
// dWp (nullable, H <= 512): the workgroup also accumulates its share of the recurrent weight
// gradient over the steps of the launch, dW_hh[q*H + j0 + m][:] += sum over its batch rows
// of dgh_t[row][q*H + j0 + m] * h_{t-1}[row][:], and stores it at the end to
// dWp[(g * RT + ty)][3H][H] (one partial sum per batch-row tile; the caller adds the RT of
// them).  That work does not depend on the other workgroups: it is done between counting
// the step in and waiting for the next one, in the time the chain of waits leaves idle.
// Wave w owns columns 64w .. 64w+63 and all 48 gate rows (3 x 4 accumulator tiles); tile
// (mt, jt) holds the columns 64w + 4*lane%16 + jt, so that a lane fetches h as four floats per
// batch row and stores its results as such.
//
// Register cap: two waves of this kernel share a SIMD, and at 256 registers each they would own
// its whole register file, so that no wave of any other kernel (the merge of the other stream,
// a short kernel queued behind) could start on a CU before this launch has ended.  The
// attribute counts in halves of the unified VGPR/AGPR file on this target: 124 caps the wave at
// 248 registers, which leaves 16 per SIMD for a co-tenant.
typedef float f4ua __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any 4-byte boundary

// The workgroup's share of dW_hh takes its operands in the order of the batch rows: a stage of the step's gate gradients,
// transposed and split, [part][gate row][batch row].
constexpr int SPT = 40;  // its pitch in values: 16-byte pieces of 16 gate rows in different banks

// The batch rows of a lane's operand: 8 of the 32 with v_mfma_f32_16x16x32_bf16, 4 of the 16 with v_mfma_f32_16x16x16_bf16.
typedef short bf16x4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ floatx4 dw_mfma(const bf16x8s& a, const bf16x8s& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 dw_mfma(const bf16x4s& a, const bf16x4s& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
// column jt of the rows v, split
__device__ __forceinline__ void split_rows(const f4ua (&v)[8], int jt, bf16x8s (&h)[3]) {
  const SplitFrag f = split_frag(make_float4(v[0][jt], v[1][jt], v[2][jt], v[3][jt]), make_float4(v[4][jt], v[5][jt], v[6][jt], v[7][jt]));
#pragma unroll
  for (int p = 0; p < 3; ++p) h[p] = f.p[p];
}
__device__ __forceinline__ void split_rows(const f4ua (&v)[4], int jt, bf16x4s (&h)[3]) {
  uint2 p[3];
  split2(v[0][jt], v[1][jt], p[0].x, p[1].x, p[2].x);
  split2(v[2][jt], v[3][jt], p[0].y, p[1].y, p[2].y);
#pragma unroll
  for (int i = 0; i < 3; ++i) h[i] = __builtin_bit_cast(bf16x4s, p[i]);
}

// How many of the three parts of the resident weights lie in LDS, the smallest first (each wave reads back only its own): with
// them in registers the kernel would spill.
__host__ __device__ constexpr int persist_bwd_nl(int ncw, int prt) { return ncw > 6 ? 0 : prt == 32 ? (ncw >= 3 ? 2 : 1) : ncw >= 6 ? 2 : ncw >= 4 ? 1 : 0; }

// NCW: chunks of the contraction per wave (3 HP <= 256 NCW)
template <int NCW, int PRT>
__global__ void __launch_bounds__(PNT) __attribute__((amdgpu_num_vgpr(124)))
gru_bwd_persist_kernel(const float* __restrict__ W_hh, long s_rep, float* __restrict__ dgh, float* dghx, long s_dghx,
                       float* __restrict__ dgx, long s_dg,
                       const float* __restrict__ D, long s_D, int d_zero, const float* __restrict__ above, long s_above,
                       const float* __restrict__ sv, long s_sv, const float* __restrict__ hs, long s_hs,
                       int B, int H, int T, int sg0, int n_sg, unsigned* sync, unsigned base,
                       unsigned spin_limit, unsigned* tickets, unsigned ticket_base, unsigned per_xcd,
                       float* __restrict__ dWp, float* __restrict__ dbp) {
  extern __shared__ __attribute__((aligned(16))) float persist_lds[];
  constexpr int RB = PRT / 16;
  constexpr int DR = PRT / 4;                                       // batch rows per lane of the dW_hh products
  using DwFrag = std::conditional_t<PRT == 32, bf16x8s, bf16x4s>;
  constexpr int JN = PRT == 32 ? 2 : 4;                             // columns split at a time (registers)
  constexpr bool DW = NCW <= 6;                                     // (8 waves x 64 columns cover H)
  constexpr int NL = persist_bwd_nl(NCW, PRT), NR = 3 - NL;         // parts of the weights in LDS, in registers
  const int NJ = (H + PJ - 1) / PJ, HP = NJ * PJ, RT = (B + PRT - 1) / PRT;
  const int H3 = 3 * H, HP3 = 3 * HP;
  const int nch = (HP3 + PC - 1) / PC;
  float* red = persist_lds;                                         // [8][RB][4][64]
  __bf16* stage = reinterpret_cast<__bf16*>(red + 8 * RB * 256);    // [3 parts][48][SPT]
  u32x4_t* wl = reinterpret_cast<u32x4_t*>(stage + 3 * 48 * SPT);   // [8 waves][NCW][NL][64 lanes]
  int* lds_flag = reinterpret_cast<int*>(wl + 8 * NCW * NL * 64);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  unsigned* abort_w = sync;
  int tx, sg;
  bool l2x;
  if (!persist_place(tickets, ticket_base, per_xcd, abort_w, spin_limit, lds_flag, NJ, n_sg, tx, sg, l2x)) return;
  sg += sg0;
  const int g = sg / RT, ty = sg - g * RT;
  const int j0 = tx * PJ, r0 = ty * PRT;
  unsigned* flags = sync + 1 + sg * PF;
  __builtin_amdgcn_s_setprio(3);
  // weight-gradient share: this lane's 4 columns (clamped: results outside H are not stored)
  const int wn = 64 * wave + 4 * lr;
  const bool dw_wave = DW && dWp != nullptr && 64 * wave < H;  // (uniform)
  const bool wn_ok = dw_wave && wn < H;
  const int wnc = wn < H ? wn : 0;
  floatx4 dw[3][4];
#pragma unroll
  for (int mt = 0; mt < 3; ++mt)
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) dw[mt][jt] = (floatx4){0.f, 0.f, 0.f, 0.f};
  // resident fragments: W_hh[q H + k][j0 + lr] for the contraction indices q HP + k of chunk wave + 8 i
  auto weight_frag = [&](int c, const float* Wh, int H, float4 (&v)[2]) {
    const float* Wj = Wh + g * s_rep + min(j0 + lr, H - 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kk = PC * c + 16 * h, q = (kk >= HP ? 1 : 0) + (kk >= 2 * HP ? 1 : 0), k = kk - q * HP + 4 * lg;
      const bool in = kk < HP3 && j0 + lr < H;
      const float* p = Wj + (long)q * H * H;
      v[h] = make_float4(in && k < H ? p[(long)k * H] : 0.f, in && k + 1 < H ? p[(long)(k + 1) * H] : 0.f,
                         in && k + 2 < H ? p[(long)(k + 2) * H] : 0.f, in && k + 3 < H ? p[(long)(k + 3) * H] : 0.f);
    }
  };
  bf16x8s w[NCW][NR];
#pragma unroll
  for (int i = 0; i < NCW; ++i) {
    float4 v[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
    if (wave + 8 * i < nch) weight_frag(wave + 8 * i, W_hh, H, v);
    const SplitFrag f = split_frag(v[0], v[1]);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (p < NR) w[i][p < NR ? p : 0] = f.p[p];
      else wl[((wave * NCW + i) * NL + p - NR) * 64 + lane] = __builtin_bit_cast(u32x4_t, f.p[p]);
    }
    __builtin_amdgcn_sched_barrier(0);  // (or the pieces of all chunks take registers at once)
  }
  float bsum[4] = {0.f, 0.f, 0.f, 0.f};  // this thread's da_r, da_z, da_n, dq summed over the steps
  const int j = j0 + lr, jc = min(j, H - 1);
  const bool act = RB == 2 || wave < 4;
  const int qv = wave & 3, rbo = RB == 2 ? wave >> 2 : 0;
  const int rt = rbo * 16 + 4 * lg + qv;  // this thread's row of the tile
  const int row = r0 + rt;
  const int rowc = min(row, B - 1);
  const bool ok = row < B && j < H;
  const int ohv = ((r0 + DR * lg) * H + wnc) * 4;
  const unsigned osv = rowc * 4 * H + jc, oh = rowc * H + jc, og = row * H3 + j;
  // where the lane's gate q goes in a step's block: word xb[q] + xl
  const unsigned xl = (((lr >> 2) << 4) + (row & 15)) * 4 + (lr & 3);
  unsigned xb[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) xb[q] = ((r0 / 16 + rbo) * nch * 2 + (q * HP + j0) / 16) * 256;
  float dcar = d_zero || !ok || !act ? 0.f : D[g * s_D + (long)rowc * H + jc];  // dh_{t+1} * z_{t+1}, carried in a register
  // (dgh: row-major, for later launches; nullptr: nobody reads it)
  float* dgxg = dghx + g * s_dghx;               // the gate gradients as the workgroups exchange them
  const long xblk = xblock_words(B, HP3);
  const int Bx = (B + 15) / 16 * 16;             // ... whole blocks of 16 rows
  int rbx[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) rbx[rb] = (r0 + rb * 16 < B ? r0 + rb * 16 : r0) >> 4;
  // The step's saved gates, h and the gradient from above are loaded one step ahead, and the rows of h that the step's share
  // of dW_hh multiplies, behind the products: a CU's loads return in the order of their issue, whichever wave's they are, and
  // operands (or the polling wave's flags) would wait for these to come from memory.
  // (uniform addresses and 32-bit offsets of the lane: a lane's own addresses would take registers this kernel has not got)
  float nr = 0.f, nz = 0.f, nn = 0.f, nq = 0.f, nhp = 0.f, nab = 0.f;
  auto prefetch = [&](int tn) {
    if (!act) return;
    const float* svt = sv + g * s_sv + (long)tn * B * 4 * H;
    nr = svt[osv], nz = (svt + H)[osv], nn = (svt + 2 * H)[osv], nq = (svt + 3 * H)[osv];
    nhp = (hs + g * s_hs + (long)tn * B * H)[oh];
    nab = above ? (above + g * s_above + (long)tn * B * H)[oh] : 0.f;
  };
  prefetch(T - 1);
  __syncthreads();
  int it = 0;
  for (int t = T - 1; t >= 0; --t, ++it) {
    const float r = nr, z = nz, n = nn, q = nq, hp = nhp, ab = nab;
    if (it > 0 && !group_wait(flags, NJ, base + (unsigned)it, abort_w, spin_limit, lds_flag)) return;
    floatx4 big[RB][1], small[RB][1];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) big[rb][0] = small[rb][0] = (floatx4){0.f, 0.f, 0.f, 0.f};
    if (t + 1 < T) {  // uniform over the grid
      const __amdgpu_buffer_rsrc_t rs = tile_rsrc(dgxg + bwd_block(t + 1, l2x) * xblk);
      constexpr int AHEAD = RB == 1 ? 6 : NCW == 6 ? 2 : 3, NA = NCW < AHEAD ? NCW : AHEAD;  // chunks in flight
      float4 a[NA][RB][2];
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          if (wave + 8 * i < nch) exchange_frag(rs, nch, HP3, rbx[rb], wave + 8 * i, a[i][rb]);  // (uniform)
      __builtin_amdgcn_sched_barrier(0);  // these loads are issued before anything waits for one
#pragma unroll
      for (int i = 0; i < NCW; ++i) {
        if (wave + 8 * i < nch) {
          SplitFrag wi[1];
#pragma unroll
          for (int p = 0; p < 3; ++p)
            wi[0].p[p] = p < NR ? w[i][p < NR ? p : 0] : __builtin_bit_cast(bf16x8s, wl[((wave * NCW + i) * NL + p - NR) * 64 + lane]);
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            const SplitFrag f = split_frag(a[i % NA][rb][0], a[i % NA][rb][1]);
            if (i + NA < NCW && wave + 8 * (i + NA) < nch) exchange_frag(rs, nch, HP3, rbx[rb], wave + 8 * (i + NA), a[i % NA][rb]);
            split_mfmas(f, wi, big[rb], small[rb]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        big[rb][0] += small[rb][0];
        if (__builtin_expect(any_beyond(big[rb][0]), 0)) {
          big[rb][0] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int c = wave; c < nch; c += 8) {
            float4 v[2], x[2];
            exchange_frag(rs, nch, HP3, rbx[rb], c, x);
            weight_frag(c, rarely(W_hh), rarely(H), v);
            plain_mfmas(x, v, PC * c + 16 < HP3, big[rb][0]);
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    f4ua hv[DR];
    if (dw_wave) {
      // (rows beyond the batch are zeros but for the first, which the block behind it holds)
      const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(hs + g * s_hs + (long)t * B * H), 0,
                                                                          (B * H + 4) * 4, 0x00020000);
#pragma unroll
      for (int e = 0; e < DR; ++e)
        hv[e] = __builtin_bit_cast(f4ua, __builtin_amdgcn_raw_buffer_load_b128(rh, ohv, e * H * 4, 0));
    }
    prefetch(max(t - 1, 0));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((wave * RB + rb) * 4 + v) * 64 + lane] = big[rb][0][v];
    __syncthreads();
    float da_r = 0.f, da_z = 0.f, dq = 0.f;
    if (act) {
      const float rec = sum_planes<8>(red, (rbo * 4 + qv) * 64 + lane, RB * 256);
      // (a unit beyond H reads another unit's gates; its gradient is forced to zero)
      const float dh = ok ? (dcar + ab) + rec : 0.f;
      const float dn = dh * (1.0f - z);
      const float dz = dh * (hp - n);
      const float da_n = dn * (1.0f - n * n);
      dq = da_n * r;
      da_r = da_n * q * r * (1.0f - r);
      da_z = dz * z * (1.0f - z);
      // (rows of the last block beyond the batch as zeros: whatever the memory held, a value there that is not finite
      // would send every step's sums to the fp32 instruction, above)
      if (row < Bx) {
        const bool in = row < B;
        float* oe = dgxg + bwd_block(t, l2x) * xblk;
        st_dev(oe + xb[0] + xl, in ? da_r : 0.f, l2x);
        st_dev(oe + xb[1] + xl, in ? da_z : 0.f, l2x);
        st_dev(oe + xb[2] + xl, in ? dq : 0.f, l2x);
      }
      if (ok) {
        float* ox = dgx + g * s_dg + (long)t * B * H3;
        ox[og] = da_r;
        (ox + H)[og] = da_z;
        (ox + 2 * H)[og] = da_n;
        if (dgh) {
          float* ohg = dgh + g * s_dg + (long)t * B * H3;
          ohg[og] = da_r;
          (ohg + H)[og] = da_z;
          (ohg + 2 * H)[og] = dq;
        }
      }
      dcar = dh * z;
      bsum[0] += da_r;
      bsum[1] += da_z;
      bsum[2] += da_n;
      bsum[3] += dq;
    }
    if (DW && dWp) {  // uniform
      // rows beyond the batch contribute nothing: their staged gradients are zero, their h is
      // read from a valid row
      if (act) {
        const float d3[3] = {da_r, da_z, dq};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          uint32_t p0, p1, p2;
          split2<true>(d3[i], 0.f, p0, p1, p2);  // (nothing is computed again here)
          __bf16* st = stage + (i * 16 + lr) * SPT + rt;
          st[0] = __builtin_bit_cast(bf16x2, p0)[0];
          st[48 * SPT] = __builtin_bit_cast(bf16x2, p1)[0];
          st[2 * 48 * SPT] = __builtin_bit_cast(bf16x2, p2)[0];
        }
      }
    }
    group_signal(flags + tx, base + (unsigned)it + 1u, l2x);  // (its barrier also publishes the staged tile to the workgroup)
    if (dw_wave) {
      // The sum over the step's rows by itself, then added: the running sum is rounded once a step.  (A gate gradient that is
      // not finite makes NaN of it, as it does in any case: it reaches every unit one step earlier in time, and h_0 is zero.)
#pragma unroll
      for (int jp = 0; jp < 4; jp += JN) {
        DwFrag h[JN][3];
#pragma unroll
        for (int i = 0; i < JN; ++i) split_rows(hv, jp + i, h[i]);
#pragma unroll
        for (int mt = 0; mt < 3; ++mt) {
          DwFrag am[3];
#pragma unroll
          for (int p = 0; p < 3; ++p) am[p] = *reinterpret_cast<const DwFrag*>(stage + (p * 48 + mt * 16 + lr) * SPT + DR * lg);
          floatx4 sm[JN];
#pragma unroll
          for (int i = 0; i < JN; ++i) sm[i] = (floatx4){0.f, 0.f, 0.f, 0.f};
          auto mul = [&](int pa, int ph) {
#pragma unroll
            for (int i = 0; i < JN; ++i) sm[i] = dw_mfma(am[pa], h[i][ph], sm[i]);
          };
          mul(1, 1);
          mul(2, 0);
          mul(0, 2);
          mul(1, 0);
          mul(0, 1);
          mul(0, 0);
#pragma unroll
          for (int i = 0; i < JN; ++i) dw[mt][jp + i] += sm[i];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (dbp) {  // uniform
    // bias gradients: sums over the tile's batch rows, in row order; one partial sum per
    // batch-row tile: [b_ih: r | z | n][b_hh: r | z | q], 6H floats
    __syncthreads();
    float* bs = reinterpret_cast<float*>(stage);  // [PRT][64]: row, then 4 sums x 16 units
    if (act) {
#pragma unroll
      for (int i = 0; i < 4; ++i) bs[rt * 64 + i * 16 + lr] = bsum[i];
    }
    __syncthreads();
    if (tid < 64) {
      float tot = 0.f;
      for (int r32 = 0; r32 < PRT; ++r32) tot += bs[r32 * 64 + tid];
      const int i = tid >> 4, jj = j0 + (tid & 15);
      float* out = dbp + (long)(g * RT + ty) * 6 * H;
      if (jj < H) {
        if (i == 0) out[jj] = out[H3 + jj] = tot;
        if (i == 1) out[H + jj] = out[H3 + H + jj] = tot;
        if (i == 2) out[2 * H + jj] = tot;
        if (i == 3) out[H3 + 2 * H + jj] = tot;
      }
    }
  }
  if (wn_ok) {
    // accumulator register v of tile (mt, jt): gate row mt*16 + 4*lg + v, column wn + jt
    float* out = dWp + ((long)(g * RT + ty) * H3) * H;
#pragma unroll
    for (int mt = 0; mt < 3; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = j0 + 4 * lg + v;
        float* o = out + ((long)mt * H + m) * H + wn;
        if (m >= H) continue;
        if (wn + 4 <= H) {
          *reinterpret_cast<f4ua*>(o) = (f4ua){dw[mt][0][v], dw[mt][1][v], dw[mt][2][v], dw[mt][3][v]};
        } else {
#pragma unroll
          for (int jt = 0; jt < 3; ++jt)
            if (wn + jt < H) o[jt] = dw[mt][jt][v];
        }
      }
  }
}

// ---------------------------------------------------------------------------- bf16 operands
// The same scheme with v_mfma_f32_16x16x32_bf16 on the bf16 copies of W_hh and of the exchanged
// activations (every operand is the nearest-even bf16 rounding of the fp32 value; accumulation,
// cell math and everything stored for later use stay fp32).  A workgroup owns 32 batch rows (or 16,
// gru_persist_bf16_rows) x 32 hidden units.  Its slice of the weights (forward: 96 gate rows x H; backward: 32 rows of
// W_hh^T x 3H; 192 KB at H = 1024) stays in REGISTERS for the whole launch: the contraction is
// cut into 32-wide chunks, wave w owns the chunks w, w + 8, .. with all the column blocks, i.e.
// up to 24 B-operand fragments of 16 bytes per lane.  Per step a wave fetches only its own A
// fragments (16 bytes per lane per chunk and row block); the 8 partial sums of every output
// meet in LDS.  MFMA 16x16x32 lane layout: A lane l holds A[m = l%16][k = 8*(l/16) .. +7],
// B lane l holds B[k = 8*(l/16) .. +7][n = l%16], accumulator as for 16x16x4.
// Epilogue: thread t owns batch row t/16 and the two units 2*(t%16), +1 of the tile, so that
// bf16 values are stored in pairs (16 rows: the first four waves).
//
// Layout of the exchanged operand.  A wave's A fragment is 16 rows x 32 contraction indices,
// 16 bytes per lane.  Read from a row-major matrix that is 64 bytes of each of 16 rows, half a
// cache line per row, and a CU then takes 5.3 us to fetch the 196 KB a backward step needs
// (measured: the same whether the lines come from L2 or past it, whatever the cache policy of the
// load and however few CUs read at once), against 1.9 us when every load instruction reads whole
// lines.  So the exchange buffers are kept fragment-major: per step, row block (16 batch rows) and
// chunk, the 1 KB that one load instruction reads, lane l's 16 bytes at byte 16 l (lane l holds row
// l % 16, contraction indices 8 (l / 16) .. + 7 of the chunk).  A workgroup's 32 units are exactly
// one chunk (per gate), so a workgroup writes whole fragments and nobody else writes into them.
// Rows of the last row block beyond the batch are never written: what a consumer reads there goes
// into output rows that are never stored.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int QJ = 32;       // hidden units per workgroup
constexpr int TP = 40;       // pitch (bf16) of a staged transposed row of 32 batch rows

__device__ __forceinline__ bf16x8 ld_frag(const __bf16* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4_t*>(p));
}
__device__ __forceinline__ bf16x8 ld_frag_dev(__amdgpu_buffer_rsrc_t rs, int byte_off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, byte_off, 0, 16 /* sc1 */));
}
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const __bf16 x = (__bf16)a, y = (__bf16)b;
  return (unsigned)__builtin_bit_cast(unsigned short, x) | ((unsigned)__builtin_bit_cast(unsigned short, y) << 16);
}
__device__ __forceinline__ void st_dev_u32(void* p, unsigned v, bool l2x) {
  if (l2x) __hip_atomic_store(reinterpret_cast<unsigned*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(reinterpret_cast<unsigned*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Element offset, inside a step's block of a fragment-major exchange buffer with nch chunks per
// row, of (row, chunk c, index u within the chunk)
__device__ __forceinline__ long xfrag(int row, int nch, int c, int u) {
  return ((long)(row >> 4) * nch + c) * 512 + (((u >> 3) << 4) + (row & 15)) * 8 + (u & 7);
}

// What a launch reads once (input projections, saved gates, the gradient from above) or leaves for
// later launches (saved gates, h, the copies for the GEMMs) goes past the L2 with the non-temporal
// hint: the L2 is where the exchanged operand lives between its stores and its loads.
typedef float f2nt_t __attribute__((ext_vector_type(2)));
typedef unsigned u4nt_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float2 ld2_nt(const float* p) {
  const f2nt_t v = __builtin_nontemporal_load(reinterpret_cast<const f2nt_t*>(p));
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ void st2_nt(float* p, float2 v) {
  const f2nt_t t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<f2nt_t*>(p));
}
__device__ __forceinline__ void st_u32_nt(void* p, unsigned v) { __builtin_nontemporal_store(v, reinterpret_cast<unsigned*>(p)); }
__device__ __forceinline__ void st16_nt(void* p, uint4 v) {
  const u4nt_t t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<u4nt_t*>(p));
}

// Forward.  Wb: bf16 W_hh [3H][H]; hx: bf16 h_0 .. h_T fragment-major (blocks of 16 ceil(B/16) x H,
// h_0 given), the exchanged operand; hb: the same row-major (blocks of B x H; written, not read);
// hs: the same in fp32; hT (nullable): bf16 transposed copy [H][ld_hT], column (t+1)*B + row.
// NCF: chunks per wave (H <= 256 * NCF).  RB: row blocks of 16 per workgroup.  EX: the gates of the fp32 launches (gru_bf16_exact_gates).
template <int NCF, int RB, bool EX>
__global__ void __launch_bounds__(PNT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_fwd_persist_bf16_kernel(const __bf16* __restrict__ Wb, long s_wb, const float* __restrict__ b_ih,
                            const float* __restrict__ b_hh, long s_rep, int Hc, const float* __restrict__ gx, long s_gx, float* __restrict__ hs, long s_hs,
                            __bf16* __restrict__ hb, long s_hb, __bf16* hx, long s_hx, float* __restrict__ sv, long s_sv, __bf16* __restrict__ hT, long ld_hT,
                            long s_hT, int Bc, int B, int H, int T, int sg0, int n_sg, unsigned* sync, unsigned base,
                            unsigned spin_limit, unsigned* tickets, unsigned ticket_base, unsigned per_xcd) {
  extern __shared__ __attribute__((aligned(16))) float persist_lds[];
  constexpr int PRB = 16 * RB;                                  // rows of the tile
  float* red = persist_lds;                                     // [8][RB][6][4][64]
  __bf16* tt = reinterpret_cast<__bf16*>(red + 8 * RB * 6 * 256);  // [32 units][TP]
  int* lds_flag = reinterpret_cast<int*>(tt + QJ * TP);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int NJ = H / QJ, RT = (B + PRB - 1) / PRB;
  unsigned* abort_w = sync;
  int tx, sg;
  bool l2x;
  if (!persist_place(tickets, ticket_base, per_xcd, abort_w, spin_limit, lds_flag, NJ, n_sg, tx, sg, l2x)) return;
  sg += sg0;
  const int g = sg / RT, ty = sg - g * RT;
  const int j0 = tx * QJ, r0 = ty * PRB;
  unsigned* flags = sync + 1 + sg * PF;
  __builtin_amdgcn_s_setprio(3);
  const int nch = H / PC;
  // resident fragments: chunk wave + 8i, column block cb = 2q + half: rows q*H + j0 + 16*half + lr
  bf16x8 wf[NCF][6];
#pragma unroll
  for (int i = 0; i < NCF; ++i) {
    const int c = wave + 8 * i;
#pragma unroll
    for (int cb = 0; cb < 6; ++cb) {
      const long wrow = (long)(cb >> 1) * H + j0 + 16 * (cb & 1) + lr;
      const bf16x8 v = ld_frag(Wb + g * s_wb + wrow * H + PC * (c < nch ? c : 0) + 8 * lg);
      const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      wf[i][cb] = c < nch ? v : zero;  // a chunk slot beyond the contraction multiplies by zero
    }
  }
  // epilogue element: row rl of the tile, units u0, u0 + 1
  const bool epi = RB == 2 || wave < 4;  // (uniform)
  const int rl = (tid >> 4) & (PRB - 1), u0 = 2 * (tid & 15);
  const int row = r0 + rl, rowc = min(row, B - 1);
  const int j = j0 + u0;
  const int ro = ((rl >> 4) * 6) * 256 + (rl & 3) * 64 + ((rl >> 2) & 3) * 16 + (u0 & 15);  // + cb * 256 + w * RB * 1536
  const int half = u0 >> 4;
  const bool ok0 = row < Bc && j < Hc, ok1 = row < Bc && j + 1 < Hc;  // of the model, not of its padding
  // the biases: arrays of the model's own width (units beyond it have none)
  float2 bias[3], biasx[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const float* bi = b_ih + g * s_rep + q * Hc;
    const float* bh = b_hh + g * s_rep + q * Hc;
    biasx[q] = make_float2(j < Hc ? bi[j] : 0.f, j + 1 < Hc ? bi[j + 1] : 0.f);
    bias[q] = make_float2(j < Hc ? bh[j] : 0.f, j + 1 < Hc ? bh[j + 1] : 0.f);
  }
  float* hsg = hs + g * s_hs;
  __bf16* hbg = hb + g * s_hb;
  __bf16* hxg = hx + g * s_hx;
  const long xblk = (long)((B + 15) / 16) * 16 * H;  // elements of a step's block of hx
  float2 hpv = *reinterpret_cast<const float2*>(hsg + (long)rowc * H + j);
  // A fragments: row blocks r0/16 + rb (one that lies beyond the batch is read from the tile's first)
  int aoff[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) aoff[rb] = (((r0 + rb * 16 < B ? r0 + rb * 16 : r0) >> 4) * nch) * 1024 + lane * 16;
  // The step's input projection is loaded one step ahead, behind the products of the step before: a CU's loads return in
  // the order of their issue, whichever wave's they are, and these come from memory, not from the L2.  Requested in front of
  // the wait, they would sit between the polling wave and its view of the flags; in front of the products, between the
  // second four waves and their operands (144 us a launch against 128).
  float2 gxn[3];
  auto prefetch = [&](int tn) {
    const float* gxr = gx + g * s_gx + ((long)tn * B + rowc) * 3 * H + j;
#pragma unroll
    for (int q = 0; q < 3; ++q) gxn[q] = ld2_nt(gxr + q * H);
  };
  if (epi) prefetch(0);
  else gxn[0] = gxn[1] = gxn[2] = make_float2(0.f, 0.f);
  for (int t = 0; t < T; ++t) {
    float2 gxv[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) gxv[q] = make_float2(gxn[q].x + biasx[q].x, gxn[q].y + biasx[q].y);
    if (t > 0 && !group_wait(flags, NJ, base + (unsigned)t, abort_w, spin_limit, lds_flag)) return;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(hxg + fwd_block(t, l2x) * xblk, 0, 0x7fffffff, 0x00020000);
    bf16x8 a[NCF][RB];
#pragma unroll
    for (int i = 0; i < NCF; ++i) {
      const int c = wave + 8 * i;
      const int co = (c < nch ? c : 0) * 1024;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) a[i][rb] = ld_frag_dev(rs, aoff[rb] + co);
    }
    floatx4 acc[RB][6];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < 6; ++cb) acc[rb][cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_sched_barrier(0);  // every load is issued before anything waits for one
#pragma unroll
    for (int i = 0; i < NCF; ++i)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < 6; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][rb], wf[i][cb], acc[rb][cb], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (epi) prefetch(min(t + 1, T - 1));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < 6; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(((wave * RB + rb) * 6 + cb) * 4 + v) * 64 + lane] = acc[rb][cb][v];
    __syncthreads();
    if (epi) {
      float2 gh[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float* rp = red + ro + (2 * q + half) * 256;
        float2 p[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) p[w] = *reinterpret_cast<const float2*>(rp + w * RB * 1536);
        gh[q].x = (((p[0].x + p[1].x) + (p[2].x + p[3].x)) + ((p[4].x + p[5].x) + (p[6].x + p[7].x))) + bias[q].x;
        gh[q].y = (((p[0].y + p[1].y) + (p[2].y + p[3].y)) + ((p[4].y + p[5].y) + (p[6].y + p[7].y))) + bias[q].y;
      }
      float r0v = sigm_of<EX>(gxv[0].x + gh[0].x), r1v = sigm_of<EX>(gxv[0].y + gh[0].y);
      float z0v = sigm_of<EX>(gxv[1].x + gh[1].x), z1v = sigm_of<EX>(gxv[1].y + gh[1].y);
      float n0v = tanh_of<EX>(gxv[2].x + r0v * gh[2].x), n1v = tanh_of<EX>(gxv[2].y + r1v * gh[2].y);
      // rows and units of the padding leave zeros, selected and not multiplied: an infinite value of the model times
      // their zero operands is NaN, which their h and gate gradients would hand to everyone
      if (!ok0) r0v = z0v = n0v = gh[2].x = 0.f;
      if (!ok1) r1v = z1v = n1v = gh[2].y = 0.f;
      const float2 hn = make_float2((1.0f - z0v) * n0v + z0v * hpv.x, (1.0f - z1v) * n1v + z1v * hpv.y);
      if (row < B) {
        const long e = ((long)(t + 1) * B + row) * H + j;
        const unsigned hp2 = pack_bf16(hn.x, hn.y);
        st_dev_u32(hxg + fwd_block(t + 1, l2x) * xblk + xfrag(row, nch, tx, u0), hp2, l2x);
        st2_nt(hsg + e, hn);
        st_u32_nt(hbg + e, hp2);
        float* svr = sv + g * s_sv + ((long)t * B + row) * 4 * H + j;
        st2_nt(svr, make_float2(r0v, r1v));
        st2_nt(svr + H, make_float2(z0v, z1v));
        st2_nt(svr + 2 * H, make_float2(n0v, n1v));
        st2_nt(svr + 3 * H, gh[2]);
      }
      if (hT) {
        tt[u0 * TP + rl] = (__bf16)hn.x;
        tt[(u0 + 1) * TP + rl] = (__bf16)hn.y;
      }
      hpv = hn;
    }
    group_signal(flags + tx, base + (unsigned)t + 1u, l2x);  // (its barrier also separates the reads of red from the next step's writes)
    if (hT && wave >= 8 - RB) {
      // 64- (or 32-) byte row segments of the transposed copy, 16 bytes per thread (the last waves: the
      // first one polls the flags next, and would see them only behind its own stores)
      const unsigned u = (unsigned)(tid - (PNT - 64 * RB)) / (2 * RB), part = (unsigned)tid % (2 * RB);
      if (r0 + 8 * (int)part < B)  // B is a multiple of 8: a piece of 8 rows is all in or all out
        st16_nt(hT + g * s_hT + (long)(j0 + u) * ld_hT + (long)(t + 1) * B + r0 + 8 * part,
                *reinterpret_cast<const uint4*>(tt + u * TP + 8 * part));
    }
  }
}

// chunks of a wave's backward weights that lie in LDS
constexpr int persist_bwd_bf16_nl(int ncb, int rb) { return rb == 2 && ncb > 8 ? ncb - ncb / 2 : 0; }

// Backward.  WT: bf16 W_hh^T [H][3H]; dghx: bf16 gate gradients of all steps, fragment-major
// (blocks of 16 ceil(B/16) x 3H), the exchanged operand; dgxb: bf16 dgx row-major; dgxT / dghT: bf16 transposed copies
// [3H][ld_T], column t*B + row; dbp: partial bias-gradient sums [(g*RT + ty)][6H] (b_ih | b_hh).
// D: dh_T * z_T on entry (the head's gradient; d_zero: zero, D is not read), dh_0 * z_0 on exit.  NCB: chunks per wave
// (3H <= 256 * NCB).  The fragments of the first half of a wave's chunks stay in registers,
// those of the second half in LDS (each wave reads back only its own): with all of them in
// registers the two waves of a SIMD would fill its register file, and no wave of any other
// kernel (a merge on the second stream) could ever share the CU.  (Tiles of 16 rows have half the operands: all of the
// weights in registers leave room for others.)
template <int NCB, int RB>
__global__ void __launch_bounds__(PNT) __attribute__((amdgpu_waves_per_eu(1, 2)))
gru_bwd_persist_bf16_kernel(const __bf16* __restrict__ WT, long s_wt, __bf16* dghx, long s_dgh, long s_dgb, float* __restrict__ D,
                            long s_D, int d_zero, const float* __restrict__ above, long s_above, const float* __restrict__ sv,
                            long s_sv, const float* __restrict__ hs, long s_hs, __bf16* __restrict__ dgxb,
                            __bf16* __restrict__ dgxT, __bf16* __restrict__ dghT, long ld_T, long s_T,
                            float* __restrict__ dbp, int Hc, int B, int H, int T, int sg0, int n_sg, unsigned* sync, unsigned base,
                            unsigned spin_limit, unsigned* tickets, unsigned ticket_base, unsigned per_xcd) {
  extern __shared__ __attribute__((aligned(16))) float persist_lds[];
  constexpr int PRB = 16 * RB;                                  // rows of the tile
  constexpr int NCL = persist_bwd_bf16_nl(NCB, RB), NCR = NCB - NCL;  // chunks in LDS / in registers
  float* red = persist_lds;                                     // [8][RB][2][4][64]
  __bf16* tt = reinterpret_cast<__bf16*>(red + 8 * RB * 2 * 256);    // [da_r | da_z | da_n | dq][32 units][TP]
  u32x4_t* wl = reinterpret_cast<u32x4_t*>(tt + 4 * QJ * TP);   // [8 waves][NCL][2][64 lanes] fragments
  int* lds_flag = reinterpret_cast<int*>(wl + 8 * NCL * 2 * 64);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int NJ = H / QJ, RT = (B + PRB - 1) / PRB;
  unsigned* abort_w = sync;
  int tx, sg;
  bool l2x;
  if (!persist_place(tickets, ticket_base, per_xcd, abort_w, spin_limit, lds_flag, NJ, n_sg, tx, sg, l2x)) return;
  sg += sg0;
  const int g = sg / RT, ty = sg - g * RT;
  const int j0 = tx * QJ, r0 = ty * PRB;
  unsigned* flags = sync + 1 + sg * PF;
  __builtin_amdgcn_s_setprio(3);
  const int H3 = 3 * H;
  const int nch = H3 / PC;
  // resident fragments: chunk wave + 8i, column block = half: rows j0 + 16*half + lr of W_hh^T
  bf16x8 wf[NCR][2];
#pragma unroll
  for (int i = 0; i < NCB; ++i) {
    const int c = wave + 8 * i;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      const bf16x8 v = ld_frag(WT + g * s_wt + (long)(j0 + 16 * cb + lr) * H3 + PC * (c < nch ? c : 0) + 8 * lg);
      const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      const bf16x8 f = c < nch ? v : zero;
      if (i < NCR)
        wf[i][cb] = f;
      else
        wl[((wave * NCL + (i - NCR)) * 2 + cb) * 64 + lane] = __builtin_bit_cast(u32x4_t, f);
    }
  }
  const bool epi = RB == 2 || wave < 4;  // (uniform)
  const int rl = (tid >> 4) & (PRB - 1), u0 = 2 * (tid & 15);
  const int row = r0 + rl, rowc = min(row, B - 1);
  const int j = j0 + u0;
  const int ro = ((rl >> 4) * 2 + (u0 >> 4)) * 256 + (rl & 3) * 64 + ((rl >> 2) & 3) * 16 + (u0 & 15);  // + w * RB * 512
  float* Dg = D + g * s_D;
  float2 dcar = make_float2(0.f, 0.f);
  if (!d_zero) dcar = *reinterpret_cast<const float2*>(Dg + (long)rowc * H + j);
  __bf16* dghg = dghx + g * s_dgh;
  const long xblk = (long)((B + 15) / 16) * 16 * H3;  // elements of a step's block of dghx
  float2 bsum[4] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};  // da_r, da_z, da_n, dq over the steps
  int aoff[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) aoff[rb] = (((r0 + rb * 16 < B ? r0 + rb * 16 : r0) >> 4) * nch) * 1024 + lane * 16;
  // The step's saved gates, h and the gradient from above are loaded one step ahead, behind the operand loads of the step
  // before (see the forward kernel: in front of the wait they would delay the polling wave's view of the flags by a trip to
  // memory; further back there is too little of the step left to cover them, 179 us a launch against 184 to 195).
  float2 nr = make_float2(0.f, 0.f), nz = nr, nn = nr, nq = nr, nhp = nr, nab = nr;
  auto prefetch = [&](int tn) {
    const long e = ((long)tn * B + rowc) * H + j;
    const float* svr = sv + g * s_sv + ((long)tn * B + rowc) * 4 * H + j;
    nr = ld2_nt(svr), nz = ld2_nt(svr + H);
    nn = ld2_nt(svr + 2 * H), nq = ld2_nt(svr + 3 * H);
    nhp = ld2_nt(hs + g * s_hs + e);
    nab = above ? ld2_nt(above + g * s_above + e) : make_float2(0.f, 0.f);
  };
  if (epi) prefetch(T - 1);
  int it = 0;
  for (int t = T - 1; t >= 0; --t, ++it) {
    const float2 r = nr, z = nz, n = nn, q = nq, hp = nhp, ab = nab;
    if (it > 0 && !group_wait(flags, NJ, base + (unsigned)it, abort_w, spin_limit, lds_flag)) return;
    floatx4 acc[RB][2];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
    if (t + 1 < T) {  // uniform over the grid
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(dghg + bwd_block(t + 1, l2x) * xblk, 0, 0x7fffffff,
                                                                          0x00020000);
      bf16x8 a[NCB][RB];
#pragma unroll
      for (int i = 0; i < NCB; ++i) {
        const int c = wave + 8 * i;
        const int co = (c < nch ? c : 0) * 1024;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) a[i][rb] = ld_frag_dev(rs, aoff[rb] + co);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (epi) prefetch(max(t - 1, 0));
      __builtin_amdgcn_sched_barrier(0);  // every load is issued before anything waits for one
#pragma unroll
      for (int i = 0; i < NCB; ++i) {
        bf16x8 w2[2];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          w2[cb] = i < NCR ? wf[i < NCR ? i : 0][cb]
                           : __builtin_bit_cast(bf16x8, wl[((wave * NCL + (i - NCR)) * 2 + cb) * 64 + lane]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < 2; ++cb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][rb], w2[cb], acc[rb][cb], 0, 0, 0);
      }
    } else {
      if (epi) prefetch(max(t - 1, 0));
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(((wave * RB + rb) * 2 + cb) * 4 + v) * 64 + lane] = acc[rb][cb][v];
    __syncthreads();
    if (epi) {
      float2 p[8];
#pragma unroll
      for (int w = 0; w < 8; ++w) p[w] = *reinterpret_cast<const float2*>(red + ro + w * RB * 512);
      const float recx = ((p[0].x + p[1].x) + (p[2].x + p[3].x)) + ((p[4].x + p[5].x) + (p[6].x + p[7].x));
      const float recy = ((p[0].y + p[1].y) + (p[2].y + p[3].y)) + ((p[4].y + p[5].y) + (p[6].y + p[7].y));
      const float2 dh = make_float2((dcar.x + ab.x) + recx, (dcar.y + ab.y) + recy);
      const float2 dn = make_float2(dh.x * (1.0f - z.x), dh.y * (1.0f - z.y));
      const float2 dz = make_float2(dh.x * (hp.x - n.x), dh.y * (hp.y - n.y));
      const float2 da_n = make_float2(dn.x * (1.0f - n.x * n.x), dn.y * (1.0f - n.y * n.y));
      const float2 dq = make_float2(da_n.x * r.x, da_n.y * r.y);
      const float2 da_r = make_float2(da_n.x * q.x * r.x * (1.0f - r.x), da_n.y * q.y * r.y * (1.0f - r.y));
      const float2 da_z = make_float2(dz.x * z.x * (1.0f - z.x), dz.y * z.y * (1.0f - z.y));
      if (row < B) {
        const long o = ((long)t * B + row) * H3 + j;
        const unsigned pr = pack_bf16(da_r.x, da_r.y), pz = pack_bf16(da_z.x, da_z.y);
        const long ox3 = bwd_block(t, l2x) * xblk + xfrag(row, nch, tx, u0);  // gate q: chunk q H/32 + tx
        st_dev_u32(dghg + ox3, pr, l2x);
        st_dev_u32(dghg + ox3 + (long)(H / PC) * 512, pz, l2x);
        st_dev_u32(dghg + ox3 + (long)(2 * H / PC) * 512, pack_bf16(dq.x, dq.y), l2x);
        __bf16* ox = dgxb + g * s_dgb + o;
        st_u32_nt(ox, pr);
        st_u32_nt(ox + H, pz);
        st_u32_nt(ox + 2 * H, pack_bf16(da_n.x, da_n.y));
        bsum[0].x += da_r.x; bsum[0].y += da_r.y;
        bsum[1].x += da_z.x; bsum[1].y += da_z.y;
        bsum[2].x += da_n.x; bsum[2].y += da_n.y;
        bsum[3].x += dq.x;   bsum[3].y += dq.y;
      }
      // the four distinct gate-gradient blocks, staged for the transposed copies
      tt[(0 * QJ + u0) * TP + rl] = (__bf16)da_r.x;
      tt[(0 * QJ + u0 + 1) * TP + rl] = (__bf16)da_r.y;
      tt[(1 * QJ + u0) * TP + rl] = (__bf16)da_z.x;
      tt[(1 * QJ + u0 + 1) * TP + rl] = (__bf16)da_z.y;
      tt[(2 * QJ + u0) * TP + rl] = (__bf16)da_n.x;
      tt[(2 * QJ + u0 + 1) * TP + rl] = (__bf16)da_n.y;
      tt[(3 * QJ + u0) * TP + rl] = (__bf16)dq.x;
      tt[(3 * QJ + u0 + 1) * TP + rl] = (__bf16)dq.y;
      dcar = make_float2(dh.x * z.x, dh.y * z.y);
    }
    group_signal(flags + tx, base + (unsigned)it + 1u, l2x);
    // transposed copies [gate unit][t*B + row] as 64- (or 32-) byte row segments, 16 bytes per piece:
    // dgx^T = (da_r, da_z, da_n), dgh^T = (da_r, da_z, dq).  256 RB pieces, by the waves 1 .. 7: wave
    // 0 polls the flags next, and would see them only behind its own stores
    for (unsigned idx = tid - 64; idx < 256u * RB; idx += PNT - 64) {  // (wave 0's wrap beyond the end)
      const unsigned blk = idx / (64 * RB), u = idx / (2 * RB) & 31, part = idx % (2 * RB);
      if (r0 + 8 * (int)part < B) {  // B is a multiple of 8
        const uint4 v = *reinterpret_cast<const uint4*>(tt + (blk * QJ + u) * TP + 8 * part);
        const unsigned gate = blk == 3 ? 2 : blk;
        const long o = g * s_T + (long)(gate * H + j0 + u) * ld_T + (long)t * B + r0 + 8 * part;
        if (blk != 3) st16_nt(dgxT + o, v);
        if (blk != 2) st16_nt(dghT + o, v);
      }
    }
  }
  if (epi && row < B) *reinterpret_cast<float2*>(Dg + (long)row * H + j) = dcar;
  // bias gradients: sums over the tile's batch rows, in row order
  __syncthreads();
  float* bs = red;  // [PRB rows][4 sums][32 units]
  if (epi) {
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<float2*>(bs + (rl * 4 + i) * QJ + u0) = bsum[i];
  }
  __syncthreads();
  if (tid < 128) {
    float tot = 0.f;
    for (int r = 0; r < PRB; ++r) tot += bs[r * 128 + tid];
    const int i = tid >> 5, jj = j0 + (tid & 31);
    float* out = dbp + (long)(g * RT + ty) * 6 * Hc;  // (the model's own width)
    if (jj < Hc) {
      if (i == 0) out[jj] = out[3 * Hc + jj] = tot;
      if (i == 1) out[Hc + jj] = out[4 * Hc + jj] = tot;
      if (i == 2) out[2 * Hc + jj] = tot;
      if (i == 3) out[5 * Hc + jj] = tot;
    }
  }
}

// How a launch places its workgroups (persist_place).  By ticket, with the exchange through the
// XCDs' L2s, when the caller allows it and the launch's groups of NJ workgroups fit the XCDs whole: the
// launch then has one workgroup per CU of the device, whether it has work for all of them or not
// (a workgroup that asks for more than half of a CU's LDS has a CU to itself, so each of the 8 XCDs
// receives cus / 8 of them).
struct Placement { unsigned* tickets; unsigned ticket_base, per_xcd; int grid; size_t lds; };
int device_cus() {
  static int cus = -1;
  if (cus < 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return 0;
    cus = n;
  }
  return cus;
}
constexpr size_t kLdsLimit = 160 * 1024;
constexpr size_t kLdsAlone = 80 * 1024 + 256;  // more than half of a CU's LDS
constexpr int kPlanCus = 256;                  // the chip's compute units: what sizes and forms are planned for

// all_groups: of the step (the counters lie behind the flag words of all of them); ticket_launches: how
// many launches of this step have drawn tickets so far (counted here)
Placement placement(unsigned* sync, int all_groups, int sync_groups, int NJ, size_t lds, bool device_scope,
                    unsigned* ticket_launches) {
  const int cus = device_cus(), per = cus / 8;
  if (device_scope || !ticket_launches || cus <= 0 || cus % 8 != 0 || NJ > per || sync_groups > 8 * (per / NJ))
    return Placement{nullptr, 0u, 0u, NJ * sync_groups, lds};
  return Placement{sync + 1 + (size_t)all_groups * PF, (*ticket_launches)++ * (unsigned)per, (unsigned)per, cus,
                   lds > kLdsAlone ? lds : kLdsAlone};
}

// The synchronisation groups of a launch: as many whole groups of NJ workgroups as the device has room
// for at one workgroup per CU.
int groups_per_launch(int NJ, int SG) {
  const int most = device_cus() / NJ;
  if (most >= SG || most < 1) return SG;
  return most >= 8 ? most / 8 * 8 : most;  // (whole rounds over the XCDs)
}

// Widths the fp32 launches take: a group's members' flags fit its words, the weight parts a wave's registers.
constexpr int kPersistMaxH = 704;
// A forward launch: the waves that share a contraction (and the batch rows per wave that follow from it, see the kernel),
// their chunks of it and of the layer input (width 0: no projection in the launch), its LDS.
struct FwdForm { int kw, ncw, xnb; size_t lds; };
constexpr FwdForm persist_fwd_form(int H, int rows, int width) {
  const int kw = rows == 32 && H <= 512 ? 4 : 8, nchw = (width + PC - 1) / PC;
  const int least = rows == 16 ? 1 : kw == 4 ? 2 : 3, need = (((H + PJ - 1) / PJ * PJ + PC - 1) / PC + kw - 1) / kw;
  const int ncw = need > least ? need : least, xnb = (nchw + kw - 1) / kw;
  const size_t lds = (size_t)kw * (rows / 16) * (width ? 4 : 3) * 1024 + (size_t)nchw * 9 * 1024 +
                     (persist_fwd_lw(ncw, xnb, rows / 16 * kw / 8) ? (size_t)kw * ncw * 3 * 1024 : 0) + 16;
  return {kw, ncw, xnb, lds};
}
// backward: chunks per wave
constexpr int persist_bwd_ncw(int H) {
  const int n = (3 * ((H + PJ - 1) / PJ * PJ) + 8 * PC - 1) / (8 * PC);
  return n <= 4 ? (n < 2 ? 2 : n) : n <= 6 ? 6 : 9;
}
constexpr size_t persist_bwd_lds(int H, int rows) {
  const int n = persist_bwd_ncw(H);
  return (size_t)8 * (rows / 16) * 1024 + (size_t)3 * 48 * SPT * 2 + (size_t)8 * n * persist_bwd_nl(n, rows) * 1024 + 16;
}
// every launch but those of a projection, which gru_persist_xproj_supported asks for by its LDS
constexpr bool persist_fits(int rows) {
  for (int H = 16; H <= kPersistMaxH; ++H)
    if (persist_fwd_form(H, rows, 0).lds > kLdsLimit || persist_bwd_lds(H, rows) > kLdsLimit) return false;
  return true;
}
static_assert(persist_fits(16) && persist_fits(32), "a launch of any width it takes fits a CU's LDS");

}  // namespace

// Batch rows per workgroup for a layer of K workers, or 0 for a width these launches do not take.  A launch has at most one
// workgroup per CU and all of them resident: 16 rows where all
// workers' workgroups then still fit the chip; more workgroups than CUs go out as several launches of
// whole synchronisation groups, of 32 rows each where a batch has more than 16.
int gru_persist_rows(int B, int H, int K) {
  if (H < 16 || B < 1 || K < 1 || H > kPersistMaxH) return 0;
  const long NJ = (H + PJ - 1) / PJ;
  return B <= 16 || NJ * ((B + 15) / 16) * K <= kPlanCus ? 16 : 32;
}

// Whether `groups` workers' layer is better off resident for its T time steps than with one launch per step.  A
// single launch always is.  Of several, each (forward and backward together) loads and splits its weights,
// 20 us and 1 us for every 20 units, and pays 4.5 us and 1 us for every 75 units per step, 21 us (16-row tiles: 12)
// where a group does not fit an XCD; a step of the launches per step costs 26 us for all workers together and
// 0.22 us per million of groups * B * H * H, with at least 16 rows for B.
// us per local step of 20 time steps, resident / per step, (H, B, workers):
//   2 launches  (256, 64, 16) 392 / 705, (160, 128, 8) 336 / 670, (144, 40, 16) 329 / 465, (200, 40, 16) 360 / 569,
//               (450, 20, 16) 537 / 857, (512, 128, 4) 554 / 1030
//   3, 4        (144, 128, 16) 492 / 919, (384, 96, 8) 670 / 1113, (300, 100, 8) 817 / 910, (512, 64, 16) 1165 / 1706
//   8           (300, 100, 16) 1653 / 1352, (320, 128, 16) 1684 / 1741, (500, 128, 16) 2312 / 2529
//   groups beyond an XCD  3 launches (640, 32, 16) 1338 / 1673, (700, 4, 12) 762 / 1246
// of 3 time steps: (144, 40, 16) 104 / 87, (256, 64, 16) 127 / 119, (384, 96, 8) 198 / 185, (300, 100, 8) 233 / 161.
// Widths off the 16-unit blocks, where the launches per step lose their wide accesses, are on par after 3 or 4 steps
// with up to 3 launches: (300, 70, 5) 150 / 156, (530, 33, 4) 158 / 145, (500, 11, 11) 159 / 194, (690, 4, 12) 270 / 276;
// so is work of about 40 million groups * B * H * H per launch, (512, 128, 4) 169 / 165: both are resident at any T.
bool gru_persist_pays(int B, int H, int T, int groups, int rows) {
  const int NJ = (H + PJ - 1) / PJ, SG = groups * ((B + rows - 1) / rows), per = groups_per_launch(NJ, SG);
  const long launches = (SG + per - 1) / per;
  const double work = (double)groups * B * H * H;
  if (launches <= (H % 16 ? 3 : 1)) return true;
  if (H % 16 == 0 && NJ * 8 <= kPlanCus && work >= 40e6 * (double)launches - 5e6) return true;
  const double step = NJ * 8 <= kPlanCus ? 4.5 + H / 75.0 : rows == 16 ? 12.0 : 21.0;
  const double steps = 26.0 + 0.22e-6 * (B < 16 ? work / B * 16 : work);
  return (double)launches * (20.0 + H / 20.0 + T * step) <= T * steps;
}

// The backward kernel can accumulate dW_hh itself when 8 waves x 64 columns cover H.
bool gru_persist_dw_supported(int H) { return H <= 512; }

// Words of device memory the kernels synchronise through: the abort word + 64 flag words per group.
size_t gru_persist_sync_words(int B, int groups, int rows) { return (size_t)groups * ((B + rows - 1) / rows) * PF + 1 + 8; }

// How much every flag advances per time step of a launch.
unsigned gru_persist_count_per_step(int) { return 1u; }

// The forward kernel can do the input projection itself when the layer input is narrow (at most 2 chunks of 32 per
// wave) and its 48 rows of W_ih fit the LDS beside the rest: with 32 rows
// and H > 512 that is 64 KB of partial sums and 72 KB of weight parts, which leaves room for an input of 64.  Beyond H = 512 a group
// spans XCDs: a step waits 2 us for the hand-off, and the projection, done before the wait, costs nothing.  Up to there a step
// waits too little to hide more than 21 chunks of both contractions.  us per local step of 20 steps, projected in the launch /
// by a product of its own:
//   beyond H = 512   16 rows, batch 16, 4 workers   H = 576, input 112  263 / 274,  256  279 / 294     H = 640, 256  291 / 311
//                    12 workers, H = 610, 128  577 / 606 (several launches)          5 steps, H = 704, 16  117 / 121
//                    32 rows, 4 workers   H = 640, 64, batch 32  397 / 409           6 workers, H = 600, 64, batch 128  1764 / 1766
//   up to it, within 21 chunks   16 rows  H = 320, 112  176 / 178,  416, 112  200 / 201     32 rows, batch 40  H = 320, 256  218 / 236,  480, 112  289 / 296
//             beyond them        16 rows  H = 448, 256  214 / 213,  512, 176  221 / 219     32 rows, batch 40  H = 448, 176  294 / 289,  500, 256  319 / 319,
//             6 workers, H = 512, 256, batch 40  585 / 569; (batches of whole 32-row tiles gain: 4 workers, 512, 256, batch 64  326 / 355)
bool gru_persist_xproj_supported(int H, int width, int rows) {
  return width >= 16 && width % 16 == 0 && width <= 256 && (H > 512 || (H + PC - 1) / PC + (width + PC - 1) / PC <= 21) &&
         persist_fwd_form(H, rows, width).lds <= kLdsLimit;
}

size_t gru_persist_exchange_words(int B, int H, int gates) { return (size_t)xblock_words(B, gates * ((H + PJ - 1) / PJ * PJ)); }

hipError_t launch_gru_fwd_persist(const float* W_hh, const float* b_hh, long s_rep, const float* gx, long s_gx,
                                  float* hs, long s_hs, float* hx, long s_hx, float* sv, long s_sv, int B, int H, int T,
                                  int groups, int rows,
                                  unsigned* sync, unsigned base, unsigned spin_limit, const float* xin, long s_x,
                                  int width, const float* W_ih, const float* b_ih, bool device_scope, unsigned* ticket_launches, hipStream_t s) {
  const int NJ = (H + PJ - 1) / PJ, SG = groups * ((B + rows - 1) / rows), per = groups_per_launch(NJ, SG);
  if ((rows != 16 && rows != 32) || T < 1 || H > kPersistMaxH || NJ > device_cus()) return hipErrorInvalidValue;
  if (!hx || ((uintptr_t)hx & 15) != 0 || (s_hx & 3) != 0) return hipErrorInvalidValue;
  if (xin && (!gru_persist_xproj_supported(H, width, rows) || !W_ih || !b_ih || ((uintptr_t)xin & 15) != 0 || (s_x & 3) != 0))
    return hipErrorInvalidValue;
  if (!xin && !gx) return hipErrorInvalidValue;
  KernelTimer kt(KID_GRU_FWD_PERSIST, 2.0 * B * 3 * H * ((double)H + (xin ? width : 0)) * T * groups, s);
#define HPSGD_FWD_PERSIST(C, N, R, KW)                                                                            \
  do {                                                                                                            \
    static std::atomic<size_t> allowed{0};                                                                        \
    const hipError_t e = allow_lds((const void*)gru_fwd_persist_kernel<C, N, R, KW>, pl.lds, allowed);            \
    if (e != hipSuccess) return e;                                                                                \
    hipLaunchKernelGGL((gru_fwd_persist_kernel<C, N, R, KW>), dim3(pl.grid), dim3(PNT), pl.lds, s, W_hh, b_hh, s_rep, gx, s_gx, hs, \
                       s_hs, hx, s_hx, sv, s_sv, B, H, T, sg0, n_sg, sync, base, spin_limit, pl.tickets, pl.ticket_base, \
                       pl.per_xcd, xin, s_x, width, W_ih, b_ih);                                                  \
  } while (0)
#define HPSGD_FWD_PERSIST_X(C, R, KW, XMAX)                \
  do {                                                     \
    if (xnb == 0) HPSGD_FWD_PERSIST(C, 0, R, KW);          \
    else if (xnb == 1) HPSGD_FWD_PERSIST(C, 1, R, KW);     \
    else HPSGD_FWD_PERSIST(C, XMAX, R, KW);                \
  } while (0)
  const FwdForm f = persist_fwd_form(H, rows, xin ? width : 0);
  const int kw = f.kw, ncw = f.ncw, xnb = f.xnb;
  for (int sg0 = 0; sg0 < SG; sg0 += per) {
    const int n_sg = SG - sg0 < per ? SG - sg0 : per;
    const Placement pl = placement(sync, SG, n_sg, NJ, f.lds, device_scope, ticket_launches);
    if (rows == 16) {
      if (ncw == 1) HPSGD_FWD_PERSIST_X(1, 16, 8, 1);
      else if (ncw == 2) HPSGD_FWD_PERSIST_X(2, 16, 8, 1);
      else HPSGD_FWD_PERSIST_X(3, 16, 8, 1);
    } else if (kw == 4) {
      if (ncw == 2) HPSGD_FWD_PERSIST_X(2, 32, 4, 2);
      else if (ncw == 3) HPSGD_FWD_PERSIST_X(3, 32, 4, 2);
      else HPSGD_FWD_PERSIST_X(4, 32, 4, 2);
    } else {
      HPSGD_FWD_PERSIST_X(3, 32, 8, 1);
    }
  }
#undef HPSGD_FWD_PERSIST_X
#undef HPSGD_FWD_PERSIST
  return hipGetLastError();
}

hipError_t launch_gru_bwd_persist(const float* W_hh, long s_rep, float* dgh, float* dghx, long s_dghx, float* dgx,
                                  long s_dg, const float* D,
                                  long s_D, bool d_zero, const float* above, long s_above, const float* sv, long s_sv,
                                  const float* hs, long s_hs, int B, int H, int T,
                                  int groups, int rows, unsigned* sync, unsigned base, unsigned spin_limit, float* dWp,
                                  float* dbp, bool device_scope, unsigned* ticket_launches, hipStream_t s) {
  const int NJ = (H + PJ - 1) / PJ, SG = groups * ((B + rows - 1) / rows), per = groups_per_launch(NJ, SG);
  if ((rows != 16 && rows != 32) || T < 1 || H > kPersistMaxH || NJ > device_cus()) return hipErrorInvalidValue;
  if ((dWp && !gru_persist_dw_supported(H)) || !dghx || ((uintptr_t)dghx & 15) != 0 || (s_dghx & 3) != 0)
    return hipErrorInvalidValue;
  KernelTimer kt(KID_GRU_BWD_PERSIST, 2.0 * B * 3 * H * (double)H * T * groups * (dWp ? 2 : 1), s);
#define HPSGD_BWD_PERSIST(C, R)                                                                                     \
  do {                                                                                                              \
    static std::atomic<size_t> allowed{0};                                                                          \
    const hipError_t e = allow_lds((const void*)gru_bwd_persist_kernel<C, R>, pl.lds, allowed);                     \
    if (e != hipSuccess) return e;                                                                                  \
    hipLaunchKernelGGL((gru_bwd_persist_kernel<C, R>), dim3(pl.grid), dim3(PNT), pl.lds, s, W_hh, s_rep, dgh, dghx, s_dghx, dgx, \
                       s_dg, D, s_D, d_zero ? 1 : 0, above, s_above, sv, s_sv, hs, s_hs, B, H, T, sg0, n_sg, sync, base, \
                       spin_limit, pl.tickets, pl.ticket_base, pl.per_xcd, dWp, dbp);                               \
  } while (0)
#define HPSGD_BWD_PERSIST_C(C)           \
  do {                                   \
    if (rows == 16) HPSGD_BWD_PERSIST(C, 16); \
    else HPSGD_BWD_PERSIST(C, 32);       \
  } while (0)
  for (int sg0 = 0; sg0 < SG; sg0 += per) {
    const int n_sg = SG - sg0 < per ? SG - sg0 : per;
    const Placement pl = placement(sync, SG, n_sg, NJ, persist_bwd_lds(H, rows), device_scope, ticket_launches);
    switch (persist_bwd_ncw(H)) {
      case 2: HPSGD_BWD_PERSIST_C(2); break;
      case 3: HPSGD_BWD_PERSIST_C(3); break;
      case 4: HPSGD_BWD_PERSIST_C(4); break;
      case 6: HPSGD_BWD_PERSIST_C(6); break;
      default: HPSGD_BWD_PERSIST_C(9); break;
    }
  }
#undef HPSGD_BWD_PERSIST_C
#undef HPSGD_BWD_PERSIST
  return hipGetLastError();
}

// Makes a given-up recurrence visible in the results: NaN in the losses and in the first
// parameter of every output replica.
__global__ void poison_on_abort_kernel(const unsigned* abort_w, float* loss, int n_loss, float* rout, long s_rout,
                                       int groups) {
  if (*abort_w == 0u) return;
  const float nan = __builtin_nanf("");
  for (int i = threadIdx.x; i < groups; i += blockDim.x) {
    rout[i * s_rout] = nan;
    if (loss && i < n_loss) loss[i] = nan;
  }
}

hipError_t launch_poison_on_abort(const unsigned* abort_w, float* loss, int n_loss, float* rout, long s_rout,
                                  int groups, hipStream_t s) {
  hipLaunchKernelGGL(poison_on_abort_kernel, dim3(1), dim3(64), 0, s, abort_w, loss, n_loss, rout, s_rout, groups);
  return hipGetLastError();
}

// bf16 operands: 32 units per workgroup, the weight slice in registers (24 fragments per wave at most)
bool gru_persist_bf16_supported(int B, int H) {
  return H % 32 == 0 && H >= 32 && H <= 1024 && B >= 8 && B % 8 == 0 && H / QJ <= device_cus();
}

// Batch rows per workgroup.  16 where all workers' workgroups then still fit one launch, and the XCDs, where they would with 32: a step's operands, its
// products, the partial sums that meet in LDS and the cells of a workgroup are half as many.  (A step is a chain of these; the chip has room for
// twice the workgroups.)  us per local step, 20 time steps, 2000 words, 32 rows / 16 (with no more chunk slots per wave than the width needs):
//   (H, batch, workers)  (1024, 32, 4) 436 / 397   (1024, 16, 8) 485 / 456   (768, 32, 2) 345 / 297   (650, 20, 4) 379 / 331
//                        (512, 64, 4) 365 / 340    (512, 16, 16) 413 / 394   (400, 24, 8) 332 / 305   (320, 8, 1) 221 / 199
// The slots alone, 32 rows: (672, 24, 5) 377 / 361, (672, 40, 5) 478 / 466, (768, 64, 5) 553 / 542.
int gru_persist_bf16_rows(int B, int H, int K) {
  if (B <= 16) return 16;
  const long NJ = (H + QJ - 1) / QJ, xcd = NJ <= kPlanCus / 8 ? 8 * (kPlanCus / 8 / NJ) : 0;  // groups that share an L2 each
  const long n16 = (long)((B + 15) / 16) * K, n32 = (long)((B + 31) / 32) * K;
  return n16 * NJ <= kPlanCus && (n16 <= xcd || n32 > xcd) ? 16 : 32;
}

// The gates of a model whose sizes are the launches' own and whose K workers fit one launch are the hardware's
// (sigm_fast, tanh_fast); every other bf16 model has those of the fp32 launches, as the step kernels that it would
// take without these launches.  (H, B: padded; padded: they are not the model's own.)
bool gru_bf16_exact_gates(int B, int H, int K, bool padded) {
  return padded || (long)(H / QJ) * ((B + 31) / 32) * K > kPlanCus;
}

unsigned gru_persist_bf16_count_per_step(int) { return 1u; }

size_t gru_persist_bf16_exchange_elems(int B, int width) { return (size_t)((B + 15) / 16) * 16 * (size_t)width; }

hipError_t launch_gru_fwd_persist_bf16(const void* Wb, long s_wb, const float* b_ih, const float* b_hh, long s_rep, int Hc,
                                       const float* gx,
                                       long s_gx, float* hs, long s_hs, void* hb, long s_hb, void* hx, long s_hx,
                                       float* sv, long s_sv, void* hT, long ld_hT, long s_hT, int Bc, int B, int H, int T,
                                       int groups, int rows, bool exact, unsigned* sync, unsigned base, unsigned spin_limit,
                                       bool device_scope, unsigned* ticket_launches, hipStream_t s) {
  if (!gru_persist_bf16_supported(B, H) || (rows != 16 && rows != 32) || Hc < 1 || Hc > H || Bc < 1 || Bc > B || T < 1) return hipErrorInvalidValue;
  auto a16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if (!hx || !a16(hx) || (s_hx & 7) != 0) return hipErrorInvalidValue;
  if (!a16(Wb) || !a16(hb) || !a16(hs) || !a16(gx) || !a16(sv) || (hT && !a16(hT)) || (s_wb & 7) != 0 ||
      (s_hb & 7) != 0 || (s_hs & 3) != 0 || (s_gx & 3) != 0 || (s_sv & 3) != 0 ||
      (hT && ((ld_hT & 7) != 0 || (s_hT & 7) != 0)))
    return hipErrorInvalidValue;
  const size_t lds = (size_t)8 * rows / 16 * 6 * 256 * sizeof(float) + (size_t)QJ * TP * 2 + 16;
  const int ncf = (H + 255) / 256;  // (a wave loads and multiplies all of its slots: those beyond the contraction are in vain)
  KernelTimer kt(KID_GRU_FWD_PERSIST_BF16, 2.0 * B * 3 * H * (double)H * T * groups, s);
#define HPSGD_FWD_PB(N, RB, EX)                                                                                    \
  do {                                                                                                             \
    static std::atomic<size_t> allowed{0};                                                                                     \
    const hipError_t e = allow_lds((const void*)gru_fwd_persist_bf16_kernel<N, RB, EX>, pl.lds, allowed);          \
    if (e != hipSuccess) return e;                                                                                 \
    hipLaunchKernelGGL((gru_fwd_persist_bf16_kernel<N, RB, EX>), dim3(pl.grid), dim3(PNT), pl.lds, s, (const __bf16*)Wb, s_wb, b_ih, \
                       b_hh, s_rep, Hc, gx, s_gx, hs, s_hs, (__bf16*)hb, s_hb, (__bf16*)hx, s_hx, sv, s_sv, (__bf16*)hT, ld_hT, \
                       s_hT, Bc, B, H, T, sg0, n_sg, sync, base, spin_limit, pl.tickets, pl.ticket_base, pl.per_xcd);  \
  } while (0)
#define HPSGD_FWD_PBN(N)                             \
  do {                                               \
    if (rows == 16 && exact) HPSGD_FWD_PB(N, 1, true);  \
    else if (rows == 16) HPSGD_FWD_PB(N, 1, false);     \
    else if (exact) HPSGD_FWD_PB(N, 2, true);           \
    else HPSGD_FWD_PB(N, 2, false);                     \
  } while (0)
  const int NJ = H / QJ, SG = groups * ((B + rows - 1) / rows), per = groups_per_launch(NJ, SG);
  for (int sg0 = 0; sg0 < SG; sg0 += per) {
    const int n_sg = SG - sg0 < per ? SG - sg0 : per;
    const Placement pl = placement(sync, SG, n_sg, NJ, lds, device_scope, ticket_launches);
    switch (ncf) {
      case 1: HPSGD_FWD_PBN(1); break;
      case 2: HPSGD_FWD_PBN(2); break;
      case 3: HPSGD_FWD_PBN(3); break;
      default: HPSGD_FWD_PBN(4); break;
    }
  }
#undef HPSGD_FWD_PBN
#undef HPSGD_FWD_PB
  return hipGetLastError();
}

hipError_t launch_gru_bwd_persist_bf16(const void* WT, long s_wt, void* dghx, long s_dgh, long s_dgb, float* D, long s_D,
                                       bool d_zero, const float* above, long s_above, const float* sv, long s_sv, const float* hs,
                                       long s_hs, void* dgxb, void* dgxT, void* dghT, long ld_T, long s_T, float* dbp,
                                       int Hc, int B, int H, int T, int groups, int rows, unsigned* sync, unsigned base,
                                       unsigned spin_limit, bool device_scope, unsigned* ticket_launches, hipStream_t s) {
  if (!gru_persist_bf16_supported(B, H) || (rows != 16 && rows != 32) || Hc < 1 || Hc > H || T < 1 || !dbp || !dgxb || !dgxT || !dghT || !dghx)
    return hipErrorInvalidValue;
  auto a16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if ((s_dgh & 7) != 0) return hipErrorInvalidValue;
  if (!a16(WT) || !a16(dghx) || !a16(dgxb) || !a16(dgxT) || !a16(dghT) || !a16(D) || !a16(sv) || !a16(hs) ||
      (above && !a16(above)) || (s_wt & 7) != 0 || (s_dgb & 7) != 0 || (ld_T & 7) != 0 || (s_T & 7) != 0 ||
      (s_D & 3) != 0 || (s_above & 3) != 0 || (s_sv & 3) != 0 || (s_hs & 3) != 0)
    return hipErrorInvalidValue;
  const int need = (3 * H / PC + 7) / 8;  // chunks per wave
  const int ncb = need <= 3 ? 3 : need <= 6 ? need : need <= 8 ? 8 : need <= 10 ? need : 12;
  const size_t lds = (size_t)8 * rows / 16 * 2 * 256 * sizeof(float) + (size_t)4 * QJ * TP * 2 +
                     (size_t)8 * persist_bwd_bf16_nl(ncb, rows / 16) * 2 * 64 * 16 + 16;
  KernelTimer kt(KID_GRU_BWD_PERSIST_BF16, 2.0 * B * 3 * H * (double)H * T * groups, s);
#define HPSGD_BWD_PB(N, RB)                                                                                        \
  do {                                                                                                             \
    static std::atomic<size_t> allowed{0};                                                                         \
    const hipError_t e = allow_lds((const void*)gru_bwd_persist_bf16_kernel<N, RB>, pl.lds, allowed);              \
    if (e != hipSuccess) return e;                                                                                 \
    hipLaunchKernelGGL((gru_bwd_persist_bf16_kernel<N, RB>), dim3(pl.grid), dim3(PNT), pl.lds, s, (const __bf16*)WT, s_wt,      \
                       (__bf16*)dghx, s_dgh, s_dgb, D, s_D, d_zero ? 1 : 0, above, s_above, sv, s_sv, hs, s_hs, (__bf16*)dgxb,  \
                       (__bf16*)dgxT, (__bf16*)dghT, ld_T, s_T, dbp, Hc, B, H, T, sg0, n_sg, sync, base, spin_limit,         \
                       pl.tickets, pl.ticket_base, pl.per_xcd);                                                    \
  } while (0)
#define HPSGD_BWD_PBN(N)                 \
  do {                                   \
    if (rows == 16) HPSGD_BWD_PB(N, 1);  \
    else HPSGD_BWD_PB(N, 2);             \
  } while (0)
  const int NJ = H / QJ, SG = groups * ((B + rows - 1) / rows), per = groups_per_launch(NJ, SG);
  for (int sg0 = 0; sg0 < SG; sg0 += per) {
    const int n_sg = SG - sg0 < per ? SG - sg0 : per;
    const Placement pl = placement(sync, SG, n_sg, NJ, lds, device_scope, ticket_launches);
    switch (ncb) {
      case 3: HPSGD_BWD_PBN(3); break;
      case 4: HPSGD_BWD_PBN(4); break;
      case 5: HPSGD_BWD_PBN(5); break;
      case 6: HPSGD_BWD_PBN(6); break;
      case 8: HPSGD_BWD_PBN(8); break;
      case 9: HPSGD_BWD_PBN(9); break;
      case 10: HPSGD_BWD_PBN(10); break;
      default: HPSGD_BWD_PBN(12); break;
    }
  }
#undef HPSGD_BWD_PBN
#undef HPSGD_BWD_PB
  return hipGetLastError();
}

}  // namespace hpsgd
