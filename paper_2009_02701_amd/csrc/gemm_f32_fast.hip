// Grouped fp32 GEMM for operands of any alignment: pipelined kernels.
//
//   C[g] (M x N) = op(A[g]) (M x Kd) * op(B[g]) (Kd x N)      (same contract as gemm_f32.hip)
//
// Products of many tiles are computed on the bf16 matrix cores from operands split into three parts, products of few tiles on
// the fp32 ones.
// v_mfma_f32_32x32x2_f32 lane layout: A lane l holds A[m = l%32][k = l/32], B lane l holds
// B[k = l/32][n = l%32], accumulator register v holds C[8*(v/4) + 4*(l/32) + v%4][l%32];
// v_mfma_f32_32x32x16_bf16 the same with 8 values of k per lane.
#include <type_traits>

#include "kernels.h"
#include "split_f32.h"

namespace hpsgd {

typedef float floatx16 __attribute__((ext_vector_type(16)));

static constexpr int FTHREADS = 256;  // of a product of few tiles, of column sums

// 16 bytes at a 4-byte boundary: one load or store instruction like the aligned kind (this target
// splits what crosses a cache line)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ld16(const float* p) {
  const f4u v = *reinterpret_cast<const f4u*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
// components sh .. 3 of v moved to the front, zeros behind them
__device__ __forceinline__ float4 shift_down(const float4& v, int sh) {
  return make_float4(sh == 0 ? v.x : sh == 1 ? v.y : sh == 2 ? v.z : v.w, sh == 0 ? v.y : sh == 1 ? v.z : sh == 2 ? v.w : 0.f,
                     sh == 0 ? v.z : sh == 1 ? v.w : 0.f, sh == 0 ? v.w : 0.f);
}

// ---------------------------------------------------------------------------- split operands
// The product as six products of bf16 parts (split_f32.h).  A workgroup has a 64 x 64 tile and k-tiles of 32; 2 x 2 waves share the
// tile, and every other group of 8 along k has four waves of its own, whose sums meet in the epilogue: with four waves for all
// of them, half as many waves were there to cover each other's loads, splits and barriers.
// An operand tile is split once, on its way to LDS, where its parts lie in the order in which the lanes of an MFMA
// read them: 16 bytes are the 8 values of k-group g (k = 8g ..) of one row, 32 rows of a group are consecutive,
// REGION keeps a row's four groups in different banks for the writes.
// Any alignment, pitch and size: rows and columns are clamped into the matrix (what that changes is never stored); along k a
// thread has half a group of 4, clamped to the last 4 of the contraction, and those that another half group has already are
// zeroed in A.  Operands of any size: a lane's offset is of 32 bits (every address a load of its own took more instructions than
// its products) from a uniform address of 64, the tile's first row or, across the contraction, the half group's.
// us, the fp32 instruction's pipelined kernel of 64 x 64 or 128 x 128 tiles before / this (GRU language model, classifier and
// MLP, operands of every worker's own):
//   128 x 1024 x 784, 16 workers  39.4 / 29.1      560 x 2000 x 256, 4  32.4 / 26.0        560 x 256 x 2000, 4  48.5 / 35.3
//   1536 x 128 x 560, 16          46.6 / 35.7      2000 x 256 x 560, 4, in place  34.1 / 25.3     1000 x 300 x 40, 4  6.9 / 7.1
//   1024 x 784 x 128, 16, in place  51.2 / 51.9 (its bytes)     4096 x 4096 x 4096  1099 / 876
// 1.4 to 2.0 us per k-tile of 256 workgroups: the LDS writes (6 bytes a value at 75 bytes a cycle) and the conversions take
// as long as the matrix work.
static constexpr int SBM = 64, SBK = 32, STHREADS = 512;
typedef float f4v __attribute__((ext_vector_type(4)));
template <bool CK>
struct SplitTile {
  static constexpr int REGION = 512 + 32, PLANE = SBM / 32 * 4 * REGION, LDS_BYTES = 3 * PLANE;
  const float* p;  // the tile's first row (CK) or column
  __amdgpu_buffer_rsrc_t rs;
  long ld;
  int off;        // the thread's row (CK) or column from there, in bytes
  float r[2][4];  // a half group each: 64 x 8 of them are one per thread

  __device__ __forceinline__ static int half(int tid) { return CK ? tid & 7 : __builtin_amdgcn_readfirstlane(tid / SBM); }
  __device__ __forceinline__ static int row(int tid) { return CK ? tid >> 3 : tid % SBM; }
  // first k of half group k4 as it is read
  __device__ __forceinline__ static int base(int k4, int Kd) { return max(min(k4, Kd - 4), 0); }
  __device__ __forceinline__ void init(const float* __restrict__ p_, long ld_, int i0, int imax, int tid) {
    ld = ld_;
    p = p_ + (CK ? i0 * ld : i0);
    rs = rsrc(p);
    off = min(row(tid), imax - 1 - i0) * (CK ? (int)ld * 4 : 4);
  }
  // (everything that is read lies inside the operand)
  __device__ __forceinline__ static __amdgpu_buffer_rsrc_t rsrc(const float* q) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(q), 0, 0x7fffffff, 0x00020000);
  }
  __device__ __forceinline__ void load(int st, int kt, int Kd, int tid) {
    const int k4 = kt * SBK + 4 * half(tid);
    const bool tail = (kt + 1) * SBK > Kd;  // (uniform; beyond the last tile everything is read from the end)
    if (CK) {
      const f4v v = __builtin_bit_cast(f4v, tail ? __builtin_amdgcn_raw_buffer_load_b128(rs, off + 4 * base(k4, Kd), 0, 0)
                                                 : __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * half(tid), kt * SBK * 4, 0));
#pragma unroll
      for (int j = 0; j < 4; ++j) r[st][j] = v[j];
    } else {
      const __amdgpu_buffer_rsrc_t rk = rsrc(p + base(k4, Kd) * ld);
#pragma unroll
      for (int j = 0; j < 4; ++j) r[st][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rk, off, min(j, Kd - 1) * (int)ld * 4, 0));
    }
  }
  __device__ __forceinline__ void mask(int st, int kt, int Kd, int tid) {
    const int k4 = kt * SBK + 4 * half(tid), kb = base(k4, Kd);
#pragma unroll
    for (int j = 0; j < 4; ++j) r[st][j] = kb + j >= k4 && kb + j < Kd ? r[st][j] : 0.f;
  }
  __device__ __forceinline__ void store(int st, char* __restrict__ lds, int tid) const {
    uint2 p0, p1, p2;
    split2(r[st][0], r[st][1], p0.x, p1.x, p2.x);
    split2(r[st][2], r[st][3], p0.y, p1.y, p2.y);
    const int i = row(tid), h = half(tid);
    char* q = lds + ((i >> 5) * 4 + (h >> 1)) * REGION + (i & 31) * 16 + (h & 1) * 8;
    *reinterpret_cast<uint2*>(q) = p0;
    *reinterpret_cast<uint2*>(q + PLANE) = p1;
    *reinterpret_cast<uint2*>(q + 2 * PLANE) = p2;
  }
  // the parts of the values of 32-row block b, k-group g, lane row `lrow`
  __device__ __forceinline__ static void frag(const char* __restrict__ lds, int b, int g, int lrow, bf16x8s (&f)[3]) {
#pragma unroll
    for (int p = 0; p < 3; ++p) f[p] = *reinterpret_cast<const bf16x8s*>(lds + p * PLANE + (b * 4 + g) * REGION + lrow * 16);
  }
};

// Contractions of up to 3 (weight gradients of so small a batch) stay with the fp32 instruction: of one term it gives the rounded
// product, the six bf16 ones an error 3 % larger in the 2-norm and up to 1.5 times as large.
static constexpr int kShort = 3;
__host__ __device__ static inline bool is_short(const GemmDesc& d) { return d.Kd <= kShort && d.splits <= 1 && d.transA && !d.transB; }

// The sums of a 32 x 32 block that are not finite, again with the fp32 instruction (rare: nothing is staged):
// the k-groups g0, g0 + dg, .. of 8
template <bool TA, bool TB>
__device__ __forceinline__ floatx16 split_redo(const float* __restrict__ A, long lda, const float* __restrict__ B, long ldb,
                                               int m, int n, int Kd, int g0, int dg, floatx16 have) {
  const int lk = (threadIdx.x & 63) >> 5;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll 1
  for (int k8 = 8 * g0; k8 < Kd; k8 += 8 * dg)
#pragma unroll 1
    for (int kk = k8; kk < min(k8 + 8, Kd); kk += 2) {
      const int k = min(kk + lk, Kd - 1);
      const float a = TA ? A[(long)k * lda + m] : A[(long)m * lda + k], b = TB ? B[(long)n * ldb + k] : B[(long)k * ldb + n];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(kk + lk < Kd ? a : 0.f, kk + lk < Kd ? b : 0.f, acc, 0, 0, 0);
    }
#pragma unroll
  for (int v = 0; v < 16; ++v) have[v] = have[v] - have[v] == 0.f ? have[v] : acc[v];
  return have;
}

template <bool TA, bool TB, bool SHORT>
__device__ __forceinline__ void split_body(GemmDesc d, unsigned bid) {
  constexpr int NT = STHREADS, BM = SBM, BN = SBM;
  using OpA = SplitTile<!TA>;
  using OpB = SplitTile<TB>;
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  char* const lds = reinterpret_cast<char*>(fast_lds);
  constexpr int BUF = OpA::LDS_BYTES + OpB::LDS_BYTES;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave & 1, wm = (wave >> 1) & 1, ks = wave >> 2;
  const int lrow = lane & 31, lk = lane >> 5;
  // Tile order.  Workgroup i runs on XCD i % 8 and every XCD has its own L2: the tiles, in
  // (group, row tile, column tile) order, are cut into 8 contiguous runs, one per XCD, so that
  // an XCD fetches the A rows of its run once and only the B operands of the groups it touches.
  const int tn = (d.N + BN - 1) / BN, tm = (d.M + BM - 1) / BM;
  const int splits = d.splits > 1 ? d.splits : 1;
  // (a grid holds them: 32 bits; with divisions in 64 a launch of one round, 256 x 2048 x 10, 2 workers, took 6.5 us instead of 5.8)
  const unsigned each = (unsigned)tn * tm, ntiles = each * d.groups * splits, per = (ntiles + 7) / 8;
  const unsigned tile = (bid & 7) * per + (bid >> 3);
  if ((bid >> 3) >= per || tile >= ntiles) return;  // padding of the last run
  const int gp = (int)(tile / each), in_g = (int)(tile - gp * each);   // group * splits + part of the contraction
  const int g = gp / splits, part = gp - g * splits;
  const int m0 = in_g / tn * BM, n0 = in_g % tn * BN;

  OpA a;
  OpB b;
  const float* Ag = d.A + (long)g * d.strideA + (long)part * d.Kd * (TA ? d.lda : 1);
  const float* Bg = d.B + (long)g * d.strideB + (long)part * d.Kd * (TB ? 1 : d.ldb);
  // a part of a split contraction starts part * Kd further along k; the last one may be shorter
  if (splits > 1) d.Kd = min(d.Kd, d.Kall - part * d.Kd);
  a.init(Ag, d.lda, m0, d.M, tid);
  b.init(Bg, d.ldb, n0, d.N, tid);

  const int nk = (d.Kd + SBK - 1) / SBK;
  a.load(0, 0, d.Kd, tid);
  b.load(0, 0, d.Kd, tid);
  a.load(1, 1, d.Kd, tid);
  b.load(1, 1, d.Kd, tid);
  // The epilogue's extra matrix operand in C's layout (the old C, the ReLU mask or the weights
  // to update) is requested here, behind the first operand tiles: it arrives during the
  // contraction instead of holding up the epilogue (a weight gradient over one batch is a few
  // k-tiles of matrix work and as many bytes of weights to update as of operands).
  float* C = d.C + (long)(splits > 1 ? gp : g) * d.strideC;
  const float* aux = d.aux ? d.aux + (long)g * d.strideAux : nullptr;
  constexpr int CP = BN + 4;                       // pitch in floats
  constexpr int RPP = NT / (BN / 4);               // rows per pass
  constexpr int PASSES = BM / RPP;
  const int c4 = (tid % (BN / 4)) << 2, rbase = tid / (BN / 4);
  const int col = n0 + c4;
  const int epi = d.epilogue;
  const float* X = epi == EPI_ACCUM ? C : (epi == EPI_RELU_MASK || epi == EPI_COMMIT) ? aux : nullptr;
  f4u x[PASSES];
  if (X && col + 3 < d.N) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int row = min(m0 + rbase + RPP * p, d.M - 1);  // clamped: not stored when outside
      x[p] = *reinterpret_cast<const f4u*>(X + (long)row * d.ldc + col);
    }
  }
  floatx16 acc, acs;  // the sum of a0 b0 and the sum of the other products
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = acs[v] = 0.f;
  if constexpr (SHORT) {
    float* q = fast_lds;  // [A, B][4 of k][64]: the first half groups, which wave 0 has
    if (wave == 0) {
      a.mask(0, 0, d.Kd, tid);
      b.mask(0, 0, d.Kd, tid);
#pragma unroll
      for (int j = 0; j < 4; ++j) q[j * BM + lane] = a.r[0][j], q[(4 + j) * BM + lane] = b.r[0][j];
    }
    __syncthreads();
    if (ks == 0)
#pragma unroll
      for (int j = 0; j < 4; j += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(q[(j + lk) * BM + wm * 32 + lrow], q[(4 + j + lk) * BM + wn * 32 + lrow], acc, 0, 0, 0);
  } else {
    if (nk == 1) a.mask(0, 0, d.Kd, tid);
    a.store(0, lds, tid);
    b.store(0, lds + OpA::LDS_BYTES, tid);
    a.load(0, 2, d.Kd, tid);
    b.load(0, 2, d.Kd, tid);

    // fragments of two tiles (this wave's groups of each): the one that is multiplied and the next one, on its way from LDS
    bf16x8s fa[2][3], fb[2][3];
    auto frags = [&](int s, int buf) {
      OpA::frag(lds + buf * BUF, wm, 2 * lk + ks, lrow, fa[s]);
      OpB::frag(lds + buf * BUF + OpA::LDS_BYTES, wn, 2 * lk + ks, lrow, fb[s]);
    };
    auto mul = [&](int s, int pa, int pb, floatx16& to) { to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][pa], fb[s][pb], to, 0, 0, 0); };
    __syncthreads();
    frags(0, 0);
    // Tile kt's fragments are in registers, tile kt + 1 in register stage (kt + 1) & 1, tile kt + 2 on its way to the other.
    // Half of the tile's products cover the splitting of the next one, the other half the first reads of it.
    auto step = [&](auto P_, int kt) {
      constexpr int P = decltype(P_)::value, Q = 1 - P;
      if (kt + 2 >= nk) a.mask(Q, kt + 1, d.Kd, tid);
      __builtin_amdgcn_sched_barrier(0);
      mul(P, 0, 0, acc);
      mul(P, 1, 0, acs);
      mul(P, 2, 0, acs);
      a.store(Q, lds + Q * BUF, tid);
      b.store(Q, lds + Q * BUF + OpA::LDS_BYTES, tid);
      a.load(Q, kt + 3, d.Kd, tid);
      b.load(Q, kt + 3, d.Kd, tid);
#pragma unroll
      for (int i = 0; i < 3; ++i) {  // (interleaved: an MFMA, 12 vector instructions)
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
      }
      __syncthreads();
      frags(Q, Q);
      mul(P, 0, 1, acs);
      mul(P, 1, 1, acs);
      mul(P, 0, 2, acs);
    };
    for (int kt = 0; kt < nk; kt += 2) {
      step(std::integral_constant<int, 0>(), kt);
      if (kt + 1 < nk) step(std::integral_constant<int, 1>(), kt + 1);
    }
  }

  bool redo = false;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    acc[v] += acs[v];
    redo = redo || !(acc[v] - acc[v] == 0.f);
  }
  if (__builtin_expect(__any(redo), 0))
    acc = split_redo<TA, TB>(Ag, d.lda, Bg, d.ldb, min(m0 + wm * 32 + lrow, d.M - 1), min(n0 + wn * 32 + lrow, d.N - 1), d.Kd, ks, 2, acc);
  __syncthreads();  // (the last fragments have been read)

  // Epilogue through LDS: the accumulators are laid out as the BM x BN tile, then every thread moves 16-byte pieces of
  // whole rows, so the stores and the loads of the extra operand (the old C, the ReLU mask or
  // the weights to update; all requested before the first is used) are fully coalesced.
  float* sC = fast_lds;
#pragma unroll
  for (int v = 0; v < 16; ++v) sC[(ks * BM + wm * 32 + 8 * (v / 4) + 4 * lk + (v % 4)) * CP + wn * 32 + lrow] = acc[v];
  __syncthreads();
  if (col + 3 < d.N) {
    f4u bv = {0.f, 0.f, 0.f, 0.f};
    if (epi == EPI_BIAS || epi == EPI_BIAS_RELU) bv = *reinterpret_cast<const f4u*>(aux + col);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int rl = rbase + RPP * p, row = m0 + rl;
      if (row >= d.M) continue;
      const float4 av = *reinterpret_cast<const float4*>(&sC[rl * CP + c4]);
      const float4 aw = *reinterpret_cast<const float4*>(&sC[(BM + rl) * CP + c4]);
      f4u o = {av.x + aw.x, av.y + aw.y, av.z + aw.z, av.w + aw.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        switch (epi) {
          case EPI_BIAS: o[e] = o[e] + bv[e]; break;
          case EPI_BIAS_RELU: o[e] = fmaxf(o[e] + bv[e], 0.f); break;
          case EPI_ACCUM: o[e] = o[e] + x[p][e]; break;
          case EPI_RELU_MASK: o[e] = x[p][e] > 0.f ? o[e] : 0.f; break;
          case EPI_COMMIT: o[e] = x[p][e] - d.alpha * o[e]; break;
          default: break;
        }
      }
      *reinterpret_cast<f4u*>(C + (long)row * d.ldc + col) = o;
    }
  } else {
    for (int p = 0; p < PASSES; ++p) {
      const int rl = rbase + RPP * p, row = m0 + rl;
      if (row >= d.M) continue;
      for (int e = 0; e < 4; ++e) {
        if (col + e >= d.N) break;
        const long off = (long)row * d.ldc + col + e;
        float val = sC[rl * CP + c4 + e] + sC[(BM + rl) * CP + c4 + e];
        switch (epi) {
          case EPI_BIAS: val += aux[col + e]; break;
          case EPI_BIAS_RELU: val = fmaxf(val + aux[col + e], 0.f); break;
          case EPI_ACCUM: val += C[off]; break;
          case EPI_RELU_MASK: val = aux[off] > 0.f ? val : 0.f; break;
          case EPI_COMMIT: val = aux[off] - d.alpha * val; break;
          default: break;
        }
        C[off] = val;
      }
    }
  }
}
// ---------------------------------------------------------------------------- both operands stored along the contraction
// C = A^T B with A stored [Kd][M] and B [Kd][N], M and N even (the weight gradients): a load of one k for 64 columns, a pair per
// lane, is whole cache lines, so every wave takes the operands of its 64 x 64 outputs straight from memory into the MFMA
// layout and splits them in registers: no LDS, no barrier, nobody to wait for.  Two waves a SIMD cover each other's loads,
// conversions and epilogues.  Columns are clamped into the matrix; rows beyond the contraction lie beyond the buffers: zeros.
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
static constexpr int DBM = 128;  // 2 x 2 waves
template <bool SHORT>
__device__ __forceinline__ void direct_body(GemmDesc d, unsigned bid) {
  constexpr int BM = DBM, BN = DBM, TM = 2, TN = 2, ST = 2;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 31, lk = lane >> 5;
  const int tn = (d.N + BN - 1) / BN, tm = (d.M + BM - 1) / BM;
  const int splits = d.splits > 1 ? d.splits : 1;
  const long ntiles = (long)tn * tm * d.groups * splits, per = (ntiles + 7) / 8;  // (a run of tiles per XCD, as above)
  const long tile = (long)(bid & 7) * per + (bid >> 3);
  if ((long)(bid >> 3) >= per || tile >= ntiles) return;
  const int gp = (int)(tile / ((long)tn * tm));
  const int g = gp / splits, part = gp - g * splits;
  const int m0 = (int)((tile / tn) % tm) * BM + (wave & 1) * 32 * TM, n0 = (int)(tile % tn) * BN + (wave >> 1) * 32 * TN;
  if (m0 >= d.M || n0 >= d.N) return;  // (no barrier follows)
  const float* Ag = d.A + (long)g * d.strideA + (long)part * d.Kd * d.lda;
  const float* Bg = d.B + (long)g * d.strideB + (long)part * d.Kd * d.ldb;
  if (splits > 1) d.Kd = min(d.Kd, d.Kall - part * d.Kd);
  // the lane's neighbouring columns, one of each 32 x 32 block: 64 columns are loaded as 32 pairs
  const int ca = m0 + 2 * lrow, cb = n0 + 2 * lrow;
  const int oa = (min(ca, d.M - 2) + lk * (int)d.lda) * 4, ob = (min(cb, d.N - 2) + lk * (int)d.ldb) * 4;
  auto rsrc = [](const float* p, long floats) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)(floats * 4), 0x00020000); };
  const __amdgpu_buffer_rsrc_t ba = rsrc(Ag, (long)(d.Kd - 1) * d.lda + d.M), bb = rsrc(Bg, (long)(d.Kd - 1) * d.ldb + d.N);
  const int nc = (d.Kd + 15) / 16;
  float ra[ST][TM][8], rb[ST][TN][8];
  // k = 16 c + 2 j + lk: the two halves of a load are neighbouring rows
  auto load = [&](int st, int c) {
    int fa = c * 16 * (int)d.lda * 4, fb = c * 16 * (int)d.ldb * 4;
#pragma unroll
    for (int j = 0; j < 8; ++j, fa += 8 * (int)d.lda, fb += 8 * (int)d.ldb) {
      const f2v va = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(ba, oa, fa, 0));
      const f2v vb = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(bb, ob, fb, 0));
      ra[st][0][j] = va.x;
      ra[st][1][j] = va.y;
      rb[st][0][j] = vb.x;
      rb[st][1][j] = vb.y;
    }
  };
#pragma unroll
  for (int st = 0; st < ST; ++st) load(st, st);
  floatx16 acc[TM][TN], acs[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = acs[i][j][v] = 0.f;
  if constexpr (SHORT) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ra[0][i][k], rb[0][j][k], acc[i][j], 0, 0, 0);
  }
  for (int c0 = SHORT ? nc : 0; c0 < nc; c0 += ST) {
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      const int c = c0 + st;
      if (c >= nc) break;
      uint4 fa[TM][3], fb[TN][3];
#pragma unroll
      for (int i = 0; i < TM; ++i) split8(ra[st][i], fa[i][0], fa[i][1], fa[i][2]);
#pragma unroll
      for (int j = 0; j < TN; ++j) split8(rb[st][j], fb[j][0], fb[j][1], fb[j][2]);
      load(st, c + ST);
      auto mul = [&](int pa, int pb, floatx16 (&to)[TM][TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            to[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8s, fa[i][pa]), __builtin_bit_cast(bf16x8s, fb[j][pb]), to[i][j], 0, 0, 0);
      };
      mul(0, 0, acc);
      mul(1, 0, acs);
      mul(2, 0, acs);
      mul(0, 1, acs);
      mul(1, 1, acs);
      mul(0, 2, acs);
    }
  }
  float* C = d.C + (long)(splits > 1 ? gp : g) * d.strideC;
  const float* aux = d.aux ? d.aux + (long)g * d.strideAux : nullptr;
  const int epi = d.epilogue;
  const float* X = epi == EPI_ACCUM ? C : (epi == EPI_RELU_MASK || epi == EPI_COMMIT) ? aux : nullptr;
  // block (i, j) holds the rows m0 + 2 r + i and the columns n0 + 2 c + j
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    float x[16][2];
    const int r0 = m0 + 8 * lk + i;  // + 2 (8 (v / 4) + v % 4)
    if (X) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = min(r0 + 2 * (8 * (v / 4) + v % 4), d.M - 1);
        const f2u t = *reinterpret_cast<const f2u*>(X + (long)r * d.ldc + min(cb, d.N - 2));
        x[v][0] = t.x;
        x[v][1] = t.y;
      }
    }
    floatx16 s[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      s[j] = acc[i][j] + acs[i][j];
      bool redo = false;
#pragma unroll
      for (int v = 0; v < 16; ++v) redo = redo || !(s[j][v] - s[j][v] == 0.f);
      if (__builtin_expect(__any(redo), 0))
        s[j] = split_redo<true, false>(Ag, d.lda, Bg, d.ldb, min(m0 + 2 * lrow + i, d.M - 1), min(cb + j, d.N - 1), d.Kd, 0, 1, s[j]);
    }
    f2u bias = {0.f, 0.f};
    if (epi == EPI_BIAS || epi == EPI_BIAS_RELU) bias = *reinterpret_cast<const f2u*>(aux + min(cb, d.N - 2));
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = r0 + 2 * (8 * (v / 4) + v % 4);
      f2u o = {s[0][v], s[1][v]};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        switch (epi) {
          case EPI_BIAS: o[e] = o[e] + bias[e]; break;
          case EPI_BIAS_RELU: o[e] = fmaxf(o[e] + bias[e], 0.f); break;
          case EPI_ACCUM: o[e] = o[e] + x[v][e]; break;
          case EPI_RELU_MASK: o[e] = x[v][e] > 0.f ? o[e] : 0.f; break;
          case EPI_COMMIT: o[e] = x[v][e] - d.alpha * o[e]; break;
          default: break;
        }
      }
      if (r < d.M && cb < d.N) *reinterpret_cast<f2u*>(C + (long)r * d.ldc + cb) = o;
    }
  }
}
template <bool SHORT>
__global__ void __launch_bounds__(FTHREADS, 2) gemm_f32_direct_kernel(GemmDesc d) { direct_body<SHORT>(d, blockIdx.x); }

// ---------------------------------------------------------------------------- few tiles
// A product of few tiles is bound by one wave's chain: in the form above a 64 x 64 tile's k-tile of 32 takes 0.8 us
// (16 MFMAs of 64 cycles per wave, two barriers' worth of waits), one after the other, while most of the chip is idle.
// Here a workgroup has a 32 x 32 tile and its four waves take a quarter of the contraction each, so that there
// are four times the workgroups and a chain is a quarter as long.  A wave loads its operands straight into the MFMA
// layout, four steps of 8 ahead, and waits for nobody before the sums of the four meet in LDS.
template <bool CK>
struct SlimOperand {
  const float* p;
  long ld;
  float4 r[4];
  __device__ __forceinline__ void init(const float* __restrict__ base, long ld_, int i, int imax) {
    ld = ld_;
    p = base + (CK ? (long)min(i, imax - 1) * ld_ : (long)min(i, imax - 1));
  }
  // the values k .. k + 3, clamped into the contraction
  __device__ __forceinline__ void load(int u, int k, int Kd) {
    if (CK) {
      r[u] = ld16(p + max(min(k, Kd - 4), 0));
    } else {
      r[u] = make_float4(p[(long)min(k, Kd - 1) * ld], p[(long)min(k + 1, Kd - 1) * ld], p[(long)min(k + 2, Kd - 1) * ld],
                         p[(long)min(k + 3, Kd - 1) * ld]);
    }
  }
  // ... with zeros beyond it
  __device__ __forceinline__ float4 tail(int u, int k, int Kd) const {
    float4 v = r[u];
    if (CK) return k >= Kd ? make_float4(0.f, 0.f, 0.f, 0.f) : shift_down(v, k - min(k, Kd - 4));
    return make_float4(k < Kd ? v.x : 0.f, k + 1 < Kd ? v.y : 0.f, k + 2 < Kd ? v.z : 0.f, k + 3 < Kd ? v.w : 0.f);
  }
};

// bid: the four waves' index among those of this product; lds: theirs
template <bool TA, bool TB>
__device__ __forceinline__ void slim_body(GemmDesc d, unsigned bid, float* lds) {
  constexpr int PITCH = 36;  // floats of a row of a wave's sums
  const int tid = threadIdx.x & (FTHREADS - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 31, lk = lane >> 5;
  const int tn = (d.N + 31) / 32, tm = (d.M + 31) / 32;
  const int splits = d.splits > 1 ? d.splits : 1;
  const long ntiles = (long)tn * tm * d.groups * splits, per = (ntiles + 7) / 8;  // (a run of tiles per XCD, as above)
  const long tile = (long)(bid & 7) * per + (bid >> 3);
  if ((long)(bid >> 3) >= per || tile >= ntiles) return;
  const int gp = (int)(tile / ((long)tn * tm));
  const int g = gp / splits, part = gp - g * splits;
  const int m0 = (int)((tile / tn) % tm) * 32, n0 = (int)(tile % tn) * 32;
  const long ka = (long)part * d.Kd * (TA ? d.lda : 1), kb = (long)part * d.Kd * (TB ? 1 : d.ldb);
  if (splits > 1) d.Kd = min(d.Kd, d.Kall - part * d.Kd);
  SlimOperand<!TA> a;
  SlimOperand<TB> b;
  a.init(d.A + (long)g * d.strideA + ka, d.lda, m0 + lrow, d.M);
  b.init(d.B + (long)g * d.strideB + kb, d.ldb, n0 + lrow, d.N);
  const int nc = (d.Kd + 7) / 8, ncw = (nc + 3) / 4, c0 = wave * ncw, c1 = min(nc, c0 + ncw);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    a.load(u, 8 * (c0 + u) + 4 * lk, d.Kd);
    b.load(u, 8 * (c0 + u) + 4 * lk, d.Kd);
  }
  // the epilogue's extra matrix operand, behind the first operands (see above)
  float* C = d.C + (long)(splits > 1 ? gp : g) * d.strideC;
  const float* aux = d.aux ? d.aux + (long)g * d.strideAux : nullptr;
  const int epi = d.epilogue;
  const float* X = epi == EPI_ACCUM ? C : (epi == EPI_RELU_MASK || epi == EPI_COMMIT) ? aux : nullptr;
  const int row = m0 + (tid >> 3), col = n0 + ((tid & 7) << 2);
  const bool in = row < d.M, whole = col + 3 < d.N;
  const long off = (long)min(row, d.M - 1) * d.ldc + col;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  if (X) {
    if (whole) x = ld16(X + off);
    else x = make_float4(X[off - max(col - d.N + 1, 0)], X[off - max(col + 1 - (d.N - 1), 0) + 1], X[off - max(col + 2 - (d.N - 1), 0) + 2], 0.f);
  }
  floatx16 acc[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
  for (int c = c0; c < c1; c += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (c + u < c1) {  // (uniform)
        const int k = 8 * (c + u) + 4 * lk;
        float4 fa = a.r[u], fb = b.r[u];
        if (8 * (c + u) + 8 > d.Kd) {  // (uniform)
          fa = a.tail(u, k, d.Kd);
          fb = b.tail(u, k, d.Kd);
        }
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.x, fb.x, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.y, fb.y, acc[1], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.z, fb.z, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.w, fb.w, acc[1], 0, 0, 0);
      }
      a.load(u, 8 * (c + 4 + u) + 4 * lk, d.Kd);
      b.load(u, 8 * (c + 4 + u) + 4 * lk, d.Kd);
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v)
    lds[(wave * 32 + 8 * (v / 4) + 4 * lk + (v % 4)) * PITCH + lrow] = acc[0][v] + acc[1][v];
  __syncthreads();
  if (!in || col >= d.N) return;
  float4 o[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) o[w] = *reinterpret_cast<const float4*>(&lds[(w * 32 + (tid >> 3)) * PITCH + ((tid & 7) << 2)]);
  const float4 s = make_float4((o[0].x + o[1].x) + (o[2].x + o[3].x), (o[0].y + o[1].y) + (o[2].y + o[3].y),
                               (o[0].z + o[1].z) + (o[2].z + o[3].z), (o[0].w + o[1].w) + (o[2].w + o[3].w));
  auto one = [&](float v, float xv, int e) -> float {
    switch (epi) {
      case EPI_BIAS: return v + aux[col + e];
      case EPI_BIAS_RELU: return fmaxf(v + aux[col + e], 0.f);
      case EPI_ACCUM: return v + xv;
      case EPI_RELU_MASK: return xv > 0.f ? v : 0.f;
      case EPI_COMMIT: return xv - d.alpha * v;
      default: return v;
    }
  };
  if (whole) {
    *reinterpret_cast<f4u*>(C + off) = (f4u){one(s.x, x.x, 0), one(s.y, x.y, 1), one(s.z, x.z, 2), one(s.w, x.w, 3)};
  } else {
    C[off] = one(s.x, x.x, 0);
    if (col + 1 < d.N) C[off + 1] = one(s.y, x.y, 1);
    if (col + 2 < d.N) C[off + 2] = one(s.z, x.z, 2);
  }
}
constexpr size_t kSlimLds = 4 * 32 * 36 * sizeof(float);

template <bool TA, bool TB>
__global__ void __launch_bounds__(FTHREADS) gemm_f32_slim_kernel(GemmDesc d) {
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  slim_body<TA, TB>(d, blockIdx.x, fast_lds);
}

template <bool TA, bool TB, bool SHORT = false>
__global__ void __launch_bounds__(STHREADS) gemm_f32_fast_kernel(GemmDesc d) {
  split_body<TA, TB, SHORT>(d, blockIdx.x);
}

// Column sums as further workgroups of a launch of products: a workgroup covers 64 columns with 4 row slices
// (slice s takes rows s, s + 4, ..), combined in a fixed order.
__device__ __forceinline__ void colsum_body(const ColsumPack& pk, unsigned bid, int g) {
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  int sgi = 0;
#pragma unroll
  for (int i = 1; i < ColsumPack::MAXSEG; ++i)
    if (i < pk.n && bid >= pk.blk0[i]) sgi = i;
  const ColsumSeg& sg = pk.seg[sgi];
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  if (sg.N == 1) {  // one column (the mean of the row losses): every thread takes rows
    float v = 0.f;
    for (int r = threadIdx.x; r < sg.R; r += FTHREADS) v += sg.in[g * sg.s_in + (long)r * sg.ld];
    fast_lds[threadIdx.x] = v;
    __syncthreads();
    for (int o = FTHREADS / 2; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) fast_lds[threadIdx.x] += fast_lds[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0)
      sg.out[g * sg.s_out] = sg.b_in ? sg.b_in[g * sg.s_bin] - pk.lr * fast_lds[0] : fast_lds[0] * sg.scale;
    return;
  }
  const int c = (int)(bid - pk.blk0[sgi]) * 64 + lane;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (c < sg.N) {
    const float* p = sg.in + g * sg.s_in + c;
    int r = slice;
    for (; r + 28 < sg.R; r += 32) {  // eight rows in flight
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] += p[(long)(r + 4 * u) * sg.ld];
    }
    for (; r < sg.R; r += 4) a[0] += p[(long)r * sg.ld];
  }
  fast_lds[slice * 64 + lane] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  __syncthreads();
  if (slice == 0 && c < sg.N) {
    const float v = (fast_lds[lane] + fast_lds[64 + lane]) + (fast_lds[128 + lane] + fast_lds[192 + lane]);
    sg.out[g * sg.s_out + c] = sg.b_in ? sg.b_in[g * sg.s_bin + c] - pk.lr * v : v * sg.scale;
  }
}

// Several products that need nothing of each other, and column sums, in one launch: each of
// them leaves most of the chip idle, and a launch of its own costs 4.5 us before it does anything.
// Product i owns the workgroups blk0[i] .. blk0[i+1]-1 (whole rounds over the XCDs), the column sums the rest.
// SLIM: those of the bits of `slim` are products of few tiles; a workgroup has room for two of them.
// SHORT: there are contractions of up to kShort.
template <bool SLIM, bool SHORT>
__global__ void __launch_bounds__(STHREADS) gemm_f32_multi_kernel(GemmPack pk, ColsumPack cs, int groups, unsigned slim) {
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  int i = 0;
  while (i < pk.n && blockIdx.x >= pk.blk0[i + 1]) ++i;  // (uniform)
  const unsigned bid = blockIdx.x - pk.blk0[i];
  if (i == pk.n) {
    if (threadIdx.x >= FTHREADS) return;
    const unsigned per = cs.blk0[cs.n];
    colsum_body(cs, bid % per, (int)(bid / per));
    return;
  }
  const GemmDesc& d = pk.d[i];
  if (SLIM && (slim >> i & 1)) {
    const unsigned half = __builtin_amdgcn_readfirstlane(threadIdx.x / FTHREADS);
    const unsigned b32 = (bid >> 3) * 16 + half * 8 + (bid & 7);
    float* lds = fast_lds + half * (kSlimLds / sizeof(float));
    if (d.transA) slim_body<true, false>(d, b32, lds);
    else if (d.transB) slim_body<false, true>(d, b32, lds);
    else slim_body<false, false>(d, b32, lds);
    return;
  }
  if (SHORT && is_short(d)) split_body<true, false, true>(d, bid);
  else if (d.transA) split_body<true, false, false>(d, bid);
  else if (d.transB) split_body<false, true, false>(d, bid);
  else split_body<false, false, false>(d, bid);
}

// ... and of products that take their operands from memory
template <bool SHORT>
__global__ void __launch_bounds__(FTHREADS, 2) gemm_f32_direct_multi_kernel(GemmPack pk, ColsumPack cs, int groups) {
  int i = 0;
  while (i < pk.n && blockIdx.x >= pk.blk0[i + 1]) ++i;  // (uniform)
  const unsigned bid = blockIdx.x - pk.blk0[i];
  if (i < pk.n) {
    if (SHORT && is_short(pk.d[i])) direct_body<true>(pk.d[i], bid);
    else direct_body<false>(pk.d[i], bid);
    return;
  }
  const unsigned per = cs.blk0[cs.n];
  colsum_body(cs, bid % per, (int)(bid / per));
}

// ... and where all of them are products of few tiles: a tile a workgroup, which waits for nobody else's k-tiles
// (two layers of H = 64 on 20 and 64 inputs, batch 80, 36 steps, one worker: weight gradients 10.9 us in the form above, 9.6 here)
__global__ void __launch_bounds__(FTHREADS) gemm_f32_slim_multi_kernel(GemmPack pk, ColsumPack cs, int groups) {
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  int i = 0;
  while (i < pk.n && blockIdx.x >= pk.blk0[i + 1]) ++i;  // (uniform)
  const unsigned bid = blockIdx.x - pk.blk0[i];
  if (i == pk.n) {
    const unsigned per = cs.blk0[cs.n];
    colsum_body(cs, bid % per, (int)(bid / per));
    return;
  }
  const GemmDesc& d = pk.d[i];
  if (d.transA) slim_body<true, false>(d, bid, fast_lds);
  else if (d.transB) slim_body<false, true>(d, bid, fast_lds);
  else slim_body<false, false>(d, bid, fast_lds);
}

hipError_t launch_gemm_f32_fast(const GemmDesc& d, hipStream_t s);

// Whether these kernels take the product: a contraction of at least one half group where an operand is unit-stride along it.
// Rows of 2^23 floats and more, of which the 64 of a tile are beyond 32-bit offsets, take the form for few tiles, whose addresses
// are of 64 bits.
static int last_part(const GemmDesc& d) { return d.splits > 1 ? d.Kall - (d.splits - 1) * d.Kd : d.Kd; }
static bool long_rows(const GemmDesc& d) { return d.lda >= 1L << 23 || d.ldb >= 1L << 23; }
static bool fast_takes(const GemmDesc& d) {
  return last_part(d) >= (d.transA && !d.transB ? 1 : 4) && !(d.transA && d.transB && long_rows(d));
}

// The form for few tiles: up to 256 tiles of 32 x 32, up to 448 where the launch holds nothing else (`shared`: it does;
// the form decides the order of a sum).  (Beyond, the chip is busy either way and the larger tile reads its
// operands fewer times.)  us, this form / the other one:
//   256 tiles  Kd =   64   4.9 /  5.4, 1024  11.9 / 18.3       288 tiles  Kd = 200  7.2 /  8.2      240 tiles of 960 x 32 outputs, Kd = 180  6.0 / 8.6
//   448 tiles  Kd =  200   7.8 /  8.7,  600  13.5 / 14.6       512 tiles  Kd = 300  10.2 /  9.5, Kd = 64  7.1 / 5.9
//   576 tiles  Kd = 2000  47.7 / 36.2                         1024 tiles  Kd = 512  23.7 / 13.0
static bool fast_slim(const GemmDesc& d, bool shared) {
  const long t = (long)((d.M + 31) / 32) * ((d.N + 31) / 32) * (d.workers ? d.workers : d.groups) * (d.splits > 1 ? d.splits : 1);
  return !(d.transA && d.transB) && (t <= (shared ? 256 : 448) || long_rows(d));
}
// Operands straight from memory: weight gradients of two rounds of workgroups and more.  us, this form / through LDS (in place,
// 16 workers): 1024 x 784, Kd = 128 (896 tiles)  45 / 53, 1024 x 1024 (1024)  49 / 62; but 1536 x 128, Kd = 560 (192)  35 / 35,
// 2000 x 256, Kd = 560, 4 workers (128)  36 / 25.
static bool fast_direct(const GemmDesc& d) {
  const long t = (long)((d.M + DBM - 1) / DBM) * ((d.N + DBM - 1) / DBM) * (d.workers ? d.workers : d.groups) * (d.splits > 1 ? d.splits : 1);
  const long most = (1L << 29) - 64;  // floats of an operand: 32-bit offsets from its first element
  return d.transA && !d.transB && ((d.M | d.N) & 1) == 0 && t >= 512 && (d.Kd - 1) * d.lda + d.M < most &&
         (d.Kd - 1) * d.ldb + d.N < most;
}
static unsigned tile_blocks(const GemmDesc& d, int tile) {
  const long t = (long)((d.N + tile - 1) / tile) * ((d.M + tile - 1) / tile) * d.groups * (d.splits > 1 ? d.splits : 1);
  return (unsigned)(8 * ((t + 7) / 8));
}
static hipError_t launch_slim(const GemmDesc& d, hipStream_t s) {
  const dim3 grid(tile_blocks(d, 32));
  KernelTimer kt(KID_GEMM_F32_FAST, 2.0 * d.M * d.N * (double)(d.splits > 1 ? d.Kall : d.Kd) * d.groups, s);
  if (d.transA) hipLaunchKernelGGL((gemm_f32_slim_kernel<true, false>), grid, dim3(FTHREADS), kSlimLds, s, d);
  else if (d.transB) hipLaunchKernelGGL((gemm_f32_slim_kernel<false, true>), grid, dim3(FTHREADS), kSlimLds, s, d);
  else hipLaunchKernelGGL((gemm_f32_slim_kernel<false, false>), grid, dim3(FTHREADS), kSlimLds, s, d);
  return hipGetLastError();
}

bool gemm_pack_push(GemmPack& pk, const GemmDesc& d) {
  if (pk.n >= GemmPack::MAX || d.bf16 || d.background || (d.transA && d.transB) || !fast_takes(d)) return false;
  if (d.M <= 0 || d.N <= 0 || d.groups <= 0) return false;
  pk.d[pk.n++] = d;
  return true;
}

// (both layouts of an operand have the same size in LDS; the epilogue tile is smaller, and so is a product of few tiles)
static constexpr size_t kSplitLds = 4 * SplitTile<true>::LDS_BYTES;
static_assert(2 * SBM * (SBM + 4) * sizeof(float) <= kSplitLds && 2 * kSlimLds <= kSplitLds && kSplitLds <= 64 * 1024,
              "the operand buffers hold the rest, within the default limit of dynamic LDS");

hipError_t launch_gemm_pack(GemmPack& pk, const ColsumPack& cs, int groups, hipStream_t s) {
  if (pk.n == 0 && cs.n == 0) return hipSuccess;
  if (pk.n == 0) return launch_colsum_pack(cs, groups, s);
  if (pk.n == 1 && cs.n == 0) return launch_gemm_f32_fast(pk.d[0], s);
  unsigned slim = 0;
  double flops = 0.;
  bool direct = true, alike = true, some_short = false;  // all of them: operands from memory, few tiles
  for (int i = 0; i < pk.n; ++i)
    direct = direct && fast_direct(pk.d[i]), alike = alike && fast_slim(pk.d[i], true), some_short = some_short || is_short(pk.d[i]);
  pk.blk0[0] = 0;
  for (int i = 0; i < pk.n; ++i) {
    const GemmDesc& d = pk.d[i];
    const bool few = !direct && fast_slim(d, true);
    slim |= few ? 1u << i : 0u;
    pk.blk0[i + 1] = pk.blk0[i] + (direct ? tile_blocks(d, DBM) : alike ? tile_blocks(d, 32) : few ? (tile_blocks(d, 32) / 8 + 1) / 2 * 8 : tile_blocks(d, SBM));
    flops += 2.0 * d.M * d.N * (double)(d.splits > 1 ? d.Kall : d.Kd) * d.groups;
  }
  dim3 grid(pk.blk0[pk.n] + (cs.n ? cs.blk0[cs.n] * (unsigned)groups : 0u));
  KernelTimer kt(KID_GEMM_F32_FAST, flops, s);
  if (direct) {
    hipLaunchKernelGGL(some_short ? gemm_f32_direct_multi_kernel<true> : gemm_f32_direct_multi_kernel<false>, grid, dim3(FTHREADS), FTHREADS * sizeof(float), s, pk, cs, groups);
    return hipGetLastError();
  }
  if (alike) {
    hipLaunchKernelGGL(gemm_f32_slim_multi_kernel, grid, dim3(FTHREADS), kSlimLds, s, pk, cs, groups);
    return hipGetLastError();
  }
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(STHREADS), kSplitLds, s, pk, cs, groups, slim); };
  if (some_short) slim ? launch(gemm_f32_multi_kernel<true, true>) : launch(gemm_f32_multi_kernel<false, true>);
  else slim ? launch(gemm_f32_multi_kernel<true, false>) : launch(gemm_f32_multi_kernel<false, false>);
  return hipGetLastError();
}

// Returns hipErrorNotSupported (nothing launched) where these kernels do not take the product; the caller then takes the
// generic one.
hipError_t launch_gemm_f32_fast(const GemmDesc& d, hipStream_t s) {
  if (d.splits > 1 && (d.epilogue != EPI_STORE || (d.Kd & 3) != 0 || d.Kall <= (d.splits - 1) * d.Kd)) return hipErrorInvalidValue;
  if (!fast_takes(d)) return hipErrorNotSupported;
  if (fast_slim(d, false)) return launch_slim(d, s);
  const bool direct = fast_direct(d);
  const dim3 grid(tile_blocks(d, direct ? DBM : SBM));
  KernelTimer kt(KID_GEMM_F32_FAST, 2.0 * d.M * d.N * (double)(d.splits > 1 ? d.Kall : d.Kd) * d.groups, s);
  if (direct) {
    hipLaunchKernelGGL(is_short(d) ? gemm_f32_direct_kernel<true> : gemm_f32_direct_kernel<false>, grid, dim3(FTHREADS), 0, s, d);
    return hipGetLastError();
  }
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(STHREADS), kSplitLds, s, d); };
  if (is_short(d)) launch(gemm_f32_fast_kernel<true, false, true>);
  else if (d.transA) d.transB ? launch(gemm_f32_fast_kernel<true, true>) : launch(gemm_f32_fast_kernel<true, false>);
  else d.transB ? launch(gemm_f32_fast_kernel<false, true>) : launch(gemm_f32_fast_kernel<false, false>);
  return hipGetLastError();
}

}  // namespace hpsgd
