// Grouped fp32 GEMM on the fp32 matrix cores: pipelined kernel for operands of any alignment.
//
//   C[g] (M x N) = op(A[g]) (M x Kd) * op(B[g]) (Kd x N)      (same contract as gemm_f32.hip)
//
// Differences from the generic kernel: k-tiles of 32 with two LDS buffers and one barrier per
// k-tile, two register prefetch stages, and a main loop without branches (rows and columns
// are clamped into the matrix, which only changes values that feed outputs never stored; the
// contraction tail is zeroed by a select when a tile is written to LDS).  Operand tiles keep
// their natural layout in LDS, so no store is transposing:
//   * an operand that is unit-stride along k is stored [i][k]; an MFMA lane then reads a
//     float4 = 4 consecutive k of its row and feeds component s to MFMA number s (the order of
//     the contraction index is free as long as both operands agree): lane half lk covers
//     k = 8c + 4*lk + s;
//   * an operand that is unit-stride along i is stored [k][i] and read one float per MFMA at
//     the same k = 8c + 4*lk + s.
// v_mfma_f32_32x32x2_f32 lane layout: A lane l holds A[m = l%32][k = l/32], B lane l holds
// B[k = l/32][n = l%32], accumulator register v holds C[8*(v/4) + 4*(l/32) + v%4][l%32].
#include "kernels.h"

namespace hpsgd {

typedef float floatx16 __attribute__((ext_vector_type(16)));

static constexpr int FBK = 32;
static constexpr int FTHREADS = 256;

// 16 bytes at a 4-byte boundary: one load or store instruction like the aligned kind (this target
// splits what crosses a cache line)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
template <bool RAG>
__device__ __forceinline__ float4 ld16(const float* p) {
  if (RAG) {
    const f4u v = *reinterpret_cast<const f4u*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
  }
  return *reinterpret_cast<const float4*>(p);
}
template <bool RAG>
__device__ __forceinline__ void st16(float* p, const float4& v) {
  if (RAG) *reinterpret_cast<f4u*>(p) = (f4u){v.x, v.y, v.z, v.w};
  else *reinterpret_cast<float4*>(p) = v;
}
// components sh .. 3 of v moved to the front, zeros behind them
__device__ __forceinline__ float4 shift_down(const float4& v, int sh) {
  return make_float4(sh == 0 ? v.x : sh == 1 ? v.y : sh == 2 ? v.z : v.w, sh == 0 ? v.y : sh == 1 ? v.z : sh == 2 ? v.w : 0.f,
                     sh == 0 ? v.z : sh == 1 ? v.w : 0.f, sh == 0 ? v.w : 0.f);
}

// One operand tile: BI rows/columns x FBK.  CK: unit-stride along k in memory.
// RAG: any base alignment, row pitch and extent (>= 4 along the unit-stride index): the vectors are
// loaded at 4-byte boundaries, and one that would reach past the end of its row is loaded from the
// row's last four values and shifted into place when it is written to LDS.
template <int BI, bool CK, bool RAG>
struct FastOperand {
  static constexpr int PITCH = CK ? FBK + 4 : BI + 4;          // floats
  static constexpr int LDS_FLOATS = CK ? BI * PITCH : FBK * PITCH;
  static constexpr int UPT = BI * FBK / 4 / FTHREADS;          // float4 units per thread
  const float* ptr[UPT];   // each unit's row (CK) or column (not CK) base, clamped into the matrix
  float4 r[2][UPT];
  int shi = 0;             // RAG, not CK: how far this thread's column base was clamped (the same for all units)

  __device__ __forceinline__ void init(const float* __restrict__ base, long ld, int i0, int imax, int tid) {
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
      const int unit = tid + u * FTHREADS;
      if (CK) {
        ptr[u] = base + (long)min(i0 + (unit >> 3), imax - 1) * ld;
      } else {
        const int i = i0 + ((unit % (BI / 4)) << 2), ic = min(i, imax - 4);
        ptr[u] = base + ic;
        if (RAG) shi = min(i - ic, 3);
      }
    }
  }
  // k index of unit u inside a k-tile
  __device__ __forceinline__ static int kofs(int u, int tid) {
    const int unit = tid + u * FTHREADS;
    return CK ? ((unit & 7) << 2) : unit / (BI / 4);
  }
  __device__ __forceinline__ void load(int st, int kt, int Kd, long ld, int tid) {
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
      // a unit past the end of the contraction re-reads k = 0 (always in bounds) and is zeroed
      // when it is stored
      const int k = kt * FBK + kofs(u, tid);
      const int kc = k >= Kd ? 0 : (RAG && CK) ? min(k, Kd - 4) : k;
      r[st][u] = ld16<RAG>(ptr[u] + (CK ? (long)kc : (long)kc * ld));
    }
  }
  __device__ __forceinline__ void store(int st, int kt, int Kd, float* __restrict__ lds, int tid) const {
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
      const int unit = tid + u * FTHREADS;
      const int k = kt * FBK + kofs(u, tid);
      const bool in = k < Kd;  // not RAG: Kd % 4 == 0 for CK, a float4 is all in or out
      float4 v = in ? r[st][u] : make_float4(0.f, 0.f, 0.f, 0.f);
      if (RAG && CK && (kt + 1) * FBK > Kd && in) v = shift_down(v, k - min(k, Kd - 4));
      if (RAG && !CK) v = shift_down(v, shi);
      if (CK)
        *reinterpret_cast<float4*>(&lds[(unit >> 3) * PITCH + ((unit & 7) << 2)]) = v;
      else
        *reinterpret_cast<float4*>(&lds[(unit / (BI / 4)) * PITCH + ((unit % (BI / 4)) << 2)]) = v;
    }
  }
  // the 4 values k = 8c + 4*lk + {0..3} of row/column `i` of the tile
  __device__ __forceinline__ static float4 frag(const float* __restrict__ lds, int i, int c, int lk) {
    if (CK) return *reinterpret_cast<const float4*>(&lds[i * PITCH + 8 * c + 4 * lk]);
    const float* p = &lds[(8 * c + 4 * lk) * PITCH + i];
    return make_float4(p[0], p[PITCH], p[2 * PITCH], p[3 * PITCH]);
  }
};

// bid: the workgroup's index among those of this product
template <int BM, int BN, bool TA, bool TB, bool RAG>
__device__ __forceinline__ void fast_body(GemmDesc d, unsigned bid) {
  using OpA = FastOperand<BM, !TA, RAG>;   // A is unit-stride along k when stored [M][Kd]
  using OpB = FastOperand<BN, TB, RAG>;    // B is unit-stride along k when stored [N][Kd]
  constexpr int TM = BM / 64, TN = BN / 64;  // 2 x 2 waves, each (BM/2) x (BN/2) in 32 x 32 blocks
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  float* sA[2] = {fast_lds, fast_lds + OpA::LDS_FLOATS};
  float* sB[2] = {fast_lds + 2 * OpA::LDS_FLOATS, fast_lds + 2 * OpA::LDS_FLOATS + OpB::LDS_FLOATS};

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int lrow = lane & 31, lk = lane >> 5;
  // Tile order.  Workgroup i runs on XCD i % 8 and every XCD has its own L2: the tiles, in
  // (group, row tile, column tile) order, are cut into 8 contiguous runs, one per XCD, so that
  // an XCD fetches the A rows of its run once and only the B operands of the groups it touches.
  const int tn = (d.N + BN - 1) / BN, tm = (d.M + BM - 1) / BM;
  const int splits = d.splits > 1 ? d.splits : 1;
  const long ntiles = (long)tn * tm * d.groups * splits, per = (ntiles + 7) / 8;
  const long tile = (long)(bid & 7) * per + (bid >> 3);
  if ((long)(bid >> 3) >= per || tile >= ntiles) return;  // padding of the last run
  const int gp = (int)(tile / ((long)tn * tm));   // group * splits + part of the contraction
  const int g = gp / splits, part = gp - g * splits;
  const int m0 = (int)((tile / tn) % tm) * BM, n0 = (int)(tile % tn) * BN;

  OpA a;
  OpB b;
  const long ka = (long)part * d.Kd * (TA ? d.lda : 1), kb = (long)part * d.Kd * (TB ? 1 : d.ldb);
  // a part of a split contraction starts part * Kd further along k; the last one may be shorter
  if (splits > 1) d.Kd = min(d.Kd, d.Kall - part * d.Kd);
  a.init(d.A + (long)g * d.strideA + ka, d.lda, m0, d.M, tid);
  b.init(d.B + (long)g * d.strideB + kb, d.ldb, n0, d.N, tid);

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto compute = [&](int buf) {
#pragma unroll
    for (int c = 0; c < FBK / 8; ++c) {
      float4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = OpA::frag(sA[buf], wm * (BM / 2) + i * 32 + lrow, c, lk);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = OpB::frag(sB[buf], wn * (BN / 2) + j * 32 + lrow, c, lk);
      // contraction steps outermost: consecutive MFMAs update different accumulator tiles
      // (a dependent MFMA waits for the previous one to leave the pipeline)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].x, fb[j].x, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].y, fb[j].y, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].z, fb[j].z, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i].w, fb[j].w, acc[i][j], 0, 0, 0);
    }
  };

  const int nk = (d.Kd + FBK - 1) / FBK;
  a.load(0, 0, d.Kd, d.lda, tid);
  b.load(0, 0, d.Kd, d.ldb, tid);
  a.store(0, 0, d.Kd, sA[0], tid);
  b.store(0, 0, d.Kd, sB[0], tid);
  a.load(0, 1, d.Kd, d.lda, tid);
  b.load(0, 1, d.Kd, d.ldb, tid);
  a.load(1, 2, d.Kd, d.lda, tid);
  b.load(1, 2, d.Kd, d.ldb, tid);
  // The epilogue's extra matrix operand in C's layout (the old C, the ReLU mask or the weights
  // to update) is requested here, behind the first operand tiles: it arrives during the
  // contraction instead of holding up the epilogue (a weight gradient over one batch is a few
  // k-tiles of matrix work and as many bytes of weights to update as of operands).
  float* C = d.C + (long)(splits > 1 ? gp : g) * d.strideC;
  const float* aux = d.aux ? d.aux + (long)g * d.strideAux : nullptr;
  constexpr int CP = BN + 4;                       // pitch in floats
  constexpr int RPP = FTHREADS / (BN / 4);         // rows per pass
  constexpr int PASSES = BM / RPP;
  const int c4 = (tid % (BN / 4)) << 2, rbase = tid / (BN / 4);
  const int col = n0 + c4;
  const int epi = d.epilogue;
  const float* X = epi == EPI_ACCUM ? C : (epi == EPI_RELU_MASK || epi == EPI_COMMIT) ? aux : nullptr;
  const long xs = epi == EPI_ACCUM ? d.strideC : d.strideAux;
  const bool vec = RAG || (((d.ldc | d.strideC) & 3) == 0 && ((uintptr_t)d.C & 15) == 0 &&
                           (!X || (((uintptr_t)(epi == EPI_ACCUM ? d.C : d.aux) & 15) == 0 && (xs & 3) == 0)));
  float4 x[PASSES];
  if (X && vec && col + 3 < d.N) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int row = min(m0 + rbase + RPP * p, d.M - 1);  // clamped: not stored when outside
      x[p] = ld16<RAG>(X + (long)row * d.ldc + col);
    }
  }
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    compute(0);                                   // tile kt
    a.store(0, kt + 1, d.Kd, sA[1], tid);         // tile kt+1 -> buffer 1
    b.store(0, kt + 1, d.Kd, sB[1], tid);
    a.load(0, kt + 3, d.Kd, d.lda, tid);
    b.load(0, kt + 3, d.Kd, d.ldb, tid);
    __syncthreads();
    compute(1);                                   // tile kt+1 (all zeros past the end)
    a.store(1, kt + 2, d.Kd, sA[0], tid);         // tile kt+2 -> buffer 0
    b.store(1, kt + 2, d.Kd, sB[0], tid);
    a.load(1, kt + 4, d.Kd, d.lda, tid);
    b.load(1, kt + 4, d.Kd, d.ldb, tid);
    __syncthreads();
  }

  // Epilogue through LDS (the operand buffers are free after the last barrier): the
  // accumulators are laid out as the BM x BN tile, then every thread moves 16-byte pieces of
  // whole rows, so the stores and the loads of the extra operand (the old C, the ReLU mask or
  // the weights to update; all requested before the first is used) are fully coalesced.
  float* sC = fast_lds;
  static_assert((size_t)BM * CP <= 2 * (OpA::LDS_FLOATS + OpB::LDS_FLOATS), "epilogue tile fits the operand buffers");
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        sC[(wm * (BM / 2) + i * 32 + 8 * (v / 4) + 4 * lk + (v % 4)) * CP + wn * (BN / 2) + j * 32 + lrow] =
            acc[i][j][v];
  __syncthreads();
  if (vec && col + 3 < d.N) {
    float4 bv = make_float4(0.f, 0.f, 0.f, 0.f);
    if (epi == EPI_BIAS || epi == EPI_BIAS_RELU) bv = make_float4(aux[col], aux[col + 1], aux[col + 2], aux[col + 3]);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int rl = rbase + RPP * p, row = m0 + rl;
      if (row >= d.M) continue;
      const float4 a = *reinterpret_cast<const float4*>(&sC[rl * CP + c4]);
      float4 o = a;
      switch (epi) {
        case EPI_BIAS: o = make_float4(a.x + bv.x, a.y + bv.y, a.z + bv.z, a.w + bv.w); break;
        case EPI_BIAS_RELU:
          o = make_float4(fmaxf(a.x + bv.x, 0.f), fmaxf(a.y + bv.y, 0.f), fmaxf(a.z + bv.z, 0.f),
                          fmaxf(a.w + bv.w, 0.f));
          break;
        case EPI_ACCUM: o = make_float4(a.x + x[p].x, a.y + x[p].y, a.z + x[p].z, a.w + x[p].w); break;
        case EPI_RELU_MASK:
          o = make_float4(x[p].x > 0.f ? a.x : 0.f, x[p].y > 0.f ? a.y : 0.f, x[p].z > 0.f ? a.z : 0.f,
                          x[p].w > 0.f ? a.w : 0.f);
          break;
        case EPI_COMMIT:
          o = make_float4(x[p].x - d.alpha * a.x, x[p].y - d.alpha * a.y, x[p].z - d.alpha * a.z,
                          x[p].w - d.alpha * a.w);
          break;
        default: break;
      }
      st16<RAG>(C + (long)row * d.ldc + col, o);
    }
  } else {
    for (int p = 0; p < PASSES; ++p) {
      const int rl = rbase + RPP * p, row = m0 + rl;
      if (row >= d.M) continue;
      for (int e = 0; e < 4; ++e) {
        if (col + e >= d.N) break;
        const long off = (long)row * d.ldc + col + e;
        float val = sC[rl * CP + c4 + e];
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

// ---------------------------------------------------------------------------- few tiles
// A product of few tiles is bound by one wave's chain: in the form above a 64 x 64 tile's k-tile of 32 takes 0.8 us
// (16 MFMAs of 64 cycles per wave, two barriers' worth of waits), one after the other, while most of the chip is idle.
// Here a workgroup has a 32 x 32 tile and its four waves take a quarter of the contraction each, so that there
// are four times the workgroups and a chain is a quarter as long.  A wave loads its operands straight into the MFMA
// layout, four steps of 8 ahead, and waits for nobody before the sums of the four meet in LDS.
template <bool CK, bool RAG>
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
      r[u] = ld16<RAG>(p + max(min(k, Kd - 4), 0));
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

template <bool TA, bool TB, bool RAG>
__device__ __forceinline__ void slim_body(GemmDesc d, unsigned bid) {
  constexpr int PITCH = 36;  // floats of a row of a wave's sums
  extern __shared__ __attribute__((aligned(16))) float fast_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  SlimOperand<!TA, RAG> a;
  SlimOperand<TB, RAG> b;
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
    if (whole) x = ld16<true>(X + off);
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
    fast_lds[(wave * 32 + 8 * (v / 4) + 4 * lk + (v % 4)) * PITCH + lrow] = acc[0][v] + acc[1][v];
  __syncthreads();
  if (!in || col >= d.N) return;
  float4 o[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) o[w] = *reinterpret_cast<const float4*>(&fast_lds[(w * 32 + (tid >> 3)) * PITCH + ((tid & 7) << 2)]);
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
    st16<true>(C + off, make_float4(one(s.x, x.x, 0), one(s.y, x.y, 1), one(s.z, x.z, 2), one(s.w, x.w, 3)));
  } else {
    C[off] = one(s.x, x.x, 0);
    if (col + 1 < d.N) C[off + 1] = one(s.y, x.y, 1);
    if (col + 2 < d.N) C[off + 2] = one(s.z, x.z, 2);
  }
}
constexpr size_t kSlimLds = 4 * 32 * 36 * sizeof(float);

template <bool TA, bool TB, bool RAG>
__global__ void __launch_bounds__(FTHREADS) gemm_f32_slim_kernel(GemmDesc d) {
  slim_body<TA, TB, RAG>(d, blockIdx.x);
}

template <int BM, int BN, bool TA, bool TB, bool RAG>
__global__ void __launch_bounds__(FTHREADS) gemm_f32_fast_kernel(GemmDesc d) {
  fast_body<BM, BN, TA, TB, RAG>(d, blockIdx.x);
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

// Several products that need nothing of each other, and column sums, in one launch (64 x 64 tiles): each of
// them leaves most of the chip idle, and a launch of its own costs 4.5 us before it does anything.
// Product i owns the workgroups blk0[i] .. blk0[i+1]-1 (whole rounds over the XCDs), the column sums the rest.
// SLIM: those of the bits of `slim` are products of few tiles.
template <bool RAG, bool SLIM>
__global__ void __launch_bounds__(FTHREADS) gemm_f32_multi_kernel(GemmPack pk, ColsumPack cs, int groups, unsigned slim) {
  int i = 0;
  while (i < pk.n && blockIdx.x >= pk.blk0[i + 1]) ++i;  // (uniform)
  const unsigned bid = blockIdx.x - pk.blk0[i];
  if (i == pk.n) {
    const unsigned per = cs.blk0[cs.n];
    colsum_body(cs, bid % per, (int)(bid / per));
    return;
  }
  const GemmDesc& d = pk.d[i];
  if (SLIM && (slim >> i & 1)) {
    if (d.transA) slim_body<true, false, RAG>(d, bid);
    else if (d.transB) slim_body<false, true, RAG>(d, bid);
    else slim_body<false, false, RAG>(d, bid);
    return;
  }
  if (d.transA) fast_body<64, 64, true, false, RAG>(d, bid);
  else if (d.transB) fast_body<64, 64, false, true, RAG>(d, bid);
  else fast_body<64, 64, false, false, RAG>(d, bid);
}

template <int BM, int BN, bool TA, bool TB, bool RAG>
static hipError_t launch_fast_cfg(const GemmDesc& d, hipStream_t s) {
  using OpA = FastOperand<BM, !TA, RAG>;
  using OpB = FastOperand<BN, TB, RAG>;
  constexpr size_t smem = (size_t)2 * (OpA::LDS_FLOATS + OpB::LDS_FLOATS) * sizeof(float);
  static std::atomic<size_t> allowed{0};  // per instantiation: allow dynamic LDS above 64 KB
  if (const hipError_t e = allow_lds((const void*)gemm_f32_fast_kernel<BM, BN, TA, TB, RAG>, smem, allowed)) return e;
  const long ntiles = (long)((d.N + BN - 1) / BN) * ((d.M + BM - 1) / BM) * d.groups * (d.splits > 1 ? d.splits : 1);
  dim3 grid((unsigned)(8 * ((ntiles + 7) / 8)));
  KernelTimer kt(KID_GEMM_F32_FAST, 2.0 * d.M * d.N * (double)(d.splits > 1 ? d.Kall : d.Kd) * d.groups, s);
  hipLaunchKernelGGL((gemm_f32_fast_kernel<BM, BN, TA, TB, RAG>), grid, dim3(FTHREADS), smem, s, d);
  return hipGetLastError();
}

template <int BM, int BN, bool RAG>
static hipError_t launch_fast_layout(const GemmDesc& d, hipStream_t s) {
  if (!d.transA && d.transB) return launch_fast_cfg<BM, BN, false, true, RAG>(d, s);
  if (!d.transA && !d.transB) return launch_fast_cfg<BM, BN, false, false, RAG>(d, s);
  if (d.transA && !d.transB) return launch_fast_cfg<BM, BN, true, false, RAG>(d, s);
  return launch_fast_cfg<BM, BN, true, true, RAG>(d, s);
}

hipError_t launch_gemm_f32_fast(const GemmDesc& d, hipStream_t s);

// 0: the pipelined kernel does not take the product (an extent along a unit-stride index below one vector);
// 1: it does; 2: it does, as a product of unaligned operands
static int fast_kind(const GemmDesc& d) {
  auto aligned = [](const float* p, long ld, long stride) {
    return ((uintptr_t)p & 15) == 0 && (ld & 3) == 0 && (stride & 3) == 0;
  };
  // extents along the unit-stride index of the two operands (the contraction's last part included)
  const int klast = d.splits > 1 ? d.Kall - (d.splits - 1) * d.Kd : d.Kd;
  const int ua = d.transA ? d.M : klast, ub = d.transB ? klast : d.N;
  if (ua < 4 || ub < 4) return 0;
  return !aligned(d.A, d.lda, d.strideA) || !aligned(d.B, d.ldb, d.strideB) || ((ua | ub) & 3) != 0 ? 2 : 1;
}
static bool fast_large(const GemmDesc& d, int groups) {
  // 128 x 128 tiles from two full rounds of workgroups on: below that the smaller tiles' better
  // balance over the CUs outweighs their extra LDS traffic (the fp32 matrix rate is low enough).
  // A contraction of a few k-tiles (a weight gradient over one batch) is mostly first loads and
  // epilogue: four small workgroups per SIMD cover those better than two large ones (matrix
  // pipes busy 52 % of the time with the large tile at Kd = 128)
  const long t = (long)((d.M + 127) / 128) * ((d.N + 127) / 128) * groups;
  return d.M > 64 && d.N > 64 && t >= 512 && d.Kd > 256;
}

// The form for few tiles: up to 64 tiles of 64 x 64, up to 256 with a contraction that makes a long chain, and
// up to 128 where the launch holds nothing else (`shared`: it does, or would with all workers' tiles: the form decides
// the order of a sum).  (Beyond, the chip is busy either way and the larger tile reads its
// operands fewer times.)  Measured, one / the other form of every product of at most that many tiles:
//   to  64: MLP 30-64-896-8, batch 224, K = 2     90 /  52 us a round; 28-832-672-32-13, batch 16, K = 3   94 /  72
//   to 256: MLP 596-928-140-7, batch 145, K = 3   83 /  74;  two GRU layers of H = 544, batch 4, K = 4  1148 / 1134
//   but     two GRU layers of H = 100, batch 20, K = 4 (128 tiles, contraction 300, beside 560 others)   311 /  315
//           fp32 language model, 248 tiles, contraction 192   233 / 240
//   to 512: MLP 784-1024-1024-10, batch 128, K = 16  288 / 375
static bool fast_slim(const GemmDesc& d, bool shared) {
  const long t = (long)((d.M + 63) / 64) * ((d.N + 63) / 64) * (d.workers ? d.workers : d.groups) * (d.splits > 1 ? d.splits : 1);
  return !(d.transA && d.transB) && (t <= 64 || (t <= 256 && d.Kd >= 512) || (t <= 128 && !shared));
}
static unsigned tile_blocks(const GemmDesc& d, int tile) {
  const long t = (long)((d.N + tile - 1) / tile) * ((d.M + tile - 1) / tile) * d.groups * (d.splits > 1 ? d.splits : 1);
  return (unsigned)(8 * ((t + 7) / 8));
}
template <bool RAG>
static hipError_t launch_slim(const GemmDesc& d, hipStream_t s) {
  const dim3 grid(tile_blocks(d, 32));
  KernelTimer kt(KID_GEMM_F32_FAST, 2.0 * d.M * d.N * (double)(d.splits > 1 ? d.Kall : d.Kd) * d.groups, s);
  if (d.transA) hipLaunchKernelGGL((gemm_f32_slim_kernel<true, false, RAG>), grid, dim3(FTHREADS), kSlimLds, s, d);
  else if (d.transB) hipLaunchKernelGGL((gemm_f32_slim_kernel<false, true, RAG>), grid, dim3(FTHREADS), kSlimLds, s, d);
  else hipLaunchKernelGGL((gemm_f32_slim_kernel<false, false, RAG>), grid, dim3(FTHREADS), kSlimLds, s, d);
  return hipGetLastError();
}

bool gemm_pack_push(GemmPack& pk, const GemmDesc& d) {
  if (pk.n >= GemmPack::MAX || d.bf16 || d.background || (d.transA && d.transB) || !fast_kind(d) || fast_large(d, d.groups)) return false;
  if (d.M <= 0 || d.N <= 0 || d.groups <= 0) return false;
  pk.d[pk.n++] = d;
  // (fewer workers than all: a product that all of them launch by itself is a guest here, which changes no other's form)
  if (!fast_large(d, d.workers ? d.workers : d.groups)) ++pk.n_all;
  return true;
}

hipError_t launch_gemm_pack(GemmPack& pk, const ColsumPack& cs, int groups, hipStream_t s) {
  if (pk.n == 0 && cs.n == 0) return hipSuccess;
  if (pk.n == 0) return launch_colsum_pack(cs, groups, s);
  if (pk.n == 1 && cs.n == 0) return launch_gemm_f32_fast(pk.d[0], s);
  bool rag = false;
  unsigned slim = 0;
  double flops = 0.;
  const bool shared = pk.n_all > 1 || cs.n > 0;
  pk.blk0[0] = 0;
  for (int i = 0; i < pk.n; ++i) {
    const GemmDesc& d = pk.d[i];
    const bool few = fast_slim(d, shared);
    rag = rag || fast_kind(d) == 2;
    slim |= few ? 1u << i : 0u;
    pk.blk0[i + 1] = pk.blk0[i] + tile_blocks(d, few ? 32 : 64);
    flops += 2.0 * d.M * d.N * (double)(d.splits > 1 ? d.Kall : d.Kd) * d.groups;
  }
  using OpC = FastOperand<64, true, false>;
  using OpN = FastOperand<64, false, false>;
  constexpr size_t op = OpC::LDS_FLOATS > OpN::LDS_FLOATS ? OpC::LDS_FLOATS : OpN::LDS_FLOATS;
  constexpr size_t smem = 4 * op * sizeof(float);  // two buffers of two operands, in their largest layout
  static_assert(smem <= 64 * 1024, "within the default limit of dynamic LDS");
  dim3 grid(pk.blk0[pk.n] + (cs.n ? cs.blk0[cs.n] * (unsigned)groups : 0u));
  KernelTimer kt(KID_GEMM_F32_FAST, flops, s);
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(FTHREADS), smem, s, pk, cs, groups, slim); };
  if (rag) slim ? launch(gemm_f32_multi_kernel<true, true>) : launch(gemm_f32_multi_kernel<true, false>);
  else slim ? launch(gemm_f32_multi_kernel<false, true>) : launch(gemm_f32_multi_kernel<false, false>);
  return hipGetLastError();
}

// Returns hipErrorNotSupported (nothing launched) when an operand's extent along its unit-stride index
// is below one vector; the caller then takes the generic kernel.
hipError_t launch_gemm_f32_fast(const GemmDesc& d, hipStream_t s) {
  if (d.splits > 1 && (d.epilogue != EPI_STORE || (d.Kd & 3) != 0 || d.Kall <= (d.splits - 1) * d.Kd)) return hipErrorInvalidValue;
  const int kind = fast_kind(d);
  if (!kind) return hipErrorNotSupported;
  const bool rag = kind == 2;
  if (fast_slim(d, false)) return rag ? launch_slim<true>(d, s) : launch_slim<false>(d, s);
  if (fast_large(d, d.groups)) return rag ? launch_fast_layout<128, 128, true>(d, s) : launch_fast_layout<128, 128, false>(d, s);
  return rag ? launch_fast_layout<64, 64, true>(d, s) : launch_fast_layout<64, 64, false>(d, s);
}

}  // namespace hpsgd
