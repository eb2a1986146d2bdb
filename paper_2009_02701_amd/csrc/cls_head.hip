// The head of a classifier with few classes in two small launches per local step (fp32):
//   logits = feats W^T + b;  loss = mean cross-entropy;  dlogits = (softmax - onehot) / N;
//   dfeat = dlogits W;  dW = dlogits^T feats;  db = column sums of dlogits;
//   then either the SGD update (W_out = W_in - lr dW, b_out = b_in - lr db) or the gradients.
// With N <= 128 rows and C <= 32 classes each of the three products is a fraction of a
// megaflop per worker: as three GEMM launches, two reductions, a softmax and a loss launch
// they cost seven launch gaps and little else.  Here the forward part is cut over the rows
// (16 per workgroup) and the backward part over the feature columns (32 per workgroup), so that a
// worker's head is spread over several CUs (a single workgroup per worker with everything in LDS was
// measured at ~95 us: bound by one CU's LDS rate).  Every sum runs in a fixed order.
//
// All three products are v_mfma_f32_16x16x4_f32 with the classes in blocks of 16 (A lane l holds A[m = l%16][k = l/16],
// B lane l holds B[k = l/16][n = l%16], accumulator register v holds C[4*(l/16) + v][l%16]); eight waves cut the
// contraction, so that a launch is one trip to memory, a handful of instructions and one or two trips through LDS.
// Measured against multiply-adds from LDS with rows, then columns, in series per thread (forward + backward launch):
// N = 128, C = 10, H = 1024, 16 workers 17.5 + 28.3 -> 6.7 + 8.5 us; N = 16, C = 21, H = 64, one worker 12.6 + 7.9 -> 4.5 + 5.0; N = 14, C = 27,
// H = 130, 6 workers 16.5 + 11.0 -> 4.9 + 7.5.
#include <cmath>

#include "kernels.h"

namespace hpsgd {

namespace {

constexpr int HMAXC = 32;     // classes
constexpr int HMAXN = 128;    // rows
constexpr int HROWS = 16;     // rows per workgroup, forward
constexpr int HCOLS = 32;     // feature columns per workgroup, backward

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// Values k .. k + 3 of a row of H, zeros beyond it (any alignment)
__device__ __forceinline__ floatx4 row4(const float* __restrict__ p, int k, int H) {
  if (k + 3 < H) {
    const f4u v = *reinterpret_cast<const f4u*>(p + k);
    return (floatx4){v.x, v.y, v.z, v.w};
  }
  floatx4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = p[min(k + e, H - 1)];
    v[e] = k + e < H ? x : 0.f;
  }
  return v;
}

// grid (ceil(N / 16), groups), 512 threads: wave w takes the contraction's chunks of 16 w, w + 8, ..; behind the
// products thread t has class t % 32 of row t / 32.  CB: blocks of 16 classes
template <int CB>
__global__ void __launch_bounds__(512)
cls_head_fwd_kernel(const float* __restrict__ feats, long s_feats, const float* __restrict__ W,
                    const float* __restrict__ b, long s_in, const int32_t* __restrict__ y, long s_y,
                    float* __restrict__ dlog, long s_dlog, float* __restrict__ rowloss, long s_rowloss, int N, int C,
                    int H) {
  constexpr int LP = 16 * CB + 1;
  __shared__ float red[8][HROWS][LP];
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const float* fr = feats + g * s_feats + (long)min((int)blockIdx.x * HROWS + lr, N - 1) * H;
  const float* wr[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) wr[cb] = W + g * s_in + (long)min(16 * cb + lr, C - 1) * H;
  // (what the last part needs arrives with the operands)
  const int c = tid & 31, row = blockIdx.x * HROWS + (tid >> 5), rowc = min(row, N - 1);
  const float bias = b[g * s_in + min(c, C - 1)];
  const int label = y[g * s_y + rowc];
  floatx4 acc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc[cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
  const int nc = (H + 15) / 16;
  for (int i = w; i < nc; i += 32) {  // four chunks at a time
    floatx4 f[4], v[4][CB];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + 8 * u < nc) {  // (uniform)
        const int k = 16 * (i + 8 * u) + 4 * lg;
        f[u] = row4(fr, k, H);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) v[u][cb] = row4(wr[cb], k, H);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + 8 * u < nc) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[u][e], v[u][cb][e], acc[cb], 0, 0, 0);
      }
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[w][4 * lg + v][16 * cb + lr] = acc[cb][v];
  __syncthreads();
  if (row >= N) return;  // (the 32 threads of a row together)
  const bool ok = c < C;
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) z += red[i][tid >> 5][min(c, 16 * CB - 1)];
  z = ok ? z + bias : -INFINITY;
  float m = z;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 32));
  const float zl = __shfl(z, label & 31, 32);
  const float ez = ok ? expf(z - m) : 0.f;
  float sum = ez;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 32);
  const float inv_sum = 1.0f / sum, inv_n = 1.0f / (float)N;
  if (c == 0) rowloss[g * s_rowloss + row] = -(((label >= 0 && label < C ? zl : 0.f) - m) - logf(sum));
  if (ok) dlog[g * s_dlog + (long)row * C + c] = (ez * inv_sum - (c == label ? 1.0f : 0.0f)) * inv_n;
}

// grid (ceil(H / 32), groups), 512 threads: wave w has the columns of block w % 2 and rows 32 (w / 2) .. + 31.  Step s of
// the weight gradient's contraction takes row 16 (s / 4) + 4 (l / 16) + s % 4 of those in lane l: the row of register s
// of the input gradient's two blocks, so that a lane's features are its outputs' ReLU mask too.
template <int CB>
__global__ void __launch_bounds__(512)
cls_head_bwd_kernel(const float* __restrict__ feats, long s_feats, const float* W_in, const float* b_in, long s_in,
                    const float* __restrict__ dlog, long s_dlog, const float* __restrict__ rowloss, long s_rowloss,
                    float* __restrict__ dfeat, long s_dfeat, float* W_out, float* b_out, long s_out, float lr,
                    int commit, float* __restrict__ loss, int N, int C, int H, int relu_mask) {
  constexpr int DP = 16 * CB + 1;
  __shared__ float sD[HMAXN * DP];                   // dlogits [N][classes], zeros beyond N and C
  __shared__ float red[4][16 * CB][HCOLS + 1];       // the weight gradient's sums per quarter of the rows
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr_ = lane & 15, lg = lane >> 4, rq = w >> 1, r0 = 32 * rq;
  const int j = blockIdx.x * HCOLS + 16 * (w & 1) + lr_, jc = min(j, H - 1);
  const float* dl = dlog + g * s_dlog;
  const float* fe = feats + g * s_feats + jc;
  const float* Wg = W_in + g * s_in;
  float f[8], wv[4 * CB];
#pragma unroll
  for (int s = 0; s < 8; ++s) f[s] = fe[(long)min(r0 + 16 * (s / 4) + 4 * lg + s % 4, N - 1) * H];
#pragma unroll
  for (int s = 0; s < 4 * CB; ++s) wv[s] = Wg[(long)min(4 * s + lg, C - 1) * H + jc];
  // the old values of this thread's outputs of the update
  float wo[CB];
#pragma unroll
  for (int u = 0; u < CB; ++u) {
    const int cc = (tid >> 5) + 16 * u, jo = blockIdx.x * HCOLS + (tid & 31);
    wo[u] = Wg[(long)min(cc, C - 1) * H + min(jo, H - 1)];
  }
  // (all loads before the first store: none waits for another's value)
  const int rows = (N + 31) / 32 * 32, n = rows * 16 * CB;
  float dv[4 * CB];
#pragma unroll
  for (int u = 0; u < 4 * CB; ++u)
    if (512 * u < n) {  // (uniform)
      const int i = tid + 512 * u, r = i / (16 * CB), c = i % (16 * CB);
      dv[u] = dl[(long)min(r, N - 1) * C + min(c, C - 1)];
    }
#pragma unroll
  for (int u = 0; u < 4 * CB; ++u) {
    const int i = tid + 512 * u, r = i / (16 * CB), c = i % (16 * CB);
    if (i < n) sD[r * DP + c] = r < N && c < C ? dv[u] : 0.f;
  }
  __syncthreads();
  floatx4 aw[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) aw[cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
  if (r0 < N) {  // (uniform)
    floatx4 ad[2];
    ad[0] = ad[1] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int r = r0 + 16 * (s / 4) + 4 * lg + s % 4;
      const float fv = r < N ? f[s] : 0.f;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) aw[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(sD[r * DP + 16 * cb + lr_], fv, aw[cb], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < 4 * CB; ++s) {
      const float v = 4 * s + lg < C ? wv[s] : 0.f;
#pragma unroll
      for (int bl = 0; bl < 2; ++bl)
        ad[bl] = __builtin_amdgcn_mfma_f32_16x16x4f32(sD[(r0 + 16 * bl + lr_) * DP + 4 * s + lg], v, ad[bl], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int r = r0 + 16 * (s / 4) + 4 * lg + s % 4;
      // the features are the output of a ReLU layer: the gradient passes where the feature is positive
      const float v = relu_mask && !(f[s] > 0.f) ? 0.f : ad[s / 4][s % 4];
      if (r < N && j < H) dfeat[g * s_dfeat + (long)r * H + j] = v;
    }
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[rq][16 * cb + 4 * lg + v][16 * (w & 1) + lr_] = aw[cb][v];
  __syncthreads();
  {
    const int jl = tid & 31, jo = blockIdx.x * HCOLS + jl;
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int c = (tid >> 5) + 16 * u;
      const float dw = (red[0][c][jl] + red[1][c][jl]) + (red[2][c][jl] + red[3][c][jl]);
      if (c < C && jo < H) W_out[g * s_out + (long)c * H + jo] = commit ? wo[u] - lr * dw : dw;
    }
  }
  if (blockIdx.x == 0) {  // bias gradient (a wave per class) and mean loss: lane l has rows l and l + 64
    for (int c = w; c < C; c += 8) {
      float a = (lane < rows ? sD[lane * DP + c] : 0.f) + (lane + 64 < rows ? sD[(lane + 64) * DP + c] : 0.f);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
      if (lane == 0) b_out[g * s_out + c] = commit ? b_in[g * s_in + c] - lr * a : a;
    }
    if (w == 7 && loss) {
      const float* rl = rowloss + g * s_rowloss;
      float a = (lane < N ? rl[min(lane, N - 1)] : 0.f) + (lane + 64 < N ? rl[min(lane + 64, N - 1)] : 0.f);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
      if (lane == 0) loss[g] = a / (float)N;
    }
  }
}

// Both launches as one for up to 32 rows: a workgroup has 128 feature columns and makes the logit gradients, which are
// little work for so few rows, for itself.  The sums of the two launches in their order (a step in place takes those where
// a worker has more than one workgroup: they would read weights that another has already updated).
// N = 4, C = 10, H = 32, 2 workers 2.5 + 3.7 us in two launches, 5.2 in one;
// N = 20, C = 7, H = 100, 4 workers 4.5 + 4.6, 7.0 in one.  A round of an MLP 320-33-790-23, batch 20, 2 workers 66 -> 45 us, of
// the first 41 -> 36 (with its bias gradients in the launch of its weight gradients).
template <int CB>
__global__ void __launch_bounds__(512)
cls_head_one_kernel(const float* __restrict__ feats, long s_feats, const float* W_in, const float* b_in, long s_in,
                    const int32_t* __restrict__ y, long s_y, float* __restrict__ dfeat, long s_dfeat, float* W_out, float* b_out,
                    long s_out, float lr, int commit, float* __restrict__ loss, int N, int C, int H, int relu_mask) {
  constexpr int DP = 16 * CB + 1;
  __shared__ float red[8][32][DP];  // the logits' sums per wave
  __shared__ float sD[32 * DP];     // dlogits, zeros beyond N and C
  __shared__ float sL[32];
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr_ = lane & 15, lg = lane >> 4;
  const int nb = (N + 15) / 16;  // blocks of rows, 1 or 2
  const float* Wg = W_in + g * s_in;
  const float* fg = feats + g * s_feats;
  // what the backward part reads arrives with the forward part's operands
  const int j = blockIdx.x * 128 + 16 * w + lr_, jc = min(j, H - 1);
  float f[8], wv[4 * CB], wo[4 * CB];
#pragma unroll
  for (int s = 0; s < 8; ++s) f[s] = fg[(long)min(16 * (s / 4) + 4 * lg + s % 4, N - 1) * H + jc];
#pragma unroll
  for (int s = 0; s < 4 * CB; ++s) {
    wv[s] = Wg[(long)min(4 * s + lg, C - 1) * H + jc];
    wo[s] = Wg[(long)min(16 * (s / 4) + 4 * lg + s % 4, C - 1) * H + jc];
  }
  const int c = tid & 31;
  const float bias = b_in[g * s_in + min(c, C - 1)];
  const float* fr[2];
  const float* wr[CB];
#pragma unroll
  for (int bl = 0; bl < 2; ++bl) fr[bl] = fg + (long)min(16 * bl + lr_, N - 1) * H;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) wr[cb] = Wg + (long)min(16 * cb + lr_, C - 1) * H;
  floatx4 acc[2][CB];
#pragma unroll
  for (int bl = 0; bl < 2; ++bl)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[bl][cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
  const int nc = (H + 15) / 16;
  for (int i = w; i < nc; i += 16) {  // two chunks at a time
    floatx4 a[2][2], v[2][CB];
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (i + 8 * u < nc) {  // (uniform)
        const int k = 16 * (i + 8 * u) + 4 * lg;
#pragma unroll
        for (int bl = 0; bl < 2; ++bl)
          if (bl < nb) a[u][bl] = row4(fr[bl], k, H);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) v[u][cb] = row4(wr[cb], k, H);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (i + 8 * u < nc) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int bl = 0; bl < 2; ++bl)
            if (bl < nb) {
#pragma unroll
              for (int cb = 0; cb < CB; ++cb)
                acc[bl][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][bl][e], v[u][cb][e], acc[bl][cb], 0, 0, 0);
            }
      }
  }
#pragma unroll
  for (int bl = 0; bl < 2; ++bl)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[w][16 * bl + 4 * lg + v][16 * cb + lr_] = acc[bl][cb][v];
  __syncthreads();
#pragma unroll
  for (int bl = 0; bl < 2; ++bl) {
    const int row = 16 * bl + (tid >> 5);
    const bool ok = c < C;
    float d = 0.f;
    if (row < N) {  // (the 32 threads of a row together)
      const int label = y[g * s_y + row];
      float z = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) z += red[i][row][min(c, 16 * CB - 1)];
      z = ok ? z + bias : -INFINITY;
      float m = z;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 32));
      const float zl = __shfl(z, label & 31, 32);
      const float ez = ok ? expf(z - m) : 0.f;
      float sum = ez;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 32);
      const float inv_sum = 1.0f / sum, inv_n = 1.0f / (float)N;
      if (c == 0) sL[row] = -(((label >= 0 && label < C ? zl : 0.f) - m) - logf(sum));
      if (ok) d = (ez * inv_sum - (c == label ? 1.0f : 0.0f)) * inv_n;
    }
    if (c < 16 * CB) sD[row * DP + c] = d;
  }
  __syncthreads();
  floatx4 aw[CB], ad[2];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) aw[cb] = (floatx4){0.f, 0.f, 0.f, 0.f};
  ad[0] = ad[1] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int r = 16 * (s / 4) + 4 * lg + s % 4;
    const float fv = r < N ? f[s] : 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) aw[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(sD[r * DP + 16 * cb + lr_], fv, aw[cb], 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < 4 * CB; ++s) {
    const float v = 4 * s + lg < C ? wv[s] : 0.f;
#pragma unroll
    for (int bl = 0; bl < 2; ++bl)
      ad[bl] = __builtin_amdgcn_mfma_f32_16x16x4f32(sD[(16 * bl + lr_) * DP + 4 * s + lg], v, ad[bl], 0, 0, 0);
  }
  if (j < H) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int r = 16 * (s / 4) + 4 * lg + s % 4;
      const float v = relu_mask && !(f[s] > 0.f) ? 0.f : ad[s / 4][s % 4];
      if (r < N) dfeat[g * s_dfeat + (long)r * H + j] = v;
    }
#pragma unroll
    for (int s = 0; s < 4 * CB; ++s) {
      const int cc = 16 * (s / 4) + 4 * lg + s % 4;
      const float dw = aw[s / 4][s % 4];
      if (cc < C) W_out[g * s_out + (long)cc * H + j] = commit ? wo[s] - lr * dw : dw;
    }
  }
  if (blockIdx.x == 0) {  // bias gradient (a wave per class) and mean loss: lane l has row l
    for (int cc = w; cc < C; cc += 8) {
      float a = lane < 32 ? sD[(lane & 31) * DP + cc] : 0.f;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
      if (lane == 0) b_out[g * s_out + cc] = commit ? b_in[g * s_in + cc] - lr * a : a;
    }
    if (w == 7 && loss) {
      float a = lane < N ? sL[lane & 31] : 0.f;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
      if (lane == 0) loss[g] = a / (float)N;
    }
  }
}

}  // namespace

// (any H: against the general products, softmax and sums a local step of an MLP of two layers, 128 rows, one worker, takes
// H = 1536, 32 classes 35 -> 28 us; H = 4096, 32 classes 57 -> 44; H = 8192, 10 classes 84 -> 50, and nothing that was tried from 1028 to 12288 longer)
bool cls_head_supported(int N, int C, int H) { return N >= 1 && N <= HMAXN && C >= 2 && C <= HMAXC && H >= 1; }

// feats: [groups][N][H] (stride s_feats); W_in / b_in: the head's parameters in the input replicas
// (stride s_in); dlog ([N][C] per group, stride s_dlog) and rowloss ([N] per group) are scratch
// that the first launch hands to the second (not written by one launch); dfeat: [N][H] per group (stride s_dfeat);
// commit != 0: W_out / b_out (stride s_out, may be W_in / b_in) receive the updated parameters,
// else the gradients; loss: per group mean cross-entropy, or nullptr.  relu_mask != 0: the features
// are the output of a ReLU layer and dfeat is the gradient in front of that ReLU (zero where the
// feature is not positive).
hipError_t launch_cls_head(const float* feats, long s_feats, const float* W_in, const float* b_in, long s_in,
                           const int32_t* y, long s_y, float* dlog, long s_dlog, float* rowloss, long s_rowloss,
                           float* dfeat, long s_dfeat, float* W_out, float* b_out, long s_out, float lr, int commit,
                           float* loss, int N, int C, int H, int groups, hipStream_t s, int relu_mask) {
  if (!cls_head_supported(N, C, H)) return hipErrorInvalidValue;
  // One launch up to the width where its logits, which every workgroup makes for itself over all features, cost more than a
  // launch.  A whole local step (an MLP of two layers), time in two launches over time in one, with 1, 4 and 16 workers:
  //   16 rows, 10 classes   H = 512  1.01 1.06 1.11   1024  0.96 1.05 1.00   2048  0.89 0.90 0.94
  //   32 rows, 10 classes   H = 256  1.01 1.02 1.09   384   0.98 0.97 1.00   512   0.96 0.98 0.96   1024  0.84 0.84 0.87
  //   32 rows, 32 classes   H = 640  1.05 1.03 1.05   768   0.98 1.02 1.02   1024  0.99 0.94 0.95
  const int one_to = N <= 16 ? 1024 : C <= 16 ? 384 : 768;
  if (N <= 32 && H <= one_to && (H <= 128 || !commit || W_out != W_in)) {
    auto one = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((H + 127) / 128, groups), dim3(512), 0, s, feats, s_feats, W_in, b_in, s_in, y, s_y, dfeat, s_dfeat,
                         W_out, b_out, s_out, lr, commit, loss, N, C, H, relu_mask);
    };
    if (C <= 16) one(cls_head_one_kernel<1>);
    else one(cls_head_one_kernel<2>);
    return hipGetLastError();
  }
  auto launch = [&](auto fwd, auto bwd) {
    hipLaunchKernelGGL(fwd, dim3((N + HROWS - 1) / HROWS, groups), dim3(512), 0, s, feats, s_feats, W_in, b_in, s_in, y, s_y, dlog,
                       s_dlog, rowloss, s_rowloss, N, C, H);
    hipLaunchKernelGGL(bwd, dim3((H + HCOLS - 1) / HCOLS, groups), dim3(512), 0, s, feats, s_feats, W_in, b_in, s_in, dlog, s_dlog,
                       rowloss, s_rowloss, dfeat, s_dfeat, W_out, b_out, s_out, lr, commit, loss, N, C, H, relu_mask);
  };
  if (C <= 16) launch(cls_head_fwd_kernel<1>, cls_head_bwd_kernel<1>);
  else launch(cls_head_fwd_kernel<2>, cls_head_bwd_kernel<2>);
  return hipGetLastError();
}

}  // namespace hpsgd
