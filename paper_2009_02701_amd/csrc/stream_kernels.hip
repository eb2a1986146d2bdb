// HBM-streaming kernels over flat fp32 parameter buffers: replica merge (Eq. 1), replica
// sync (Alg. 2 "make replica"), SGD commit (Alg. 2 "update replica"), zero fill and the
// time-major batch gather.  All work on 16-byte vectors: every lane keeps K+2 independent
// loads in flight and every wave reads and writes 1 KiB contiguous per stream.  They are launched
// with a grid as long as the buffer: on this chip
// that measured 10-20% faster than a resident grid-stride grid, and the merge's operands,
// each touched exactly once, are read and written with non-temporal hints.
#include "kernels.h"

namespace hpsgd {

static constexpr int kThreads = 256;
static constexpr int kMaxBlocks = 256 * 8;  // 256 CUs, up to 8 resident blocks each

// one 256-lane workgroup per 256 vectors (the kernels still stride, should the cap bind)
static inline int onepass_blocks(size_t n_items) {
  size_t b = (n_items + kThreads - 1) / kThreads;
  if (b > (size_t)1 << 30) b = (size_t)1 << 30;
  if (b < 1) b = 1;
  return (int)b;
}

typedef float f4v __attribute__((ext_vector_type(4)));

static inline int stream_blocks(size_t n_items) {
  size_t b = (n_items + kThreads - 1) / kThreads;
  if (b > (size_t)kMaxBlocks) b = kMaxBlocks;
  if (b < 1) b = 1;
  return (int)b;
}

// The merges and the clone below are bound by HBM: 5.5 TB/s where as much is written as read, up to 6.4 where most of it
// is read.  What is left to choose is how many buffers are in flight at a time: V, the vectors of 256 lanes per
// workgroup and buffer (4 KB x V contiguous), and UN, how far the loop over the replicas is unrolled (0: as far as the
// compiler will), or KT > 0, their number, known when compiled.  Short runs of many buffers at once cost more in HBM than they hide once there are enough
// workgroups; a small model wants everything requested at once.  Measured (us, one vector and all replicas at
// once -> what is taken; replicas x parameters):
//   merge          8 x 100M 752 -> 688, 12 x 50M 523 -> 455, 5 x 45M 244 -> 229, 16 x 20M 255 -> 230 (UN 2, V 4);
//                  4 x 9M 41 (42.7), 7 x 7.5M 47.5 (52.8), 5 x 1M 8.5 (11.5) stay: the line is at 16M
//                  (one replica keeps one vector: 90M 227 against 232, 60M 151 against 155)
//   sync           8 x 100M 755 -> 722, 12 x 50M 602 -> 525, 5 x 45M 233 -> 224, 4 x 3M 12.0 -> 12.1 (UN 1, V 1)
//   merge + clone  8 x 100M 1505 -> 1454, 5 x 45M 475 -> 439, 4 x 9M 82 -> 74, 5 x 1M 9.4 -> 8.4 (UN 4, V 2)
//   merge + snapshot  8 x 100M 825 -> 779, 12 x 50M 588 -> 496, 5 x 45M 281 -> 259 (UN 2, V 4, from 16M on;
//                  two or three replicas keep one vector: 2 x 24M 92 against 96, 2 x 90M 341 against 357, 3 x 90M 407 against 417)
// Where one vector and all replicas at once stays, K known when compiled is the shortest form (merge + snapshot,
// 5 x 1M: 7.1 -> 6.5, 12 x 800k 10.3 -> 9.2, 5 x 2.2M 13.4 -> 11.6; merge, 5 x 2.2M 11.9 -> 9.9; merge + clone,
// 6 x 600k 8.3 -> 7.1), with two exceptions where K is no power of two, that is, for loops that the compiler unrolls no
// further than eight replicas: merge + clone from 32 MB of buffers on (6 x 1.2M 12.5 known, 11.8 not, 7 x 1.6M 20.2 and
// 17.3, 12 x 1.2M 24.2 and 22.6; 5 x 900k 7.1 and 7.8), and the merge of gradients from 4M parameters on (6 x 13M 68.6
// and 66.4, 5 x 5M 22.5 and 21.7; 6 x 2.2M 10.1 and 12.4, 5 x 3M 12.3 and 13.3).  The latter reads one buffer less and
// from 16M on never wants K known (8 x 100M 687 and 649, 4 x 60M 235 and 229; below, 8 x 4.5M 27.9 and 30.1,
// 16 x 9M 103 and 108).
static constexpr size_t kManyVectors = (size_t)1 << 22, kFewVectors = (size_t)1 << 19;

static inline bool power_of_two(int K) { return (K & (K - 1)) == 0; }

#define HPSGD_K_CASES(M)                                                                          \
  switch (K) {                                                                                    \
    case 1: M(1); break;   case 2: M(2); break;   case 3: M(3); break;   case 4: M(4); break;     \
    case 5: M(5); break;   case 6: M(6); break;   case 7: M(7); break;   case 8: M(8); break;     \
    case 9: M(9); break;   case 10: M(10); break; case 11: M(11); break; case 12: M(12); break;   \
    case 13: M(13); break; case 14: M(14); break; case 15: M(15); break; case 16: M(16); break;   \
    default: M(0); break;                                                                         \
  }

// V vectors of a lane, kThreads apart; one beyond the buffer is read as the first and not written
template <int V>
struct Vectors {
  size_t i[V];
  __device__ __forceinline__ Vectors(size_t i0, size_t n4) {
#pragma unroll
    for (int v = 0; v < V; ++v) i[v] = i0 + v * kThreads < n4 ? i0 + v * kThreads : i0;
  }
  __device__ __forceinline__ bool in(int v) const { return v == 0 || i[v] != i[0]; }
  __device__ __forceinline__ void load(f4v (&x)[V], const float* p) const {
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(p) + i[v]);
  }
  __device__ __forceinline__ void store(const f4v (&x)[V], float* p) const {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (in(v)) __builtin_nontemporal_store(x[v], reinterpret_cast<f4v*>(p) + i[v]);
  }
  // x += replica - snapshot
  __device__ __forceinline__ void add_diff(f4v (&x)[V], const float* p, const f4v (&sn)[V]) const {
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] += __builtin_nontemporal_load(reinterpret_cast<const f4v*>(p) + i[v]) - sn[v];
  }
};
template <int KT, int UN, typename F>
__device__ __forceinline__ void each_replica(int K, F f) {
  if (KT > 0) {
#pragma unroll
    for (int k = 0; k < KT; ++k) f(k);
  } else if (UN > 0) {
#pragma unroll UN
    for (int k = 0; k < K; ++k) f(k);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) f(k);
  }
}

// ---------------------------------------------------------------------------- merge
// global[j] += (1/K) * sum_k (replica_k[j] - snapshot[j]); the sum over k runs in order.
template <int KT, int UN, int V>
__global__ void __launch_bounds__(kThreads)
merge_kernel(float* global, PtrPack rep, const float* snapshot, int K, float inv_k, size_t n4, size_t P) {
  const size_t stride = (size_t)gridDim.x * kThreads * V;
  for (size_t i = (size_t)blockIdx.x * kThreads * V + threadIdx.x; i < n4; i += stride) {
    const Vectors<V> at(i, n4);
    f4v sn[V], g[V], acc[V];
    at.load(sn, snapshot);
    at.load(g, global);
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = (f4v){0.f, 0.f, 0.f, 0.f};
    each_replica<KT, UN>(K, [&](int k) { at.add_diff(acc, rep.p[k], sn); });
#pragma unroll
    for (int v = 0; v < V; ++v) g[v] += acc[v] * inv_k;
    at.store(g, global);
  }
  // ragged tail (P not a multiple of 4): the first block's first lanes
  if (blockIdx.x == 0) {
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < P) {
      const float s = snapshot[j];
      float acc = 0.f;
      for (int k = 0; k < K; ++k) acc += rep.p[k][j] - s;
      global[j] = global[j] + acc * inv_k;
    }
  }
}

hipError_t launch_merge(float* global, const PtrPack& replicas, const float* snapshot, int K,
                        size_t P, hipStream_t s) {
  if (P == 0) return hipSuccess;
  const size_t n4 = P / 4;
  const float inv_k = 1.0f / (float)K;
#define HPSGD_MERGE(KT, UN, V)                                                                                       \
  hipLaunchKernelGGL((merge_kernel<KT, UN, V>), dim3(onepass_blocks((n4 + V - 1) / V)), dim3(kThreads), 0, s, global, replicas, \
                     snapshot, K, inv_k, n4, P)
#define HPSGD_MERGE_FEW(KT) HPSGD_MERGE(KT, 0, 1)
  if (n4 >= kManyVectors && K > 1) HPSGD_MERGE(0, 2, 4);
  else HPSGD_K_CASES(HPSGD_MERGE_FEW)
#undef HPSGD_MERGE_FEW
#undef HPSGD_MERGE
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- sync
__global__ void __launch_bounds__(kThreads)
sync_kernel(const float* __restrict__ global, PtrPack rep, int K, float* snapshot, size_t n4, size_t P) {
  const size_t stride = (size_t)gridDim.x * kThreads;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += stride) {
    const float4 g = reinterpret_cast<const float4*>(global)[i];
    each_replica<0, 1>(K, [&](int k) { reinterpret_cast<float4*>(rep.p[k])[i] = g; });
    if (snapshot) reinterpret_cast<float4*>(snapshot)[i] = g;
  }
  if (blockIdx.x == 0) {
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < P) {
      const float g = global[j];
      for (int k = 0; k < K; ++k) rep.p[k][j] = g;
      if (snapshot) snapshot[j] = g;
    }
  }
}

hipError_t launch_sync_all(const float* global, const PtrPack& replicas, int K, float* snapshot,
                           size_t P, hipStream_t s) {
  if (P == 0) return hipSuccess;
  const size_t n4 = P / 4;
  hipLaunchKernelGGL(sync_kernel, dim3(onepass_blocks(n4)), dim3(kThreads), 0, s, global, replicas, K, snapshot, n4, P);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- merge + sync in one pass
// global[j] += (1/K) * sum_k (replica_k[j] - snapshot[j]), then replica_k[j] = snapshot[j] = global[j]:
// what merge_kernel followed by sync_kernel leaves, with every buffer read once and written once
// (4 (2K + 4) bytes per parameter instead of 4 (2K + 5)).  A lane reads its elements of all K + 2
// buffers before it writes any of them, so the update in place is safe.
// CLONE = false: the replicas are only read (the snapshot alone is taken: 4 (K + 4) bytes per
// parameter, against 4 (K + 3) + 8 for the merge followed by a copy of its result).
template <bool CLONE, int KT, int UN, int V>
__global__ void __launch_bounds__(kThreads)
merge_sync_kernel(float* global, PtrPack rep, float* snapshot, int K, float inv_k, size_t n4, size_t P) {
  const size_t stride = (size_t)gridDim.x * kThreads * V;
  for (size_t i = (size_t)blockIdx.x * kThreads * V + threadIdx.x; i < n4; i += stride) {
    const Vectors<V> at(i, n4);
    f4v sn[V], g[V], acc[V];
    at.load(sn, snapshot);
    at.load(g, global);
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = (f4v){0.f, 0.f, 0.f, 0.f};
    each_replica<KT, UN>(K, [&](int k) { at.add_diff(acc, rep.p[k], sn); });
#pragma unroll
    for (int v = 0; v < V; ++v) g[v] += acc[v] * inv_k;
    at.store(g, global);
    if (CLONE) each_replica<KT, UN>(K, [&](int k) { at.store(g, rep.p[k]); });
    at.store(g, snapshot);
  }
  if (blockIdx.x == 0) {
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < P) {
      const float s = snapshot[j];
      float acc = 0.f;
      for (int k = 0; k < K; ++k) acc += rep.p[k][j] - s;
      const float o = global[j] + acc * inv_k;
      global[j] = o;
      if (CLONE)
        for (int k = 0; k < K; ++k) rep.p[k][j] = o;
      snapshot[j] = o;
    }
  }
}

hipError_t launch_merge_sync(float* global, const PtrPack& replicas, float* snapshot, int K, size_t P,
                             hipStream_t s, bool clone) {
  if (P == 0) return hipSuccess;
  const size_t n4 = P / 4;
  const float inv_k = 1.0f / (float)K;
#define HPSGD_MS(CL, KT, UN, V)                                                                                         \
  hipLaunchKernelGGL((merge_sync_kernel<CL, KT, UN, V>), dim3(onepass_blocks((n4 + V - 1) / V)), dim3(kThreads), 0, s, global, \
                     replicas, snapshot, K, inv_k, n4, P)
#define HPSGD_MS_CLONE_FEW(KT) HPSGD_MS(true, KT, 0, 1)
#define HPSGD_MS_SNAP_FEW(KT) HPSGD_MS(false, KT, 0, 1)
  if (clone) {
    if (n4 >= kFewVectors) HPSGD_MS(true, 0, 4, 2);
    else if (!power_of_two(K) && (K + 2) * n4 >= (size_t)1 << 21) HPSGD_MS(true, 0, 0, 1);
    else HPSGD_K_CASES(HPSGD_MS_CLONE_FEW)
  } else {
    if (n4 >= kManyVectors && K != 2 && K != 3) HPSGD_MS(false, 0, 2, 4);
    else HPSGD_K_CASES(HPSGD_MS_SNAP_FEW)
  }
#undef HPSGD_MS_SNAP_FEW
#undef HPSGD_MS_CLONE_FEW
#undef HPSGD_MS
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- commit
// out[k][j] = in[k][j] - lr * grad[k][j]  (in_stride 0: every worker starts from the one model `in`)
__global__ void __launch_bounds__(kThreads)
commit_kernel(const float* in, size_t in_stride, float* out, size_t stride, const float* __restrict__ grad,
              size_t grad_stride, float lr, size_t n4, size_t P) {
  const int k = blockIdx.y;
  const float* ink = in + (size_t)k * in_stride;
  float* outk = out + (size_t)k * stride;
  const float* gk = grad + (size_t)k * grad_stride;
  const size_t step = (size_t)gridDim.x * kThreads;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += step) {
    const float4 w = reinterpret_cast<const float4*>(ink)[i];
    const float4 g = reinterpret_cast<const float4*>(gk)[i];
    float4 o;
    o.x = w.x - lr * g.x;
    o.y = w.y - lr * g.y;
    o.z = w.z - lr * g.z;
    o.w = w.w - lr * g.w;
    reinterpret_cast<float4*>(outk)[i] = o;
  }
  if (blockIdx.x == 0) {
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < P) outk[j] = ink[j] - lr * gk[j];
  }
}

// Several ranges of the flat buffers in one launch (a dependent launch costs 4.5 us however little it
// does); segment i owns the grid columns blk0[i] .. blk0[i+1]-1.  Buffers and strides are 16-byte
// aligned, a range may start anywhere: its head and tail elements go one per thread.
__global__ void __launch_bounds__(kThreads)
commit_multi_kernel(CommitPack pk, const float* in, size_t in_stride, float* out, size_t stride,
                    const float* __restrict__ grad, size_t grad_stride, float lr) {
  int sgi = 0;
#pragma unroll
  for (int i = 1; i < CommitPack::MAXSEG; ++i)
    if (i < pk.n_seg && blockIdx.x >= pk.blk0[i]) sgi = i;
  const size_t k = blockIdx.y, lo = pk.lo[sgi], n = pk.n[sgi];
  const float* ink = in + k * in_stride + lo;
  float* outk = out + k * stride + lo;
  const float* gk = grad + k * grad_stride + lo;
  const unsigned b0 = blockIdx.x - pk.blk0[sgi], nblk = pk.blk0[sgi + 1] - pk.blk0[sgi];
  const size_t head = min((size_t)((4 - (lo & 3)) & 3), n), n4 = (n - head) / 4;
  const float4* in4 = reinterpret_cast<const float4*>(ink + head);
  const float4* g4 = reinterpret_cast<const float4*>(gk + head);
  for (size_t i = (size_t)b0 * kThreads + threadIdx.x; i < n4; i += (size_t)nblk * kThreads) {
    const float4 w = in4[i], g = g4[i];
    reinterpret_cast<float4*>(outk + head)[i] = make_float4(w.x - lr * g.x, w.y - lr * g.y, w.z - lr * g.z, w.w - lr * g.w);
  }
  if (b0 == 0) {
    if (threadIdx.x < head) outk[threadIdx.x] = ink[threadIdx.x] - lr * gk[threadIdx.x];
    const size_t j = head + 4 * n4 + threadIdx.x;
    if (j < n) outk[j] = ink[j] - lr * gk[j];
  }
}

// the same, one element per thread: for buffers that are not 16-byte aligned
__global__ void __launch_bounds__(kThreads)
commit_scalar_kernel(const float* in, size_t in_stride, float* out, size_t stride, const float* __restrict__ grad,
                     size_t grad_stride, float lr, size_t P) {
  const size_t k = blockIdx.y;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < P; i += (size_t)gridDim.x * kThreads)
    out[k * stride + i] = in[k * in_stride + i] - lr * grad[k * grad_stride + i];
}

bool commit_pack_push(CommitPack& pk, size_t lo, size_t n) {
  if (pk.n_seg >= CommitPack::MAXSEG || n == 0) return false;
  pk.lo[pk.n_seg] = lo;
  pk.n[pk.n_seg] = n;
  pk.blk0[pk.n_seg + 1] = (pk.n_seg ? pk.blk0[pk.n_seg] : 0u) + (unsigned)onepass_blocks(n / 4);
  if (pk.n_seg == 0) pk.blk0[0] = 0;
  ++pk.n_seg;
  return true;
}

hipError_t launch_commit_pack(const CommitPack& pk, const float* in, size_t in_stride, float* out, size_t stride,
                              const float* grad, size_t grad_stride, float lr, int K, hipStream_t s) {
  if (pk.n_seg == 0 || K <= 0) return hipSuccess;
  size_t total = 0;
  for (int i = 0; i < pk.n_seg; ++i) total += pk.n[i];
  KernelTimer kt(KID_COMMIT, 12.0 * (double)total * K, s);
  if ((((uintptr_t)in | (uintptr_t)out | (uintptr_t)grad) & 15) != 0 || ((in_stride | stride | grad_stride) & 3) != 0) {
    for (int i = 0; i < pk.n_seg; ++i) {
      size_t blocks = (pk.n[i] + kThreads - 1) / kThreads;
      if (blocks > 1024) blocks = 1024;
      hipLaunchKernelGGL(commit_scalar_kernel, dim3((unsigned)blocks, K), dim3(kThreads), 0, s, in + pk.lo[i], in_stride,
                         out + pk.lo[i], stride, grad + pk.lo[i], grad_stride, lr, pk.n[i]);
    }
    return hipGetLastError();
  }
  if (pk.n_seg == 1 && (pk.lo[0] & 3) == 0) {
    const size_t lo = pk.lo[0], n4 = pk.n[0] / 4;
    hipLaunchKernelGGL(commit_kernel, dim3(onepass_blocks(n4), K), dim3(kThreads), 0, s, in + lo, in_stride, out + lo, stride,
                       grad + lo, grad_stride, lr, n4, pk.n[0]);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(commit_multi_kernel, dim3(pk.blk0[pk.n_seg], K), dim3(kThreads), 0, s, pk, in, in_stride, out, stride,
                     grad, grad_stride, lr);
  return hipGetLastError();
}

// sum + p[n4] + p[2 n4] + .. + p[(n_parts-1) n4], added in that order; the loads of 16 parts are in
// flight together (with one load per trip a sum over 140 parts waits out 140 memory latencies)
__device__ __forceinline__ float4 add_parts_in_order(const float4* p, size_t n4, int n_parts, float4 sum) {
  int q = 1;
  for (; q + 16 <= n_parts; q += 16) {
    float4 v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(size_t)(q + u) * n4];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      sum.x += v[u].x;
      sum.y += v[u].y;
      sum.z += v[u].z;
      sum.w += v[u].w;
    }
  }
  for (; q < n_parts; ++q) {
    const float4 v = p[(size_t)q * n4];
    sum.x += v.x;
    sum.y += v.y;
    sum.z += v.z;
    sum.w += v.w;
  }
  return sum;
}

// Partial sums of a weight gradient (one per batch-row tile of the recurrence kernel), added in
// tile order, then either committed (out = in - lr * sum) or stored (out = sum).  n % 4 == 0.
__global__ void __launch_bounds__(kThreads)
reduce_parts_kernel(const float* __restrict__ parts, int n_parts, size_t n4, const float* in, size_t s_in,
                    float* out, size_t s_out, float lr, int commit) {
  const size_t k = blockIdx.y;
  const float4* pk = reinterpret_cast<const float4*>(parts) + k * n_parts * n4;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += (size_t)gridDim.x * kThreads) {
    const float4 sum0 = pk[i];
    float4 sum = add_parts_in_order(pk + i, n4, n_parts, sum0);
    if (commit) {
      const float4 w = reinterpret_cast<const float4*>(in + k * s_in)[i];
      sum = make_float4(w.x - lr * sum.x, w.y - lr * sum.y, w.z - lr * sum.z, w.w - lr * sum.w);
    }
    reinterpret_cast<float4*>(out + k * s_out)[i] = sum;
  }
}

// Several such sums in one launch (each of these kernels is a few microseconds of work behind
// a launch): segment i owns the grid columns blk0[i] .. blk0[i+1]-1.  A segment whose length or buffers
// are not in whole 16-byte words is added one element per thread.
__global__ void __launch_bounds__(kThreads) reduce_parts_multi_kernel(ReducePack pk) {
  if (pk.rowloss && blockIdx.x == gridDim.x - 1) {  // the mean loss, in a fixed order
    __shared__ float red[kThreads];
    const int tid = threadIdx.x;
    float v = 0.f;
    for (int i = tid; i < pk.rows; i += kThreads) v += pk.rowloss[blockIdx.y * pk.s_rowloss + i];
    red[tid] = v;
    __syncthreads();
    for (int o = kThreads / 2; o > 0; o >>= 1) {
      if (tid < o) red[tid] += red[tid + o];
      __syncthreads();
    }
    if (tid == 0) pk.loss[blockIdx.y] = red[0] / (float)pk.count;
    return;
  }
  int sgi = 0;
#pragma unroll
  for (int i = 1; i < ReducePack::MAXSEG; ++i)
    if (i < pk.n && blockIdx.x >= pk.blk0[i]) sgi = i;
  const ReduceSeg& sg = pk.seg[sgi];
  const size_t k = blockIdx.y;
  const unsigned nblk = pk.blk0[sgi + 1] - pk.blk0[sgi];
  const size_t i0 = (size_t)(blockIdx.x - pk.blk0[sgi]) * kThreads + threadIdx.x;
  if (!sg.vec) {
    const float* p = sg.parts + k * sg.n_parts * sg.pitch;
    for (size_t i = i0; i < sg.n; i += (size_t)nblk * kThreads) {
      float sum = p[i];
#pragma unroll 8
      for (int q = 1; q < sg.n_parts; ++q) sum += p[(size_t)q * sg.pitch + i];
      if (sg.commit) sum = sg.in[k * sg.s_in + i] - pk.lr * sum;
      sg.out[k * sg.s_out + i] = sum;
    }
    return;
  }
  const size_t n4 = sg.n / 4, p4 = sg.pitch / 4;
  const float4* pkp = reinterpret_cast<const float4*>(sg.parts) + k * sg.n_parts * p4;
  for (size_t i = i0; i < n4; i += (size_t)nblk * kThreads) {
    const float4 sum0 = pkp[i];
    float4 sum = add_parts_in_order(pkp + i, p4, sg.n_parts, sum0);
    if (sg.commit) {
      const float4 w = reinterpret_cast<const float4*>(sg.in + k * sg.s_in)[i];
      sum = make_float4(w.x - pk.lr * sum.x, w.y - pk.lr * sum.y, w.z - pk.lr * sum.z, w.w - pk.lr * sum.w);
    }
    reinterpret_cast<float4*>(sg.out + k * sg.s_out)[i] = sum;
  }
}

bool reduce_pack_push(ReducePack& pk, const float* parts, int n_parts, size_t n, const float* in, size_t s_in,
                      float* out, size_t s_out, int commit, size_t pitch) {
  if (pk.n >= ReducePack::MAXSEG || n == 0 || n_parts < 1 || (commit && !in)) return false;
  ReduceSeg& sg = pk.seg[pk.n];
  sg.parts = parts; sg.n_parts = n_parts; sg.n = n; sg.in = in; sg.s_in = s_in; sg.out = out; sg.s_out = s_out;
  sg.commit = commit;
  sg.pitch = pitch ? pitch : n;
  sg.vec = ((n | sg.pitch) & 3) == 0 && ((uintptr_t)parts & 15) == 0 && ((uintptr_t)out & 15) == 0 && (s_out & 3) == 0 &&
           (!commit || (((uintptr_t)in & 15) == 0 && (s_in & 3) == 0));
  pk.blk0[pk.n + 1] = pk.blk0[pk.n] + (unsigned)onepass_blocks(sg.vec ? n / 4 : n);
  ++pk.n;
  return true;
}

hipError_t launch_reduce_pack(const ReducePack& pk, int groups, hipStream_t s) {
  const unsigned blocks = pk.blk0[pk.n] + (pk.rowloss ? 1u : 0u);
  if (blocks == 0 || groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_parts_multi_kernel, dim3(blocks, groups), dim3(kThreads), 0, s, pk);
  return hipGetLastError();
}

hipError_t launch_reduce_parts(const float* parts, int n_parts, size_t n, const float* in, size_t s_in,
                               float* out, size_t s_out, float lr, int commit, int groups, hipStream_t s, size_t pitch) {
  if (n == 0 || groups <= 0) return hipSuccess;
  ReducePack pk;
  pk.n = 0;
  pk.blk0[0] = 0;
  pk.lr = lr;
  if (!reduce_pack_push(pk, parts, n_parts, n, in, s_in, out, s_out, commit, pitch)) return hipErrorInvalidValue;
  if (!pk.seg[0].vec || pk.seg[0].pitch != n) return launch_reduce_pack(pk, groups, s);
  const size_t n4 = n / 4;
  const int blocks = onepass_blocks(n4);
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(blocks, groups), dim3(kThreads), 0, s, parts, n_parts, n4, in, s_in,
                     out, s_out, lr, commit);
  return hipGetLastError();
}

// out[k][j] = in[k][j] - lr * grad[k][j];  acc[k][j] += grad[k][j]  (Alg. 2: update the replica and
// accumulate the gradient in one pass, 20 B/param)
__global__ void __launch_bounds__(kThreads)
commit_acc_kernel(const float* in, size_t in_stride, float* out, size_t stride, const float* __restrict__ grad,
                  size_t grad_stride, float* __restrict__ acc, size_t acc_stride, float lr, size_t P) {
  const size_t k = blockIdx.y;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < P; i += (size_t)gridDim.x * kThreads) {
    const float g = grad[k * grad_stride + i];
    out[k * stride + i] = in[k * in_stride + i] - lr * g;
    acc[k * acc_stride + i] += g;
  }
}

// The same on 16-byte vectors, one per lane (all four buffers 16-byte aligned, strides multiples
// of 4): three loads in flight per lane, every wave reads and writes 1 KiB contiguous per stream.
__global__ void __launch_bounds__(kThreads)
commit_acc4_kernel(const float* in, size_t in_stride, float* out, size_t stride, const float* __restrict__ grad,
                   size_t grad_stride, float* __restrict__ acc, size_t acc_stride, float lr, size_t n4, size_t P) {
  const size_t k = blockIdx.y;
  const f4v* in4 = reinterpret_cast<const f4v*>(in + k * in_stride);
  f4v* out4 = reinterpret_cast<f4v*>(out + k * stride);
  const f4v* g4 = reinterpret_cast<const f4v*>(grad + k * grad_stride);
  f4v* a4 = reinterpret_cast<f4v*>(acc + k * acc_stride);
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += (size_t)gridDim.x * kThreads) {
    const f4v g = __builtin_nontemporal_load(g4 + i);
    const f4v w = __builtin_nontemporal_load(in4 + i);
    const f4v a = __builtin_nontemporal_load(a4 + i);
    __builtin_nontemporal_store(w - g * lr, out4 + i);
    __builtin_nontemporal_store(a + g, a4 + i);
  }
  if (blockIdx.x == 0) {  // ragged tail
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < P) {
      const float g = grad[k * grad_stride + j];
      out[k * stride + j] = in[k * in_stride + j] - lr * g;
      acc[k * acc_stride + j] += g;
    }
  }
}

hipError_t launch_commit_acc(const float* in, size_t in_stride, float* out, size_t stride, const float* grad,
                             size_t grad_stride, float* acc, size_t acc_stride, float lr, int K, size_t P, hipStream_t s) {
  if (P == 0) return hipSuccess;
  const bool vec = ((((uintptr_t)in | (uintptr_t)out | (uintptr_t)grad | (uintptr_t)acc) & 15) == 0) &&
                   ((in_stride | stride | grad_stride | acc_stride) & 3) == 0 && P >= 4;
  KernelTimer kt(KID_COMMIT_ACC, 20.0 * (double)P * K, s);
  if (vec) {
    const size_t n4 = P / 4;
    hipLaunchKernelGGL(commit_acc4_kernel, dim3(onepass_blocks(n4), K), dim3(kThreads), 0, s, in, in_stride, out, stride, grad,
                       grad_stride, acc, acc_stride, lr, n4, P);
    return hipGetLastError();
  }
  size_t blocks = (P + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(commit_acc_kernel, dim3((unsigned)blocks, K), dim3(kThreads), 0, s, in, in_stride, out, stride, grad,
                     grad_stride, acc, acc_stride, lr, P);
  return hipGetLastError();
}

// global[j] -= lr * (1/K) * sum_k acc_k[j], the sum in worker order (Eq. 1 as printed)
// (KT: their number, known when compiled, 0: it is not)
template <int KT>
__global__ void __launch_bounds__(kThreads)
merge_grad_kernel(float* global, PtrPack acc, int Krt, float scale, size_t n4, size_t P) {
  const int K = KT > 0 ? KT : Krt;
  const size_t stride = (size_t)gridDim.x * kThreads;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += stride) {
    f4v t = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(acc.p[0]) + i);
#pragma unroll
    for (int k = 1; k < K; ++k) t += __builtin_nontemporal_load(reinterpret_cast<const f4v*>(acc.p[k]) + i);
    const f4v g = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(global) + i);
    __builtin_nontemporal_store(g - t * scale, reinterpret_cast<f4v*>(global) + i);
  }
  if (blockIdx.x == 0) {
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < P) {
      float t = acc.p[0][j];
      for (int k = 1; k < K; ++k) t += acc.p[k][j];
      global[j] = global[j] - t * scale;
    }
  }
}

hipError_t launch_merge_grad(float* global, const PtrPack& accs, float lr, int K, size_t P, hipStream_t s) {
  if (P == 0) return hipSuccess;
  const size_t n4 = P / 4;
  const int blocks = onepass_blocks(n4);
  const float scale = lr / (float)K;
#define HPSGD_MG(KT) hipLaunchKernelGGL(merge_grad_kernel<KT>, dim3(blocks), dim3(kThreads), 0, s, global, accs, K, scale, n4, P)
  if (n4 >= (power_of_two(K) ? kManyVectors : (size_t)1 << 20)) HPSGD_MG(0);
  else HPSGD_K_CASES(HPSGD_MG)
#undef HPSGD_MG
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- fill
// p[g*stride + i] = 0 for i < n, g < groups; grid row `groups`, if launched, clears a second
// range extra[0 .. n_extra) instead
__global__ void __launch_bounds__(kThreads)
fill_zero_kernel(float* p, size_t n4, size_t n, size_t stride, int groups, float* extra, size_t n_extra) {
  float* pg = p + (size_t)blockIdx.y * stride;
  if ((int)blockIdx.y == groups) {
    pg = extra;
    n = n_extra;
    n4 = n_extra / 4;
  }
  const size_t step = (size_t)gridDim.x * kThreads;
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += step)
    reinterpret_cast<float4*>(pg)[i] = z;
  if (blockIdx.x == 0) {
    const size_t j = n4 * 4 + threadIdx.x;
    if (j < n) pg[j] = 0.f;
  }
}

// extra (nullable, 16-byte aligned): a second range of n_extra floats cleared by the same launch
hipError_t launch_fill_zero(float* p, size_t n, size_t stride, int groups, hipStream_t s, float* extra,
                            size_t n_extra) {
  if (n == 0 || groups == 0) {
    if (!extra || n_extra == 0) return hipSuccess;
    return launch_fill_zero(extra, n_extra, n_extra, 1, s, nullptr, 0);
  }
  if (extra && ((uintptr_t)extra & 15) != 0) return hipErrorInvalidValue;
  const size_t n4 = n / 4;
  const size_t big4 = (extra && n_extra / 4 > n4) ? n_extra / 4 : n4;
  int blocks = stream_blocks(big4);
  const int rows = groups + ((extra && n_extra) ? 1 : 0);
  if (blocks * rows > kMaxBlocks) blocks = (kMaxBlocks + rows - 1) / rows;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks, rows), dim3(kThreads), 0, s, p, n4, n, stride, groups, extra,
                     n_extra);
  return hipGetLastError();
}

// Several such clears in one launch (the h_0 slots and flag words a step clears before its first
// layer: each a few microseconds behind a launch); segment i owns grid columns blk0[i] .. blk0[i+1]-1.
// Segment: p[g*stride + r*ld + c] = 0 for r < rows, c < cols, g < its groups.
__global__ void __launch_bounds__(kThreads) fill_zero_multi_kernel(FillPack pk) {
  int sgi = 0;
#pragma unroll
  for (int i = 1; i < FillPack::MAXSEG; ++i)
    if (i < pk.n && blockIdx.x >= pk.blk0[i]) sgi = i;
  const FillSeg& sg = pk.seg[sgi];
  if ((int)blockIdx.y >= sg.groups) return;
  float* pg = sg.p + (size_t)blockIdx.y * sg.stride;
  const long n = (long)sg.rows * sg.cols;
  const unsigned nblk = pk.blk0[sgi + 1] - pk.blk0[sgi];
  for (long i = (long)(blockIdx.x - pk.blk0[sgi]) * kThreads + threadIdx.x; i < n; i += (long)nblk * kThreads)
    pg[(i / sg.cols) * sg.ld + i % sg.cols] = 0.f;
}

bool fill_pack_push(FillPack& pk, float* p, long ld, int rows, long cols, size_t stride, int groups) {
  if (pk.n >= FillPack::MAXSEG || !p || rows <= 0 || cols <= 0 || groups <= 0) return false;
  FillSeg& sg = pk.seg[pk.n];
  sg.p = p; sg.ld = ld; sg.rows = rows; sg.cols = cols; sg.stride = stride; sg.groups = groups;
  const long n = (long)rows * cols;
  long blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 64) blocks = 64;
  pk.blk0[pk.n + 1] = pk.blk0[pk.n] + (unsigned)blocks;
  if (groups > pk.max_groups) pk.max_groups = groups;
  ++pk.n;
  return true;
}

hipError_t launch_fill_pack(const FillPack& pk, hipStream_t s) {
  if (pk.n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_multi_kernel, dim3(pk.blk0[pk.n], pk.max_groups), dim3(kThreads), 0, s, pk);
  return hipGetLastError();
}

// p[g*stride + r*ld + c] = 0 for r < rows, c < cols: a column block of a row-major matrix
__global__ void __launch_bounds__(kThreads)
fill_zero_2d_kernel(float* p, long ld, int rows, int cols, size_t stride) {
  float* pg = p + (size_t)blockIdx.y * stride;
  const long n = (long)rows * cols;
  for (long i = (long)blockIdx.x * kThreads + threadIdx.x; i < n; i += (long)gridDim.x * kThreads)
    pg[(i / cols) * ld + i % cols] = 0.f;
}

hipError_t launch_fill_zero_2d(float* p, long ld, int rows, int cols, size_t stride, int groups,
                               hipStream_t s) {
  if (rows <= 0 || cols <= 0 || groups <= 0) return hipSuccess;
  const long n = (long)rows * cols;
  int blocks = (int)((n + kThreads - 1) / kThreads);
  if (blocks > 256) blocks = 256;
  hipLaunchKernelGGL(fill_zero_2d_kernel, dim3(blocks, groups), dim3(kThreads), 0, s, p, ld, rows, cols, stride);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- delay
// Ends when the 100 MHz wall clock has advanced by `ticks`: the wait is bounded by construction.
__global__ void __launch_bounds__(64) delay_kernel(long long ticks) {
  const long long t0 = wall_clock64();
  while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(32);
}

hipError_t launch_delay(unsigned us, hipStream_t s) {
  if (us == 0) return hipSuccess;
  hipLaunchKernelGGL(delay_kernel, dim3(1), dim3(64), 0, s, (long long)us * 100);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- gather
// out[(c*n_idx + b)*chunk ...] = shard[idx[b]*row + c*chunk ...], in 4-byte words.
__global__ void __launch_bounds__(kThreads)
gather_kernel(const uint32_t* __restrict__ shard, const int32_t* __restrict__ idx, int n_idx,
              size_t row_w, int n_chunks, size_t chunk_w, uint32_t* __restrict__ out) {
  const size_t b = blockIdx.x;           // sample
  const size_t c = blockIdx.y;           // chunk (time step)
  const uint32_t* src = shard + (size_t)idx[b] * row_w + c * chunk_w;
  uint32_t* dst = out + (c * (size_t)n_idx + b) * chunk_w;
  for (size_t w = threadIdx.x; w < chunk_w; w += kThreads) dst[w] = src[w];
}

// The same for K workers and up to two arrays of the same samples in one launch: worker k = blockIdx.y,
// array p the workgroups blk0[p] .. blk0[p+1]-1.  A thread moves one unit of `vec` words (four where rows,
// chunks and buffers are in whole 16-byte pieces): output unit o = (c*n_idx + b)*units + u.
struct GatherArgs {
  static constexpr int MAX = 2;
  const uint32_t* shard[MAX][HPSGD_KMAX];
  uint32_t* out[MAX][HPSGD_KMAX];
  const int32_t* idx[HPSGD_KMAX];
  size_t row_w[MAX];
  unsigned units[MAX], total[MAX], blk0[MAX + 1];  // units of a chunk, of the whole output
  int vec[MAX];
  int n_parts, n_idx;
};

__global__ void __launch_bounds__(kThreads) gather_parts_kernel(GatherArgs a) {
  const int p = a.n_parts > 1 && blockIdx.x >= a.blk0[1] ? 1 : 0, k = blockIdx.y;  // (uniform)
  const unsigned o = (blockIdx.x - a.blk0[p]) * kThreads + threadIdx.x;
  if (o >= a.total[p]) return;
  const unsigned cb = o / a.units[p], u = o - cb * a.units[p];
  const unsigned c = cb / (unsigned)a.n_idx, b = cb - c * (unsigned)a.n_idx;
  const size_t src = (size_t)a.idx[k][b] * a.row_w[p];
  if (a.vec[p] == 4) {
    typedef uint32_t u4g __attribute__((ext_vector_type(4)));
    reinterpret_cast<u4g*>(a.out[p][k])[o] =
        reinterpret_cast<const u4g*>(a.shard[p][k] + src)[(size_t)c * a.units[p] + u];
  } else {
    a.out[p][k][o] = a.shard[p][k][src + (size_t)c * a.units[p] + u];
  }
}

hipError_t launch_gather_parts(const GatherPart* parts, int n_parts, const int32_t* const* idx, int K, int n_idx, hipStream_t s) {
  if (K == 0 || n_idx == 0) return hipSuccess;
  GatherArgs a;
  a.n_parts = 0;
  a.n_idx = n_idx;
  a.blk0[0] = 0;
  for (int k = 0; k < K; ++k) a.idx[k] = idx[k];
  for (int i = 0; i < n_parts; ++i) {
    const GatherPart& q = parts[i];
    if (q.n_chunks == 0 || q.chunk_bytes == 0) continue;
    const int p = a.n_parts++;
    bool v4 = ((q.row_bytes | q.chunk_bytes) & 15) == 0;
    for (int k = 0; k < K; ++k) {
      a.shard[p][k] = (const uint32_t*)q.shards[k];
      a.out[p][k] = (uint32_t*)q.outs[k];
      v4 = v4 && (((uintptr_t)q.shards[k] | (uintptr_t)q.outs[k]) & 15) == 0;
    }
    a.vec[p] = v4 ? 4 : 1;
    a.row_w[p] = q.row_bytes / 4;
    a.units[p] = (unsigned)(q.chunk_bytes / 4 / a.vec[p]);
    const size_t total = (size_t)q.n_chunks * n_idx * (q.chunk_bytes / 4 / a.vec[p]);
    if (total >= (size_t)1 << 31) return hipErrorInvalidValue;  // (the caller checks)
    a.total[p] = (unsigned)total;
    a.blk0[p + 1] = a.blk0[p] + (unsigned)((total + kThreads - 1) / kThreads);
  }
  if (a.n_parts == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_parts_kernel, dim3(a.blk0[a.n_parts], K), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

// An output of 2^31 words or more per worker, which the launch above does not index: one workgroup per chunk.
struct GatherPack {
  const uint32_t* shard[HPSGD_KMAX];
  const int32_t* idx[HPSGD_KMAX];
  uint32_t* out[HPSGD_KMAX];
};

__global__ void __launch_bounds__(kThreads)
gather_all_kernel(GatherPack pk, int n_idx, size_t row_w, size_t chunk_w) {
  const size_t b = blockIdx.x, c = blockIdx.y;
  const int k = blockIdx.z;
  const uint32_t* src = pk.shard[k] + (size_t)pk.idx[k][b] * row_w + c * chunk_w;
  uint32_t* dst = pk.out[k] + (c * (size_t)n_idx + b) * chunk_w;
  for (size_t w = threadIdx.x; w < chunk_w; w += kThreads) dst[w] = src[w];
}

hipError_t launch_gather_all(const void* const* shards, const int32_t* const* idx, int K, int n_idx,
                             size_t row_bytes, int n_chunks, size_t chunk_bytes, void* const* outs,
                             hipStream_t s) {
  if (K == 0 || n_idx == 0 || n_chunks == 0 || chunk_bytes == 0) return hipSuccess;
  if ((size_t)n_chunks * n_idx * (chunk_bytes / 4) < (size_t)1 << 31) {
    const GatherPart part{shards, outs, row_bytes, chunk_bytes, n_chunks};
    return launch_gather_parts(&part, 1, idx, K, n_idx, s);
  }
  GatherPack pk;
  for (int k = 0; k < K; ++k) {
    pk.shard[k] = (const uint32_t*)shards[k];
    pk.idx[k] = idx[k];
    pk.out[k] = (uint32_t*)outs[k];
  }
  hipLaunchKernelGGL(gather_all_kernel, dim3(n_idx, n_chunks, K), dim3(kThreads), 0, s, pk, n_idx,
                     row_bytes / 4, chunk_bytes / 4);
  return hipGetLastError();
}

hipError_t launch_gather(const void* shard, const int32_t* idx, int n_idx, size_t row_bytes,
                         int n_chunks, size_t chunk_bytes, void* out, hipStream_t s) {
  if (n_idx == 0 || n_chunks == 0 || chunk_bytes == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_kernel, dim3(n_idx, n_chunks), dim3(kThreads), 0, s,
                     (const uint32_t*)shard, idx, n_idx, row_bytes / 4, n_chunks, chunk_bytes / 4,
                     (uint32_t*)out);
  return hipGetLastError();
}

}  // namespace hpsgd
