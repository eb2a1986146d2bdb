// Internal launch interface between the C-ABI layer and the HIP kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <atomic>
#include <mutex>

#define HPSGD_KMAX 32

namespace hpsgd {

// Allows kernel fn `lds` bytes of dynamic LDS.  `allowed` (one per kernel): what it may have already; any thread may
// come first, and a smaller amount never replaces a larger one.
inline hipError_t allow_lds(const void* fn, size_t lds, std::atomic<size_t>& allowed) {
  if (lds <= allowed.load(std::memory_order_acquire)) return hipSuccess;
  static std::mutex mu;
  std::lock_guard<std::mutex> lock(mu);
  if (lds <= allowed.load(std::memory_order_relaxed)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess) allowed.store(lds, std::memory_order_release);
  return e;
}

struct PtrPack {  // K device pointers passed by value as a kernel argument
  float* p[HPSGD_KMAX];
};

// ---- per-kernel timing (benchmarks) ----
// The kernels whose launches can be timed one by one (enum hpsgd_kernel in hpsgd.h has the
// same numbering).  A launcher creates a KernelTimer around its launch: when the calling
// thread is inside a local step whose context has that kernel's timing enabled, a HIP event
// pair is recorded on the launch's own stream, together with the launch's algorithmic work
// (flops for the contractions, bytes for the streaming kernels); otherwise it does nothing.
enum KernelId : int {
  KID_NONE = 0,
  KID_GRU_FWD_PERSIST = 1,        // gru_fwd_persist_kernel (fp32, any input-projection form)
  KID_GRU_BWD_PERSIST = 2,        // gru_bwd_persist_kernel
  KID_GRU_FWD_PERSIST_BF16 = 3,   // gru_fwd_persist_bf16_kernel
  KID_GRU_BWD_PERSIST_BF16 = 4,   // gru_bwd_persist_bf16_kernel
  KID_GEMM_BF16_DL = 5,           // gemm_bf16_dl_kernel<false>   (128 x 128)
  KID_GEMM_BF16_DL_COMMIT = 6,    // gemm_bf16_dl_kernel<true>
  KID_GEMM_BF16_DLX128 = 7,       // gemm_bf16_dlx_kernel<false, 2, 4, 2, 2, 3>  (128 x 256)
  KID_GEMM_BF16_DLX128_COMMIT = 8,
  KID_GEMM_BF16_DLX192 = 9,       // gemm_bf16_dlx_kernel<false, 2, 4, 3, 2, 2>  (192 x 256)
  KID_GEMM_BF16_DLX192_COMMIT = 10,  // (also gemm_bf16_dlx_pair_kernel<true, 2, 4, 3, 2, 2>: two such products in one launch)
  KID_GEMM_BF16_DLX256 = 11,      // gemm_bf16_dlx_kernel<false, 2, 4, 4, 2, 2>  (256 x 256)
  KID_GEMM_BF16_DLX256_COMMIT = 12,
  KID_GEMM_BF16_NT = 13,          // gemm_bf16_nt_kernel (an fp32 operand rounded while staged)
  KID_GEMM_F32_FAST = 14,         // gemm_f32_fast, _slim, _direct kernels and their joint launches
  KID_GEMM_F32 = 15,              // gemm_f32_kernel / gemm_bf16_kernel (generic fallbacks)
  KID_CVT2 = 16,                  // cvt2_kernel, embed_bf16_kernel (bf16 copy, transposed copy or both)
  KID_SOFTMAX_CE_BF16 = 17,       // softmax_ce_bf16_rows_kernel / softmax_ce_bf16_kernel
  KID_GRU_STEP = 18,              // gru_{fwd,bwd}_step(_bf16)_kernel: one launch per time step
  KID_COMMIT_ACC = 19,            // commit_acc4_kernel / commit_acc_kernel (update + accumulate, 20 B/param)
  KID_COMMIT = 20,                // commit_kernel (update of what no GEMM epilogue updated, 12 B/param)
  KID_CVT2_PACK = 21,             // cvt2_pack_kernel (the copies of several matrices in one launch)
  KID_COUNT = 22
};
struct KernelTimer {
  // launches: what the launch counts as (the products it holds, where it holds several)
  KernelTimer(int kid, double work, hipStream_t s, int launches = 1);
  ~KernelTimer();
  KernelTimer(const KernelTimer&) = delete;
  KernelTimer& operator=(const KernelTimer&) = delete;
 private:
  void* ctx_;  // the context that holds the open stamp, or nullptr
  int idx_;    // its index there
  hipStream_t s_;
};

// ---- HBM-streaming kernels over flat parameter buffers ----
hipError_t launch_merge(float* global, const PtrPack& replicas, const float* snapshot, int K,
                        size_t P, hipStream_t s);
hipError_t launch_sync_all(const float* global, const PtrPack& replicas, int K, float* snapshot,
                           size_t P, hipStream_t s);
// merge, then sync of the same replicas and snapshot, in one pass
// (clone = false: the replicas are only read, the snapshot alone is taken)
hipError_t launch_merge_sync(float* global, const PtrPack& replicas, float* snapshot, int K, size_t P,
                             hipStream_t s, bool clone = true);
// out[k] = in[k] - lr * grad[k] for K strided slices of P floats (in_stride 0: one model for all)
// for up to MAXSEG ranges [lo, lo + n) of the flat buffers in one launch (16-byte accesses where a range allows them)
struct CommitPack {
  static constexpr int MAXSEG = 16;
  size_t lo[MAXSEG], n[MAXSEG];
  unsigned blk0[MAXSEG + 1];
  int n_seg;
};
bool commit_pack_push(CommitPack& pk, size_t lo, size_t n);
hipError_t launch_commit_pack(const CommitPack& pk, const float* in, size_t in_stride, float* out, size_t stride,
                              const float* grad, size_t grad_stride, float lr, int K, hipStream_t s);
// p[g*stride + i] = 0 for i < n (p 16-byte aligned, stride a multiple of 4)
hipError_t launch_commit_acc(const float* in, size_t in_stride, float* out, size_t stride, const float* grad,
                             size_t grad_stride, float* acc, size_t acc_stride, float lr, int K, size_t P, hipStream_t s);
hipError_t launch_merge_grad(float* global, const PtrPack& accs, float lr, int K, size_t P, hipStream_t s);
hipError_t launch_fill_zero(float* p, size_t n, size_t stride, int groups, hipStream_t s, float* extra = nullptr,
                            size_t n_extra = 0);
// p[g*stride + r*ld + c] = 0 for r < rows, c < cols (4-byte words)
// Up to MAXSEG clears in one launch.  pk.n = 0, pk.blk0[0] = 0, pk.max_groups = 0 are set by the caller.
struct FillSeg {
  float* p; long ld; int rows; long cols; size_t stride; int groups;
};
struct FillPack {
  static constexpr int MAXSEG = 12;
  FillSeg seg[MAXSEG];
  unsigned blk0[MAXSEG + 1];
  int n, max_groups;
};
bool fill_pack_push(FillPack& pk, float* p, long ld, int rows, long cols, size_t stride, int groups);
hipError_t launch_fill_pack(const FillPack& pk, hipStream_t s);
hipError_t launch_fill_zero_2d(float* p, long ld, int rows, int cols, size_t stride, int groups,
                               hipStream_t s);
hipError_t launch_gather(const void* shard, const int32_t* idx, int n_idx, size_t row_bytes,
                         int n_chunks, size_t chunk_bytes, void* out, hipStream_t s);

hipError_t launch_gather_all(const void* const* shards, const int32_t* const* idx, int K, int n_idx,
                             size_t row_bytes, int n_chunks, size_t chunk_bytes, void* const* outs,
                             hipStream_t s);

// one array of the gathered samples; gather_parts: all arrays of all K workers in one launch
struct GatherPart {
  const void* const* shards; void* const* outs;
  size_t row_bytes, chunk_bytes;
  int n_chunks;
};
hipError_t launch_gather_parts(const GatherPart* parts, int n_parts, const int32_t* const* idx, int K, int n_idx, hipStream_t s);

// ---- grouped GEMM on the fp32 / bf16 matrix cores ----
enum Epilogue : int {
  EPI_STORE = 0,      // C = acc
  EPI_BIAS = 1,       // C = acc + bias[n]
  EPI_BIAS_RELU = 2,  // C = max(acc + bias[n], 0)
  EPI_ACCUM = 3,      // C += acc
  EPI_RELU_MASK = 4,  // C = acc * (mask[m,n] > 0)      (mask has C's layout)
  EPI_COMMIT = 5      // C = W[m,n] - alpha * acc       (W = aux, C's layout; C may be W itself):
                      // the SGD update of a weight matrix applied where its gradient is produced
};

struct GemmDesc {
  // C[g] (M x N, row-major, ldc) = op(A[g]) (M x Kd) * op(B[g]) (Kd x N)
  const float* A; long lda; long strideA; int transA;  // transA=0: A stored [M][Kd]; 1: stored [Kd][M]
  const float* B; long ldb; long strideB; int transB;  // transB=0: B stored [Kd][N]; 1: stored [N][Kd]
  float* C; long ldc; long strideC;
  const float* aux; long strideAux;                    // bias [N] or mask [M][N] (ldc)
  int M, N, Kd, groups;
  // splits > 1 (pipelined fp32 kernel only): the contraction of Kall is cut into `splits` parts of Kd
  // each (a multiple of 4; the last one may be shorter), part p of group g reads A and B advanced by
  // p * Kd along the contraction and writes its own C at C + (g * splits + p) * strideC
  // (strideC is then the distance between two parts; the epilogue must be EPI_STORE)
  int splits, Kall;
  int epilogue;
  int bf16;                                            // round operands to bf16, use the bf16 MFMA
  float alpha;                                         // EPI_COMMIT: the learning rate
  int background;                                      // runs beside latency-critical kernels: keep the
                                                       // LDS footprint small so both fit on a CU
  // all workers of the context, of which `groups` are stepped (0: groups): what decides the order of a sum goes by
  // it, so that a worker's result is the same however many are stepped with it
  int workers;
};
hipError_t launch_gemm(const GemmDesc& d, hipStream_t s);

// Column sums of up to MAXSEG matrices, optionally applied as out = b_in - lr * sum.
// pk.n = 0, pk.blk0[0] = 0 and pk.lr are set by the caller.
struct ColsumSeg {
  const float* in; long ld, s_in;
  float* out; long s_out;
  const float* b_in; long s_bin;
  int R, N;
  float scale;  // applied when b_in is null
};
struct ColsumPack {
  static constexpr int MAXSEG = 8;
  ColsumSeg seg[MAXSEG];
  unsigned blk0[MAXSEG + 1];
  int n;
  float lr;
};
bool colsum_pack_push(ColsumPack& pk, const float* in, long ld, long s_in, float* out, long s_out, const float* b_in,
                      long s_bin, int R, int N, float scale = 1.0f);
hipError_t launch_colsum_pack(const ColsumPack& pk, int groups, hipStream_t s);

// fp32 products that need nothing of each other, and column sums beside them, in one launch.
// gemm_pack_push returns false for a product the shared launch does not take or has no room for (nothing
// is added: launch it by itself).  pk.n = 0 is set by the caller.
struct GemmPack {
  static constexpr int MAX = 4;
  GemmDesc d[MAX];
  unsigned blk0[MAX + 1];  // filled by the launch
  int n;
};
bool gemm_pack_push(GemmPack& pk, const GemmDesc& d);
hipError_t launch_gemm_pack(GemmPack& pk, const ColsumPack& cs, int groups, hipStream_t s);

// ---- classifier head with few classes in two small launches (fp32), see cls_head.hip ----
bool cls_head_supported(int N, int C, int H);
hipError_t launch_cls_head(const float* feats, long s_feats, const float* W_in, const float* b_in, long s_in,
                           const int32_t* y, long s_y, float* dlog, long s_dlog, float* rowloss, long s_rowloss,
                           float* dfeat, long s_dfeat, float* W_out, float* b_out, long s_out, float lr, int commit,
                           float* loss, int N, int C, int H, int groups, hipStream_t s, int relu_mask = 0);

// ---- GRU cell, loss, reductions ----
// forward cell for one time step of all groups:
//   gx [B][3H] (b_ih included), gh [B][3H] (b_hh included), h_prev [B][H] -> h [B][H], saved [B][4H] = r|z|n|q
hipError_t launch_gru_cell_fwd(const float* gx, long s_gx, const float* gh, long s_gh,
                               const float* h_prev, float* h, long s_h, float* saved, long s_saved,
                               int B, int H, int groups, hipStream_t s);
// backward cell: dh = D + above (above nullable); writes dgx [B][3H], dgh [B][3H], D = dh*z
hipError_t launch_gru_cell_bwd(float* D, long s_D, const float* above, long s_above,
                               const float* saved, long s_saved, const float* h_prev, long s_h,
                               float* dgx, float* dgh, long s_dg, int B, int H, int groups,
                               hipStream_t s);
// ---- fused recurrent steps (recurrent GEMM + cell math in one launch), see gru_fused.hip ----
bool gru_fused_supported(int H);
hipError_t launch_gru_fwd_step(const float* W_hh, const float* b_hh, long s_rep, const float* gx_t,
                               long s_gx, const float* h_prev, float* h_out, long s_hs, float* sv_t,
                               long s_sv, int B, int H, int groups, hipStream_t s);
hipError_t launch_gru_bwd_step(const float* WT, long s_wt, const float* dgh_next, long s_dg, float* D,
                               long s_D, const float* above, long s_above, const float* sv_t,
                               long s_sv, const float* h_prev, long s_hs, float* dgx_t, float* dgh_t,
                               int B, int H, int groups, hipStream_t s);
// ---- all time steps of a narrow layer in one launch without any exchange between workgroups (fp32), see gru_solo.hip ----
// (workers: all of the context's, of which `groups` are stepped)
bool gru_solo_supported(int B, int H);
int gru_solo_row_tiles(int B, int H, int workers);                    // partial sums of the bias gradients per worker
size_t gru_solo_saved_words(int B, int H, int T, int workers);        // floats of `sv` per worker (a layout of its own)
hipError_t launch_gru_solo_fwd(const float* W_hh, const float* b_hh, long s_rep, const float* gx, long s_gx, float* hs,
                               long s_hs, float* sv, long s_sv, int B, int H, int T, int groups, int workers, hipStream_t s);
// D == nullptr: no gradient is carried into the last step; dbp[(g * row tiles + tile)][6H] receives the
// partial bias-gradient sums (b_ih: r z n, then b_hh: r z q)
hipError_t launch_gru_solo_bwd(const float* W_hh, long s_rep, float* dgx, float* dgh, long s_dg, const float* D, long s_D,
                               const float* above, long s_above, const float* sv, long s_sv, const float* hs, long s_hs,
                               float* dbp, int B, int H, int T, int groups, int workers, hipStream_t s);
// Both layers of a model of two in one launch (each way), the upper one a few steps behind: gx and dgh are each layer's own (gx: the
// upper layer's is written by the forward launch; the gate gradients replace it), dx receives the gradient that the upper layer passes on.
// sync: gru_stack_sync_words() words, zero; sync[0] is the abort word.  A wait that was given up sets it and
// leaves NaN in everything behind it in the chain (launch_poison_on_abort behind the step shows it in the results).
struct GruStackLayer {
  const float *W_hh, *b_hh;
  float *gx, *dgh, *hs, *sv, *dbp;
};
bool gru_stack_supported(int B, int H, int T, int layers, int workers, bool lm);  // lm: of a language model
size_t gru_stack_sync_words(int B, int groups);
hipError_t launch_gru_stack_fwd(const GruStackLayer& lo, const GruStackLayer& up, const float* W_ih, const float* b_ih, long s_rep, long s_gx,
                                long s_hs, long s_sv, int B, int H, int T, int groups, unsigned* sync, unsigned limit, hipStream_t s);
hipError_t launch_gru_stack_bwd(const GruStackLayer& lo, const GruStackLayer& up, const float* W_ih, long s_rep, const float* D, long s_D,
                                const float* above, long s_above, float* dx, long s_dx, long s_gx, long s_hs, long s_sv,
                                int B, int H, int T, int groups, unsigned* sync, unsigned limit, hipStream_t s);
// the same with bf16 operands (H a multiple of 32 up to 256, B of 8): writes hb, hT (h_0 = 0 included) and dbp as the
// resident-weight launches below do, and the gate gradients row-major as dg4 [T B][4H] = r | z | n | q; hs
// and sv hold h_{t-1} and the gates in lane order (T B H and 4 T B H floats), for the backward launch only
bool gru_solo_bf16_supported(int B, int H);
int gru_solo_bf16_row_tiles(int B, int workers);
hipError_t launch_gru_solo_fwd_bf16(const void* Wb, long s_wb, const float* b_ih, const float* b_hh, long s_rep, int Hc,
                                    const float* gx, long s_gx, void* hb, long s_hb, float* hs, long s_hs, float* sv, long s_sv,
                                    void* hT, long ld_hT, long s_hT, int Bc, int B, int H, int T, int groups, int workers, bool exact,
                                    hipStream_t s);
hipError_t launch_gru_solo_bwd_bf16(const void* WT, long s_wt, const float* above, long s_above, const float* sv, long s_sv,
                                    const float* hs, long s_hs, void* dg4, long s_dg4, float* dbp, int Hc, int B, int H, int T,
                                    int groups, int workers, hipStream_t s);
// two such layers in one launch (each way), as launch_gru_stack_*: hb and dg4 are each layer's own; W_ih [3H][H] and WT_ih = W_ih^T [H][3H] are the
// upper layer's
struct GruStackLayerB {
  const void *W, *WT;  // W_hh and W_hh^T
  const float *b_ih, *b_hh;
  float* gx;
  void* hb;
  float *hs, *sv;
  void *hT, *dg4;
  float* dbp;
};
bool gru_stack_bf16_supported(int B, int H, int T, int layers, int workers);
size_t gru_stack_bf16_sync_words(int B, int groups);
hipError_t launch_gru_stack_fwd_bf16(const GruStackLayerB& lo, const GruStackLayerB& up, const void* W_ih, long s_wih, long s_wb, long s_rep,
                                     int Hc, long s_gx, long s_hb, long s_hs, long s_sv, long ld_hT, long s_hT, int Bc, int B, int H, int T,
                                     int groups, bool exact, unsigned* sync, unsigned limit, hipStream_t s);
hipError_t launch_gru_stack_bwd_bf16(const GruStackLayerB& lo, const GruStackLayerB& up, const void* WT_ih, long s_wih, long s_wt,
                                     const float* above, long s_above, float* dx, long s_dx, long s_hs, long s_sv, long s_dg4,
                                     int Hc, int B, int H, int T, int groups, unsigned* sync, unsigned limit, hipStream_t s);
// its transposes: dgxT [3H][ld_T] = (r | z | n)^T, dghT = (r | z | q)^T over R = T B rows, in one launch
hipError_t launch_transpose_dg4(const void* dg4, long s_dg4, void* dgxT, void* dghT, long ld_T, long s_T, int R, int H, int groups,
                                hipStream_t s);
// ---- whole runs of time steps in one launch, W_hh resident on the chip (fp32), see gru_persist.hip ----
// sync: gru_persist_sync_words() words of device memory (the abort word, the flag words of the
// synchronisation groups, 8 ticket counters); base: what the flags read when the launch starts; every launch
// advances them by steps * gru_persist_count_per_step().  spin_limit bounds every wait.
// any H from 16 to 704; rows: batch rows per workgroup, as gru_persist_rows gives them
// for the context's K workers, however many of them a call steps (0: does not fit).  More workgroups than the chip
// has CUs run as several launches where that pays, which goes by the time steps and by the workers of the call (gru_persist_pays): stepping
// one worker and stepping all of them may take different forms, whose sums differ in their order.
int gru_persist_rows(int B, int H, int K);
bool gru_persist_pays(int B, int H, int T, int groups, int rows);
size_t gru_persist_sync_words(int B, int groups, int rows);
unsigned gru_persist_count_per_step(int H);
// device_scope: the workgroups exchange through memory that every XCD sees; false lets a launch
// that fills the chip with one workgroup per CU exchange through the L2 of the XCD a
// synchronisation group runs on (the workgroups then take their tiles by where they run: they draw
// tickets from 8 counters at the end of the sync words, zero at the start of a step).
// ticket_launches: the step's count of launches that have drawn tickets (advanced by the launcher;
// all launches of a step that share the sync words must share it).
// hx / dghx: h_0 .. h_T and the gate gradients of all steps as the workgroups exchange them,
// fragment-major, gru_persist_exchange_words floats per time step (hx: T + 1
// steps, the first one, h_0, given); hs / dgh are the row-major copies for the other kernels
// (dgh may be nullptr in the backward launch when nothing reads it later).
size_t gru_persist_exchange_words(int B, int H, int gates);  // gates: 1 for h, 3 for the gate gradients
hipError_t launch_gru_fwd_persist(const float* W_hh, const float* b_hh, long s_rep, const float* gx, long s_gx,
                                  float* hs, long s_hs, float* hx, long s_hx, float* sv, long s_sv, int B, int H, int T,
                                  int groups, int rows,
                                  unsigned* sync, unsigned base, unsigned spin_limit, const float* xin, long s_x,
                                  int width, const float* W_ih, const float* b_ih, bool device_scope, unsigned* ticket_launches, hipStream_t s);
// xin != nullptr (allowed when gru_persist_xproj_supported(H, width, rows)): the launch computes the input
// projection itself from the layer input xin (T blocks of B x width per worker, stride s_x) and W_ih,
// b_ih (in the replica, like W_hh); gx is then unused and may be nullptr.
bool gru_persist_xproj_supported(int H, int width, int rows);
// d_zero: the gradient carried into the last step is zero (D is not read)
hipError_t launch_gru_bwd_persist(const float* W_hh, long s_rep, float* dgh, float* dghx, long s_dghx, float* dgx,
                                  long s_dg, const float* D,
                                  long s_D, bool d_zero, const float* above, long s_above, const float* sv, long s_sv,
                                  const float* hs, long s_hs, int B, int H, int T,
                                  int groups, int rows, unsigned* sync, unsigned base, unsigned spin_limit, float* dWp,
                                  float* dbp, bool device_scope, unsigned* ticket_launches, hipStream_t s);
// dbp != nullptr: the launch also leaves dbp[(g * RT + ty)][6H], partial sums over its steps of the
// bias gradients (b_ih: sum of dgx, then b_hh: sum of dgh)
// dWp != nullptr (allowed when gru_persist_dw_supported(H)): the launch also leaves
// dWp[(g * RT + ty)][3H][H], RT = ceil(B / rows) partial sums of dW_hh over its steps per worker.
bool gru_persist_dw_supported(int H);
// out[g][i] = in[g][i] - lr * sum_p parts[(g * n_parts + p)][i]  (commit != 0; in may be out)
// out[g][i] = sum_p parts[(g * n_parts + p)][i]                   (commit == 0)
// Up to MAXSEG sums of partial results in one launch: reduce_pack_push (false: the pack is full;
// nothing is added), then launch_reduce_pack.  Any n and alignment (16-byte accesses where they allow it).  pk.n = 0, pk.blk0[0] = 0 and pk.lr are set by the caller.
struct ReduceSeg {
  const float* parts; int n_parts; size_t n, pitch; int vec;  // pitch: floats from one part to the next
  const float* in; size_t s_in; float* out; size_t s_out; int commit;
};
struct ReducePack {
  static constexpr int MAXSEG = 6;  // two layers' parts of both weight gradients and of the bias gradients
  unsigned blk0[MAXSEG + 1];  // (what every workgroup reads lies in front of the segments, of which it reads one)
  int n;
  float lr;
  // beside the sums (nullptr: none): loss[g] = the sum of group g's `rows` row losses over `count`
  const float* rowloss = nullptr;
  long s_rowloss = 0;
  float* loss = nullptr;
  int rows = 0, count = 0;
  ReduceSeg seg[MAXSEG];
};
bool reduce_pack_push(ReducePack& pk, const float* parts, int n_parts, size_t n, const float* in, size_t s_in,
                      float* out, size_t s_out, int commit, size_t pitch = 0);
hipError_t launch_reduce_pack(const ReducePack& pk, int groups, hipStream_t s);
hipError_t launch_reduce_parts(const float* parts, int n_parts, size_t n, const float* in, size_t s_in,
                               float* out, size_t s_out, float lr, int commit, int groups, hipStream_t s,
                               size_t pitch = 0);
// bf16 operands (strides of bf16 buffers in bf16 elements): hx / dghx hold all time steps and are the
// operands the workgroups exchange, kept fragment-major (per step a block of 16 ceil(B/16) rows;
// gru_persist_bf16_exchange_elems gives a step's block); hb is the row-major copy of h for the
// GEMMs; hT, dgxT, dghT are the transposed copies [unit][time * B + row].
// The backward launch always leaves the partial bias-gradient sums in dbp and writes no fp32
// gate gradients.  Counters advance by steps * gru_persist_bf16_count_per_step().
// H: the width of every internal buffer (a multiple of 32); Hc <= H: the width of the model's own
// arrays (b_ih, b_hh, dbp).  Bc <= B: the batch rows that are the model's own.  Of units beyond Hc and rows
// beyond Bc the forward launch leaves zeros, whatever their input projections are.  b_ih is added by the forward launch.
// More workgroups than the chip has CUs are issued as several launches of whole synchronisation groups.
bool gru_persist_bf16_supported(int B, int H);
// batch rows per workgroup (16 or 32: the launches' argument `rows`) of a layer of K workers
int gru_persist_bf16_rows(int B, int H, int K);
// whether the bf16 forward launches compute a model's gates as the fp32 ones do (their argument `exact`)
bool gru_bf16_exact_gates(int B, int H, int K, bool padded);
unsigned gru_persist_bf16_count_per_step(int H);
hipError_t launch_gru_fwd_persist_bf16(const void* Wb, long s_wb, const float* b_ih, const float* b_hh, long s_rep, int Hc, const float* gx,
                                       long s_gx, float* hs, long s_hs, void* hb, long s_hb, void* hx, long s_hx,
                                       float* sv, long s_sv, void* hT, long ld_hT, long s_hT, int Bc, int B, int H, int T,
                                       int groups, int rows, bool exact, unsigned* sync, unsigned base, unsigned spin_limit,
                                       bool device_scope, unsigned* ticket_launches, hipStream_t s);
// bf16 elements of one time step's block of an exchange buffer whose rows are `width` wide
size_t gru_persist_bf16_exchange_elems(int B, int width);
hipError_t launch_gru_bwd_persist_bf16(const void* WT, long s_wt, void* dghx, long s_dgh, long s_dgb, float* D, long s_D,
                                       bool d_zero, const float* above, long s_above, const float* sv, long s_sv, const float* hs,
                                       long s_hs, void* dgxb, void* dgxT, void* dghT, long ld_T, long s_T, float* dbp, int Hc,
                                       int B, int H, int T, int groups, int rows, unsigned* sync, unsigned base,
                                       unsigned spin_limit, bool device_scope, unsigned* ticket_launches, hipStream_t s);
// NaN into loss[0..n_loss) and into rout[g * s_rout] for every group if *abort_w != 0
hipError_t launch_poison_on_abort(const unsigned* abort_w, float* loss, int n_loss, float* rout, long s_rout,
                                  int groups, hipStream_t s);
// bf16-operand variants (strides of bf16 buffers are in bf16 elements)
bool gru_fused_bf16_supported(int H);
hipError_t launch_gru_fwd_step_bf16(const void* Wb, long s_wb, const float* b_hh, long s_rep,
                                    const float* gx_t, long s_gx, const float* h_prev, float* h_out,
                                    long s_hs, const void* hb_prev, void* hb_out, long s_hb, float* sv_t,
                                    long s_sv, void* hT_out, long ld_hT, long s_hT, int B, int H,
                                    int groups, hipStream_t s);
hipError_t launch_gru_bwd_step_bf16(const void* WTb, long s_wt, const void* dghb_next, void* dghb_t,
                                    long s_dgb, float* D, long s_D, const float* above, long s_above,
                                    const float* sv_t, long s_sv, const float* h_prev, long s_hs,
                                    float* dgx_t, float* dgh_t, long s_dg, void* dgxb_t, void* dgxT_t,
                                    void* dghT_t, long ld_T, long s_T, int B, int H, int groups,
                                    hipStream_t s);
// out(bf16) = round(in), in is R x C with row pitch ld_in; transpose: out[c][r] = in[r][c];
// ld_out is the row pitch of out, strides of out in bf16 elements
hipError_t launch_cvt_bf16(const float* in, long ld_in, long s_in, void* out, long ld_out, long s_out,
                           int R, int C, bool transpose, int groups, hipStream_t s);
// in (fp32, or bf16 when in_bf16) R x C -> out_p = bf16 rounding (nullable), out_t = its
// transpose (nullable), one read of `in`; strides of each buffer in its own elements
bool cvt2_supported(const void* in, int in_bf16, long ld_in, long s_in, const void* out_p, long ld_p,
                    long s_p, const void* out_t, long ld_t, long s_t, int R, int C);
hipError_t launch_cvt2(const void* in, int in_bf16, long ld_in, long s_in, void* out_p, long ld_p, long s_p,
                       void* out_t, long ld_t, long s_t, int R, int C, int groups, hipStream_t s);
// several fp32 matrices through one launch of the same copies (one group count for all of them)
// R x C: the extents of the copies.  gp != 0: a source of any alignment and size, Cs <= C columns wide and
// with gh rows per block of gp rows of the copies (row r of a copy is source row (r / gp) gh + r % gp);
// what the source does not have is zero in the copies.
struct Cvt2Job {
  const float* in;
  long ld_in, s_in;
  void* out_p;
  long ld_p, s_p;
  void* out_t;
  long ld_t, s_t;
  int R, C, tiles_x, gp, gh, Cs;
};
struct Cvt2Pack {
  static constexpr int MAX = 8;
  int n = 0;
  int tile0[MAX + 1] = {0};  // first tile of job j in blockIdx.x; tile0[n] = all tiles
  double bytes = 0;          // per group, for the launch timer
  Cvt2Job job[MAX];
};
// false: the pack is full or the job is not one cvt2_supported takes (launch it by itself)
bool cvt2_pack_push(Cvt2Pack& p, const float* in, long ld_in, long s_in, void* out_p, long ld_p, long s_p,
                    void* out_t, long ld_t, long s_t, int R, int C);
// a source the plain copies do not take: rows in blocks of gh, padded to gp per block in the copies, Cs
// columns padded to C (out_p: row pitch C or more, a multiple of 4; out_t: ld_t a multiple of 8, R a multiple of 8)
bool cvt2_pack_push_padded(Cvt2Pack& p, const float* in, long ld_in, long s_in, void* out_p, long ld_p, long s_p,
                           void* out_t, long ld_t, long s_t, int R, int C, int gp, int gh, int Cs);
hipError_t launch_cvt2_pack(const Cvt2Pack& p, int groups, hipStream_t s);
// The first layer's input of a language model, rounded: row r = t Bp + b of the copies is the embedding
// row of token tok[t B + b] (zero for b >= B and beyond column Ew), as xb (row pitch Ep) and transposed
// as xT ([Ep][ld_T]); Bp and Ep are multiples of 8.
hipError_t launch_embed_bf16(const float* E, long s_E, const int32_t* tok, long s_tok, void* xb, long s_xb, void* xT,
                             long ld_T, long s_xT, int T, int B, int Bp, int Ew, int Ep, int groups, hipStream_t s);
// mean softmax-CE of N = T Bp rows of C logits (row pitch ld_l, a multiple of 4 and at least C rounded up to
// 8; what lies beyond C may be anything), whose gradient is written rounded to bf16 (row pitch ld_d), zero
// from C up to the next multiple of 8; logits intact.  Row t Bp + b has the label y[t B + b]; rows with
// b >= B are padding: zero gradient, zero loss.  The mean runs over the T B real rows.
bool softmax_ce_bf16_supported(const float* logits, long ld_l, long s_logits, const void* dlog, long ld_d, long s_d,
                               int C);
// colpart receives one partial sum of the unrounded gradient's columns per block of rows, C rounded up to
// 8 floats apart: softmax_ce_bf16_row_blocks(N, sizing_groups) blocks per group, where sizing_groups is the
// number of workers the launch is sized for (the same value must go to the launch); 0 gives the upper
// bound, for allocations
hipError_t launch_softmax_ce_bf16(const float* logits, long ld_l, long s_logits, const int32_t* y, long s_y, void* dlog,
                                  long ld_d, long s_d, float* rowloss, long s_rowloss, int N, int B, int Bp, int C,
                                  int groups, hipStream_t s, float* colpart, long s_colpart, int sizing_groups);
int softmax_ce_bf16_row_blocks(int N, int sizing_groups = 0, int C = 0);
// one wave that sleeps until the wall clock has advanced by `us` microseconds
hipError_t launch_delay(unsigned us, hipStream_t s);
// pure-MFMA loop, one wave on every SIMD, operands from `operands` (16 KiB); see hpsgd.h
hipError_t launch_mfma_probe(bool bf16, const void* operands, int iterations, double* result, float* sink,
                             hipStream_t s);
// bf16 GEMM with both operands unit-stride along the contraction (gemm_bf16_nt.hip)
bool gemm_bf16_nt_supported(const void* p, int is_bf16, long ld, long stride, int Kd);
hipError_t launch_gemm_bf16_nt(const void* A, int a_bf16, long lda, long sA, const void* B, int b_bf16,
                               long ldb, long sB, float* C, long ldc, long sC, const float* bias,
                               long sBias, const float* win, long sWin, float lr, int M, int N, int Kd,
                               int groups, hipStream_t s, int form = 0, int gp = 0, int gh = 0, int splits = 1,
                               int Kall = 0, int outer = 0);
// (splits > 1, two bf16 operands, no bias and no update: the contraction of Kall in parts of Kd, a multiple
// of 64; part p of group g writes its own C at C + (g splits + p) sC)
// (gp != 0: the operands' rows come in up to three gate blocks of gp, C and win have gh rows per block)
// (outer: 2 for a B that is stored [Kd][N], without an update; 3 for such a B and an A that is stored [Kd][M]; both
// bf16, gp == 0, a pitch that covers the row rounded up to 8)
// Two products with bf16 operands and the update epilogue (C = win - lr * A B^T) in ONE launch of
// the 192 x 256 form: for two that neither need each other nor fill the chip alone.  Strides in
// elements of each buffer's own type; the same conditions as launch_gemm_bf16_nt per product.
struct GemmBf16Args {
  const void* A; long lda, sA;
  const void* B; long ldb, sB;
  float* C; long ldc, sC;
  const float* win; long sWin;
  float lr;
  int M, N, Kd, groups;
  int gp, gh;
  int outer = 0, splits = 1, Kall = 0;  // (the pair: as they are here)
};
// Up to three products with bf16 operands, as updates (win) or plain, in one launch of 128 x 128 tiles
bool gemm_bf16_multi_pays(const GemmBf16Args* p, int n);
hipError_t launch_gemm_bf16_multi(const GemmBf16Args* p, int n, hipStream_t s);
bool gemm_bf16_update_pair_supported(const GemmBf16Args& p0, const GemmBf16Args& p1);
hipError_t launch_gemm_bf16_update_pair(const GemmBf16Args& p0, const GemmBf16Args& p1, hipStream_t s);

// out[c][r] = in[r][c], R x C per group
hipError_t launch_transpose(const float* in, long s_in, float* out, long s_out, int R, int C,
                            int groups, hipStream_t s);

// mean softmax cross-entropy over N rows of C logits; dlogits = (p - onehot)/N; row losses to rowloss
hipError_t launch_softmax_ce(const float* logits, long s_logits, const int32_t* y, long s_y,
                             float* dlogits, float* rowloss, long s_rowloss, int N, int C,
                             int groups, hipStream_t s);
// loss[g] = (1/N) sum_i rowloss[g][i], fixed order
// (count: what the sum is divided by, when not N)
hipError_t launch_loss_mean(const float* rowloss, long s_rowloss, float* loss, int N, int groups,
                            hipStream_t s, int count = 0);
// out[g][n] = sum_r in[g][r][n]
hipError_t launch_colsum(const float* in, long ld, long s_in, float* out, long s_out, int R, int N,
                         int groups, hipStream_t s);
// embedding rows: out[g][i][:] = E[g][tok[g][i]][:]
hipError_t launch_embed_fwd(const float* E, long s_E, const int32_t* tok, long s_tok, float* out,
                            long s_out, int N, int Ew, int groups, hipStream_t s);
// dE[g][v][:] = sum over positions i with tok[g][i]==v of dx[g][i][:], in increasing i; other rows untouched
// (ld_dx: row pitch of dx; B, Bp: position t B + b has its gradient in row t Bp + b)
hipError_t launch_embed_bwd(const float* dx, long ld_dx, long s_dx, const int32_t* tok, long s_tok, float* dE,
                            long s_dE, int N, int B, int Bp, int Ew, int groups, hipStream_t s, const float* E_in = nullptr,
                            long s_E = 0, float lr = 0.f);

}  // namespace hpsgd
