// Internal launcher interface between the stage orchestrator and the kernels.
// Every launcher only enqueues on `st` and returns hipGetLastError().
#pragma once
#include "../../include/gpt_stage.h"
#include "common.hpp"

namespace gpts {

// dtype: 0 = fp32 storage, 1 = bf16 storage (fp32 arithmetic in both).

// Several micro-batches in one launch (a window of them): the operators below take the tensors of the first
// one and how far those of the next one lie, in bytes: a multiple of 16 below 64 GiB, which some kernels are told in 32 bits.
// A micro-batch's share is computed as by a launch of its own, bit for bit.
constexpr int kMaxWindow = 8;
inline bool window_stride_ok(size_t s) { return s % 16 == 0 && s < ((size_t)1 << 36); }

// x_f32: the normalised tensor x (the residual stream) is fp32 even when dtype is bf16.
// out_f16 (bf16 stages only): out is written as fp16 instead of bf16.
// xcopy (may be null): receives x as fp32.
// n micro-batches: out, mean, rstd, xcopy lie `stride` apart, x `x_stride`.
hipError_t ln_fwd(int dtype, bool x_f32, int T_rows, int H, float eps, const void* x,
                  const void* gamma, const void* beta, void* out, float* mean, float* rstd,
                  hipStream_t st, bool out_f16 = false, float* xcopy = nullptr, int n = 1, size_t stride = 0,
                  size_t x_stride = 0);
// Partial column sums waiting to be added up: out[c] += sum_{g<G} partial[g*stride + c], the columns
// c < N being split at n0 and n1 over out0 (c < n0), out1 (n0 <= c < n1) and out2 (n1 <= c).
// N, n0, n1 and stride are multiples of 4.  batch > 1: as many groups of G rows, one after the other in memory, each
// added up as above and then to out, in order.
struct ReduceSeg {
  const float* partial;
  size_t stride;
  int G, N, n0, n1;
  float *out0, *out1, *out2;
  int batch = 1;
};
constexpr int kMaxReduceSegs = 5;
// adds up n <= kMaxReduceSegs segments in one launch, each in fixed order
hipError_t reduce_partials(const ReduceSeg* segs, int n, hipStream_t st);
size_t ln_bwd_scratch_bytes(int T_rows, int H);
// a matrix whose columns are summed, see colsum_partials()
struct ColsumMat {
  const void* A;
  int N;
  float *out, *partial;
};
constexpr int kMaxColsums = 3;
// dxsum (may be null): += column sums of dx as stored.  ln_bwd_partials leaves the three sums in
// `partial` (ln_bwd_scratch_bytes(), for each micro-batch) and describes them in *seg; ln_bwd adds them up as well.
// cols, n_cols, col_segs: what colsum_partials would do for n_cols <= kMaxColsums matrices of as many rows, in the same
// launch (only where ln_bwd_takes_colsums(), of the rows of all micro-batches).  dx must not overlap them.
bool ln_bwd_takes_colsums(int dtype, int T_rows, int H, const ColsumMat* cols, int n);
struct LnBwdWindow {
  int n = 1;
  size_t act = 0, dres = 0, dx = 0, cols = 0;   // strides of dout, x, mean and rstd; of dres; of dx; of the matrices `cols`
};
hipError_t ln_bwd_partials(int dtype, bool x_f32, int T_rows, int H, const void* dout, const void* x,
                           const float* mean, const float* rstd, const void* gamma, const void* dres, void* dx,
                           float* dgamma, float* dbeta, float* dxsum, float* partial, ReduceSeg* seg, hipStream_t st,
                           const LnBwdWindow* win = nullptr, const ColsumMat* cols = nullptr, int n_cols = 0,
                           ReduceSeg* col_segs = nullptr);
hipError_t ln_bwd(int dtype, bool x_f32, int T_rows, int H, const void* dout, const void* x,
                  const float* mean, const float* rstd, const void* gamma, const void* dres, void* dx,
                  float* dgamma, float* dbeta, float* dxsum, float* partial, hipStream_t st);
// g = gelu(u) elementwise (kind 0 tanh form, 1 erf form); n a multiple of 8
// u_f16 (bf16 stages): u is fp16, g is still written as bf16
hipError_t gelu_fwd(int dtype, int kind, const void* u, void* g, size_t n, hipStream_t st, bool u_f16 = false);
// out[i] = bf16(in[i]) for n fp16 elements (n a multiple of 8)
hipError_t f16_to_bf16(const void* in, void* out, size_t n, hipStream_t st);
size_t colsum_scratch_bytes(int M, int N);
// out += column sums of A [M,N].  colsum_partials takes n <= kMaxColsums matrices of M rows in one launch
// and leaves their sums in each one's `partial` (colsum_scratch_bytes(), for each micro-batch) and segs[0 .. n-1],
// as above.  A's of `batch` micro-batches lie `stride` bytes apart.
hipError_t colsum_partials(int dtype, int M, const ColsumMat* mats, int n, ReduceSeg* segs, hipStream_t st, int batch = 1,
                           size_t stride = 0);
// dst[m] = src[m] for n buffers of `bytes` (a multiple of 16) each
hipError_t window_copy(int n, const void* const* src, void* const* dst, size_t bytes, hipStream_t st);
hipError_t colsum(int dtype, int M, int N, const void* A, float* out, float* partial, hipStream_t st);
// the segment of G rows of N partial sums each, added to out
ReduceSeg colsum_segment(const float* partial, int G, int N, float* out);

// Epilogue description shared by all GEMM implementations.
struct GemmEpilogue {
  const void* bias = nullptr;      // [N], storage dtype, added to every row
  const void* residual = nullptr;  // [M,N], added; storage dtype unless residual_f32
  bool residual_f32 = false;       // bf16 stages: residual is fp32
  bool out_f32 = false;            // bf16 stages: C is written as fp32 (forms 0 with residual only)
  void* gelu_out = nullptr;        // [M,N]: if set, C keeps the pre-activation and this gets gelu(C)
  const void* dgelu_u = nullptr;   // [M,N]: if set, C *= gelu'(u)
  int gelu_kind = 0;               // 0 tanh, 1 erf
  float* colsum_partial = nullptr; // with dgelu_u, MFMA path only: [gemm_mfma_colsum_rows()][N] fp32,
                                   // written (not added to): column sums of C (fp32, before it is
                                   // rounded for storage), one row per group of tile rows; their sum
                                   // over the rows is sum_m C[m, :]
  const void* b_image = nullptr;   // form 0, bf16: B re-laid-out by gemm_prepare_image() (optional)
  // form 2, bf16 MFMA path only (gemm_wgrad_segments_supported): the contraction runs over
  // k_segments pieces of K rows each; piece s of A (B) starts seg_stride_a (seg_stride_b)
  // ELEMENTS after piece s-1.  One launch, one read-modify-write of C.
  int k_segments = 1;
  size_t seg_stride_a = 0, seg_stride_b = 0;
  // forms 0 and 1, bf16 MFMA path only: `batch` products of M rows each with the same B.  A's lie stride_a bytes
  // apart, C's and gelu_out's stride_c, residuals or dgelu_u's stride_r; the rows of colsum_partial follow on.
  int batch = 1;
  size_t stride_a = 0, stride_c = 0, stride_r = 0;
};
// form 0: C[M,N] = A[M,K] B[N,K]^T ; form 1: C[M,N] = A[M,K] B[K,N] ;
// form 2: Cf32[M,N] += A[K,M]^T B[K,N].
hipError_t gemm_simple(int dtype, int form, int M, int N, int K, const void* A, const void* B,
                       void* C, const GemmEpilogue& ep, hipStream_t st);
// fp32 products on the matrix cores (gemm_f32.hip): contiguous dimensions multiples of 4, pointers
// 16-byte aligned; any M, N, K otherwise.
bool gemm_f32_supported(int form, int M, int N, int K, const void* A, const void* B, const void* C,
                        const GemmEpilogue& ep);
hipError_t gemm_f32(int form, int M, int N, int K, const void* A, const void* B, void* C,
                    const GemmEpilogue& ep, hipStream_t st);
// bf16 MFMA path, for every shape gemm_mfma_supported(); hipErrorInvalidValue for others, nothing launched.
bool gemm_mfma_supported(int form, int M, int N, int K);
// Tiled image of a weight src [N,K] as the B operand of form 0; K % 64 == 0 (else the rest of K is
// left out).  N any.
size_t gemm_image_elems(int N, int K);
// to_f16: the image holds the bf16 source values converted to fp16.
hipError_t gemm_prepare_image(const void* src, void* img, int N, int K, hipStream_t st, bool to_f16 = false);
// Forward product with fp16 operands on the matrix cores' f16 instructions:
// C[M,N] = A[M,K] (fp16) W^T, W given as its fp16 image (gemm_prepare_image(.., to_f16 = true));
// epilogues as form 0: bias; bias + GeLU (C and gelu_out written as fp16); bias + fp32 residual
// (C fp32 or bf16 as ep.out_f32 says).  Without a residual C is written as fp16.  Any M, N % 8 == 0,
// K % 128 == 0.
bool gemm_fwd_f16_supported(int M, int N, int K);
hipError_t gemm_fwd_f16(int M, int N, int K, const void* A, const void* b_image, void* C,
                        const GemmEpilogue& ep, hipStream_t st);
hipError_t gemm_mfma(int form, int M, int N, int K, const void* A, const void* B, void* C,
                     const GemmEpilogue& ep, hipStream_t st);
// Weight gradients dw[M,N] += dout[K,M]^T in[K,N] of n <= kMaxWgrads linears over the same tokens, in one
// launch where that gains, bit for bit what gemm_mfma() gives for each; every shape gemm_mfma_supported(), with segments
// (see GemmEpilogue) gemm_wgrad_segments_supported().
struct WgradItem {
  int M, N;
  const void* dout;
  const void* in;
  float* dw;
};
// sums (n_sums of them, each of one micro-batch): what reduce_partials() would do, in the launch of the products, or in one of
// its own behind them where they are a launch each.
constexpr int kMaxWgrads = 4;
hipError_t gemm_wgrad_group(const WgradItem* items, int n, int K, int segments, size_t seg_stride_dout,
                            size_t seg_stride_in, hipStream_t st, const ReduceSeg* sums = nullptr, int n_sums = 0);
// the same for fp32 buffers, every shape and buffer gemm_f32_supported(); the sums in the last launch, whatever their number
hipError_t gemm_f32_wgrad_group(const WgradItem* items, int n, int K, hipStream_t st, const ReduceSeg* sums = nullptr,
                                int n_sums = 0);
bool gemm_wgrad_segments_supported(int M, int N, int K, int segments);
// rows of GemmEpilogue::colsum_partial that gemm_mfma() writes for an [M,N] product
int gemm_mfma_colsum_rows(int M, int N, int K);

hipError_t attention_fwd_simple(int dtype, int B, int S, int a, int d, const void* qkv, void* out,
                                float* lse, hipStream_t st);
hipError_t attention_bwd_simple(int dtype, int B, int S, int a, int d, const void* qkv,
                                const void* out, const float* lse, const void* dout, void* dqkv,
                                float* delta, hipStream_t st);

// fp32 attention on the matrix cores (head_dim 32, 64 or 128): every buffer 16-byte aligned (null
// pointers count as aligned).  No scratch memory.
bool attention_f32_supported(const void* qkv, const void* out, const void* dout, const void* dqkv);
hipError_t attention_fwd_f32(int B, int S, int a, int d, const void* qkv, void* out, float* lse, hipStream_t st);
hipError_t attention_bwd_f32(int B, int S, int a, int d, const void* qkv, const void* out, const float* lse,
                             const void* dout, void* dqkv, hipStream_t st);

// bf16 MFMA attention (head_dim 32, 64 or 128).  scratch (backward: delta): device memory of
// attention_mfma_scratch_bytes(B, S, a, d, 1) bytes; phase 0: what the forward entry points ask for, see there.
bool attention_mfma_supported(int B, int S, int a, int d);   // head_dim 32/64/128 and index ranges
size_t attention_mfma_scratch_bytes(int B, int S, int a, int d, int phase);
// f16: qkv and out are fp16 (forward activations kept in fp16); lse is fp32 either way.
// n micro-batches of B sequences: qkv, out and lse lie `stride` bytes apart.
hipError_t attention_fwd_mfma(int B, int S, int a, int d, const void* qkv, void* out, float* lse,
                              hipStream_t st, bool f16 = false, int n = 1, size_t stride = 0);
// qkv_f16 (optional): the fp16 qkv of an fp16 forward pass; the logits are then recomputed from
// its Q and K, `out` is that pass's fp16 output (it only enters delta = rowsum(dO * O)), and
// qkv is the bf16 copy that every other product reads.
// n micro-batches: qkv, out, lse, dout and scratch lie `act` bytes apart, dqkv `grad`.
hipError_t attention_bwd_mfma(int B, int S, int a, int d, const void* qkv, const void* out,
                              const float* lse, const void* dout, void* dqkv, void* scratch,
                              hipStream_t st, const void* qkv_f16 = nullptr, int n = 1, size_t act = 0, size_t grad = 0);

// ---- a chunk's window of micro-batches as one pass per operator (stage.hip, for dpp.hip) ----
// How many of a window of W micro-batches, their stashes `act_stride` and `grad_stride` bytes apart, a pass takes; 1:
// none, they go one by one.
int stage_window(const gpt_stage_params* p, int W, size_t act_stride, size_t grad_stride);
// The forward phase of n micro-batches, their stashes `act_stride` and `grad_stride` bytes apart.  y[m] may be x[m].  The
// gradient stashes only lend room: buffers that are not equally spaced go through it.
int stage_fwd_window(const gpt_stage_params* p, int n, const void* const* x, void* act_stash, size_t act_stride,
                     void* const* y, void* grad_stash, size_t grad_stride, hipStream_t st);
// Their backward data phase.  It overwrites the parts of the activation stashes that the weight phase does not read.
// dx[m] may be dy[m].
int stage_bwd_window(const gpt_stage_params* p, int n, void* act_stash, size_t act_stride, const void* const* dy,
                     void* const* dx, void* dparams, void* grad_stash, size_t grad_stride, hipStream_t st);

// Records the thread's error text and returns `code` (for sources outside stage.hip).
int set_error(int code, const char* msg);

}  // namespace gpts
