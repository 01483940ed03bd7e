// Internal launch interface between the kernel files and the module / C-ABI layer.
// Every function enqueues on `s` and returns without synchronising.  `quota` is the CU
// count the persistent grid is sized for.
#pragma once
#include "common.h"

// whether pn bytes at p and qn bytes at q share any; nothing overlaps a null pointer
inline bool overlap(const void* p, int64_t pn, const void* q, int64_t qn) {
  return p && q && (uintptr_t)p < (uintptr_t)q + (uintptr_t)qn && (uintptr_t)q < (uintptr_t)p + (uintptr_t)pn;
}

// ------------------------------------------------------------------------------ GEMM
// C[M,N] = op(A) op(B) (+ bias[N]) (+ R[M,N]), fp32 accumulation in ascending k.
//   a_kc: A is stored [M,K] (K contiguous) else [K,M];  b_kc: B is stored [N,K] else [K,N].
// fprop  Y = X W      : A = X  [T,k] a_kc=1, B = W  [k,n] b_kc=0
// dgrad  dX = dY W^T  : A = dY [T,n] a_kc=1, B = W  [k,n] b_kc=1 (contraction over n)
// wgrad  dW = X^T dY  : A = X  [T,k] a_kc=0, B = dY [T,n] b_kc=0 (contraction over T)
// Padded rows: with lda >= M rounded up to 8, a K-strided A may have any M (its rows must be
// readable up to that width).  b_rows >= 0: a K-strided B has only that many of its K rows; the
// columns of A past them must hold zeros.
mosaic_status launch_gemm(hipStream_t s, int quota, int dtype, bool a_kc, bool b_kc,
                          int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                          const void* B, int64_t ldb, void* C, int64_t ldc,
                          const void* bias, const void* R, void* splitk_scratch = nullptr, int64_t b_rows = -1);
// Bytes of fp32 scratch the weight-gradient form wants for a deterministic split of a long
// contraction over few output tiles (0 when no split is used for this shape).
size_t gemm_splitk_scratch_bytes(int64_t M, int64_t N, int64_t K);
// Y[b, t, :] = X[b, t, :] W + bias + table[t, :]: B x rows patches of k values, ldx apart (zeros past k), W [k, n].  One rounding
// where the bf16 matrix-core kernel takes the product and the table in its epilogue, else the product and add_pos.
mosaic_status launch_embed_fwd(hipStream_t s, int quota, int dtype, int64_t B, int64_t rows, int64_t n, int64_t k, int64_t ldx, const void* X,
                               const void* W, const void* bias, const void* table, void* Y);
// Z[T,n] = X[T,k] W[k,n] (+ bias[n]) and A = act(Z): GELU / tanh GELU give A[T,n]; SwiGLU reads Z
// as [gate | up] halves and gives A[T,n/2] = silu(gate) * up.  Where the bf16 matrix-core kernel
// takes the product, and for small fp32 products, the activation is applied in its epilogue (same bits as the separate pass);
// otherwise the elementwise kernel follows the product.  fp32: A may lie on X, W or the bias, or be Z (GELU); the elementwise kernel then follows.
mosaic_status launch_linear_act_fwd(hipStream_t s, int quota, int dtype, int act, int64_t T, int64_t k, int64_t n,
                                    const void* X, const void* W, const void* bias, void* Z, void* A);
// Z = X W + bias over samples of 2 lo rows (of X, ldx apart, zeros past k), and P [B lo, 3n] = the gathered input of a three-tap convolution of stride 2 over
// gelu(Z) (launch_im2col1d): written by the epilogue where the bf16 matrix-core kernel takes the product, else through A [2 B lo, n];
// the same bits.
mosaic_status launch_gelu_taps_fwd(hipStream_t s, int quota, int dtype, int64_t B, int64_t lo, int64_t n, int64_t k, int64_t ldx, const void* X, const void* W,
                                   const void* bias, void* Z, void* A, void* P);
// dW[k,n] = X^T dY and dX[T,k] = dY W^T, dense rows (X's ldx apart; 0: k); one launch where that is the faster way, else two, the input gradient's
// first or last (1 - 2 % of a layer either way, by what the caches still hold)
mosaic_status launch_linear_bwd(hipStream_t s, int quota, int dtype, int64_t T, int64_t k, int64_t n, const void* X, const void* dY,
                                const void* W, void* dX, void* dW, void* splitk_scratch, bool dx_first, int64_t ldx = 0);

// U = norm(X), stats, then Z[T,n] = U W (+ bias) and, act >= 0, A = act(Z): one launch for small fp32 layers, else launch_norm_fwd and
// launch_gemm or launch_linear_act_fwd
mosaic_status launch_norm_linear_fwd(hipStream_t s, int quota, int dtype, int norm, int act, int64_t T, int64_t h, int64_t n, float eps, const void* X,
                                     const void* gamma, const void* beta, void* U, float* stats, const void* W, const void* bias, void* Z, void* A);
// The backward pass of Y = act(Z) W: dW = act(Z)^T dY with A = act(Z)[T,k], and dZ = act'(Z) (dY W^T) in one launch with it for small fp32 layers, else
// through dA[T,k].  colsum (may be null; GELU): the column sums of dZ, partial sums in `scratch`, the last pass in `later`.
struct ColReduceList;
mosaic_status launch_act_linear_bwd(hipStream_t s, int quota, int dtype, int act, int64_t T, int64_t k, int64_t n, const void* Z, const void* A, const void* dY,
                                    const void* W, void* dA, void* dZ, void* dW, void* splitk_scratch, void* colsum, void* scratch, ColReduceList* later);

// ------------------------------------------------------------------------- attention
// packed rows [q (H heads) | k (Hkv heads) | v (Hkv heads)]; Hkv divides H; query head t
// attends to key/value head t / (H/Hkv)
mosaic_status launch_attention_fwd(hipStream_t s, int quota, int dtype, int B, int N, int H, int Hkv,
                                   int d, int causal, const void* qkv, void* O, float* lse);
mosaic_status launch_attention_bwd(hipStream_t s, int quota, int dtype, int B, int N, int H, int Hkv,
                                   int d, int causal, const void* qkv, const void* O,
                                   const float* lse, const void* dO, void* dqkv, float* delta);

// ----------------------------------------------------------- norms and elementwise
mosaic_status launch_norm_fwd(hipStream_t s, int quota, int dtype, int norm, int64_t T,
                              int64_t h, float eps, const void* x, const void* gamma,
                              const void* beta, void* y, float* stats);
// A column reduction whose partial sums are written and whose final pass is not: out[col] = sum_p partial[p * ld + col] for
// col < ncols, columns from `split` on to out1, from `split2` on to out2 (a null destination skips its columns).  The backward
// pass of a layer collects those of its norms and biases and launches them together; each keeps its partial sums
// in scratch of its own until then.
struct ColReduce {
  const float* partial;
  int np;
  int64_t ld, ncols, split, split2;
  void *out0, *out1, *out2;
};
// Partial column sums of X[rows, n] that have not been formed yet: the next byte-bound kernel of the list's layer takes them along in its
// launch (a pass of its own costs 4 to 5 us however small), or the final reduction launches them first.  np == 0: none.
struct ColSumJob {
  const void* X = nullptr;
  float* partial = nullptr;
  int64_t rows = 0, n = 0;
  int rp = 0, np = 0, ctiles = 0;
};
struct ColReduceList {
  static constexpr int kMax = 6;
  ColReduce job[kMax];
  int n = 0;
  ColSumJob pending;
  // a loss whose partial sums launch_mse left here: loss = loss_scale * their sum, formed beside the column sums
  const float* loss_partial = nullptr;
  float* loss = nullptr;
  int loss_np = 0;
  float loss_scale = 0.f;
};
mosaic_status launch_col_reduce(hipStream_t s, int quota, int dtype, const ColReduceList& list);
// scratch of launch_norm_bwd: two slabs of partial sums per row partition, a third when dxsum is asked for
size_t norm_bwd_scratch_bytes(int64_t h, bool with_dxsum = true);
mosaic_status launch_norm_bwd(hipStream_t s, int quota, int dtype, int norm, int64_t T,
                              int64_t h, const void* x, const void* gamma, const float* stats,
                              const void* dy, const void* R, void* dx, void* dgamma,
                              void* dbeta, void* scratch, void* dxsum = nullptr, ColReduceList* later = nullptr);
// dxsum (may be null): receives the column sums of dx[T,h] as stored, in the fixed two-level
// order of launch_colsum's partitions; formed inside the norm kernel where it has a variant
// for that (LayerNorm rows of up to 2048 bf16 / 1024 fp32 elements), by a pass over dx otherwise.
// later (here and below; may be null): the final pass of the column sums is appended there and not launched
mosaic_status launch_gelu_fwd(hipStream_t s, int quota, int dtype, int64_t n, const void* z, void* a);
mosaic_status launch_gelu_bwd(hipStream_t s, int quota, int dtype, int64_t n, const void* z,
                              const void* da, void* dz);
// dz = da * gelu'(z) and colsum[n] = column sums of dz[T,n] as stored (same bits as launch_colsum
// over dz); scratch: colsum_scratch_bytes(n).  taps_lo > 0: T rows are samples of 2 * taps_lo positions, the input of a three-tap
// convolution of stride 2, and da is the gradient [T / 2, 3n] of its gathered input (launch_im2col1d)
mosaic_status launch_gelu_bwd_colsum(hipStream_t s, int quota, int dtype, int64_t T, int64_t n, const void* z,
                                     const void* da, void* dz, void* colsum, void* scratch, ColReduceList* later = nullptr, int taps_lo = 0);
mosaic_status launch_swiglu_fwd(hipStream_t s, int quota, int dtype, int64_t T, int64_t f,
                                const void* gu, void* a);
mosaic_status launch_swiglu_bwd(hipStream_t s, int quota, int dtype, int64_t T, int64_t f,
                                const void* gu, const void* da, void* dgu);
// ------------------------------------------------------------------- layer variants
mosaic_status launch_gelu_tanh_fwd(hipStream_t s, int quota, int dtype, int64_t n, const void* z, void* a);
mosaic_status launch_gelu_tanh_bwd(hipStream_t s, int quota, int dtype, int64_t n, const void* z,
                                   const void* da, void* dz);
// (cos, sin) of n * base^(-2i/d) for n < N, i < d/2, as float2[N][d/2]
size_t rope_table_bytes(int N, int d);
mosaic_status launch_rope_table(hipStream_t s, int quota, int N, int d, float base, void* table);
// rotates the q and k parts of packed [B*N, (H+2*Hkv)*d] rows in place; direction -1 turns back
mosaic_status launch_rope(hipStream_t s, int quota, int dtype, int B, int N, int H, int Hkv, int d,
                          int direction, void* qkv, const void* table);
// p, m, v (and master, if not null) updated in place; m, v, master are fp32
mosaic_status launch_adamw(hipStream_t s, int quota, int dtype, int64_t n, void* p, const void* g,
                           float* m, float* v, float* master, float lr, float beta1, float beta2,
                           float eps, float weight_decay, int64_t step);
// k=3, pad=1 convolution over frames-major [B, L, C] as gather + GEMM: out [B*Lo, 3*C] with
// column index tap*C + channel; col2im1d is the transposed gather at stride 1 (one owner per element)
mosaic_status launch_im2col1d(hipStream_t s, int quota, int dtype, int64_t B, int L, int Lo, int C,
                              int stride, const void* x, void* out, int64_t ld = 0);      // rows ld >= 3C apart (0: 3C), zeros between
mosaic_status launch_col2im1d(hipStream_t s, int quota, int dtype, int64_t B, int L, int C, const void* dP, void* dx);
size_t mse_scratch_bytes();
mosaic_status launch_mse(hipStream_t s, int quota, int dtype, int64_t n, const void* y,
                         const void* target, void* dy, float* loss, void* scratch, ColReduceList* later = nullptr);
size_t colsum_scratch_bytes(int64_t n);
int64_t colsum_partition_rows(int64_t T);      // rows of a partition; each is summed in ascending order (colsum_quarters aside)
// out[n] = sum over T rows of X[T,n] in a fixed two-level order.
// in_passing: the partial sums may be left to a later kernel (ColSumJob); X has to stay as it is until then
mosaic_status launch_colsum(hipStream_t s, int quota, int dtype, int64_t T, int64_t n,
                            const void* X, void* out, void* scratch, ColReduceList* later = nullptr, bool in_passing = false);

// ----------------------------------------------------------------------------- stems
// rows of `out` are ld elements apart (whole 16-byte pieces), zeros past 3*patch*patch
mosaic_status launch_unfold(hipStream_t s, int quota, int dtype, int B, int side, int patch,
                            const void* img, void* out, int ld);
// y[b*N+t, :] += pos[t, :]
mosaic_status launch_add_pos(hipStream_t s, int quota, int dtype, int B, int N, int h,
                             const void* pos, void* y);
// dpos[t,:] = sum_b dy[b*N+t,:] in ascending b
mosaic_status launch_pos_grad(hipStream_t s, int quota, int dtype, int B, int N, int h,
                              const void* dy, void* dpos);
// launch_pos_grad, and colsum[h] = the column sums of dy over all positions and samples; scratch: colsum_scratch_bytes(h)
mosaic_status launch_stem_grad(hipStream_t s, int quota, int dtype, int B, int N, int h, const void* dy, void* dpos, void* colsum, void* scratch);
// out rows: per sample b, [0,n_b) from img_tok, [n_b,N) from table[ids]; n_b = n_img, or
// counts[b] (clamped to [0,n_img]) when counts is given; ids is [B, N-n_img] without counts and
// one id per sequence position, [B, N], with them
mosaic_status launch_text_stem_fwd(hipStream_t s, int quota, int dtype, int B, int N, int n_img,
                                   int h, int vocab, const void* img_tok, const int32_t* ids,
                                   const int32_t* counts, const void* table, void* out);
// d_img rows from dy (zero for image tokens a sample did not use); dtable[v] = sum over
// occurrences of v in an order that the ids alone fix.  scratch: text_stem_scratch_bytes, 256-byte aligned
size_t text_stem_scratch_bytes(int64_t T, int64_t h);
mosaic_status launch_text_stem_bwd(hipStream_t s, int quota, int dtype, int B, int N, int n_img,
                                   int h, int vocab, const void* dy, const int32_t* ids,
                                   const int32_t* counts, void* d_img, void* dtable, void* scratch);
