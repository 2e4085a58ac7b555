// Internal interface of the surrogate-network kernels (k_mlp.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pcmd.h"

namespace pcmd {

enum { EPI_STORE = 0, EPI_BIAS = 1, EPI_BIAS_GELU = 2, EPI_GELU_GRAD = 3, EPI_BIAS_MSE = 4 };

// C[M][N] = sum_k A(m, k) B(n, k) with the operand layouts of k_gemm and a fused epilogue.
struct GemmArgs {
  int M, N, K;
  const __bf16 *A;
  int lda;
  const __bf16 *B;
  int ldb;
  float *C;           // FP32 output (EPI_STORE, EPI_BIAS; EPI_BIAS_GELU unless NULL)
  int ldc;
  __bf16 *Cb;         // BF16 output (EPI_BIAS_GELU: GELU(z); EPI_GELU_GRAD: dz_prev)
  int ldcb;
  const float *bias;  // [N]
  const float *Z;     // FP32 pre-activations for GELU' (EPI_GELU_GRAD)
  int ldz;
  float *part;        // split-K partial products [splits][M][N] (set by launch_gemm)
  int kchunk;         // K elements per split (a multiple of the K step; set by launch_gemm)
  int nz;             // K ranges over blocks (set by launch_gemm)
  // A given in FP32 instead (A unused): row m is row rows[m] of A32 (m when rows is NULL; a row outside
  // [0, n_total) is taken as row 0 and sets STATUS_BAD_ROW), rounded to BF16 and, unless Aout is NULL,
  // also written there [M][lda].  Only where gemm_reads_f32(M, N, K).
  const float *A32;
  const int32_t *rows;
  int64_t n_total;
  __bf16 *Aout;
  uint32_t *status;
  // EPI_BIAS_MSE: y = product + bias is compared with the target rows (by the row vector, as A32's) of
  // T [n_total][N]: 2 (y - T) scale = gscale (y - T) in BF16 to Cb (unless NULL) and the squared errors'
  // sums to lpart[gemm_loss_parts(M, N, K)]; y itself is not stored
  const float *T;
  float gscale;
  double *lpart;
};

// Every layer's parameters, packed as in pcmd_mlp (off: W_l in master, adam_m, adam_v and grad, b_l
// after it; woff: in the BF16 copies).
struct AdamArgs {
  int n_layers, update;
  int dims[PCMD_MLP_MAX_LAYERS + 1];
  int first[PCMD_MLP_MAX_LAYERS + 1];  // set by launch_adam
  int64_t off[PCMD_MLP_MAX_LAYERS], woff[PCMD_MLP_MAX_LAYERS];
  float *master, *m, *v;
  const float *grad;
  void *w_bf16, *wt_bf16;
  float lr, beta1, beta2, eps, bc1, bc2;
};

// Partial sums that an EPI_BIAS_MSE product writes (0: this shape cannot take that epilogue).
int64_t gemm_loss_parts(int M, int N, int K);
// Whether a product of these sizes takes A in FP32 (A32): where that is faster than rounding it first.
bool gemm_reads_f32(int M, int N, int K);
// Workspace (bytes) launch_gemm needs for an M x N x K product: transposed copies of K-major
// operands (at: A(m, k) = A[k][m]; bt: B(n, k) = B[k][n]) where its tiles do not read them in place, and split-K
// partials.
size_t gemm_workspace_bytes(int M, int N, int K, bool at, bool bt);
hipError_t launch_gemm(const GemmArgs &g, bool at, bool bt, int epi, void *ws, size_t ws_bytes, hipStream_t s);
hipError_t launch_f32_to_bf16(const float *x, void *y, int64_t n, hipStream_t s);
// y[k][j] = bf16(x[row k][j]), row k = rows[k] (or k when rows is NULL; rows outside [0, n_total)
// read row 0 and set STATUS_BAD_ROW).
hipError_t launch_gather_f32_to_bf16(const float *x, const int32_t *rows, int64_t n_total, int d, int64_t n, void *y,
                                     uint32_t *status, hipStream_t s);
// Per-block partial sums of the squared error of y [n / M][M] against the target rows (as in the
// gather) and the BF16 gradient 2 (y - t) scale into dy (unless NULL).  part holds MSE_BLOCKS doubles.
constexpr int MSE_BLOCKS = 256;
hipError_t launch_mse_grad(const float *y, const float *t, int64_t n, int M, const int32_t *rows, int64_t n_total,
                           double scale, void *dy, double *part, uint32_t *status, hipStream_t s);
// out[0] = scale x the sum of part[0 .. nb) in an order fixed by nb.
hipError_t launch_sum_partials(const double *part, int64_t nb, double scale, double *out, hipStream_t s);
hipError_t launch_sum_partials(const double *part, int64_t nb, double scale, float *out, hipStream_t s);
// out[r][j] = ln((h[r][j] + 1/2) / (N_r + nbins / 2)) for n rows of nbins counts.
hipError_t launch_log_hess_target(const uint32_t *h, int n, int nbins, float *out, hipStream_t s);
// One layer's backward pass: the weight gradient w (EPI_STORE, both operands K-major), the bias gradient c
// and, unless x is NULL, the layer below's dz (EPI_GELU_GRAD); in one launch where that pays.
struct ColsumArgs {  // db[m] = sum_n dz[n][m]
  const __bf16 *dz;
  int n, m;
  float *db;
};
hipError_t launch_backward(const GemmArgs &w, const GemmArgs *x, const ColsumArgs &c, void *ws, size_t ws_bytes, hipStream_t s);
hipError_t launch_adam(AdamArgs a, hipStream_t s);
// lnfact64[k] = ln k! for k < nlf (Stirling's series beyond; nlf >= 1000)
hipError_t launch_surrogate_loglike(const float *y, int n, int nbins, const uint32_t *d, double *out,
                                   const double *lnfact64, int nlf, hipStream_t s);

}  // namespace pcmd
