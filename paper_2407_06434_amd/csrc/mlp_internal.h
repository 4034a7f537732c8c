// Internal declarations of the learned support proposal (network kernels and
// their host driver). Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "omp_internal.h"

namespace bomp {

// Epilogues of the BF16 "NT" product C[m][n] = sum_k P[m][k] Q[n][k].
enum {
  EPI_FEATURES = 0,  // out bf16 = |c| * colscale[n] * rowscale[m] * scale
  EPI_BIAS_RELU = 1, // out bf16 = relu(c + bias[n])
  EPI_BIAS = 2,      // out f32  = c + bias[n]
  EPI_BCE = 3,       // out bf16 = (sigmoid(c + bias[n]) - t[m][n]) * scale; loss terms per block
  EPI_RELU_MASK = 4, // out bf16 = c where mask[m][n] > 0, else 0
  EPI_PARTIAL = 5,   // out f32 [split][m][n] = this split's partial sum
};

struct GemmEpi {
  void *out;
  int64_t ldo;               // output row stride (elements)
  const float *bias;         // [n]
  const float *colscale;     // [n]
  const float *rowscale;     // [m]
  const uint16_t *mask;      // [m][ldo] BF16 activations (EPI_RELU_MASK)
  const uint32_t *labels;    // [m][ldl] multi-hot bits (EPI_BCE)
  int64_t ldl;
  int64_t mvalid;            // rows below this are real signals (EPI_BCE)
  float scale;               // EPI_BCE: 1 / batch; EPI_FEATURES: sqrt(M)
  float *loss_part;          // EPI_BCE: one partial per block
};

// One layer's parameters and optimiser state (device pointers).
struct LayerView {
  int64_t n_in, n_out;
  float *W32;      // [out][in] FP32 master weights
  uint16_t *W16;   // [out][in] BF16 copy (forward operand)
  uint16_t *W16T;  // [in][out] BF16 transposed copy (backward operand)
  float *b32;      // [out]
  float *mW, *vW;  // Adam moments of W
  float *mb, *vb;  // Adam moments of b
};

int64_t loss_blocks(int64_t M, int64_t N);  // workgroups, so loss partials, of an EPI_BCE product
hipError_t launch_gemm_bf16(int epi, const uint16_t *P, int64_t ldp, const uint16_t *Q, int64_t ldq, int64_t M,
                            int64_t N, int64_t K, const GemmEpi &e, hipStream_t st);
hipError_t launch_prep_signals(const float *Y, int64_t ldy, int64_t B, int64_t M, int64_t Mp, int64_t Bp,
                               uint16_t *Y16, float *yinv, hipStream_t st);
// With `sup`: the rows' multi-hot labels into bits [Bp][n_out / 32] too.
hipError_t launch_pad_rows16(const uint16_t *src, int64_t ld, const int32_t *rows, int64_t B, int64_t cols,
                             int64_t Bp, uint16_t *dst, hipStream_t st, const int32_t *sup = nullptr, int S = 0,
                             int64_t n_out = 0, uint32_t *bits = nullptr);
// Six transposes in one launch, with column sums per group of transpose_rows(R) rows where
// `part` is set (at most COLSUM_GROUPS groups).
constexpr int COLSUM_GROUPS = 16;
struct TransposeBatch {
  const uint16_t *src[6];  // [R][cols]
  uint16_t *dst[6];        // [cols][R]
  float *part[6];          // [groups][cols] or nullptr
  int64_t cols[6], end[6];  // end: filled by the launcher
};
int64_t transpose_rows(int64_t R);
hipError_t launch_transposes16(TransposeBatch g, int64_t R, hipStream_t st);
// dW_l [rows][in] = dOutT_l [rows][K] InT_l [in][K]^T for the three layers; with `splits`
// slices of K, out_l holds [splits][rows][in] partial sums.
constexpr int WSPLITS_MAX = 4;
struct WgradBatch {
  const uint16_t *dOutT[3], *InT[3];
  float *out[3];
  int64_t rows[3], in[3], end[3];  // end: filled by the launcher
};
int wgrad_splits(const WgradBatch &g, int64_t K);
hipError_t launch_wgrad(const WgradBatch &g, int64_t K, int splits, hipStream_t st);
// out_m[i] = sum over parts_m (at most 16) of part_m[.][i] (out nullptr: left out), and the loss.
struct SumBatch {
  const float *part[6];
  float *out[6];
  int64_t n[6], end[6];  // end: filled by the launcher
  int parts[6];
};
hipError_t launch_grad_sums(SumBatch g, const float *loss_part, int64_t nloss, float scale, float *loss_out,
                            hipStream_t st);
hipError_t launch_adam_w(const LayerView &L, const float *gpart, int splits, float lr, float b1, float b2, float eps,
                         float c1, float c2, int update, hipStream_t st);
hipError_t launch_adam_b(const LayerView &L, const float *gpart, int chunks, float lr, float b1, float b2, float eps,
                         float c1, float c2, hipStream_t st);
hipError_t launch_copy32(const float *src, int64_t n, float *dst, hipStream_t st);
hipError_t launch_topk(const float *Z, int64_t ldz, int64_t N, int64_t B, int S, int32_t *P, hipStream_t st);
hipError_t launch_ls_check(const DictView &d, const float *Y, int64_t ldy, int64_t B, const int32_t *P, int S,
                           const float *eps_per, float eps, int32_t *support_out, float *coef_out, int32_t *status_out,
                           float *rnorm_out, int32_t *accept, hipStream_t st);
hipError_t launch_compact(const int32_t *accept, int64_t B, int32_t *idx, int32_t *count, hipStream_t st);
hipError_t launch_gather_rejects(const float *Y, int64_t ldy, int64_t M, const float *eps_per, float eps,
                                 const int32_t *idx, int64_t n, float *Yr, float *eps_r, hipStream_t st);
hipError_t launch_scatter_fallback(const int32_t *idx, int64_t n, int S, const int32_t *sup_r, const float *coef_r,
                                   const int32_t *st_r, const float *rn_r, int32_t *support_out, float *coef_out,
                                   int32_t *status_out, float *rnorm_out, hipStream_t st);

}  // namespace bomp
