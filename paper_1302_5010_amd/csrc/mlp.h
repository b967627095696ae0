// Launchers of the learned-proposal kernels (mlp.hip).  Internal; the public
// entry points are the bmpl_mlp_* calls of include/bmpl.h.
//
// Matrix products C = X W^T: X [M][ldx] and W [N][ldw] bfloat16 (raw 16-bit storage), both
// K-contiguous with kpad % 64 == 0 and zeros in columns past the true contraction length.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bmpl {

constexpr int TOPK_MAX = 38912;   // entries per row of the top-k kernel (38 float4 per thread)

hipError_t mlp_project(const float* At, int64_t lda, int n, int m, const float* P, int d, uint16_t* APt, int npad,
                       hipStream_t s);
hipError_t mlp_signals_bf16(const float* B, int64_t ldb, int n, int p, uint16_t* B16, int npad, hipStream_t s);
// C[r][c] = (X W^T)[r][c] (+ bias[c])
hipError_t mlp_gemm_store(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                          float* C, int64_t ldc, const float* bias, hipStream_t s);
// u = (X W^T)[r][c] + bias[c]; U[r][c] = u when U != null; H[r][c] = bf16(gelu(u))
hipError_t mlp_gemm_bias_gelu(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                              const float* bias, float* U, int64_t ldu, uint16_t* H, int64_t ldh, hipStream_t s);
// d = (X W^T)[r][c] * gelu'(U[r][c]); D = d (float32), D16 = bf16(d)
hipError_t mlp_gemm_gelu_back(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                              const float* U, int64_t ldu, float* D, int64_t ldd, uint16_t* D16, int64_t ld16,
                              hipStream_t s);
// X0[r] = bf16(Z[r] sqrt(d) / ||Z[r]||); Zout (optional) receives X0 widened to float32
hipError_t mlp_embed_norm(const float* Z, int d, int p, uint16_t* X0, float* Zout, int64_t ldz_out, hipStream_t s);
// Weighted BCE with logits S [rows][lds >= mpad], mpad % 64 == 0: D16 = bf16(dl/ds / rows) (zero past m), DT its
// transpose [m][ldt] (zero for rows up to the next multiple of 64), colpart [ceil(rows / 64)][ldc] and rowpart
// [mpad / 64][ldr] the 64 x 64 tiles' sums of dl/ds over rows and of the loss over columns (mlp_partial_sums).
hipError_t mlp_bce_tiles(const float* S, int64_t lds, uint16_t* D16, int64_t ld16, uint16_t* DT, int64_t ldt, int m,
                         int mpad, int rows, const int* supp, int64_t ld_supp, const int* supp_len, float pos_w,
                         double* colpart, int64_t ldc, double* rowpart, int64_t ldr, hipStream_t s);
// DT[c][r] = bf16(in[r][c]) (zero rows as above), colpart the tiles' column sums; cols % 64 == 0
hipError_t mlp_transpose_colsum(const float* in, int64_t ld, int rows, int cols, uint16_t* DT, int64_t ldt,
                                double* colpart, int64_t ldc, hipStream_t s);
// The bias gradients out[q][c < cols[q]] and the mean loss from the tiles' partial sums.
struct PartialSums {
    const double* part[3]; int64_t ldc[3]; int cols[3]; float* out[3];
    const double* rowpart; int64_t ldr; int tile_cols; int rows; float* rowloss;
    int start[4]; int tile_rows;   // set by the launcher
};
hipError_t mlp_partial_sums(PartialSums a, double* loss, hipStream_t s);
// out[c][r] = in[r][c]; zero for rows <= r < ldo (ldo % 64 == 0, cols % 8 == 0); up to three in one launch
struct TransposeJob { const uint16_t* in; int64_t ldi; int rows, cols; uint16_t* out; int64_t ldo; };
struct TransposeJobs { TransposeJob job[3]; int start[3]; };
hipError_t mlp_transposes(const TransposeJob* jobs, int count, hipStream_t s);
hipError_t mlp_adam(float* P, float* m1, float* m2, const float* g, uint16_t* P16, int64_t count, float lr,
                    float beta1, float beta2, float eps, float bc1, float bc2, hipStream_t s);
hipError_t mlp_params_bf16(const float* P, uint16_t* P16, int64_t count, hipStream_t s);
// top-k indices per row of S [rows][lds] (first L columns), ascending by index, -1 padded
hipError_t mlp_topk(const float* S, int64_t lds, int rows, int L, int k, int* out, int64_t ldo, hipStream_t s);

}  // namespace bmpl
