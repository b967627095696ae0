// Kernels of the learned support proposal: a small network that scores every
// atom for a signal so that the pursuit can start from a good active set
// (the warm start of Algorithm 1, step 5, taken from outside the method; the
// natural stopping condition, Eq. (9), still certifies the result).
//
//   embedding   z = (A P)^T b, then scaled to unit root-mean-square
//   network     h1 = gelu(W1 z + b1), h2 = gelu(W2 h1 + b2), s = W3 h2 + b3
//   loss        binary cross-entropy with logits, positive-class weight w
//   training    gradients by the chain rule, Adam with float32 master weights
//   proposal    the k largest scores per signal (radix select, ties to the lower index)
//
// Precision: weights and activations in bfloat16 for the matrix products,
// float32 accumulation, float32 pre-activations, logits, gradients and
// optimiser state.  All products C = X W^T run on the shared MFMA tile loop
// with both operands K-contiguous; the backward products that contract over
// the batch or the output width use bfloat16 transposes made for them.
#include <float.h>
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "bmpl_internal.h"
#include "gemm_tile.h"
#include "mlp.h"
#include "wave_ops.h"

namespace bmpl {
namespace {

__device__ inline float bf16_to_f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline float gelu_f(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)); }

__device__ inline float gelu_prime_f(float u)
{
    return 0.5f * (1.0f + erff(u * 0.70710678118654752f)) + u * 0.39894228040143268f * expf(-0.5f * u * u);
}

// ---------------------------------------------------------------------------
// Epilogues of C = X W^T, called once per 32 x 32 block of a wave: column c = c0 + l32 (a column below N), rows
// r0 + 4 h + 8 (r / 4) + r % 4 for r < 16 with values v[r], rows below M stored (all of them when FULL).  r0 and c0
// are the same in every lane, so a row's address is scalar arithmetic and a lane's part of it one 32-bit offset.
// What a column shares (col: the bias) is loaded before the tile's first store and what a block needs from memory
// (U) before the block's: a load behind a store waits until the store has been acknowledged, and the compiler has to
// assume that a store changes what is loaded, so the bias read at each element cost 128 such waits per tile (scores
// of 4096 signals, 2048 -> 20000: 446 -> 352 us with the loop of mfma_tile_loop_pipe, of which 15 are the loop's).
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ T* epi_row(T* base, int64_t ld, int r0, int c0, int r)
{
    return base + (int64_t)(r0 + 8 * (r >> 2) + (r & 3)) * ld + c0;
}
// The 32-bit lane offset holds for rows of at most EPI_LD_MAX entries (16 ldc + 128 bytes).
constexpr int64_t EPI_LD_MAX = 1 << 26;
// FAR: rows longer than that, a 64-bit offset per lane.
template <bool BIAS, bool FAR = false>
struct EpiStore {            // C[r][c] = v (+ bias[c])
    static constexpr bool TILE256 = !FAR;   // (rows of 256 MB: not worth kernels of its own)
    float* C; int64_t ldc; const float* bias;
    __device__ __forceinline__ float col(int c) const { return BIAS ? bias[c] : 0.f; }
    template <bool FULL>
    __device__ __forceinline__ void block(const floatx16& v, float b, int r0, int c0, int h, int l32, int M) const
    {
        using Off = std::conditional_t<FAR, uint64_t, uint32_t>;
        const Off off = 4 * ((Off)(4 * h) * (Off)ldc + (Off)l32);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (FULL || r0 + 4 * h + 8 * (r >> 2) + (r & 3) < M)
                at_bytes(epi_row(C, ldc, r0, c0, r), off) = BIAS ? v[r] + b : v[r];
    }
};
struct EpiBiasGelu {         // u = v + bias[c]; U[r][c] = u (if kept); H[r][c] = bf16(gelu(u))
    static constexpr bool TILE256 = true;
    const float* bias; float* U; int64_t ldu; uint16_t* H; int64_t ldh;
    __device__ __forceinline__ float col(int c) const { return bias[c]; }
    template <bool FULL>
    __device__ __forceinline__ void block(const floatx16& v, float b, int r0, int c0, int h, int l32, int M) const
    {
        const uint32_t offu = 4u * (uint32_t)(4 * h * (int)ldu + l32), offh = 2u * (uint32_t)(4 * h * (int)ldh + l32);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (!FULL && r0 + 4 * h + 8 * (r >> 2) + (r & 3) >= M) continue;
            const float u = v[r] + b;
            if (U) at_bytes(epi_row(U, ldu, r0, c0, r), offu) = u;
            at_bytes(epi_row(H, ldh, r0, c0, r), offh) = bf16_round(gelu_f(u));
        }
    }
};
struct EpiGeluBack {         // d = v * gelu'(U[r][c]); D[r][c] = d; D16[r][c] = bf16(d)
    static constexpr bool TILE256 = false;   // its loads on top of 128 x 64 per wave would spill
    const float* U; int64_t ldu; float* D; int64_t ldd; uint16_t* D16; int64_t ld16;
    __device__ __forceinline__ float col(int) const { return 0.f; }
    template <bool FULL>
    __device__ __forceinline__ void block(const floatx16& v, float, int r0, int c0, int h, int l32, int M) const
    {
        const uint32_t offd = 4u * (uint32_t)(4 * h * (int)ldd + l32), off16 = 2u * (uint32_t)(4 * h * (int)ld16 + l32);
        float u[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = r0 + 4 * h + 8 * (r >> 2) + (r & 3);
            u[r] = U[(int64_t)(FULL || row < M ? row : M - 1) * ldu + c0 + l32];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (!FULL && r0 + 4 * h + 8 * (r >> 2) + (r & 3) >= M) continue;
            const float d = v[r] * gelu_prime_f(u[r]);
            at_bytes(epi_row(D, ldd, r0, c0, r), offd) = d;
            at_bytes(epi_row(D16, ld16, r0, c0, r), off16) = bf16_round(d);
        }
    }
};

// C[r][c] = sum_k X[r][k] W[c][k] for r < M, c < N; kpad % 64 == 0 and both operands hold
// zeros in columns past the true contraction length.  Rows past M (N) re-read row M-1 (N-1);
// their results are never stored.
template <int BM, int BN, int WM, int WN, int NBUF, class Epi>
__global__ __launch_bounds__((TileShape<BM, BN, WM, WN>::THREADS)) void mlp_gemm_kernel(
    const __bf16* __restrict__ X, int64_t ldx, int M, const __bf16* __restrict__ W, int64_t ldw, int N, int kpad,
    int tiles_m, int tiles_n, Epi epi)
{
    using S = TileShape<BM, BN, WM, WN>;
    using D = DmaShape<BM, BN, WM, WN>;
    const int tile = xcd_tile_index(blockIdx.x, gridDim.x);
    int tm, tn;                              // grouped order: an XCD's concurrent tiles share X and W rows
    grouped_tile<8>(tile, tiles_m, tiles_n, tm, tn);
    if (tn >= tiles_n) return;
    const int row0 = tm * BM, col0 = tn * BN;

    __shared__ __attribute__((aligned(1024))) PipeLds<BM, BN, NBUF> lds;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    int64_t oX[D::GX], oW[D::GW];
#pragma unroll
    for (int i = 0; i < D::GX; ++i) {
        const int g = wave + S::WAVES * i;
        const int r = row0 + dma_row(g, lane);
        oX[i] = (int64_t)(r < M ? r : M - 1) * ldx + 8 * dma_chunk(g, lane);
    }
#pragma unroll
    for (int i = 0; i < D::GW; ++i) {
        const int g = wave + S::WAVES * i;
        const int c = col0 + dma_row(g, lane);
        oW[i] = (int64_t)(c < N ? c : N - 1) * ldw + 8 * dma_chunk(g, lane);
    }
    const int ws = (wave % S::WAVES_M) * WM;
    const int wa = (wave / S::WAVES_M) * WN;
    floatx16 acc[S::TI][S::TJ];
    mfma_tile_loop_pipe<BM, BN, WM, WN, NBUF>(X, oX, W, oW, kpad, lds, ws, wa, acc);

    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int r0 = __builtin_amdgcn_readfirstlane(row0 + ws), c0 = __builtin_amdgcn_readfirstlane(col0 + wa);
    float cv[S::TJ];
#pragma unroll
    for (int j = 0; j < S::TJ; ++j) cv[j] = epi.col(c0 + 32 * j + l32 < N ? c0 + 32 * j + l32 : N - 1);
#pragma unroll
    for (int i = 0; i < S::TI; ++i)
#pragma unroll
        for (int j = 0; j < S::TJ; ++j) {
            if (c0 + 32 * j + l32 >= N) continue;
            if (r0 + 32 * i + 32 <= M) epi.template block<true>(acc[i][j], cv[j], r0 + 32 * i, c0 + 32 * j, h, l32, M);
            else epi.template block<false>(acc[i][j], cv[j], r0 + 32 * i, c0 + 32 * j, h, l32, M);
        }
}

template <int BM, int BN, int WM, int WN, int NBUF, class Epi>
hipError_t launch_gemm_shape(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                             const Epi& epi, hipStream_t s)
{
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int64_t nwg = (int64_t)tiles_m * tiles_n;
    if (nwg > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((mlp_gemm_kernel<BM, BN, WM, WN, NBUF, Epi>), dim3((unsigned)nwg),
                       dim3(TileShape<BM, BN, WM, WN>::THREADS), 0, s, reinterpret_cast<const __bf16*>(X), ldx, M,
                       reinterpret_cast<const __bf16*>(W), ldw, N, kpad, tiles_m, tiles_n, epi);
    return hipGetLastError();
}

template <class Epi>
hipError_t launch_gemm(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                       const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    if (kpad <= 0 || kpad % 64 || ldx % 8 || ldw % 8 || ldx < kpad || ldw < kpad ||
        (reinterpret_cast<uintptr_t>(X) & 15) || (reinterpret_cast<uintptr_t>(W) & 15) || N > (1 << 26))
        return hipErrorInvalidValue;
    // very large outputs (four or more rounds of 256 x 256 tiles on 256 CUs): eight 128 x 64 waves per
    // tile; large ones (two or more 128 x 128 tiles per CU): four 64 x 64 waves; below that 64 x 128 tiles of eight
    // 32 x 32 waves while they still give every CU one, else 64 x 64 tiles of four (512 x 2048 x 2048: 11.3 us against
    // 13.7; 1024 x 2048 x 20032: 64 x 128 128 us, 64 x 64 125, at 2048 x 2048 x 1024 15.5 against 17.9)
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if constexpr (Epi::TILE256)
        if (tiles(256, 256) >= 1024)
            return launch_gemm_shape<256, 256, 128, 64, 2>(X, ldx, M, W, ldw, N, kpad, epi, s);
    if (tiles(128, 128) >= 512)
        return launch_gemm_shape<128, 128, 64, 64, 2>(X, ldx, M, W, ldw, N, kpad, epi, s);
    if (tiles(64, 128) >= 256)
        return launch_gemm_shape<64, 128, 32, 32, 3>(X, ldx, M, W, ldw, N, kpad, epi, s);
    return launch_gemm_shape<64, 64, 32, 32, 3>(X, ldx, M, W, ldw, N, kpad, epi, s);
}

// ---------------------------------------------------------------------------
// (A P)^T: APt[c][i] = sum_j P[j][c] A[j][i] in float32, written as bfloat16 [d][npad]
// (zeros past n).  A one-time precomputation: a plain 64 x 64 LDS-tiled product.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void project_kernel(const float* __restrict__ At, int64_t lda, int n, int m,
                                                      const float* __restrict__ P, int d, uint16_t* __restrict__ APt,
                                                      int npad)
{
    __shared__ float sP[16][64];
    __shared__ float sA[16][64];
    const int c0 = blockIdx.y * 64, i0 = blockIdx.x * 64;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    float acc[4][4] = {};
    for (int j0 = 0; j0 < m; j0 += 16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = tid + 256 * q, jj = e >> 6, cc = e & 63;
            const int j = j0 + jj;
            sP[jj][cc] = (j < m && c0 + cc < d) ? P[(int64_t)j * d + c0 + cc] : 0.f;
            sA[jj][cc] = (j < m && i0 + cc < n) ? At[(int64_t)j * lda + i0 + cc] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            float pv[4], av[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) { pv[a] = sP[jj][4 * ty + a]; av[a] = sA[jj][4 * tx + a]; }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) acc[a][b] = fmaf(pv[a], av[b], acc[a][b]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int c = c0 + 4 * ty + a;
        if (c >= d) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int i = i0 + 4 * tx + b;
            if (i < npad) APt[(int64_t)c * npad + i] = i < n ? bf16_round(acc[a][b]) : (uint16_t)0;
        }
    }
}

// Signals to bfloat16 rows [p][npad], zeros past n.
__global__ __launch_bounds__(256) void signals_bf16_kernel(const float* __restrict__ B, int64_t ldb, int n,
                                                           uint16_t* __restrict__ B16, int npad)
{
    const int r = blockIdx.x;
    for (int i = threadIdx.x; i < npad; i += 256)
        B16[(int64_t)r * npad + i] = i < n ? bf16_round(B[(int64_t)r * ldb + i]) : (uint16_t)0;
}

// X0[r] = bf16(Z[r] * sqrt(d) / ||Z[r]||) (a zero row stays zero); optionally X0 widened to Zout.
__global__ __launch_bounds__(256) void embed_norm_kernel(const float* __restrict__ Z, int d,
                                                         uint16_t* __restrict__ X0, float* __restrict__ Zout,
                                                         int64_t ldz_out)
{
    __shared__ double red[4];
    const int r = blockIdx.x;
    const float* z = Z + (int64_t)r * d;
    double s = 0.0;
    for (int c = threadIdx.x; c < d; c += 256) s += (double)z[c] * z[c];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    const double nrm = sqrt(red[0] + red[1] + red[2] + red[3]);
    const float scale = nrm > 0.0 ? (float)(sqrt((double)d) / nrm) : 0.f;
    for (int c = threadIdx.x; c < d; c += 256) {
        const uint16_t v = bf16_round(z[c] * scale);
        X0[(int64_t)r * d + c] = v;
        if (Zout) Zout[(int64_t)r * ldz_out + c] = bf16_to_f(v);
    }
}

// The passes of the backward that read whole activation matrices work on 64 x 64 tiles (LT), a workgroup of
// 256 threads each: a matrix is read once, in float4 / 16-byte rows, and its bfloat16 transpose leaves through
// LDS in 128-byte rows, while the tile's sums over its rows or columns go to partial arrays that one small
// kernel adds up at the end of the step.  One workgroup per 256 columns that walks every row by itself (the
// plain column sum) leaves 8 to 79 of the 256 CUs with work: 246 us for 1024 x 2048 as for 1024 x 20000.  As
// tiles: 5.7 us for 1024 x 2048 with its transpose, 88 us for the loss of 1024 x 20000 (bound by its expf, log1pf
// and division; 377 us as loss, column sum and transpose before), and 12 us for the partial sums; a training step
// at 1024 signals, d = h = 2048, m = 20000: 1.93 -> 1.11 ms.
constexpr int LT = 64;
constexpr int LTS = LT + 8;   // LDS row of bfloat16 values: 16-byte aligned, rows 4 banks apart

// Write the transposed tile t[row][col] (bfloat16): out[c0 + col][r0 + row], col rows below `cols`, 16 bytes per
// lane (ldo % 64 == 0 and r0 % 64 == 0, so a tile's 64 entries always lie inside a row of out).
__device__ __forceinline__ void store_tile_transposed(const uint16_t (&t)[LT][LTS], uint16_t* __restrict__ out,
                                                      int64_t ldo, int r0, int c0, int cols)
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = threadIdx.x + 256 * q, col = e >> 3, rr = 8 * (e & 7);
        if (c0 + col >= cols) continue;
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (uint32_t)t[rr + 2 * i][col] | ((uint32_t)t[rr + 2 * i + 1][col] << 16);
        *reinterpret_cast<uint4*>(out + (int64_t)(c0 + col) * ldo + r0 + rr) = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

// Column sums of a tile held by its threads (thread: columns 4 (tid % 16) .. + 3, rows tid / 16 + 16 q, already
// added over q into cs) into part[col] (float64), through s_col.
__device__ __forceinline__ void tile_column_sums(const double (&cs)[4], double (&s_col)[16][LT + 1],
                                                 double* __restrict__ part, int c0, int cols)
{
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) s_col[tid >> 4][4 * (tid & 15) + i] = cs[i];
    __syncthreads();
    if (tid < LT && c0 + tid < cols) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) v += s_col[q][tid];
        part[c0 + tid] = v;
    }
}

// Weighted binary cross-entropy with logits on one tile of S (logits, [rows][lds], lds = mpad): with g = dl/ds
// divided by the batch size, D16[r][j] = bf16(g) (zero in columns m..mpad-1), DT[j][r] = bf16(g) (zero for
// rows..64 ceil(rows / 64) - 1), colpart[tile row][j] = the tile's sum of g over its rows, rowpart[tile col][r] =
// its sum of l(s_j, y_j).  Targets y_j = 1 for the atoms listed in supp[r][0..len[r]).
__global__ __launch_bounds__(256) void bce_tile_kernel(const float* __restrict__ S, int64_t lds,
                                                       uint16_t* __restrict__ D16, int64_t ld16,
                                                       uint16_t* __restrict__ DT, int64_t ldt, int m, int rows,
                                                       const int* __restrict__ supp, int64_t ld_supp,
                                                       const int* __restrict__ supp_len, float pos_w, float inv_batch,
                                                       double* __restrict__ colpart, int64_t ldc,
                                                       double* __restrict__ rowpart, int64_t ldr)
{
    __shared__ uint32_t bits[LT][2];
    __shared__ __attribute__((aligned(16))) uint16_t t[LT][LTS];
    __shared__ double s_col[16][LT + 1];
    const int c0 = blockIdx.x * LT, r0 = blockIdx.y * LT;
    const int tid = threadIdx.x, tc = 4 * (tid & 15), tr = tid >> 4;
    float4 x[4];   // four rows of four logits (mpad is a multiple of 64: every column is readable)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = r0 + tr + 16 * q;
        x[q] = *reinterpret_cast<const float4*>(S + (int64_t)(r < rows ? r : rows - 1) * lds + c0 + tc);
    }
    if (tid < 2 * LT) bits[tid >> 1][tid & 1] = 0u;
    __syncthreads();
    for (int q = tid >> 2; q < LT; q += 64) {   // four lanes walk a row's support list
        const int r = r0 + q;
        if (r >= rows) continue;
        const int len = min(supp_len[r], (int)ld_supp);
        for (int e = tid & 3; e < len; e += 4) {
            const int j = supp[(int64_t)r * ld_supp + e] - c0;
            if (j >= 0 && j < LT && c0 + j < m) atomicOr(&bits[q][j >> 5], 1u << (j & 31));
        }
    }
    __syncthreads();
    double cs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = tr + 16 * q, r = r0 + row;
        const float xv[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
        const uint32_t yb = bits[row][tc >> 5] >> (tc & 31);
        uint16_t hv[4];
        double part = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = r < rows && c0 + tc + i < m;
            const float v = xv[i];
            const bool y = (yb >> i) & 1u;
            const float e = expf(-fabsf(v));
            const float l1 = log1pf(e);
            const float sp = fmaxf(y ? -v : v, 0.f) + l1;           // log(1 + e^-v) for a target, else log(1 + e^v)
            const float sig = (v >= 0.f ? 1.f : e) / (1.f + e);
            const float g = (y ? sig * pos_w - pos_w : sig) * inv_batch;
            part += in ? (y ? (double)pos_w * sp : (double)sp) : 0.0;
            cs[i] += in ? (double)g : 0.0;
            hv[i] = in ? bf16_round(g) : (uint16_t)0;
            t[row][tc + i] = hv[i];
        }
        part = row16_sum(part);                                      // the row's 16 threads
        if (r < rows) {
            *reinterpret_cast<uint2*>(D16 + (int64_t)r * ld16 + c0 + tc) =
                make_uint2((uint32_t)hv[0] | ((uint32_t)hv[1] << 16), (uint32_t)hv[2] | ((uint32_t)hv[3] << 16));
            if ((tid & 15) == 0) rowpart[(int64_t)blockIdx.x * ldr + r] = part;
        }
    }
    tile_column_sums(cs, s_col, colpart + (int64_t)blockIdx.y * ldc, c0, m);   // its barrier also publishes t
    store_tile_transposed(t, DT, ldt, r0, c0, m);
}

// One tile of a float32 matrix: DT[c][r] = bf16(in[r][c]) (zero for rows past `rows`, up to a multiple of 64) and
// colpart[tile row][c] = the tile's column sum.  cols is a multiple of 64.
__global__ __launch_bounds__(256) void transpose_colsum_kernel(const float* __restrict__ in, int64_t ld, int rows,
                                                               int cols, uint16_t* __restrict__ DT, int64_t ldt,
                                                               double* __restrict__ colpart, int64_t ldc)
{
    __shared__ __attribute__((aligned(16))) uint16_t t[LT][LTS];
    __shared__ double s_col[16][LT + 1];
    const int c0 = blockIdx.x * LT, r0 = blockIdx.y * LT;
    const int tid = threadIdx.x, tc = 4 * (tid & 15), tr = tid >> 4;
    float4 x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = r0 + tr + 16 * q;
        x[q] = *reinterpret_cast<const float4*>(in + (int64_t)(r < rows ? r : rows - 1) * ld + c0 + tc);
    }
    double cs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = tr + 16 * q;
        const bool in_rows = r0 + row < rows;
        const float xv[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            cs[i] += in_rows ? (double)xv[i] : 0.0;
            t[row][tc + i] = in_rows ? bf16_round(xv[i]) : (uint16_t)0;
        }
    }
    tile_column_sums(cs, s_col, colpart + (int64_t)blockIdx.y * ldc, c0, cols);
    store_tile_transposed(t, DT, ldt, r0, c0, cols);
}

// The step's sums from the tiles' partial ones: out[c] = sum over the tile rows of colpart[.][c] for up to three
// matrices (the bias gradients) and rowloss[r] = sum over the tile columns of rowpart[.][r] (four threads per
// row).  Blocks [start[q], start[q + 1]) take job q, the last job the rows.
__global__ __launch_bounds__(256) void partial_sums_kernel(PartialSums a)
{
    __shared__ double s_p[4][LT];
    const int tid = threadIdx.x;
    int q = 0;
    while (q < 3 && (int)blockIdx.x >= a.start[q + 1]) ++q;
    const int b = blockIdx.x - a.start[q];
    if (q < 3) {
        const int c = b * 256 + tid;
        if (c >= a.cols[q]) return;
        double s = 0.0;
#pragma unroll 8
        for (int r = 0; r < a.tile_rows; ++r) s += a.part[q][(int64_t)r * a.ldc[q] + c];
        a.out[q][c] = (float)s;
        return;
    }
    const int r = b * LT + (tid & (LT - 1)), g = tid >> 6;
    double s = 0.0;
    if (r < a.rows) {
#pragma unroll 8
        for (int c = g; c < a.tile_cols; c += 4) s += a.rowpart[(int64_t)c * a.ldr + r];
    }
    s_p[g][tid & (LT - 1)] = s;
    __syncthreads();
    if (g == 0 && r < a.rows) a.rowloss[r] = (float)(((s_p[0][tid] + s_p[1][tid]) + s_p[2][tid]) + s_p[3][tid]);
}

// loss = sum_r rowloss[r] / rows (one workgroup).
__global__ __launch_bounds__(256) void loss_sum_kernel(const float* __restrict__ rowloss, int rows, double* loss)
{
    __shared__ double red[4];
    double s = 0.0;
    for (int r = threadIdx.x; r < rows; r += 256) s += rowloss[r];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *loss = (red[0] + red[1] + red[2] + red[3]) / rows;
}

// out[c][r] = in[r][c] for c < cols, r < rows; out[c][r] = 0 for rows <= r < ldo, for up to three matrices in one
// launch (ldo % 64 == 0, ldi % 8 == 0; blocks [start[q], start[q + 1]) take matrix q, tile columns fastest).  A
// thread moves 16 bytes each way: 90 -> 43 us for 20000 x 2048 and 2048 x 2048 (two bytes per access before).
__global__ __launch_bounds__(256) void transpose_bf16_kernel(TransposeJobs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t t[LT][LTS];
    int q = 0;
    while (q < 2 && (int)blockIdx.x >= a.start[q + 1]) ++q;
    const TransposeJob& J = a.job[q];
    const int b = blockIdx.x - a.start[q];
    const int tiles_c = (J.cols + LT - 1) / LT;
    const int r0 = b / tiles_c * LT, c0 = b % tiles_c * LT;
    const int tid = threadIdx.x;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int e = tid + 256 * h, row = e >> 3, cc = 8 * (e & 7);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (r0 + row < J.rows && c0 + cc < J.cols)   // cols % 8 == 0
            v = *reinterpret_cast<const uint4*>(J.in + (int64_t)(r0 + row) * J.ldi + c0 + cc);
        *reinterpret_cast<uint4*>(&t[row][cc]) = v;
    }
    __syncthreads();
    store_tile_transposed(t, J.out, J.ldo, r0, c0, J.cols);
}

// Adam with bias correction (bc1 = 1 - beta1^t, bc2 = 1 - beta2^t); refreshes the bfloat16 copy.
__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ P, float* __restrict__ m1,
                                                   float* __restrict__ m2, const float* __restrict__ g,
                                                   uint16_t* __restrict__ P16, int64_t count, float lr, float beta1,
                                                   float beta2, float eps, float bc1, float bc2)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
        const float gi = g[i];
        const float a = beta1 * m1[i] + (1.f - beta1) * gi;
        const float b = beta2 * m2[i] + (1.f - beta2) * gi * gi;
        m1[i] = a;
        m2[i] = b;
        const float v = P[i] - lr * (a / bc1) / (sqrtf(b / bc2) + eps);
        P[i] = v;
        P16[i] = bf16_round(v);
    }
}

__global__ __launch_bounds__(256) void params_bf16_kernel(const float* __restrict__ P, uint16_t* __restrict__ P16,
                                                          int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
        P16[i] = bf16_round(P[i]);
}

// ---------------------------------------------------------------------------
// Top-k per row (k <= 256), ties to the lower index, output ascending by atom index,
// padded with -1 when the row is shorter than k.  One workgroup per row.
//   1. Each thread keeps the two largest order keys of its entries; the k-th largest of
//      those 512 keys, T, is at most the row's k-th largest key (they are distinct
//      entries of the row), so every entry of the top k has a key >= T.
//   2. The entries with a key >= T (typically a few hundred) are appended to an LDS list.
//   3. A radix select over the list finds the k-th largest key; the entries above it and the lowest-indexed
//      ones equal to it are the answer, each placed by counting the answer's entries below it.  The indices of equal
//      entries take a radix select too, and a wave counts a digit's entries at once: with 1400 of 20000 scores equal,
//      4096 rows, a count per equal entry and a list of 1024 took 602 us, the sorts before them 220, this 110.
// If more entries pass than the list holds (many equal keys), the row is done by an exact radix select over the
// keys in global memory instead.
// With 16-byte rows the whole row stays in registers between steps 1 and 2 (NQ float4 per thread, all loads in flight
// at once), so it is read once; the k-th of a list costs 4 digit passes of three barriers where a bitonic sort took 36
// to 66 steps of one.  4096 rows of 20000, k = 64: 161 -> 73 us (328 MB: 4.5 TB/s), k = 256: 165 -> 91 us.
// ---------------------------------------------------------------------------
__device__ inline uint32_t order_key(float x)
{
    if (x != x) return 0u;                     // NaN ranks below everything
    uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);   // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix count of `flag` over the workgroup (256 threads) and the total.
__device__ inline int block_excl_count(bool flag, int* s_wave, int& total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t bal = __ballot(flag);
    const int within = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) s_wave[wave] = __popcll(bal);
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    __syncthreads();
    return before + within;
}

constexpr int TOPK_CAP = 2048;   // list entries per row
static_assert(TOPK_MAX <= 65536, "the list's indices have 16 bits");

// (Kept small: it decides how many workgroups of short rows share a CU.  4096 rows of 1000: 26 us with 12 KB, 27 with
// these 13, 33 with 20.)
struct TopkLds {
    uint32_t key[TOPK_CAP];      // the threads' two largest first (512), then the list
    uint16_t idx[TOPK_CAP];
    int hist[256];               // digit counts, then the answer before it is put in order
    int wave[4];
    int n, digit, need, ties;
};

// One entry per lane (`left`: this lane has one) into the digit counts.  Where many entries share a digit (sign and
// exponent, or equal values) lanes would queue at one address, so a wave adds all entries of a digit at once: for the
// digit of its first lane, or with ALL for every digit.
template <bool ALL>
__device__ __forceinline__ void count_digits(int* hist, bool left, uint32_t d)
{
    unsigned long long rest = __ballot(left);
    while (rest) {
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, __ffsll((long long)rest) - 1);
        const unsigned long long same = __ballot(left && d == d0);
        if ((threadIdx.x & 63) == 0) atomicAdd(&hist[d0], __popcll(same));
        left = left && d != d0;
        rest &= ~same;
        if (!ALL) break;
    }
    if (!ALL && left) atomicAdd(&hist[d], 1);
}

// The digit that holds the need-th entry in order of falling digits (s.digit), its rank there (s.need) and how many
// entries it has (s.ties).  Between barriers, called by the whole workgroup.
__device__ __forceinline__ void pick_digit(TopkLds& s, int need)
{
    const int tid = threadIdx.x;
    if (tid >= 64) return;
    // lane l owns digits 255 - 4 l .. 252 - 4 l, so the lanes before it hold the larger ones
    const int4 hv = *reinterpret_cast<const int4*>(&s.hist[252 - 4 * tid]);
    const int c[4] = {hv.w, hv.z, hv.y, hv.x};
    const int own = c[0] + c[1] + c[2] + c[3];
    int incl = own;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        incl += tid >= o ? v : 0;
    }
    int above = incl - own;
    if (above < need && need <= incl) {      // exactly one lane
        int q = 0, cq = c[0];
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (q == e && above + c[e] < need) { above += c[e]; q = e + 1; cq = c[e + 1]; }
        s.digit = 255 - 4 * tid - q;
        s.need = need - above;
        s.ties = cq;
    }
}

// The k-th largest of key[0 .. n) (1 <= k <= n) by 8-bit digits from the top; `need` receives how many entries equal to
// it belong to the k largest, `ties` how many there are.  Called by the whole workgroup (256 threads).
__device__ inline uint32_t radix_kth(const uint32_t* key, int n, int k, TopkLds& s, int& need, int& ties)
{
    const int tid = threadIdx.x;
    uint32_t prefix = 0u, mask = 0u;
    need = k;
    for (int shift = 24; shift >= 0; shift -= 8) {
        s.hist[tid] = 0;
        __syncthreads();
        for (int e0 = 0; e0 < n; e0 += 256) {
            const int e = e0 + tid;
            const uint32_t u = e < n ? key[e] : 0u;
            const bool left = e < n && (u & mask) == prefix;
            const uint32_t d = (u >> shift) & 255u;
            if (shift == 24) count_digits<true>(s.hist, left, d);
            else if (shift < 16 && ties > 64) count_digits<false>(s.hist, left, d);   // equal in 16 bits: equal values
            else if (left) atomicAdd(&s.hist[d], 1);
        }
        __syncthreads();
        pick_digit(s, need);
        __syncthreads();
        prefix |= (uint32_t)s.digit << shift;
        mask |= 0xFFu << shift;
        need = s.need;
        ties = s.ties;
    }
    return prefix;
}

// The k-th lowest index among the list's entries with key P (at least k of them), by its two bytes.
__device__ inline int kth_lowest_index(int n, uint32_t P, int k, TopkLds& s)
{
    const int tid = threadIdx.x;
    int prefix = 0, need = k;
    for (int shift = 8; shift >= 0; shift -= 8) {
        s.hist[tid] = 0;
        __syncthreads();
        for (int e0 = 0; e0 < n; e0 += 256) {
            const int e = e0 + tid;
            const int j = e < n ? s.idx[e] : 0;
            const bool left = e < n && s.key[e] == P && (shift == 8 || (j >> 8) == prefix);
            count_digits<false>(s.hist, left, 255u - ((uint32_t)(j >> shift) & 255u));   // lowest first
        }
        __syncthreads();
        pick_digit(s, need);
        __syncthreads();
        prefix = (prefix << 8) | (255 - s.digit);
        need = s.need;
    }
    return prefix;
}

// The exact radix select of a row over its keys in global memory.
__device__ void topk_sweeps(const float* s, int L, int k, int kk, int* o, int* hist, int* s_wave, int& s_digit, int& s_need)
{
    const int tid = threadIdx.x;
    __syncthreads();
    // Fallback: exact radix select over the keys in global memory.  Four 8-bit passes find the
    // kk-th largest key P and how many keys equal to P to take; a final pass compacts in index order.
    uint32_t prefix = 0u, mask = 0u;
    int need = kk;
    if (need > 0) {
        for (int shift = 24; shift >= 0; shift -= 8) {
            hist[tid] = 0;
            __syncthreads();
            for (int j = tid; j < L; j += 256) {
                const uint32_t u = order_key(s[j]);
                if ((u & mask) == prefix) atomicAdd(&hist[(u >> shift) & 255u], 1);
            }
            __syncthreads();
            if (tid == 0) {
                int above = 0, d = 255;
                for (; d > 0; --d) {
                    if (above + hist[d] >= need) break;
                    above += hist[d];
                }
                s_digit = d;
                s_need = need - above;
            }
            __syncthreads();
            prefix |= (uint32_t)s_digit << shift;
            mask |= 0xFFu << shift;
            need = s_need;
            __syncthreads();
        }
    }
    // keys > prefix are all taken; `need` keys equal to prefix, the lowest indices first
    int base_out = 0, base_tie = 0;
    for (int c0 = 0; c0 < L && kk > 0; c0 += 256) {
        const int j = c0 + tid;
        const uint32_t u = j < L ? order_key(s[j]) : 0u;
        const bool gt = j < L && u > prefix;
        const bool eq = j < L && u == prefix;
        int tot_eq, tot_sel;
        const int tie_rank = base_tie + block_excl_count(eq, s_wave, tot_eq);
        const bool sel = gt || (eq && tie_rank < need);
        const int pos = base_out + block_excl_count(sel, s_wave, tot_sel);
        if (sel) o[pos] = j;
        base_tie += tot_eq;
        base_out += tot_sel;
    }
    for (int q = base_out + tid; q < k; q += 256) o[q] = -1;
}

template <int NQ>   // 0: any row alignment and length, read twice
__global__ __launch_bounds__(256, NQ > 20 ? 2 : 4) void topk_kernel(const float* __restrict__ S, int64_t lds, int L, int k,
                                                                    int* __restrict__ out, int64_t ldo)
{
    __shared__ __attribute__((aligned(16))) TopkLds w;
    const int row = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const float* s = S + (int64_t)row * lds;
    int* o = out + (int64_t)row * ldo;
    const int kk = k < L ? k : L;                  // >= 1

    // 1. per-thread two largest values, then the kk-th largest over the workgroup.  With t1 >= t2 the median of t1, t2
    //    and v is the new second largest; a NaN changes neither (the median instruction returns the least of the others)
    float t1 = -INFINITY, t2 = -INFINITY;
    auto top2 = [&](float v) {
        t2 = __builtin_amdgcn_fmed3f(t1, t2, v);
        t1 = fmaxf(t1, v);
    };
    constexpr int NR = NQ > 0 ? NQ : 1;
    float4 f[NR];
    if constexpr (NQ > 0) {
        // chunks past the row read its last one, the 16 aligned bytes that hold the row's last entry (of the last row
        // they can lie past the caller's matrix, never past its page: the values are not used)
        const int last = (L - 1) / 4;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int c = tid + 256 * q;
            f[q] = reinterpret_cast<const float4*>(s)[c < last ? c : last];
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int j = 4 * (tid + 256 * q);
            if (4 * 256 * (q + 1) > L) {           // the row's end (the same for the whole workgroup): NaN past it
                f[q].x = j < L ? f[q].x : NAN;
                f[q].y = j + 1 < L ? f[q].y : NAN;
                f[q].z = j + 2 < L ? f[q].z : NAN;
                f[q].w = j + 3 < L ? f[q].w : NAN;
            }
            top2(f[q].x);
            top2(f[q].y);
            top2(f[q].z);
            top2(f[q].w);
        }
    } else {
        for (int j0 = tid; j0 < L; j0 += 256 * 8) {   // eight loads in flight (clamped: no branch waits for them)
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = s[j0 + 256 * e < L ? j0 + 256 * e : L - 1];
#pragma unroll
            for (int e = 0; e < 8; ++e) top2(j0 + 256 * e < L ? v[e] : NAN);
        }
    }
    w.key[tid] = order_key(t1);
    w.key[256 + tid] = order_key(t2);
    if (tid == 0) w.n = 0;
    __syncthreads();
    int need, ties;
    const uint32_t Tk = radix_kth(w.key, 512, kk, w, need, ties);
    // the value of a key (of +0 for the zeros, which compare equal)
    const float T = __uint_as_float((Tk & 0x80000000u) ? Tk & 0x7fffffffu : ~Tk);

    // 2. the entries at or above T (never NaN) into the list, in any order
    if constexpr (NQ > 0) {
        // which of the thread's entries pass, as bits (straight-line code: appending at each of the 4 NQ places would be
        // larger than the instruction cache); the few that do are read again
        constexpr int NW = (NQ + 7) / 8;
        uint32_t bits[NW];
        int cnt = 0;
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            bits[v] = 0u;
#pragma unroll
            for (int q = 8 * v; q < NQ && q < 8 * v + 8; ++q) {
                const int b = 4 * (q - 8 * v);
                bits[v] |= (f[q].x >= T ? 1u << b : 0u) | (f[q].y >= T ? 2u << b : 0u) | (f[q].z >= T ? 4u << b : 0u) |
                           (f[q].w >= T ? 8u << b : 0u);
            }
            cnt += __popc(bits[v]);
        }
        int incl = cnt;
        for (int o2 = 1; o2 < 64; o2 <<= 1) {
            const int v = __shfl_up(incl, o2);
            incl += lane >= o2 ? v : 0;
        }
        int base = 0;
        if (lane == 63) base = atomicAdd(&w.n, incl);
        int pos = __shfl(base, 63) + incl - cnt;
#pragma unroll
        for (int v = 0; v < NW; ++v)
            for (uint32_t m = bits[v]; m; m &= m - 1u) {
                const int b = __ffs(m) - 1;
                const int j = 4 * (tid + 256 * (8 * v + (b >> 2))) + (b & 3);
                if (pos < TOPK_CAP) { w.key[pos] = order_key(s[j]); w.idx[pos] = (uint16_t)j; }
                ++pos;
            }
    } else {
        for (int j0 = 0; j0 < L; j0 += 256 * 8) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = s[j0 + 256 * e + tid < L ? j0 + 256 * e + tid : L - 1];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int j = j0 + 256 * e + tid;
                const bool t = j < L && v[e] >= T;
                const unsigned long long bal = __ballot(t);
                if (!bal) continue;
                int base = 0;
                if (lane == 0) base = atomicAdd(&w.n, __popcll(bal));
                base = __builtin_amdgcn_readfirstlane(base);
                const int pos = base + __popcll(bal & ((1ull << lane) - 1ull));
                if (t && pos < TOPK_CAP) { w.key[pos] = order_key(v[e]); w.idx[pos] = (uint16_t)j; }
            }
        }
    }
    __syncthreads();
    const int n = w.n;
    if (n > TOPK_CAP || n < kk) {                  // many equal values, or fewer than kk that are not NaN
        topk_sweeps(s, L, k, kk, o, w.hist, w.wave, w.digit, w.need);
        return;
    }
    // 3. the kk-th largest key P of the list (n >= kk: T is a lower bound); entries above P are in, and the `need`
    //    lowest-indexed of the entries equal to it
    const uint32_t P = radix_kth(w.key, n, kk, w, need, ties);
    const int cut = ties > need ? kth_lowest_index(n, P, need, w) : INT_MAX;   // the same test in every thread
    int* sel = w.hist;
    if (tid == 0) w.n = 0;
    __syncthreads();
    for (int e0 = 0; e0 < n; e0 += 256) {          // the same number of steps in every lane
        const int e = e0 + tid;
        const uint32_t u = e < n ? w.key[e] : 0u;
        const int j = e < n ? w.idx[e] : 0;
        const bool in = e < n && (u > P || (u == P && j <= cut));
        const unsigned long long bal = __ballot(in);
        int base = 0;
        if (lane == 0 && bal) base = atomicAdd(&w.n, __popcll(bal));
        base = __builtin_amdgcn_readfirstlane(base);
        if (in) sel[base + __popcll(bal & ((1ull << lane) - 1ull))] = j;
    }
    __syncthreads();
    if (tid < kk) {
        const int j = sel[tid];
        int rank = 0;
        for (int d = 0; d < kk; ++d) rank += sel[d] < j;
        o[rank] = j;
    } else if (tid < k) {
        o[tid] = -1;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t mlp_project(const float* At, int64_t lda, int n, int m, const float* P, int d, uint16_t* APt, int npad,
                       hipStream_t s)
{
    dim3 grid((npad + 63) / 64, (d + 63) / 64);
    hipLaunchKernelGGL(project_kernel, grid, dim3(256), 0, s, At, lda, n, m, P, d, APt, npad);
    return hipGetLastError();
}

hipError_t mlp_signals_bf16(const float* B, int64_t ldb, int n, int p, uint16_t* B16, int npad, hipStream_t s)
{
    if (p <= 0) return hipSuccess;
    hipLaunchKernelGGL(signals_bf16_kernel, dim3(p), dim3(256), 0, s, B, ldb, n, B16, npad);
    return hipGetLastError();
}

hipError_t mlp_gemm_store(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                          float* C, int64_t ldc, const float* bias, hipStream_t s)
{
    if (bias && ldc > EPI_LD_MAX) return launch_gemm(X, ldx, M, W, ldw, N, kpad, EpiStore<true, true>{C, ldc, bias}, s);
    if (ldc > EPI_LD_MAX) return hipErrorInvalidValue;
    if (bias) return launch_gemm(X, ldx, M, W, ldw, N, kpad, EpiStore<true>{C, ldc, bias}, s);
    return launch_gemm(X, ldx, M, W, ldw, N, kpad, EpiStore<false>{C, ldc, nullptr}, s);
}

hipError_t mlp_gemm_bias_gelu(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                              const float* bias, float* U, int64_t ldu, uint16_t* H, int64_t ldh, hipStream_t s)
{
    return launch_gemm(X, ldx, M, W, ldw, N, kpad, EpiBiasGelu{bias, U, ldu, H, ldh}, s);
}

hipError_t mlp_gemm_gelu_back(const uint16_t* X, int64_t ldx, int M, const uint16_t* W, int64_t ldw, int N, int kpad,
                              const float* U, int64_t ldu, float* D, int64_t ldd, uint16_t* D16, int64_t ld16,
                              hipStream_t s)
{
    return launch_gemm(X, ldx, M, W, ldw, N, kpad, EpiGeluBack{U, ldu, D, ldd, D16, ld16}, s);
}

hipError_t mlp_embed_norm(const float* Z, int d, int p, uint16_t* X0, float* Zout, int64_t ldz_out, hipStream_t s)
{
    if (p <= 0) return hipSuccess;
    hipLaunchKernelGGL(embed_norm_kernel, dim3(p), dim3(256), 0, s, Z, d, X0, Zout, ldz_out);
    return hipGetLastError();
}

hipError_t mlp_bce_tiles(const float* S, int64_t lds, uint16_t* D16, int64_t ld16, uint16_t* DT, int64_t ldt, int m,
                         int mpad, int rows, const int* supp, int64_t ld_supp, const int* supp_len, float pos_w,
                         double* colpart, int64_t ldc, double* rowpart, int64_t ldr, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    if (mpad % LT || lds < mpad || ld16 < mpad || lds % 4 || ld16 % 4 || ldt % LT || ldt < (rows + LT - 1) / LT * LT)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(bce_tile_kernel, dim3(mpad / LT, (rows + LT - 1) / LT), dim3(256), 0, s, S, lds, D16, ld16, DT,
                       ldt, m, rows, supp, ld_supp, supp_len, pos_w, 1.0f / rows, colpart, ldc, rowpart, ldr);
    return hipGetLastError();
}

hipError_t mlp_transpose_colsum(const float* in, int64_t ld, int rows, int cols, uint16_t* DT, int64_t ldt,
                                double* colpart, int64_t ldc, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    if (cols % LT || ld % 4 || ldt % LT || ldt < (rows + LT - 1) / LT * LT) return hipErrorInvalidValue;
    hipLaunchKernelGGL(transpose_colsum_kernel, dim3(cols / LT, (rows + LT - 1) / LT), dim3(256), 0, s, in, ld, rows,
                       cols, DT, ldt, colpart, ldc);
    return hipGetLastError();
}

hipError_t mlp_partial_sums(PartialSums a, double* loss, hipStream_t s)
{
    if (a.rows <= 0) return hipSuccess;
    a.start[0] = 0;
    for (int q = 0; q < 3; ++q) a.start[q + 1] = a.start[q] + (a.cols[q] + 255) / 256;
    a.tile_rows = (a.rows + LT - 1) / LT;
    const int blocks = a.start[3] + a.tile_rows;
    hipLaunchKernelGGL(partial_sums_kernel, dim3(blocks), dim3(256), 0, s, a);
    hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(256), 0, s, a.rowloss, a.rows, loss);
    return hipGetLastError();
}

hipError_t mlp_transposes(const TransposeJob* jobs, int count, hipStream_t s)
{
    if (count < 1 || count > 3) return hipErrorInvalidValue;
    TransposeJobs a{};
    int64_t at = 0;
    for (int q = 0; q < 3; ++q) {
        a.start[q] = (int)at;
        if (q >= count) continue;
        const TransposeJob& J = jobs[q];
        if (J.ldo % LT || J.ldo < J.rows || J.cols % 8 || J.ldi % 8) return hipErrorInvalidValue;
        a.job[q] = J;
        at += (J.ldo / LT) * ((J.cols + LT - 1) / LT);   // every tile row of out, the zero rows included
        if (at > 0x7fffffff) return hipErrorInvalidValue;
    }
    for (int q = count; q < 3; ++q) a.start[q] = (int)at;
    hipLaunchKernelGGL(transpose_bf16_kernel, dim3((unsigned)at), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t mlp_adam(float* P, float* m1, float* m2, const float* g, uint16_t* P16, int64_t count, float lr,
                    float beta1, float beta2, float eps, float bc1, float bc2, hipStream_t s)
{
    const int64_t blocks = std::min<int64_t>((count + 255) / 256, 16384);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)blocks), dim3(256), 0, s, P, m1, m2, g, P16, count, lr, beta1,
                       beta2, eps, bc1, bc2);
    return hipGetLastError();
}

hipError_t mlp_params_bf16(const float* P, uint16_t* P16, int64_t count, hipStream_t s)
{
    const int64_t blocks = std::min<int64_t>((count + 255) / 256, 16384);
    hipLaunchKernelGGL(params_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, P, P16, count);
    return hipGetLastError();
}

hipError_t mlp_topk(const float* S, int64_t lds, int rows, int L, int k, int* out, int64_t ldo, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    if (k < 1 || k > 256 || L < 1 || ldo < k) return hipErrorInvalidValue;
    if (L > TOPK_MAX) return hipErrorInvalidValue;
    // rows on 16-byte boundaries stay in registers: 4, 8, 20 or 38 float4 per thread by the row's length
    auto launch = [&](auto nq) {
        hipLaunchKernelGGL(topk_kernel<decltype(nq)::value>, dim3(rows), dim3(256), 0, s, S, lds, L, k, out, ldo);
    };
    if (lds % 4 || (reinterpret_cast<uintptr_t>(S) & 15)) launch(std::integral_constant<int, 0>());
    else if (L <= 4096) launch(std::integral_constant<int, 4>());
    else if (L <= 8192) launch(std::integral_constant<int, 8>());
    else if (L <= 20480) launch(std::integral_constant<int, 20>());
    else launch(std::integral_constant<int, 38>());
    return hipGetLastError();
}

}  // namespace bmpl
