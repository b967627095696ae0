// Gram table Q = A^T A in float64 (the precomputed Q of Section III, Eq. (12)).
//
// The batch mode of the paper precomputes Q once per dictionary and amortises
// it over all signals (Remark 1).  Here Q serves the master problem: the Gram
// rows G_{J,I} of the atoms entering an active set become gathers from Q
// instead of n-long float64 dot products per pair.  Entries are accumulated in
// float64 from the float32 atoms (every product is exact in float64), so they
// equal the directly computed Gram entries up to summation order.
//
// A dense symmetric rank-n update on the float64 matrix cores (v_mfma_f64_16x16x4f64), TB x TB output tiles per
// 256-thread workgroup, four waves of TB/2 x TB/2.  The matrix instruction runs 64 cycles per SIMD, so the bound
// is keeping it fed: K is staged 32 at a time through two LDS buffers as float32 (half the LDS of float64 values;
// a lane converts what it reads), the next slice loaded into registers while the current one is multiplied, one
// barrier per slice.  In LDS a row's 32 values are ordered [k % 4][k / 4], so the 8 values that a lane supplies to
// the slice's 8 matrix steps (k = 4 t + lane / 16) are two 16-byte reads; rows are 144 bytes apart, which puts 16
// lanes' reads on distinct banks.  Each step still sums k = 4 t .. 4 t + 3 in order of t.
// Only tiles on or below the diagonal are computed; each entry on or below the diagonal is written to
// both triangles, so Q is exactly symmetric.
// Measured (atoms x values): 6000 x 1000 0.74 ms, 20000 x 1024 7.3 ms, 16384 x 2048 9.3 ms (59 TFLOP/s of 78.6);
// with float64 slices of 16 loaded, stored and multiplied in turn: 1.29, 11.7 and 15.3 ms.
#include "bmpl_internal.h"

namespace bmpl {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int KB = 32;           // k per LDS stage
constexpr int LS = KB + 4;       // LDS row stride (floats)

template <int TB>
__global__ __launch_bounds__(256) void gram_table_kernel(const float* __restrict__ At, int64_t lda, int m,
                                                         int kpad, double* __restrict__ Q, int64_t ldq, int T)
{
    // blockIdx.x enumerates lower-triangle tiles (ti >= tj) row by row.
    const int64_t b = blockIdx.x;
    int ti = (int)((sqrt(8.0 * (double)b + 1.0) - 1.0) / 2.0);
    while ((int64_t)ti * (ti + 1) / 2 > b) --ti;
    while ((int64_t)(ti + 1) * (ti + 2) / 2 <= b) ++ti;
    const int tj = (int)(b - (int64_t)ti * (ti + 1) / 2);
    if (ti >= T || tj > ti) return;
    const int i0 = ti * TB, j0 = tj * TB;
    constexpr int W = TB / 32;   // 16 x 16 blocks per wave and side
    constexpr int LD = TB / 32;  // 16-byte loads per thread, operand and stage

    __shared__ __attribute__((aligned(16))) float sI[2][TB * LS];
    __shared__ __attribute__((aligned(16))) float sJ[2][TB * LS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = (wave >> 1) * (TB / 2), wj = (wave & 1) * (TB / 2);
    const int lr = tid >> 3, lt = tid & 7;   // this thread's loads: rows lr + 32 q, k = 4 lt .. 4 lt + 3

    doublex4 acc[W][W];
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int c = 0; c < W; ++c) acc[a][c] = doublex4{0.0, 0.0, 0.0, 0.0};

    // rows past the end read the dictionary's zero row m
    const float *pI[LD], *pJ[LD];
#pragma unroll
    for (int q = 0; q < LD; ++q) {
        const int ai = i0 + lr + 32 * q, aj = j0 + lr + 32 * q;
        pI[q] = At + (int64_t)(ai < m ? ai : m) * lda + 4 * lt;
        pJ[q] = At + (int64_t)(aj < m ? aj : m) * lda + 4 * lt;
    }
    float4 gI[LD], gJ[LD];
    auto load = [&](int k0) {
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            gI[q] = *reinterpret_cast<const float4*>(pI[q] + k0);
            gJ[q] = *reinterpret_cast<const float4*>(pJ[q] + k0);
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            float* di = &sI[buf][(lr + 32 * q) * LS + lt];
            float* dj = &sJ[buf][(lr + 32 * q) * LS + lt];
            di[0] = gI[q].x; di[8] = gI[q].y; di[16] = gI[q].z; di[24] = gI[q].w;
            dj[0] = gJ[q].x; dj[8] = gJ[q].y; dj[16] = gJ[q].z; dj[24] = gJ[q].w;
        }
    };
    load(0);
    store(0);
    __syncthreads();
    int cur = 0;
    for (int k0 = 0; k0 < kpad; k0 += KB) {
        load(k0 + KB < kpad ? k0 + KB : k0);   // the last stage re-reads itself (never used)
        asm volatile("" ::: "memory");         // issue the loads before the matrix work
        const int off = 8 * (lane >> 4);
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {       // matrix steps t = 4 hf .. 4 hf + 3
            float4 fa[W], fb[W];
#pragma unroll
            for (int a = 0; a < W; ++a)
                fa[a] = *reinterpret_cast<const float4*>(&sI[cur][(wi + 16 * a + (lane & 15)) * LS + off + 4 * hf]);
#pragma unroll
            for (int c = 0; c < W; ++c)
                fb[c] = *reinterpret_cast<const float4*>(&sJ[cur][(wj + 16 * c + (lane & 15)) * LS + off + 4 * hf]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                double da[W], db[W];
#pragma unroll
                for (int a = 0; a < W; ++a) da[a] = (double)(t == 0 ? fa[a].x : t == 1 ? fa[a].y : t == 2 ? fa[a].z : fa[a].w);
#pragma unroll
                for (int c = 0; c < W; ++c) db[c] = (double)(t == 0 ? fb[c].x : t == 1 ? fb[c].y : t == 2 ? fb[c].z : fb[c].w);
#pragma unroll
                for (int a = 0; a < W; ++a)
#pragma unroll
                    for (int c = 0; c < W; ++c)
                        acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(da[a], db[c], acc[a][c], 0, 0, 0);
            }
        }
        asm volatile("" ::: "memory");
        store(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    }
    // D of a float64 16x16x4 block: lane l, element r -> row l/16 + 4r, column l%16.
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int c = 0; c < W; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gi = i0 + wi + 16 * a + (lane >> 4) + 4 * r;
                const int gj = j0 + wj + 16 * c + (lane & 15);
                if (gi < m && gj < m && !(ti == tj && gi < gj)) {
                    Q[(int64_t)gi * ldq + gj] = acc[a][c][r];
                    Q[(int64_t)gj * ldq + gi] = acc[a][c][r];
                }
            }
}

template <int TB>
hipError_t launch_tiles(const float* At, int64_t lda, int m, int kpad, double* Q, int64_t ldq, hipStream_t stream)
{
    const int T = (m + TB - 1) / TB;
    const int64_t nblk = (int64_t)T * (T + 1) / 2;
    if (nblk > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gram_table_kernel<TB>, dim3((unsigned)nblk), dim3(256), 0, stream, At, lda, m, kpad, Q, ldq, T);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gram_table(const float* At, int64_t lda, int m, int kpad, double* Q, int64_t ldq,
                             hipStream_t stream)
{
    if (kpad % KB || lda % 4) return hipErrorInvalidValue;
    // the largest tile that still gives every CU four workgroups' worth of tiles, so the last round is short
    auto tiles = [&](int64_t tb) { const int64_t T = (m + tb - 1) / tb; return T * (T + 1) / 2; };
    if (tiles(128) >= 1024) return launch_tiles<128>(At, lda, m, kpad, Q, ldq, stream);
    if (tiles(64) >= 512) return launch_tiles<64>(At, lda, m, kpad, Q, ldq, stream);
    return launch_tiles<32>(At, lda, m, kpad, Q, ldq, stream);
}

}  // namespace bmpl
