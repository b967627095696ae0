// Batched correlation G = A^T Xi on MFMA (float32).
//
// One outer iteration of the batched pursuit needs g_i = A^T xi_i for every
// running signal i: the full matrix-vector product of the worst-case analysis
// (Algorithm 1, step 3), done for all signals at once.  It is a dense
// contraction over the signal length n, so it runs on the matrix cores:
// M = running signals, N = atoms, K = n, both operands K-contiguous (the
// dictionary is stored atom by atom, residuals signal by signal).
//
// The K loop is the shared double-buffered MFMA tile loop of gemm_tile.h.
//
// Output: G[a*ldg + j], a = compact index of the running signal, j = atom.  The
// MFMA's row index carries the signal and its lane index the atom, so each
// accumulator register stores 32 consecutive atoms of one signal per
// half-wave (coalesced 128-byte stores).
//
// Several tile shapes are instantiated; the host picks one per launch from the
// number of running signals (autotuned, see bmpl_autotune).  The large-wave shapes
// (128 x 128 and 64 x 128 per wave) issue more matrix instructions per LDS fragment
// read, which the short bfloat16 and e4m3 instructions need.
#include <algorithm>
#include <type_traits>

#include "bmpl_internal.h"
#include "gemm_tile.h"
#include "wave_ops.h"

namespace bmpl {
namespace {

// Store a finished tile: D[row][col] of a 32x32 block (both instructions): lane l, register r -> row
// 8(r/4) + 4(l/32) + r%4, col l%32.  e4m3 operands carry power-of-two scales: one per atom, one per signal.
// A wave whose rows are all running signals stores without a test per row: the row's address is the same in every
// lane (scalar arithmetic), the lane's part of it one 32-bit offset, so a store is one instruction; with the test
// and a 64-bit address per store each was a dozen (bfloat16, 4096 x 20000 x 1024: 215 -> 207 us with the loop below).
// The float32 64 x 64 waves keep the tests: 16 of them share a CU and cover each other's (without: 491 -> 494 us).
struct CorrEpi {
    const float* ascale; const float* rscale;   // e4m3: power-of-two scales, one per atom and one per signal
    float* gm; int64_t ldgm;                    // the groups' largest |g| of each row, or null (not e4m3)
};

template <class E, int TI, int TJ>
__device__ __forceinline__ void store_tile(const floatx16 (&acc)[TI][TJ], int sig0, int ws, int atom0, int wa, int l32,
                                           int h, int m, int n_act, const int* __restrict__ act, float* __restrict__ G,
                                           int64_t ldg, CorrEpi epi)
{
    if constexpr (sizeof(E) != 1 && TJ % 2 == 0) {
        if (epi.gm) {   // the largest |g| of every group, for the selection: a row of 16 lanes by 2 columns of blocks
            const int l16 = l32 & 15;
            const bool b0 = l16 & 1, b1 = (l16 >> 1) & 1, b2 = (l16 >> 2) & 1, b3 = (l16 >> 3) & 1;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; j += 2) {
                    // sixteen rows over sixteen lanes: every exchange halves the rows a lane carries (of its
                    // partners across the row, the half and the quads), lane l16 ends with register l16's row
                    float x8[8], x4[4], x2[2];
                    auto top = [&](int r) { return fmaxf(fabsf(acc[i][j][r]), fabsf(acc[i][j + 1][r])); };
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const float lo = top(r), hi = top(r + 8);
                        x8[r] = fmaxf(b3 ? hi : lo, lane_move<DPP_MIRROR>(b3 ? lo : hi));
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        x4[r] = fmaxf(b2 ? x8[r + 4] : x8[r], lane_move<DPP_HALF_MIRROR>(b2 ? x8[r] : x8[r + 4]));
#pragma unroll
                    for (int r = 0; r < 2; ++r)
                        x2[r] = fmaxf(b1 ? x4[r + 2] : x4[r], lane_move<DPP_XOR2>(b1 ? x4[r] : x4[r + 2]));
                    const float mine = fmaxf(b0 ? x2[1] : x2[0], lane_move<DPP_XOR1>(b0 ? x2[0] : x2[1]));
                    const int a = sig0 + ws + 32 * i + 8 * (l16 >> 2) + 4 * h + (l16 & 3), atom = atom0 + wa + 32 * j;
                    if (a < n_act && atom < m) epi.gm[(int64_t)a * epi.ldgm + 2 * (atom / 64) + (l32 >> 4)] = mine;
                }
        }
    }
    if constexpr (sizeof(E) == 2 || (sizeof(E) == 4 && TI * TJ > 4)) {
        const int r0 = __builtin_amdgcn_readfirstlane(sig0 + ws);
        if (r0 + 32 * TI <= n_act && ldg <= (1 << 26)) {      // the same for the whole wave
            const uint32_t lane_off = 4u * (uint32_t)(4 * h * (int)ldg + l32);
            const int a0 = __builtin_amdgcn_readfirstlane(atom0 + wa);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    if (a0 + 32 * j + l32 >= m) continue;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        float* row = G + (int64_t)(r0 + 32 * i + 8 * (r >> 2) + (r & 3)) * ldg + a0 + 32 * j;
                        at_bytes(row, lane_off) = acc[i][j][r];
                    }
                }
            return;
        }
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int atom = atom0 + wa + 32 * j + l32;
            if (atom >= m) continue;
            const float sa = sizeof(E) == 1 ? epi.ascale[atom] : 1.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int a = sig0 + ws + 32 * i + 8 * (r >> 2) + 4 * h + (r & 3);
                if (a < n_act) {
                    if constexpr (sizeof(E) == 1)
                        G[(int64_t)a * ldg + atom] = acc[i][j][r] * sa * epi.rscale[act ? act[a] : a];
                    else
                        G[(int64_t)a * ldg + atom] = acc[i][j][r];
                }
            }
        }
}

template <class E, int BM, int BN, int WM, int WN, int DEPTH>
__global__ __launch_bounds__((TileShape<BM, BN, WM, WN>::THREADS)) void corr_gemm_kernel(
    const E* __restrict__ At, int64_t lda, int m, int kpad,
    const E* __restrict__ Rbuf, int64_t ldr, const int* __restrict__ act,
    const int* __restrict__ n_act_dev, int p_grid, float* __restrict__ G, int64_t ldg, int tiles_n, int zero_row,
    int n_lo, int n_hi, CorrEpi epi)
{
    using S = TileShape<BM, BN, WM, WN>;
    const int n_act = n_act_dev ? *n_act_dev : p_grid;
    if (n_act < n_lo || n_act >= n_hi) return;   // another tile shape serves this running count
    // Only the signal tiles that hold running signals are numbered (the grid is sized for p_grid, the
    // count at capture time), so the working tiles are dealt evenly to the XCDs at every running count.
    const int tiles_m = ((n_act < p_grid ? n_act : p_grid) + BM - 1) / BM;
    const int nwg = tiles_m * tiles_n;
    if ((int)blockIdx.x >= nwg) return;
    const int tile = xcd_tile_index(blockIdx.x, nwg);
    int tm, tn;                             // signal tile, atom tile (grouped order, see grouped_tile)
    grouped_tile<8>(tile, tiles_m, tiles_n, tm, tn);
    if (tn >= tiles_n) return;
    const int sig0 = tm * BM;
    const int atom0 = tn * BN;
    if (sig0 >= n_act) return;

    __shared__ __attribute__((aligned(16))) TileLds<BM, BN> lds;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    constexpr int VE = 16 / (int)sizeof(E);          // k per 16-byte chunk

    // Rows past the end point at an all-zero row (row `zero_row` of the residuals, row m of
    // the dictionary), so every staging load is unconditional.
    const int c4 = tile_c4(tid);
    const int r0 = tile_r0(tid);
    int64_t oR[S::LX], oA[S::LW];
#pragma unroll
    for (int q = 0; q < S::LX; ++q) {
        const int a = sig0 + r0 + S::RSTEP * q;
        const int s = a < n_act ? (act ? act[a] : a) : zero_row;
        oR[q] = (int64_t)s * ldr + VE * c4;
    }
#pragma unroll
    for (int q = 0; q < S::LW; ++q) {
        const int j = atom0 + r0 + S::RSTEP * q;
        oA[q] = (int64_t)(j < m ? j : m) * lda + VE * c4;
    }
    const int ws = (wave % S::WAVES_M) * WM;   // wave's signal offset in the tile
    const int wa = (wave / S::WAVES_M) * WN;   // wave's atom offset in the tile
    const int l32 = lane & 31;
    const int h = lane >> 5;
    floatx16 acc[S::TI][S::TJ];
    mfma_tile_loop<E, BM, BN, WM, WN, DEPTH>(Rbuf, oR, At, oA, kpad, lds, ws, wa, acc);

    store_tile<E, S::TI, S::TJ>(acc, sig0, ws, atom0, wa, l32, h, m, n_act, act, G, ldg, epi);
}

// The same product with both operand tiles copied straight into swizzled LDS buffers (mfma_tile_loop_dma; bfloat16
// mfma_tile_loop_pipe).
template <class E, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__((TileShape<BM, BN, WM, WN>::THREADS)) void corr_gemm_dma_kernel(
    const E* __restrict__ At, int64_t lda, int m, int kpad,
    const E* __restrict__ Rbuf, int64_t ldr, const int* __restrict__ act,
    const int* __restrict__ n_act_dev, int p_grid, float* __restrict__ G, int64_t ldg, int tiles_n, int zero_row,
    int n_lo, int n_hi, CorrEpi epi)
{
    using S = TileShape<BM, BN, WM, WN>;
    using D = DmaShape<BM, BN, WM, WN>;
    const int n_act = n_act_dev ? *n_act_dev : p_grid;
    if (n_act < n_lo || n_act >= n_hi) return;   // another tile shape serves this running count
    const int tiles_m = ((n_act < p_grid ? n_act : p_grid) + BM - 1) / BM;   // as in corr_gemm_kernel
    const int nwg = tiles_m * tiles_n;
    if ((int)blockIdx.x >= nwg) return;
    const int tile = xcd_tile_index(blockIdx.x, nwg);
    int tm, tn;
    grouped_tile<8>(tile, tiles_m, tiles_n, tm, tn);
    if (tn >= tiles_n) return;
    const int sig0 = tm * BM;
    const int atom0 = tn * BN;
    if (sig0 >= n_act) return;

    using Lds = std::conditional_t<sizeof(E) == 2, PipeLds<BM, BN, 2>, DmaLds<BM, BN>>;
    __shared__ __attribute__((aligned(1024))) Lds lds;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    constexpr int VE = 16 / (int)sizeof(E);          // k per 16-byte chunk
    // rows past the end read an all-zero row (row zero_row of the residuals, row m of the dictionary)
    int64_t oR[D::GX], oA[D::GW];
#pragma unroll
    for (int i = 0; i < D::GX; ++i) {
        const int g = wave + S::WAVES * i;
        const int a = sig0 + dma_row(g, lane);
        const int sg = a < n_act ? (act ? act[a] : a) : zero_row;
        oR[i] = (int64_t)sg * ldr + VE * dma_chunk(g, lane);
    }
#pragma unroll
    for (int i = 0; i < D::GW; ++i) {
        const int g = wave + S::WAVES * i;
        const int j = atom0 + dma_row(g, lane);
        oA[i] = (int64_t)(j < m ? j : m) * lda + VE * dma_chunk(g, lane);
    }
    const int ws = (wave % S::WAVES_M) * WM;
    const int wa = (wave / S::WAVES_M) * WN;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    floatx16 acc[S::TI][S::TJ];
    if constexpr (sizeof(E) == 2)
        mfma_tile_loop_pipe<BM, BN, WM, WN, 2>(Rbuf, oR, At, oA, kpad, lds, ws, wa, acc);
    else
        mfma_tile_loop_dma<E, BM, BN, WM, WN>(Rbuf, oR, At, oA, kpad, lds, ws, wa, acc);
    store_tile<E, S::TI, S::TJ>(acc, sig0, ws, atom0, wa, l32, h, m, n_act, act, G, ldg, epi);
}

// ---------------------------------------------------------------------------------------------------
// bfloat16 product with the dictionary operand read straight from global memory into registers.
//
// The dictionary is fixed for a context, so its bfloat16 copy is also stored in the matrix
// instruction's fragment order (pack_bf16_fragments_kernel): for a block of 32 atoms and a chunk of 16
// k, the 64 lanes' 16-byte B fragments are one contiguous kilobyte (lane l: atom 32 jb + l % 32,
// k = 16 c + 8 (l / 32) .. + 8).  A wave loads its fragments with fully coalesced 16-byte loads, a
// whole stage (four chunks) ahead, and only the residual tile goes through LDS; this removes the
// dictionary's LDS stores and fragment reads, which bound the all-LDS loop for 16-bit operands.
// Atoms are padded to a multiple of 256 with zero fragments, so no load is predicated.
// ---------------------------------------------------------------------------------------------------
constexpr int PACK_ATOMS = 256;   // atom padding of the packed copy

__global__ __launch_bounds__(256) void pack_bf16_fragments_kernel(const uint16_t* __restrict__ A16, int64_t lda,
                                                                  int m, int kpad, uint4* __restrict__ Apk,
                                                                  int m_pad)
{
    const int nkc = kpad / 16;
    const int64_t total = (int64_t)(m_pad / 32) * nkc * 64;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int lane = (int)(e & 63);
        const int64_t fc = e >> 6;             // fragment index = jb * nkc + c
        const int c = (int)(fc % nkc);
        const int jb = (int)(fc / nkc);
        const int atom = 32 * jb + (lane & 31);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (atom < m) v = *reinterpret_cast<const uint4*>(A16 + (int64_t)atom * lda + 16 * c + 8 * (lane >> 5));
        Apk[e] = v;
    }
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__((TileShape<BM, BN, WM, WN>::THREADS)) void corr_gemm_direct_kernel(
    const uint4* __restrict__ Apk, int m, int kpad, const __bf16* __restrict__ Rbuf, int64_t ldr,
    const int* __restrict__ act, const int* __restrict__ n_act_dev, int p_grid, float* __restrict__ G,
    int64_t ldg, int tiles_n, int zero_row, int n_lo, int n_hi, CorrEpi epi)
{
    using S = TileShape<BM, BN, WM, WN>;
    constexpr int TI = S::TI, TJ = S::TJ;
    constexpr int LR = BM * 8 / S::THREADS;            // 16-byte residual loads per thread and stage
    static_assert(LR * S::THREADS == BM * 8, "residual staging");
    const int n_act = n_act_dev ? *n_act_dev : p_grid;
    if (n_act < n_lo || n_act >= n_hi) return;   // another tile shape serves this running count
    const int tiles_m = ((n_act < p_grid ? n_act : p_grid) + BM - 1) / BM;   // as in corr_gemm_kernel
    const int nwg = tiles_m * tiles_n;
    if ((int)blockIdx.x >= nwg) return;
    const int tile = xcd_tile_index(blockIdx.x, nwg);
    int tm, tn;
    grouped_tile<8>(tile, tiles_m, tiles_n, tm, tn);
    if (tn >= tiles_n) return;
    const int sig0 = tm * BM;
    const int atom0 = tn * BN;
    if (sig0 >= n_act) return;

    __shared__ __attribute__((aligned(16))) char ldsR[2][BM * TILE_LDS_ROW];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int c4 = tile_c4(tid);
    const int r0 = tile_r0(tid);
    int64_t oR[LR];
#pragma unroll
    for (int q = 0; q < LR; ++q) {
        const int a = sig0 + r0 + S::RSTEP * q;
        const int sg = a < n_act ? (act ? act[a] : a) : zero_row;
        oR[q] = (int64_t)sg * ldr + 8 * c4;
    }
    const int ws = (wave % S::WAVES_M) * WM;
    const int wa = (wave / S::WAVES_M) * WN;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int nkc = kpad / 16;
    const uint4* aP[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) aP[j] = Apk + ((int64_t)((atom0 + wa) / 32 + j) * nkc) * 64 + lane;

    floatx16 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    float4 gR[LR];
    uint4 aC[4][TJ], aN[4][TJ];
#pragma unroll
    for (int q = 0; q < LR; ++q) gR[q] = *reinterpret_cast<const float4*>(Rbuf + oR[q]);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int j = 0; j < TJ; ++j) aC[kb][j] = aP[j][64 * kb];
#pragma unroll
    for (int q = 0; q < LR; ++q)
        *reinterpret_cast<float4*>(&ldsR[0][(r0 + S::RSTEP * q) * TILE_LDS_ROW + 16 * c4]) = gR[q];
    __syncthreads();
    int cur = 0;
    for (int k0 = 0; k0 < kpad; k0 += 64) {
        // next stage: residual slice into registers, dictionary fragments (the last stage re-reads itself)
        const int kn = k0 + 64 < kpad ? k0 + 64 : k0;
        const int cn = kn / 16;
#pragma unroll
        for (int q = 0; q < LR; ++q) gR[q] = *reinterpret_cast<const float4*>(Rbuf + oR[q] + kn);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int j = 0; j < TJ; ++j) aN[kb][j] = aP[j][64 * (cn + kb)];
        asm volatile("" ::: "memory");
        const char* cR = ldsR[cur];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            float4 fx[TI];
#pragma unroll
            for (int i = 0; i < TI; ++i)
                fx[i] = *reinterpret_cast<const float4*>(&cR[(ws + 32 * i + l32) * TILE_LDS_ROW + kb * 32 + 16 * h]);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fx[i]),
                                                                       __builtin_bit_cast(bf16x8, aC[kb][j]),
                                                                       acc[i][j], 0, 0, 0);
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < LR; ++q) {
            staged(gR[q]);   // see gemm_tile.h: keeps the residual load a stage ahead
            *reinterpret_cast<float4*>(&ldsR[cur ^ 1][(r0 + S::RSTEP * q) * TILE_LDS_ROW + 16 * c4]) = gR[q];
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int j = 0; j < TJ; ++j) aC[kb][j] = aN[kb][j];
        __syncthreads();
        cur ^= 1;
    }
    store_tile<__bf16, TI, TJ>(acc, sig0, ws, atom0, wa, l32, h, m, n_act, act, G, ldg, epi);
}

// ---------------------------------------------------------------------------------------------------
// The product for a few running signals (shape 4).  Below a few dozen signals the product reads the dictionary
// once and does little with it: the bound is HBM (134 MB of float32 at 2048 x 16384), so what counts is how many
// bytes are in flight and that no matrix work is done for padding.  One wave per workgroup, all its operands
// straight from global memory into registers (16 bytes per lane, two or three stages of 256 or 128 bytes per row in
// flight), no LDS and no barrier, so the waves of a CU drift freely; the signals' rows are shared through L1.
// 8 residuals against 2048 x 16384: 43.7 -> 27.7 us (4.9 TB/s), one against 1000 x 5001: 22.8 -> 9.3 us (before: 32 x 64
// tiles of two 32 x 32 waves through LDS).
//
// float32: 16 atoms x 32 signals per wave (16 when no more are running) by v_mfma_f32_16x16x4f32.  The float32
// matrix instructions accumulate their k in order of the lane groups, one fused multiply-add each, so taking k in
// the order of the 32 x 32 x 2 steps of the other shapes (8 b + t, 8 b + 4 + t, t = 0..3) gives the same bits: two
// steps of four k, k = 8 b + {0, 4, 1, 5} and {2, 6, 3, 7} over the lane groups q = 0..3.  A lane loads k = 16 B +
// 4 q .. + 3 of its row; v_permlane32_swap of the loaded .x and .y (.z and .w) pairs the lane groups 0, 1 with 2, 3
// as those steps want them, for b = 2 B and 2 B + 1 at once.
// ---------------------------------------------------------------------------------------------------
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void swap_halves(float& x, float& y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);   // lanes 0..31 of x, then lanes 0..31 of y
    y = __uint_as_float(r[1]);   // lanes 32..63 of x, then lanes 32..63 of y
}

constexpr int FEW_M = 32;        // signals per wave

template <int GROUPS>
__device__ __forceinline__ void few_f32_loop(const float* pa, const float* (&pr)[2], int stages, floatx4 (&acc)[2])
{
    constexpr int BUF = 3;       // stages of 64 k in registers
    floatx4 a[BUF][4], r[BUF][GROUPS][4];   // native vectors: the compiler keeps each in one register tuple
    auto load = [&](int st, floatx4 (&fa)[4], floatx4 (&fr)[GROUPS][4]) {
        const int k0 = 64 * (st < stages ? st : stages - 1);   // past the end: re-read the last, never used
#pragma unroll
        for (int e = 0; e < 4; ++e) fa[e] = *reinterpret_cast<const floatx4*>(pa + k0 + 16 * e);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) fr[g][e] = *reinterpret_cast<const floatx4*>(pr[g] + k0 + 16 * e);
    };
    auto compute = [&](const floatx4 (&va)[4], const floatx4 (&vr)[GROUPS][4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            floatx4 fa = va[e];
            asm volatile("" : "+v"(fa));         // consumed here, not where it was loaded
            float a0 = fa[0], a1 = fa[1], a2 = fa[2], a3 = fa[3];
            swap_halves(a0, a1);
            swap_halves(a2, a3);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                floatx4 fr = vr[g][e];
                asm volatile("" : "+v"(fr));
                float r0 = fr[0], r1 = fr[1], r2 = fr[2], r3 = fr[3];
                swap_halves(r0, r1);
                swap_halves(r2, r3);
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(r0, a0, acc[g], 0, 0, 0);
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(r2, a2, acc[g], 0, 0, 0);
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(r1, a1, acc[g], 0, 0, 0);
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(r3, a3, acc[g], 0, 0, 0);
            }
        }
    };
    // whole groups of BUF stages without a branch (a join would make the loads before it wait), then the rest
#pragma unroll
    for (int d = 0; d < BUF - 1; ++d) load(d, a[d], r[d]);
    int s0 = 0;
    for (; s0 + BUF <= stages; s0 += BUF) {
#pragma unroll
        for (int d = 0; d < BUF; ++d) {
            load(s0 + d + BUF - 1, a[(d + BUF - 1) % BUF], r[(d + BUF - 1) % BUF]);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay ahead of this stage's matrix work
            compute(a[d], r[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < BUF - 1; ++d)
        if (s0 + d < stages) compute(a[d], r[d]);
}

__global__ __launch_bounds__(64) void corr_few_f32_kernel(
    const float* __restrict__ At, int64_t lda, int m, int kpad, const float* __restrict__ Rbuf, int64_t ldr,
    const int* __restrict__ act, const int* __restrict__ n_act_dev, int p_grid, float* __restrict__ G, int64_t ldg,
    int tiles_n, int zero_row, int n_lo, int n_hi)
{
    const int n_act = n_act_dev ? *n_act_dev : p_grid;
    if (n_act < n_lo || n_act >= n_hi) return;   // another tile shape serves this running count
    const int tiles_m = ((n_act < p_grid ? n_act : p_grid) + FEW_M - 1) / FEW_M;   // as in corr_gemm_kernel
    const int nwg = tiles_m * tiles_n;
    if ((int)blockIdx.x >= nwg) return;
    const int tile = xcd_tile_index(blockIdx.x, nwg);
    const int tm = tile % tiles_m, tn = tile / tiles_m;
    const int sig0 = tm * FEW_M, atom0 = tn * 16;
    const int lane = threadIdx.x, l16 = lane & 15, q = lane >> 4;
    const float* pr[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int i = sig0 + 16 * g + l16;
        pr[g] = Rbuf + (int64_t)(i < n_act ? (act ? act[i] : i) : zero_row) * ldr + 4 * q;
    }
    const int ja = atom0 + l16;
    const float* pa = At + (int64_t)(ja < m ? ja : m) * lda + 4 * q;
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    const bool two = sig0 + 16 < n_act;          // the same for the whole wave
    if (two) few_f32_loop<2>(pa, pr, kpad / 64, acc);
    else few_f32_loop<1>(pa, pr, kpad / 64, acc);
    if (ja >= m) return;
    // D of a 16 x 16 block: lane l, register r -> row (signal) 4 (l / 16) + r, column (atom) l % 16
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = sig0 + 16 * g + 4 * q + r;
            if (i < n_act) G[(int64_t)i * ldg + ja] = acc[g][r];
        }
}

// 16- and 8-bit operands: 32 atoms x 32 signals per wave, the matrix steps and their k order of mfma_tile_stage.
template <class E>
__global__ __launch_bounds__(64) void corr_few_kernel(
    const E* __restrict__ At, int64_t lda, int m, int kpad, const E* __restrict__ Rbuf, int64_t ldr,
    const int* __restrict__ act, const int* __restrict__ n_act_dev, int p_grid, float* __restrict__ G, int64_t ldg,
    int tiles_n, int zero_row, int n_lo, int n_hi, CorrEpi epi)
{
    const int n_act = n_act_dev ? *n_act_dev : p_grid;
    if (n_act < n_lo || n_act >= n_hi) return;   // another tile shape serves this running count
    const int tiles_m = ((n_act < p_grid ? n_act : p_grid) + FEW_M - 1) / FEW_M;   // as in corr_gemm_kernel
    const int nwg = tiles_m * tiles_n;
    if ((int)blockIdx.x >= nwg) return;
    const int tile = xcd_tile_index(blockIdx.x, nwg);
    const int tm = tile % tiles_m, tn = tile / tiles_m;
    const int sig0 = tm * FEW_M, atom0 = tn * 32;
    const int lane = threadIdx.x, l32 = lane & 31, h = lane >> 5;
    const int is = sig0 + l32, ja = atom0 + l32;
    const char* pr = reinterpret_cast<const char*>(Rbuf + (int64_t)(is < n_act ? (act ? act[is] : is) : zero_row) * ldr);
    const char* pa = reinterpret_cast<const char*>(At + (int64_t)(ja < m ? ja : m) * lda);
    const int stages = kpad * (int)sizeof(E) / TILE_ROW_BYTES;
    constexpr int BUF = 4;       // stages of 128 bytes per row in registers
    // chunk e of a stage (16 bytes per lane): bfloat16 k = 64 st + 16 e + 8 h, e4m3 bytes 64 (e / 2) + 32 h + 16 (e % 2)
    floatx4 a[BUF][4], r[BUF][4];
    auto load = [&](int st, floatx4 (&fa)[4], floatx4 (&fr)[4]) {
        const int b0 = TILE_ROW_BYTES * (st < stages ? st : stages - 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int o = b0 + (sizeof(E) == 1 ? 64 * (e >> 1) + 32 * h + 16 * (e & 1) : 32 * e + 16 * h);
            fa[e] = *reinterpret_cast<const floatx4*>(pa + o);
            fr[e] = *reinterpret_cast<const floatx4*>(pr + o);
        }
    };
    floatx16 acc[1][1];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[0][0][i] = 0.f;
    auto compute = [&](const floatx4 (&va)[4], const floatx4 (&vr)[4]) {
        if constexpr (sizeof(E) == 1) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                // the two 16-byte halves of each operand as one 32-byte fragment
                const auto wide = [](floatx4 lo, floatx4 hi) {
                    return __builtin_bit_cast(intx8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                };
                const intx8 fx = wide(vr[2 * t], vr[2 * t + 1]), fw = wide(va[2 * t], va[2 * t + 1]);
                acc[0][0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fx, fw, acc[0][0], 0, 0, 0, 127, 0, 127);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, vr[e]), __builtin_bit_cast(bf16x8, va[e]), acc[0][0], 0, 0, 0);
        }
    };
    // as in few_f32_loop
#pragma unroll
    for (int d = 0; d < BUF - 1; ++d) load(d, a[d], r[d]);
    int s0 = 0;
    for (; s0 + BUF <= stages; s0 += BUF) {
#pragma unroll
        for (int d = 0; d < BUF; ++d) {
            load(s0 + d + BUF - 1, a[(d + BUF - 1) % BUF], r[(d + BUF - 1) % BUF]);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay ahead of this stage's matrix work
            compute(a[d], r[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < BUF - 1; ++d)
        if (s0 + d < stages) compute(a[d], r[d]);
    store_tile<E, 1, 1>(acc, sig0, 0, atom0, 0, l32, h, m, n_act, act, G, ldg, epi);
}

template <class E>
hipError_t launch_few(const E* At, int64_t lda, int m, int kpad, const E* Rbuf, int64_t ldr, const int* act,
                      const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row, int n_lo, int n_hi,
                      CorrEpi epi, hipStream_t stream)
{
    constexpr int BN = sizeof(E) == 4 ? 16 : 32;
    const int tiles_m = (p_grid + FEW_M - 1) / FEW_M;
    const int tiles_n = (m + BN - 1) / BN;
    const int64_t nwg = (int64_t)tiles_m * tiles_n;
    if (nwg > 0x7fffffff) return hipErrorInvalidValue;
    if constexpr (sizeof(E) == 4) {
        if (kpad % 64) return hipErrorInvalidValue;
        hipLaunchKernelGGL(corr_few_f32_kernel, dim3((unsigned)nwg), dim3(64), 0, stream, At, lda, m, kpad, Rbuf, ldr, act,
                           n_act_dev, p_grid, G, ldg, tiles_n, zero_row, n_lo, n_hi);
    } else {
        hipLaunchKernelGGL(corr_few_kernel<E>, dim3((unsigned)nwg), dim3(64), 0, stream, At, lda, m, kpad, Rbuf, ldr, act,
                           n_act_dev, p_grid, G, ldg, tiles_n, zero_row, n_lo, n_hi, epi);
    }
    return hipGetLastError();
}

template <int BM, int BN, int WM, int WN>
hipError_t launch_direct(const uint16_t* Apk, int m, int kpad, const uint16_t* Rbuf, int64_t ldr, const int* act,
                         const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row, int n_lo, int n_hi,
                         CorrEpi epi, hipStream_t stream)
{
    static_assert(PACK_ATOMS % BN == 0, "atom tiles must lie inside the packed padding");
    const int tiles_m = (p_grid + BM - 1) / BM;
    const int tiles_n = (m + BN - 1) / BN;
    const int64_t nwg = (int64_t)tiles_m * tiles_n;
    if (nwg > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((corr_gemm_direct_kernel<BM, BN, WM, WN>), dim3((unsigned)nwg),
                       dim3(TileShape<BM, BN, WM, WN>::THREADS), 0, stream, reinterpret_cast<const uint4*>(Apk), m,
                       kpad, reinterpret_cast<const __bf16*>(Rbuf), ldr, act, n_act_dev, p_grid, G, ldg, tiles_n,
                       zero_row, n_lo, n_hi, epi);
    return hipGetLastError();
}

template <class E, int BM, int BN, int WM, int WN, int DEPTH = 1>
hipError_t launch_shape(const E* At, int64_t lda, int m, int kpad, const E* Rbuf, int64_t ldr,
                        const int* act, const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row,
                        int n_lo, int n_hi, CorrEpi epi, hipStream_t stream)
{
    const int tiles_m = (p_grid + BM - 1) / BM;
    const int tiles_n = (m + BN - 1) / BN;
    const int64_t nwg = (int64_t)tiles_m * tiles_n;
    if (nwg > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((corr_gemm_kernel<E, BM, BN, WM, WN, DEPTH>), dim3((unsigned)nwg),
                       dim3(TileShape<BM, BN, WM, WN>::THREADS), 0, stream, At, lda, m, kpad, Rbuf, ldr, act,
                       n_act_dev, p_grid, G, ldg, tiles_n, zero_row, n_lo, n_hi, epi);
    return hipGetLastError();
}

template <class E, int BM, int BN, int WM, int WN>
hipError_t launch_dma(const E* At, int64_t lda, int m, int kpad, const E* Rbuf, int64_t ldr, const int* act,
                      const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row, int n_lo, int n_hi,
                      CorrEpi epi, hipStream_t stream)
{
    const int tiles_m = (p_grid + BM - 1) / BM;
    const int tiles_n = (m + BN - 1) / BN;
    const int64_t nwg = (int64_t)tiles_m * tiles_n;
    if (nwg > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((corr_gemm_dma_kernel<E, BM, BN, WM, WN>), dim3((unsigned)nwg),
                       dim3(TileShape<BM, BN, WM, WN>::THREADS), 0, stream, At, lda, m, kpad, Rbuf, ldr, act,
                       n_act_dev, p_grid, G, ldg, tiles_n, zero_row, n_lo, n_hi, epi);
    return hipGetLastError();
}

template <class E>
hipError_t launch_variant(int variant, const E* At, int64_t lda, int m, int kpad, const E* Rbuf, int64_t ldr,
                          const int* act, const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row,
                          int n_lo, int n_hi, hipStream_t stream, CorrEpi epi)
{
    if (p_grid <= 0 || m <= 0) return hipSuccess;
    if (kpad % (TILE_ROW_BYTES / (int)sizeof(E))) return hipErrorInvalidValue;
    // float32 stages of the shapes with registers to spare load two stages ahead (faster: 604 -> 514 us
    // for the 256 x 128 tile at 1024 signals); 16- and 8-bit stages measured slower that way
    constexpr int DEEP = sizeof(E) == 4 ? 2 : 1;
    switch (variant) {
    case 0: return launch_shape<E, 128, 128, 64, 64, DEEP>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 1: return launch_shape<E, 256, 256, 64, 64>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 2: return launch_shape<E, 256, 128, 64, 64, DEEP>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 3: return launch_shape<E, 64, 128, 32, 64, DEEP>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 4: return launch_few<E>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 5: return launch_shape<E, 64, 64, 32, 32, DEEP>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 6: return launch_shape<E, 256, 256, 128, 128>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 7: return launch_shape<E, 256, 256, 128, 64>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 11: return launch_dma<E, 256, 256, 128, 64>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 12: return launch_dma<E, 256, 256, 64, 64>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 13: return launch_dma<E, 128, 128, 64, 64>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    case 14: return launch_dma<E, 256, 256, 128, 128>(At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

const char* corr_shape_name(int v)
{
    switch (v) {
    case 8: return "256x256 (8 waves of 128x64), dictionary fragments from global memory";
    case 9: return "128x256 (8 waves of 64x64), dictionary fragments from global memory";
    case 10: return "256x128 (4 waves of 128x64), dictionary fragments from global memory";
    case 0: return "128x128 (4 waves of 64x64)";
    case 1: return "256x256 (16 waves of 64x64)";
    case 2: return "256x128 (8 waves of 64x64)";
    case 3: return "64x128 (4 waves of 32x64)";
    case 4: return "32x16 (float32) or 32x32 (one wave, operands from global memory)";
    case 5: return "64x64 (4 waves of 32x32)";
    case 6: return "256x256 (4 waves of 128x128)";
    case 7: return "256x256 (8 waves of 128x64)";
    case 11: return "256x256 (8 waves of 128x64), operand tiles copied straight into LDS";
    case 12: return "256x256 (16 waves of 64x64), operand tiles copied straight into LDS";
    case 13: return "128x128 (4 waves of 64x64), operand tiles copied straight into LDS";
    case 14: return "256x256 (4 waves of 128x128), operand tiles copied straight into LDS";
    default: return "?";
    }
}

bool corr_shape_has_groups(int variant) { return variant != 4 && variant != 5; }   // waves of 64 atoms or more

// The tile shape of p signals when none was set.  A launch takes rounds of tiles over the card's 256 CUs, so the best
// shape follows from how many rounds its tile count leaves: each candidate's time is modelled as a start plus
// the rounds times a round's time, both measured at kpad = 2048 and scaled by kpad.  Measured at 1000 signals
// (us): float32, 1024 x 20000: shape 13 337, 5 363, 12 493 (two rounds for 316 tiles); 2048 x 16384: 12 491, 13 521,
// 5 572, and 0, which every batch from 512 on took, 542; bfloat16: 62, 79, 75 and 77, 117, 75 (11: 72).  100 signals
// of 512 x 4096, float32: 4 18, 5 19, 3 27; 64: 4 13.5, 5 18, 3 26.5; 40 signals of 2048 x 16384: 5 56, 4 93.
int corr_default_shape(bool bf16, int m, int kpad, int p)
{
    struct Shape { int id, bm, bn, at_once; double start, round; };
    static const Shape f32[] = {{5, 64, 64, 256, 20.0, 34.5}, {3, 64, 128, 256, 20.0, 67.0},
                                {13, 128, 128, 256, 20.0, 126.0}, {12, 256, 256, 256, 5.0, 487.0}};
    static const Shape b16[] = {{5, 64, 64, 256, 6.0, 6.5}, {3, 64, 128, 256, 8.0, 11.0},
                                {13, 128, 128, 512, 0.0, 33.0}, {11, 256, 256, 256, 0.0, 61.0}};
    // the few-signals shape: the dictionary once per 32 signals, at about 3 TB/s
    const int groups = (p + 31) / 32;
    int best = 4;
    double t = 5.0 + (bf16 ? 2.0 : 4.0) * m * kpad * groups / (bf16 ? 2.0e6 : 2.9e6);
    if (p <= 32) return best;
    for (const Shape& c : bf16 ? b16 : f32) {
        const int64_t tiles = (int64_t)((p + c.bm - 1) / c.bm) * ((m + c.bn - 1) / c.bn);
        const double u = (c.start + c.round * (double)((tiles + c.at_once - 1) / c.at_once)) * kpad / 2048.0;
        if (u < t) { t = u; best = c.id; }
    }
    return best;
}

hipError_t launch_corr_gemm_f32(int variant, const float* At, int64_t lda, int m, int kpad,
                                const float* Rbuf, int64_t ldr, const int* act,
                                const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row,
                                int n_lo, int n_hi, hipStream_t stream, float* gm, int64_t ldgm)
{
    return launch_variant<float>(variant, At, lda, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row,
                                 n_lo, n_hi, stream, CorrEpi{nullptr, nullptr, gm, ldgm});
}

hipError_t launch_corr_gemm_fp8(int variant, const uint8_t* A8, int64_t lda, int m, int kpad,
                                const uint8_t* R8, int64_t ldr, const int* act,
                                const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row,
                                int n_lo, int n_hi, const float* ascale, const float* rscale, hipStream_t stream)
{
    if (!ascale || !rscale) return hipErrorInvalidValue;
    return launch_variant<uint8_t>(variant, A8, lda, m, kpad, R8, ldr, act, n_act_dev, p_grid, G, ldg, zero_row,
                                   n_lo, n_hi, stream, CorrEpi{ascale, rscale, nullptr, 0});
}

size_t packed_bf16_elems(int m, int kpad)
{
    return (size_t)((m + PACK_ATOMS - 1) / PACK_ATOMS * PACK_ATOMS) * (size_t)kpad;
}

hipError_t launch_pack_bf16(const uint16_t* A16, int64_t lda, int m, int kpad, uint16_t* Apk, hipStream_t stream)
{
    if (kpad % 64) return hipErrorInvalidValue;
    const int m_pad = (m + PACK_ATOMS - 1) / PACK_ATOMS * PACK_ATOMS;
    const int64_t total = (int64_t)(m_pad / 32) * (kpad / 16) * 64;
    const int grid = (int)std::min<int64_t>((total + 255) / 256, 65536);
    hipLaunchKernelGGL(pack_bf16_fragments_kernel, dim3(grid), dim3(256), 0, stream, A16, lda, m, kpad,
                       reinterpret_cast<uint4*>(Apk), m_pad);
    return hipGetLastError();
}

hipError_t launch_corr_gemm_bf16(int variant, const uint16_t* At, const uint16_t* Apk, int64_t lda, int m, int kpad,
                                 const uint16_t* Rbuf, int64_t ldr, const int* act,
                                 const int* n_act_dev, int p_grid, float* G, int64_t ldg, int zero_row,
                                 int n_lo, int n_hi, hipStream_t stream, float* gm, int64_t ldgm)
{
    const CorrEpi epi{nullptr, nullptr, gm, ldgm};
    if (variant >= 8 && variant <= 10) {
        if (!Apk || p_grid <= 0 || m <= 0) return Apk ? hipSuccess : hipErrorInvalidValue;
        if (kpad % 64) return hipErrorInvalidValue;
        switch (variant) {
        case 8: return launch_direct<256, 256, 128, 64>(Apk, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
        case 9: return launch_direct<128, 256, 64, 64>(Apk, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
        case 10: return launch_direct<256, 128, 128, 64>(Apk, m, kpad, Rbuf, ldr, act, n_act_dev, p_grid, G, ldg, zero_row, n_lo, n_hi, epi, stream);
        default: return hipErrorInvalidValue;
        }
    }
    return launch_variant<__bf16>(variant, reinterpret_cast<const __bf16*>(At), lda, m, kpad,
                                  reinterpret_cast<const __bf16*>(Rbuf), ldr, act, n_act_dev, p_grid, G, ldg,
                                  zero_row, n_lo, n_hi, stream, epi);
}

}  // namespace bmpl
