// Worst-case analysis (Algorithm 1, step 3): per running signal, pick the atoms
// outside the active set I with the largest |g_j| that violate |g_j| > lambda
// (the natural stopping condition, Eq. (9), fails exactly for these), at most k
// of them, largest first, ties to the lower atom index.
//
// One 256-thread workgroup per signal reads its row of correlations once
// (coalesced).  Each thread's first eight 16-byte loads stay in registers; the
// k-th largest of the threads' maxima over them bounds the row's k-th largest from
// below (they are k distinct entries of the row).  The registered entries and the
// rest of the row as it streams in are tested against that bound and lambda; the
// few that pass are appended to an LDS buffer (one atomic per wave and step) and
// ranked by (|g|, lower index): by counting for up to 256 entries, else by a bitonic sort.
// On the first pass of the relative lambda rule the row maximum is reduced first
// and lambda_i = c * ||A^T b_i||_inf is set from it (Section IV-A).
#include <float.h>
#include <limits.h>
#include <stdint.h>

#include "bmpl_internal.h"
#include "wave_ops.h"

namespace bmpl {
namespace {

__device__ inline bool better(float v, int i, float w, int j)
{
    return v > w || (v == w && i < j);
}

// With a float32 band: a signal that admitted nothing although it had room, and whose largest |g~| is
// within its band eps_i of lambda, takes the exact re-score of certify_row.
__device__ inline bool needs_certification(const SelectArgs& a, int sig, int k, int nsel, float vmax, double lam)
{
    return a.band > 0.0 && nsel == 0 && k > 0 && (double)vmax + a.band * sqrt(a.rr2[sig]) > lam;
}

// The selection of one signal; *certify is set by thread 0.
// Latency bounds it, not the bytes: 1024 rows of 16 384 are 22 us (3 TB/s), a short row 8 us (10.6 before the loads of
// its tail were issued together and the words of the bitmap stopped waiting for the values before them).
// GROUPS: the launch may have the groups' largest values (the kernel without them keeps its registers).
template <int KMAX, bool GROUPS>
__device__ __forceinline__ void select_row(const SelectArgs& a, int row, int sig, bool grouped, bool* certify)
{
    const float* g = a.G + (int64_t)row * a.ldg;
    const uint32_t* ex = a.excl ? a.excl + (int64_t)sig * a.words : nullptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    __shared__ float s_red[4];
    __shared__ float s_val[4 * KMAX];
    __shared__ int s_idx[4 * KMAX];
    __shared__ double s_lam;

    // Per-signal cap on the number of atoms admitted this pass.
    int k = a.k;
    if (a.nI && a.max_active > 0) {
        int room = a.max_active - a.nI[sig];
        k = room < k ? (room > 0 ? room : 0) : k;
    }

    // Rows are read as float4 when the layout allows it (the internal buffers always do).
    const bool vec4 = ((a.ldg & 3) == 0) && ((reinterpret_cast<uintptr_t>(a.G) & 15) == 0);
    const int m4 = vec4 ? (a.m & ~3) : 0;

    // Each thread's first CH float4 of the row stay in registers (issued before lambda is read, so the
    // loads are in flight meanwhile); the rest is streamed once later.
    constexpr int CH = 8;
    constexpr int CAPG = GROUPS ? 1024 : 1;
    __shared__ int s_gl[CAPG];
    __shared__ int s_ng;
    const float* gm = a.gm + (int64_t)row * a.ldgm;
    float4 f0[CH];
    uint32_t w0[CH];
    if (!grouped) row_chunks<CH>(g, ex, 0, m4, f0, w0);   // 4 atoms share one word
    // The rest of the row streams in chunks of CS float4 per thread, each chunk's loads issued one chunk
    // ahead (the first before the bound is computed), so a workgroup waits for memory about once.
    constexpr int CS = 4;
    float4 fa[CS];
    uint32_t wa[CS];
    auto load_chunk = [&](int base0, float4 (&f)[CS], uint32_t (&word)[CS]) {
        row_chunks<CS>(g, ex, base0, m4, f, word);
    };
    if (!grouped) load_chunk(1024 * CH, fa, wa);
    float tmax = -1.f, gall = 0.f;
    if (grouped) group_maxima(gm, corr_groups(a.m), ex, a.words, tmax, gall);

    // Pass 1 (relative lambda rule only): lambda_i = c * max_j |g_j|.
    if (a.lam_rel > 0.0) {
        float mx = gall;
        if (!grouped) {
#pragma unroll 4
            for (int j0 = 4 * tid; j0 < m4; j0 += 1024) {
                const float4 f = *reinterpret_cast<const float4*>(g + j0);
                mx = fmaxf(mx, fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w))));
            }
            for (int j = m4 + tid; j < a.m; j += 256) mx = fmaxf(mx, fabsf(g[j]));
        }
        mx = wave_max(mx);
        if (lane == 0) s_red[wave] = mx;
        __syncthreads();
        if (tid == 0) {
            float v = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
            a.lam[sig] = a.lam_rel * (double)v;
        }
        __syncthreads();
    }
    if (tid == 0) s_lam = a.lam[sig];
    __syncthreads();
    const double lam = s_lam;
    // (double)v > lam  <=>  v > lamf for every float v, with lamf the largest float <= lam
    float lamf = (float)lam;
    if ((double)lamf > lam) lamf = nextafterf(lamf, -INFINITY);

    // The k-th largest of the 256 threads' maxima over their registered entries is at most the k-th
    // largest |g_j| of the row (they are k distinct entries of it), so only entries >= T can be among
    // the k largest: the insertions below skip the rest.
    if (!grouped) {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        w0[q] = chunk_bits(ex, w0[q], 4 * tid + 1024 * q, m4);
        if (!(w0[q] & 1u)) tmax = fmaxf(tmax, fabsf(f0[q].x));
        if (!(w0[q] & 2u)) tmax = fmaxf(tmax, fabsf(f0[q].y));
        if (!(w0[q] & 4u)) tmax = fmaxf(tmax, fabsf(f0[q].z));
        if (!(w0[q] & 8u)) tmax = fmaxf(tmax, fabsf(f0[q].w));
    }
    }
    float vmx = fmaxf(tmax, 0.f);
    {
        float cur = tmax;
        for (int r = 0; r < k; ++r) {
            const float b = wave_max(cur);
            if (lane == 0) s_val[wave * KMAX + r] = b;
            const unsigned long long owners = __ballot(cur == b);
            if (lane == __ffsll((long long)owners) - 1) cur = -2.f;   // pop one holder
        }
    }
    if (tid == 0) s_red[0] = INFINITY;           // k = 0: nothing is admitted
    __syncthreads();
    if (tid < 4 * k) {
        // T = the k-th largest of the 4k listed maxima: the value with fewer than k larger ones and at
        // least k at or above it (equal values write the same T)
        const int tw = tid / k;
        const float v = s_val[tw * KMAX + (tid - tw * k)];
        int gt = 0, ge = 0;
        for (int w2 = 0; w2 < 4; ++w2)
            for (int r = 0; r < k; ++r) {
                const float w = s_val[w2 * KMAX + r];
                gt += w > v;
                ge += w >= v;
            }
        if (gt < k && ge >= k) s_red[0] = v;
    }
    __syncthreads();
    const float T = s_red[0];
    __syncthreads();

    {
        // The entries at or above the bound (a few dozen to a few hundred) are appended to an LDS buffer and
        // bitonic-sorted by (|g|, lower index).  A buffer overflow (many equal values) is resolved by the
        // exact rounds of argmax below, which need no buffer.
        constexpr int CAP = 2048;
        __shared__ float s_cv[CAP];
        __shared__ int s_ci[CAP];
        __shared__ int s_n;
        if (tid == 0) { s_n = 0; s_ng = 0; }
        __syncthreads();
        auto take = [&](bool t, int j, float v) {   // called by the whole wave
            const unsigned long long bal = __ballot(t);
            if (!bal) return;
            int base = 0;
            if (lane == 0) base = atomicAdd(&s_n, __popcll(bal));
            base = __shfl(base, 0);
            const int pos = base + __popcll(bal & ((1ull << lane) - 1ull));
            if (t && pos < CAP) { s_cv[pos] = v; s_ci[pos] = j; }
        };
        auto ok = [&](float v) { return v > lamf && v >= T; };
        // Most groups of four hold neither an entry nor a value above the largest of the registered ones: one
        // comparison of their largest value decides that for the wave.
        const float quick = fminf(fmaxf(T, lamf), wave_max(vmx));
        auto four = [&](const float4& f, uint32_t w, int j0) {
            const float v0 = fabsf(f.x), v1 = fabsf(f.y), v2 = fabsf(f.z), v3 = fabsf(f.w);
            if (!__ballot(fmaxf(fmaxf(v0, v1), fmaxf(v2, v3)) >= quick)) return;
            if (!(w & 1u)) vmx = fmaxf(vmx, v0);
            if (!(w & 2u)) vmx = fmaxf(vmx, v1);
            if (!(w & 4u)) vmx = fmaxf(vmx, v2);
            if (!(w & 8u)) vmx = fmaxf(vmx, v3);
            take(!(w & 1u) && ok(v0), j0, v0);
            take(!(w & 2u) && ok(v1), j0 + 1, v1);
            take(!(w & 4u) && ok(v2), j0 + 2, v2);
            take(!(w & 8u) && ok(v3), j0 + 3, v3);
        };
        if (grouped) {
            // the groups that can hold an entry or the largest value outside I
            visit_groups<CAPG>(gm, corr_groups(a.m), g, ex, a.m, quick, s_gl, &s_ng, [&](int j, float v, bool out) {
                if (out) vmx = fmaxf(vmx, v);
                take(out && ok(v), j, v);
            });
        } else {
#pragma unroll
        for (int q = 0; q < CH; ++q) four(f0[q], w0[q], 4 * tid + 1024 * q);
        // two chunks that take turns by name (a copied register would wait for its load); every lane runs the same
        // number of steps (the ballots need the whole wave)
        auto chunk = [&](const float4 (&f)[CS], const uint32_t (&w)[CS], int base0) {
#pragma unroll
            for (int q = 0; q < CS; ++q) four(f[q], chunk_bits(ex, w[q], base0 + 4 * tid + 1024 * q, m4), base0 + 4 * tid + 1024 * q);
        };
        for (int base0 = 1024 * CH; base0 < m4; base0 += 2 * 1024 * CS) {
            float4 fb[CS];
            uint32_t wb[CS];
            load_chunk(base0 + 1024 * CS, fb, wb);   // the next chunk (past the row: zeros, no load)
            chunk(fa, wa, base0);
            if (base0 + 1024 * CS >= m4) break;
            load_chunk(base0 + 2 * 1024 * CS, fa, wa);
            chunk(fb, wb, base0 + 1024 * CS);
        }
        for (int j0 = m4; j0 < a.m; j0 += 256) {
            const int j = j0 + tid;
            const bool in = j < a.m && !(ex && ((ex[j >> 5] >> (j & 31)) & 1u));
            const float v = in ? fabsf(g[j]) : 0.f;
            if (in) vmx = fmaxf(vmx, v);
            take(in && ok(v), j, v);
        }
        }
        __syncthreads();
        const int nc = s_n;
        if (nc <= 256) {
            // few entries: each thread ranks one by counting the better ones (entries are distinct
            // atoms, so the ranks are a permutation), no sort and one barrier
            const int nsel = nc < k ? nc : k;
            if (tid < nc) {
                const float v = s_cv[tid];
                const int j = s_ci[tid];
                int rank = 0;
                for (int d = 0; d < nc; ++d) rank += better(s_cv[d], s_ci[d], v, j) ? 1 : 0;
                if (rank < nsel) a.sel[(int64_t)sig * a.selcap + rank] = j;
            }
            for (int q = nsel + tid; q < a.selcap && q < k; q += 256) a.sel[(int64_t)sig * a.selcap + q] = -1;
            vmx = wave_max(vmx);
            if (lane == 0) s_red[wave] = vmx;
            __syncthreads();
            if (tid == 0) {
                const float vm = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
                a.nsel[sig] = nsel;
                a.vmax[sig] = vm;
                *certify = needs_certification(a, sig, k, nsel, vm, lam);
            }
            return;
        }
        if (nc <= CAP) {
            int N = 64;
            while (N < nc) N <<= 1;
            for (int e = nc + tid; e < N; e += 256) { s_cv[e] = -1.f; s_ci[e] = INT_MAX; }
            __syncthreads();
            for (int size = 2; size <= N; size <<= 1)
                for (int stride = size >> 1; stride > 0; stride >>= 1) {
                    for (int t = tid; t < N / 2; t += 256) {
                        const int i = ((t & ~(stride - 1)) << 1) | (t & (stride - 1)), j = i + stride;
                        const float vi = s_cv[i], vj = s_cv[j];
                        const int ii = s_ci[i], ij = s_ci[j];
                        const bool i_first = better(vi, ii, vj, ij);
                        if (((i & size) == 0) ? !i_first : i_first) {   // best first overall
                            s_cv[i] = vj; s_cv[j] = vi;
                            s_ci[i] = ij; s_ci[j] = ii;
                        }
                    }
                    __syncthreads();
                }
            vmx = wave_max(vmx);
            if (lane == 0) s_red[wave] = vmx;
            __syncthreads();
            const int nsel = nc < k ? nc : k;
            for (int q = tid; q < a.selcap && q < k; q += 256) a.sel[(int64_t)sig * a.selcap + q] = q < nsel ? s_ci[q] : -1;
            if (tid == 0) {
                const float vm = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
                a.nsel[sig] = nsel;
                a.vmax[sig] = vm;
                *certify = needs_certification(a, sig, k, nsel, vm, lam);
            }
            return;
        }
        // Buffer overflow (more than CAP entries at or above the bound: many equal values): k rounds of
        // a workgroup argmax over the row, each taking the best (|g|, index) pair after the previous one.
        vmx = wave_max(vmx);
        if (lane == 0) s_red[wave] = vmx;
        __syncthreads();
        const float vmax_all = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
        float pv = INFINITY;
        int pi = -1;
        int nsel = 0;
        for (int r = 0; r < k; ++r) {
            float bv = -1.f;
            int bi = INT_MAX;
            for (int j = tid; j < a.m; j += 256) {
                if (ex && ((ex[j >> 5] >> (j & 31)) & 1u)) continue;
                const float v = fabsf(g[j]);
                const bool after = v < pv || (v == pv && j > pi);
                if (v > lamf && after && better(v, j, bv, bi)) { bv = v; bi = j; }
            }
            for (int o = 32; o > 0; o >>= 1) {
                const float ov = __shfl_xor(bv, o);
                const int oi = __shfl_xor(bi, o);
                if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
            }
            __syncthreads();
            if (lane == 0) { s_val[wave] = bv; s_idx[wave] = bi; }
            __syncthreads();
            bv = s_val[0];
            bi = s_idx[0];
            for (int w2 = 1; w2 < 4; ++w2)
                if (better(s_val[w2], s_idx[w2], bv, bi)) { bv = s_val[w2]; bi = s_idx[w2]; }
            if (bv < 0.f) break;
            if (tid == 0) a.sel[(int64_t)sig * a.selcap + r] = bi;
            pv = bv;
            pi = bi;
            ++nsel;
        }
        for (int q = nsel + tid; q < a.selcap && q < k; q += 256) a.sel[(int64_t)sig * a.selcap + q] = -1;
        if (tid == 0) {
            a.nsel[sig] = nsel;
            a.vmax[sig] = vmax_all;
            *certify = needs_certification(a, sig, k, nsel, vmax_all, lam);
        }
        return;
    }
}

// Certification of the natural stop under the float32 product.  For a running signal whose selection
// admitted nothing although it had room, every float32 |g~_j| outside I is at most lambda, but the
// exact |g_j| may exceed it by up to the product's rounding error eps_i = band ||xi_i||.  If the
// largest |g~_j| is within eps_i of lambda, the atoms with |g~_j| >= lambda - eps_i (the only ones whose
// exact correlation can exceed lambda) are re-scored exactly: float32 data, float64 sums.  The exact
// violators among them are admitted, largest first (ties to the lower index), and the signal goes on;
// with none, vmax becomes the largest exact value (<= lambda), so the stop and the certificate's
// off-I term are exact.  The row is swept in chunks of the LDS buffer, so any number of atoms in the
// band is handled; at most EXB exact violators are kept (the lowest-indexed ones, all of them violators).
// (Usually no signal or a handful of them: a kernel of its own over their list took longer to launch, 4 us a pass.)
__device__ __forceinline__ void certify_row(const SelectArgs& a, int row, int sig)
{
    int k = a.k;
    if (a.nI && a.max_active > 0) {
        const int room = a.max_active - a.nI[sig];
        k = room < k ? room : k;
    }
    const double lam = a.lam[sig];
    const double eps = a.band * sqrt(a.rr2[sig]);
    const double lo = lam - eps;
    const float* g = a.G + (int64_t)row * a.ldg;
    const uint32_t* ex = a.excl + (int64_t)sig * a.words;
    const float* r = a.R + (int64_t)sig * a.ldr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int CB = 256, EXB = 256;
    __shared__ int s_c[CB];
    __shared__ int s_n, s_next;
    __shared__ float s_ev[EXB];
    __shared__ int s_ei[EXB];
    __shared__ int s_ne;
    __shared__ int s_wc[4];
    __shared__ double s_mx[4];
    if (tid == 0) s_ne = 0;
    double emax = 0.0;
    int start = 0;
    for (;;) {
        // collect up to CB atoms of the band with index >= start, in index order
        if (tid == 0) { s_n = 0; s_next = a.m; }
        __syncthreads();
        for (int j0 = start; j0 < a.m; j0 += 256) {
            const int j = j0 + tid;
            const bool t = j < a.m && !((ex[j >> 5] >> (j & 31)) & 1u) && (double)fabsf(g[j]) >= lo;
            const unsigned long long bal = __ballot(t);
            if (lane == 0) s_wc[wave] = __popcll(bal);
            __syncthreads();
            const int before = (wave > 0 ? s_wc[0] : 0) + (wave > 1 ? s_wc[1] : 0) + (wave > 2 ? s_wc[2] : 0);
            const int tot = s_wc[0] + s_wc[1] + s_wc[2] + s_wc[3];
            const int base = s_n;
            const int pos = base + before + __popcll(bal & ((1ull << lane) - 1ull));
            if (t && pos < CB) s_c[pos] = j;
            if (t && pos == CB) s_next = j;          // the first atom that did not fit
            __syncthreads();
            if (tid == 0) s_n = base + tot;
            __syncthreads();
            if (base + tot > CB) break;              // uniform: every thread read the same s_n
        }
        const int nc = s_n < CB ? s_n : CB;
        // exact re-score, one wave per atom: float32 products summed in float64
        for (int c = wave; c < nc; c += 4) {
            const int j = s_c[c];
            const float* aj = a.At + (int64_t)j * a.lda;
            double acc = 0.0;
            for (int q = lane; q < a.n; q += 64) acc += (double)aj[q] * (double)r[q];
            acc = fabs(wave_sum(acc));
            emax = fmax(emax, acc);
            if (lane == 0 && acc > lam) {
                const int pos = atomicAdd(&s_ne, 1);
                if (pos < EXB) { s_ev[pos] = (float)acc; s_ei[pos] = j; }
            }
        }
        __syncthreads();
        if (s_n <= CB) break;
        start = s_next;
        __syncthreads();
    }
    emax = wave_max(emax);
    if (lane == 0) s_mx[wave] = emax;
    __syncthreads();
    const double vmx = fmax(fmax(s_mx[0], s_mx[1]), fmax(s_mx[2], s_mx[3]));
    const int ne = s_ne < EXB ? s_ne : EXB;
    const int nsel = ne < k ? ne : k;
    if (tid < ne) {
        const float v = s_ev[tid];
        const int j = s_ei[tid];
        int rank = 0;
        for (int d = 0; d < ne; ++d) rank += better(s_ev[d], s_ei[d], v, j) ? 1 : 0;
        if (rank < nsel) a.sel[(int64_t)sig * a.selcap + rank] = j;
    }
    if (tid == 0) {
        a.nsel[sig] = nsel;
        // with no violator every exact |g_j| is <= lambda: round down, so the stop test in float64 holds
        a.vmax[sig] = nsel > 0 ? (float)vmx : __double2float_rd(vmx);
    }
}

template <int KMAX, bool GROUPS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void select_kernel(SelectArgs a)
{
    __shared__ bool s_certify;
    if (a.clear_count && blockIdx.x == 0 && threadIdx.x == 0) *a.clear_count = 0;   // a later kernel's list
    const int n_act = a.n_act_dev ? *a.n_act_dev : a.p_grid;
    const int row = blockIdx.x;
    if (row >= n_act) return;
    const int sig = a.act ? a.act[row] : row;
    select_row<KMAX, GROUPS>(a, row, sig, GROUPS && a.excl != nullptr && n_act >= a.gm_lo, &s_certify);
    __syncthreads();
    if (s_certify) certify_row(a, row, sig);
}

}  // namespace

hipError_t launch_select(const SelectArgs& a, hipStream_t stream)
{
    if (a.p_grid <= 0) return hipSuccess;
    if (a.k <= 0 || a.k > 64 || a.k > a.selcap) return hipErrorInvalidValue;
    const bool groups = a.gm != nullptr && a.gm_lo <= a.p_grid;
    const auto kernel = a.k <= 32 ? (groups ? select_kernel<32, true> : select_kernel<32, false>)
                                  : (groups ? select_kernel<64, true> : select_kernel<64, false>);
    hipLaunchKernelGGL(kernel, dim3(a.p_grid), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace bmpl
