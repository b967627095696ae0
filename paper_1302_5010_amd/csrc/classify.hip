// Sparse-representation classification: the face-recognition use of the batch
// solver (Section V follows the class-residual rule of sparse-representation-based
// classification).  For signal i with code x_i, every class with an atom in the
// support is scored by ||b_i - A delta_c(x_i)||_2 (delta_c keeps that class's
// coefficients); the label is the class with the smallest residual, ties to the
// lower class index, -1 for an empty support.  Float64 sums from float32 data.
//
// W waves per signal: one (four signals per workgroup, no barrier at all) when there are enough signals to fill the
// chip that way, else four.  The classes are visited in increasing order; a class's atoms are listed once, in support
// order, and every lane then streams its rows of them, several 16-byte loads in flight, with the signal read beside
// them.  Bound by the atoms' rows (32 KB per signal at 8 atoms of 1024 values, from L2 and the Infinity cache) and the
// latency of the list: 8192 signals x 8 atoms x 1024 values 130 -> 52 us (before, every row scanned the whole
// support for the class's atoms, one load after another, between block-wide reductions).
#include <float.h>
#include <limits.h>

#include <algorithm>

#include "bmpl_internal.h"
#include "classify.h"
#include "wave_ops.h"

namespace bmpl {
namespace {

constexpr int LCAP = 512;        // atoms of one class listed at a time

struct ClassList {
    int n;                       // entries listed
    int atom[LCAP];
    double val[LCAP];
};

__device__ inline int wave_min(int v)
{
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
    return v;
}

// A barrier of the signal's W waves that also orders their LDS accesses (one wave: its own order suffices).
template <int W>
__device__ __forceinline__ void group_sync()
{
    if constexpr (W > 1) __syncthreads();
    else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

template <int W>
__global__ __launch_bounds__(256) void classify_kernel(ClassifyArgs a)
{
    constexpr int SPB = 4 / W;           // signals per workgroup
    constexpr int NT = 64 * W;           // threads per signal
    constexpr int NV = 4 / W;            // 16-byte row chunks per thread: 1024 rows at a time
    __shared__ ClassList s_list[SPB];
    __shared__ int s_min[4];
    __shared__ double s_sum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = W == 1 ? wave : 0;
    const int t = W == 1 ? lane : (int)threadIdx.x;
    const int sig = blockIdx.x * SPB + grp;
    if (sig >= a.p) return;              // the whole wave (W = 1); never with W = 4
    ClassList& list = s_list[grp];
    const int len = min(a.supp_len[sig], a.ld_x);
    const int* idx = a.x_idx + (int64_t)sig * a.ld_x;
    const float* val = a.x_val + (int64_t)sig * a.ld_x;
    const float* b = a.B + (int64_t)sig * a.ldb;
    const bool b4 = (a.ldb & 3) == 0 && (reinterpret_cast<uintptr_t>(a.B) & 15) == 0;
    const int n4 = (a.n + 3) / 4;        // 16-byte chunks of an atom's row (zeros past n)
    auto entry = [&](int k, int& j, int& c) {   // support entry k: its atom and class (INT_MAX: none)
        j = idx[k < len ? k : len - 1];
        const bool ok = k < len && j >= 0 && j < a.m;
        c = a.class_of_atom[ok ? j : 0];
        c = ok ? c : INT_MAX;
    };
    int best = -1;
    double best_r = DBL_MAX;
    int prev = INT_MIN;
    while (len > 0) {
        // next class: the smallest class index above `prev` among the support's atoms
        int c = INT_MAX;
        for (int k0 = 0; k0 < len; k0 += NT) {
            int j, cj;
            entry(k0 + t, j, cj);
            if (cj > prev && cj < c) c = cj;
        }
        c = wave_min(c);
        if constexpr (W > 1) {
            __syncthreads();
            if (lane == 0) s_min[wave] = c;
            __syncthreads();
            c = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
        }
        if (c == INT_MAX) break;
        // its atoms and values in support order, listed by the group's first wave from entry `from` on; returns the
        // entry to go on from (len when all are listed)
        auto gather = [&](int from) {
            group_sync<W>();             // the list's readers are done
            int next = len;
            if (t < 64) {
                int n = 0;
                for (int k0 = from; k0 < len; k0 += 64) {
                    int j, cj;
                    entry(k0 + lane, j, cj);
                    const float v = val[k0 + lane < len ? k0 + lane : len - 1];
                    const unsigned long long bal = __ballot(cj == c);
                    if (n + __popcll(bal) > LCAP) {
                        next = k0;
                        break;
                    }
                    if (cj == c) {
                        const int pos = n + __popcll(bal & ((1ull << lane) - 1ull));
                        list.atom[pos] = j;
                        list.val[pos] = (double)v;
                    }
                    n += __popcll(bal);
                }
                if (lane == 0) list.n = n;
                if (W > 1 && lane == 0) s_min[0] = next;
            }
            group_sync<W>();
            return W > 1 ? s_min[0] : next;
        };
        int next = gather(0);
        const bool whole = next >= len;  // the class fits one list (the usual case): listed once for all rows
        double part = 0.0;
        for (int q0 = 0; q0 < n4; q0 += NT * NV) {
            double v[NV][4];
            int qi[NV];
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const int q = q0 + t + NT * u;
                qi[u] = q < n4 ? q : 0;  // chunks past the end re-read the first and count nothing
                if (b4 && 4 * q + 4 <= a.n) {
                    const float4 f = *reinterpret_cast<const float4*>(b + 4 * q);
                    v[u][0] = f.x; v[u][1] = f.y; v[u][2] = f.z; v[u][3] = f.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[u][e] = 4 * q + e < a.n ? (double)b[4 * q + e] : 0.0;
                }
            }
            if (!whole) next = gather(0);
            for (;;) {
                const int n = list.n;
                int k = 0;
                for (; k + 2 <= n; k += 2) {
                    float4 f[2][NV];
#pragma unroll
                    for (int z = 0; z < 2; ++z) {
                        const float4* row = reinterpret_cast<const float4*>(a.At + (int64_t)list.atom[k + z] * a.lda);
#pragma unroll
                        for (int u = 0; u < NV; ++u) f[z][u] = row[qi[u]];
                    }
#pragma unroll
                    for (int z = 0; z < 2; ++z) {
                        const double x = list.val[k + z];
#pragma unroll
                        for (int u = 0; u < NV; ++u) {
                            v[u][0] -= x * (double)f[z][u].x;
                            v[u][1] -= x * (double)f[z][u].y;
                            v[u][2] -= x * (double)f[z][u].z;
                            v[u][3] -= x * (double)f[z][u].w;
                        }
                    }
                }
                if (k < n) {
                    const float4* row = reinterpret_cast<const float4*>(a.At + (int64_t)list.atom[k] * a.lda);
                    const double x = list.val[k];
#pragma unroll
                    for (int u = 0; u < NV; ++u) {
                        const float4 f = row[qi[u]];
                        v[u][0] -= x * (double)f.x;
                        v[u][1] -= x * (double)f.y;
                        v[u][2] -= x * (double)f.z;
                        v[u][3] -= x * (double)f.w;
                    }
                }
                if (whole || next >= len) break;
                next = gather(next);
            }
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const int q = q0 + t + NT * u;
                const double s2 = v[u][0] * v[u][0] + v[u][1] * v[u][1] + v[u][2] * v[u][2] + v[u][3] * v[u][3];
                part += q < n4 ? s2 : 0.0;
            }
        }
        part = wave_sum(part);
        if constexpr (W > 1) {
            __syncthreads();
            if (lane == 0) s_sum[wave] = part;
            __syncthreads();
            part = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        }
        const double rr = sqrt(part);
        if (rr < best_r) { best_r = rr; best = c; }   // classes in increasing order: ties keep the lower
        prev = c;
    }
    if (t == 0) {
        a.labels[sig] = best;
        if (a.resid) a.resid[sig] = best >= 0 ? best_r : 0.0;
    }
}

}  // namespace

hipError_t launch_classify(const ClassifyArgs& a, hipStream_t stream)
{
    if (a.p <= 0) return hipSuccess;
    // One wave per signal once that gives every CU eight waves; fewer signals get four each, which a long support (the
    // class lists) and long rows also repay.  us with one wave and with four, support entries of random classes:
    // n = 1024: 1536 signals 8 entries 31 and 29, 300 entries 1106 and 849; 2048: 32 and 32, 1161 and 965; 3072: 37 and
    // 50, 1451 and 1658.  n = 2048: 2048 signals 55 and 43; 4096 80 and 80, 64 entries 498 and 480.  Rows of up to 128
    // values leave half of four waves idle: n = 64, 8 entries: 1024 signals 22 and 23, 2048 24 and 29 (27 before waves).
    if (a.p >= (a.n <= 128 ? 1536 : 2048)) hipLaunchKernelGGL(classify_kernel<1>, dim3((a.p + 3) / 4), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(classify_kernel<4>, dim3(a.p), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace bmpl
