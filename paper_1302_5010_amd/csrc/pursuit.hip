// Per-signal kernels of the batched pursuit: set-up, the stop/compaction step,
// the master problem on the ragged active sets, and result packing.
//
// Master problem (Eq. (7)): min_x lambda ||x||_1 + 1/2 ||b - A x||^2 with
// x = 0 outside the active set I.  The paper runs proximal gradient on it; here
// it is solved exactly, warm-started from the previous outer iteration
// (Algorithm 1, step 4), by a sign-fixed active-set method on the support
// S subset of I:
//   * for a fixed support S and signs theta the minimiser is
//     x_S = G_SS^{-1} (c_S - lambda theta_S), with G = A_I^T A_I and c = A_I^T b;
//   * atoms of I \ S whose gradient c_u - G_uS x_S exceeds lambda in magnitude
//     enter S with the sign of that gradient;
//   * if the new minimiser flips the sign of a coordinate, the step stops at the
//     first zero crossing and that atom leaves S.
// The objective decreases strictly at every non-zero step, so the loop ends at
// the restricted optimum, the point proximal gradient converges to.
//
// G_II is accumulated in float64 from the float32 atoms (products exact, sums in
// float64) and kept packed per signal, grown by rows as atoms enter I (atoms
// never leave I).  G_SS is represented by its inverse Cholesky factor
// Rinv = L^{-1} (G_SS = L L^T, so G_SS^{-1} = Rinv^T Rinv): adding an atom is a
// Cholesky row append computed from Rinv^T (Rinv g), a solve is Rinv^T (Rinv w)
// (two matrix-vector products), several appends of one step as a block, and
// removing position q is a Givens downdate of the rows below it.
//
// One 256-thread workgroup per signal (a wave per signal: pursuit_wave.hip); signals are independent.  The device
// code of the master problem is in master_body.h.
#include <float.h>
#include <limits.h>

#include <type_traits>

#include "../../include/bmpl.h"
#include "bmpl_internal.h"
#include "pursuit.h"
#include "wave_ops.h"

namespace bmpl {
namespace {

constexpr int NT = 256;
}  // namespace
}  // namespace bmpl

#include "master_body.h"

namespace bmpl {

// ---------------------------------------------------------------------------
// Set-up: copy b_i into the padded signal and residual buffers, ||b_i||^2,
// finiteness, lambda (absolute rule), and clear the per-signal state.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prep_kernel(PrepArgs a)
{
    const int sig = blockIdx.x;
    const Workspace& w = a.w;
    __shared__ double red[4];
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    const float* b = a.B + (int64_t)sig * a.ldb;
    float* Bw = a.Bw + (int64_t)sig * w.kpad;
    float* R = w.R + (int64_t)sig * w.kpad;
    double part = 0.0, dpart = 0.0;
    int bad = 0;
    for (int r = threadIdx.x; r < w.kpad; r += 256) {
        float v = r < w.n ? b[r] : 0.f;
        if (!isfinite(v)) bad = 1;
        Bw[r] = v;
        R[r] = v;
        if (w.R16) {
            const uint16_t h = bf16_round(v);
            w.R16[(int64_t)sig * w.kpad + r] = h;
            const double d = (double)bf16_value(h) - (double)v;
            dpart += d * d;
        }
        part += (double)v * (double)v;
    }
    if (bad) atomicOr(&s_bad, 1);
    for (int q = threadIdx.x; q < w.words; q += 256) w.inI[(int64_t)sig * w.words + q] = 0u;
    const double bb = block_sum(part, red);
    const double bd = w.R16 ? block_sum(dpart, red) : 0.0;
    if (threadIdx.x == 0) {
        double lam = a.lambda_dev ? a.lambda_dev[sig] : a.lambda_abs;
        int st = 0;
        if (s_bad || !isfinite(lam) || lam < 0.0) st = BMPL_SIG_NONFINITE;
        w.status[sig] = st;
        w.lam[sig] = a.lam_rel_mode ? 0.0 : lam;
        w.bnorm2[sig] = bb;
        w.iters[sig] = 0;
        w.nI[sig] = 0;
        w.nS[sig] = 0;
        w.nsel[sig] = 0;
        w.glazy[sig] = 0;
        w.jadd[sig] = JADD0;
        w.vmax[sig] = 0.f;
        w.kkt_on[sig] = 0.0;
        w.kkt[sig] = 0.0;
        w.obj[sig] = 0.5 * bb;
        w.obj_prev[sig] = 0.5 * bb;
        w.rr2[sig] = bb;
        w.g0max[sig] = 0.f;
        w.cap[sig] = 0;
        w.blk[sig] = nullptr;
        if (sig == 0) {   // a new solve hands out slot blocks from the start of the arena
            w.arena->top = 0;
            w.arena->starved = 0;
        }
        if (w.rnorm) w.rnorm[sig] = sqrt(bb);
        if (w.dxnorm) w.dxnorm[sig] = sqrt(bd);
    }
    if (w.R8) write_residual_fp8(w, sig, red);
}

// ---------------------------------------------------------------------------
// Stop test and compaction.  For each running signal after a selection pass:
// no violator left -> natural stop; an early-stop rule (Eq. (10), Eq. (13))
// holds -> early stop; no admitted atom -> the active-set cap was hit;
// iteration cap -> stop; otherwise keep it running.
// One workgroup; the running list stays in signal order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void status_compact_kernel(StatusArgs a)
{
    const Workspace& w = a.w;
    const int n_in = a.n_in_dev ? *a.n_in_dev : a.n_in;
    __shared__ int s_scan[1024];
    __shared__ int s_base;
    __shared__ unsigned long long s_res[16];
    __shared__ int s_ng;
    __shared__ unsigned long long s_goff;   // doubles of the grow list's new blocks
    __shared__ int s_maxb;                  // largest support bucket (256 positions each) among kept signals
    if (threadIdx.x == 0) { s_base = 0; s_ng = 0; s_goff = 0; s_maxb = 0; }
    __syncthreads();
    unsigned long long res = 0;   // this thread's share of the slot-block reserve
    int mbk = 0;                  // largest support bucket among this thread's kept signals
    // RPT signals per thread at a time (thread t: r0 + 1024 j + t): their state is loaded together, so a long list
    // waits for memory a few times and not once per 1024 signals (8192 signals: 62 us a call with one at a time)
    auto round = [&](auto rpt, int r0) {
        constexpr int RPT = decltype(rpt)::value;
        int sg[RPT], st[RPT], ns[RPT], it[RPT], nI[RPT], nS[RPT], cap[RPT], keep[RPT];
        double lam[RPT];
        float vm[RPT];
#pragma unroll
        for (int j = 0; j < RPT; ++j) {          // clamped, so that no load is guarded
            const int r = min(r0 + 1024 * j + (int)threadIdx.x, n_in - 1);
            sg[j] = a.act_in ? a.act_in[r] : r;
        }
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            st[j] = w.status[sg[j]];
            ns[j] = w.nsel[sg[j]];
            it[j] = w.iters[sg[j]];
            nI[j] = w.nI[sg[j]];
            nS[j] = w.nS[sg[j]];
            cap[j] = w.cap[sg[j]];
            lam[j] = w.lam[sg[j]];
            vm[j] = w.vmax[sg[j]];
        }
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int sig = sg[j];
            keep[j] = 0;
            if (r0 + 1024 * j + (int)threadIdx.x < n_in) {
                if (a.initial) {
                    keep[j] = !(st[j] & BMPL_SIG_NONFINITE);
                } else {
                    int s1 = st[j];
                    const double vmd = (double)vm[j];
                    if (it[j] == 0) w.g0max[sig] = vm[j];   // first pass: I is empty, so this is ||A^T b||_inf
                    const bool natural = ns[j] == 0 && vmd <= lam[j];
                    bool early = false;
                    if (!natural && (a.r_inf_rel > 0.0 || a.r2_rel > 0.0 || a.eps_early > 0.0)) {
                        const double bb = w.bnorm2[sig];
                        const float g0 = it[j] == 0 ? vm[j] : w.g0max[sig];
                        if (a.r_inf_rel > 0.0 && vmd <= a.r_inf_rel * (double)g0)
                            early = true;                                             // Eq. (10), correlations
                        else if (a.r2_rel > 0.0 && sqrt(w.rr2[sig]) <= a.r2_rel * sqrt(bb))
                            early = true;                                             // Eq. (10), residual norm
                        else if (a.eps_early > 0.0 && it[j] >= 1 &&
                                 fabs(w.obj_prev[sig] - w.obj[sig]) <= a.eps_early * a.rho * bb)
                            early = true;                                             // Eq. (13)
                    }
                    const bool halt = (s1 & ST_HALT) != 0;   // the solve kernel stopped it (reported inexact)
                    s1 &= ~ST_HALT;
                    if (ns[j] == 0 || it[j] >= a.max_outer || early || halt) {
                        double off = vmd - lam[j];
                        off = off > 0.0 ? off : 0.0;
                        double kk = fmax(off, w.kkt_on[sig]);
                        kk = lam[j] > 0.0 ? kk / lam[j] : kk;
                        w.kkt[sig] = kk;
                        if (a.warm_check && ns[j] != 0) s1 |= BMPL_SIG_FALLBACK;
                        if (halt) {
                            // INEXACT is set already
                        } else if (natural) {
                            if (kk <= a.kkt_tol) s1 |= BMPL_SIG_CONVERGED;
                        } else if (early) {
                            s1 |= BMPL_SIG_EARLY;
                        } else if (ns[j] == 0) {
                            if (!(s1 & BMPL_SIG_INEXACT)) s1 |= BMPL_SIG_CAP_ACTIVE;
                        } else {
                            s1 |= BMPL_SIG_CAP_ITERS;
                        }
                        w.status[sig] = s1;
                        if (ns[j] != 0) w.nsel[sig] = 0;
                    } else {
                        if (a.warm_check) w.status[sig] = s1 | BMPL_SIG_FALLBACK;
                        keep[j] = 1;
                    }
                }
            }
            if (keep[j]) mbk = max(mbk, min(3, nS[j] / 256));
            const bool grows = keep[j] && a.grow_list && nI[j] + ns[j] > cap[j];
            const unsigned long long gb = __ballot(grows);
            if (gb) {   // the same on every lane
                // their blocks grow before the master problem; the new blocks of the whole list are placed here
                // with one fetch-and-add on the arena's offset (below), each at its share of the total: a sum
                // over the wave's lanes before, and one LDS atomic per wave
                const int ln = threadIdx.x & 63;
                const int K2 = max(grow_capacity(cap[j], nI[j] + ns[j], a.slack, a.kcap), min(a.kmin, a.kcap));
                const unsigned long long sz = grows ? (unsigned long long)block_doubles(K2, w.n) : 0ull;
                unsigned long long inc = sz;
                for (int o = 1; o < 64; o <<= 1) {
                    const unsigned long long up = __shfl_up(inc, o);
                    inc += ln >= o ? up : 0ull;
                }
                int e0 = 0;
                unsigned long long off0 = 0;
                if (ln == 63) {
                    e0 = atomicAdd(&s_ng, __popcll(gb));
                    off0 = atomicAdd(&s_goff, inc);
                }
                e0 = __shfl(e0, 63);
                off0 = __shfl(off0, 63);
                if (grows) {
                    const int e = e0 + __popcll(gb & ((1ull << ln) - 1ull));
                    a.grow_list[e] = sig;
                    a.grow_off[e] = off0 + inc - sz;
                }
            }
            if (keep[j] && a.reserve_iters > 0) {
                // the blocks this signal may take while its |I| grows by up to reserve_iters * rho_pass slots
                int Kc = cap[j];
                const int target = min(a.kcap, nI[j] + a.reserve_iters * a.rho_pass);
                while (Kc < target) {
                    Kc = grow_capacity(Kc, min(target, Kc + a.rho_pass), a.slack, a.kcap);
                    res += (unsigned long long)block_doubles(Kc, w.n);
                }
            }
        }
        // order-preserving compaction: position = kept signals before this one (a ballot within the wave, the
        // counts of the earlier waves and rows from LDS), two barriers
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        unsigned long long bal[RPT];
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            bal[j] = __ballot(keep[j]);
            if (lane == 0) s_scan[16 * j + wv] = __popcll(bal[j]);
        }
        __syncthreads();
        int total = 0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            int before = s_base + total;
            for (int q = 0; q < 16; ++q) {
                const int c = s_scan[16 * j + q];
                before += q < wv ? c : 0;
                total += c;
            }
            if (keep[j]) a.act_out[before + __popcll(bal[j] & ((1ull << lane) - 1ull))] = sg[j];
        }
        __syncthreads();   // every wave has read s_scan and s_base
        if (threadIdx.x == 0) s_base += total;
    };
    if (n_in <= 1024) {
        if (n_in > 0) round(std::integral_constant<int, 1>{}, 0);
    } else {
        for (int r0 = 0; r0 < n_in; r0 += 4096) round(std::integral_constant<int, 4>{}, r0);
    }
    if (mbk > 0) atomicMax(&s_maxb, mbk);
    __syncthreads();
    {
        // The running list, largest supports first (buckets of 256 support positions, kept in signal
        // order within a bucket): the master problem's workgroups start with the longest problems and
        // the short ones fill the end of the launch.  Only when some support has 256 positions or more,
        // and for lists of at most 16 entries per thread (longer lists keep their order).
        constexpr int RMAX = 16;
        const int n = s_base;
        const bool reorder = !a.initial && s_maxb > 0 && n <= RMAX * 1024;   // the same in every thread
        int v[RMAX], bk[RMAX];
        if (reorder) {
#pragma unroll
            for (int j = 0; j < RMAX; ++j) {
                const int r = threadIdx.x + 1024 * j;
                v[j] = r < n ? a.act_out[r] : -1;
                bk[j] = v[j] >= 0 ? min(3, w.nS[v[j]] / 256) : -1;
            }
            __syncthreads();                  // every entry is read before any is rewritten
            const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
            int base = 0;
            for (int b = 3; b >= 0; --b) {
#pragma unroll
                for (int j = 0; j < RMAX; ++j) {
                    if (1024 * j >= n) break;  // the same in every thread
                    const bool in = bk[j] == b;
                    const unsigned long long bal = __ballot(in);
                    if (lane == 0) s_scan[wv] = __popcll(bal);
                    __syncthreads();
                    int before = base, total = 0;
                    for (int q = 0; q < 16; ++q) {
                        const int c = s_scan[q];
                        before += q < wv ? c : 0;
                        total += c;
                    }
                    if (in) a.act_out[before + __popcll(bal & ((1ull << lane) - 1ull))] = v[j];
                    __syncthreads();           // every wave has read s_scan
                    base += total;
                }
            }
        }
    }
    if (threadIdx.x == 0) {
        *a.n_out_dev = s_base;
        if (a.n_grow) *a.n_grow = s_ng;
        if (s_ng > 0) w.arena->grow_base = atomicAdd(&w.arena->top, s_goff);
    }
    if (a.reserve_iters > 0) {
        for (int o = 32; o > 0; o >>= 1) res += __shfl_xor(res, o);
        if ((threadIdx.x & 63) == 0) s_res[threadIdx.x >> 6] = res;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long t = 0;
            for (int q = 0; q < 16; ++q) t += s_res[q];
            w.arena->reserve = t;
            if (a.report) {
                // straight to host memory, the number last: the host sees the count about 2 us after this store;
                // a copy behind the kernel and a wait for the stream take about 25 us
                a.report->top = w.arena->top;
                a.report->reserve = t;
                a.report->n_act = s_base;
                __hip_atomic_store(&a.report->seq, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Warm start: replace this pass's selection with the proposed atoms.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void warm_select_kernel(WarmArgs a)
{
    __shared__ int s_w[256];
    __shared__ int s_cnt[4];
    const int n_act = *a.n_act_dev;
    const int row = blockIdx.x;
    if (row >= n_act) return;
    const int sig = a.act[row];
    const Workspace& w = a.w;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int cap = a.max_active < w.selcap ? a.max_active : w.selcap;
    cap = cap < 256 ? cap : 256;
    // proposal entry tid: valid atom, first occurrence in the list
    const int j = tid < a.warm_k ? a.warm[(int64_t)sig * a.warm_k + tid] : -1;
    s_w[tid] = j;
    __syncthreads();
    bool keep = j >= 0 && j < w.m;
    for (int t = 0; t < tid && keep; ++t) keep = s_w[t] != j;
    const unsigned long long bal = __ballot(keep);
    if (lane == 0) s_cnt[wave] = __popcll(bal);
    __syncthreads();
    int before = 0;
    for (int w2 = 0; w2 < wave; ++w2) before += s_cnt[w2];
    const int total = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    const int pos = before + __popcll(bal & ((1ull << lane) - 1ull));
    // an empty proposal keeps this pass's own selection
    if (total > 0) {
        if (keep && pos < cap) w.sel[(int64_t)sig * w.selcap + pos] = j;
        if (tid == 0) w.nsel[sig] = total < cap ? total : cap;
    }
}

// ---------------------------------------------------------------------------
// Slot-block growth: a running signal whose active set, with this pass's selection, outgrows its block
// takes a larger one from the arena (grow_capacity) and copies its state over: slots, support order,
// the inverse factor and the Gram matrix of I (restrided).  A request that finds no room is counted in
// the arena's `starved` and leaves the signal as it is (the master-problem kernel then skips it).
// ---------------------------------------------------------------------------
// The stop test lists the signals that need it and places their new blocks with one fetch-and-add
// (one per listed signal on that single address kept the first master problem of 16 384 signals
// waiting half a millisecond); a block that would straddle two chunks is requested again on its own.
// A grid of at most a few hundred workgroups loops over the list.
__global__ __launch_bounds__(256) void grow_kernel(GrowArgs a)
{
    const int n_list = *a.n_list;
    const Workspace& w = a.w;
    const int tid = threadIdx.x;
    __shared__ double* s_blk;
    for (int li = blockIdx.x; li < n_list; li += gridDim.x) {
        const int sig = a.list[li];
        const int nI0 = w.nI[sig], nS = w.nS[sig];
        const int nI = nI0 + w.nsel[sig];
        const int K = w.cap[sig];
        const int K2 = max(grow_capacity(K, nI, a.slack, a.kcap), min(a.kmin, a.kcap));
        if (tid == 0) {
            const unsigned long long sz = (unsigned long long)block_doubles(K2, w.n);
            const Arena& A = *w.arena;
            const unsigned long long off = A.grow_base + a.off[li];
            int c = 0;
            while (c < A.nchunks && off >= A.start[c] + A.size[c]) ++c;
            double* p = nullptr;
            if (c < A.nchunks && off + sz <= A.start[c] + A.size[c]) p = A.base[c] + (off - A.start[c]);
            else p = arena_alloc(w.arena, sz);   // straddles a chunk boundary, or past the last chunk
            if (!p) atomicAdd(&w.arena->starved, 1ull);
            s_blk = p;
        }
        __syncthreads();
        double* nb = s_blk;
        __syncthreads();   // s_blk is rewritten for the next signal
        if (!nb) continue;
        if (K > 0) {
            const SlotBlock o = slot_block(w.blk[sig], K, w.n), d = slot_block(nb, K2, w.n);
            for (int u = tid; u < nI0; u += 256) {
                d.x[u] = o.x[u]; d.c[u] = o.c[u]; d.atom[u] = o.atom[u]; d.theta[u] = o.theta[u];
                d.excl[u] = o.excl[u];
            }
            for (int k = tid; k < nS; k += 256) d.sord[k] = o.sord[k];
            const int tr = (int)tri(nS), tot = nI0 * nI0;
            for (int e0 = tid; e0 < tr; e0 += 8 * 256) {   // eight loads in flight per thread
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = o.Rinv[e0 + q * 256 < tr ? e0 + q * 256 : tr - 1];   // clamped
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (e0 + q * 256 < tr) d.Rinv[e0 + q * 256] = v[q];
            }
            for (int e0 = tid; e0 < tot; e0 += 8 * 256) {   // G restrided from K to K2
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {   // clamped, so all eight loads are issued
                    const int e = e0 + q * 256 < tot ? e0 + q * 256 : tot - 1, u = e / nI0;
                    v[q] = o.G[(int64_t)u * K + (e - u * nI0)];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int e = e0 + q * 256, u = e / nI0;
                    if (e < tot) d.G[(int64_t)u * K2 + (e - u * nI0)] = v[q];
                }
            }
        }
        if (tid == 0) {
            w.blk[sig] = nb;
            w.cap[sig] = K2;
        }
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void solve_kernel(SolveArgs a) { solve_body<false, false, 1>(a); }
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void solve_fold_kernel(SolveArgs a) { solve_body<false, true, 1>(a); }
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void solve_fold_far_kernel(SolveArgs a) { solve_body<false, true, 2>(a); }
__global__ __launch_bounds__(256) void solve_block_kernel(SolveArgs a) { solve_body<true, false, 0>(a); }

// ---------------------------------------------------------------------------
// Results: support sorted by atom index, float32 values, per-signal scalars.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_kernel(PackArgs a)
{
    const int sig = blockIdx.x;
    const Workspace& w = a.w;
    const int nS = (w.status[sig] & BMPL_SIG_NONFINITE) || !w.blk[sig] ? 0 : w.nS[sig];
    const SlotBlock b = slot_block(w.blk[sig], w.cap[sig], w.n);   // only read when nS > 0
    const int* so = b.sord;
    const double* xs = b.x;
    const int* at = b.atom;
    const int64_t K = a.stage_max;
    int cnt = 0;
    if (a.stage && nS <= a.stage_max) {
        // the support's values and atoms (INT_MAX for a zero value) in LDS, then ranks from LDS
        extern __shared__ double s_px[];
        int* s_pa = reinterpret_cast<int*>(s_px + K);
        for (int k = threadIdx.x; k < nS; k += 256) {
            const int u = so[k];
            const double xu = xs[u];
            s_px[k] = xu;
            s_pa[k] = xu != 0.0 ? at[u] : INT_MAX;
        }
        __syncthreads();
        for (int k = threadIdx.x; k < nS; k += 256) {
            const int atom = s_pa[k];
            if (atom == INT_MAX) continue;
            int rank = 0;
            for (int k2 = 0; k2 < nS; ++k2) rank += s_pa[k2] < atom;
            if (rank < a.ld_x) {
                a.x_idx[(int64_t)sig * a.ld_x + rank] = atom;
                a.x_val[(int64_t)sig * a.ld_x + rank] = (float)s_px[k];
            }
        }
    } else {
        // rank by atom index among the support positions with a nonzero value
        for (int k = threadIdx.x; k < nS; k += 256) {
            const int u = so[k];
            const double xu = xs[u];
            if (xu == 0.0) continue;
            const int atom = at[u];
            int rank = 0;
            for (int k2 = 0; k2 < nS; ++k2) {
                const int u2 = so[k2];
                if (xs[u2] != 0.0 && at[u2] < atom) ++rank;
            }
            if (rank < a.ld_x) {
                a.x_idx[(int64_t)sig * a.ld_x + rank] = atom;
                a.x_val[(int64_t)sig * a.ld_x + rank] = (float)xu;
            }
        }
    }
    for (int k = threadIdx.x; k < nS; k += 256) cnt += xs[so[k]] != 0.0;
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
    __shared__ int s_c[4];
    if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = cnt;
    __syncthreads();
    const int tot = s_c[0] + s_c[1] + s_c[2] + s_c[3];
    for (int s = tot + threadIdx.x; s < a.ld_x; s += 256) {   // the rest of the row: -1 / 0
        a.x_idx[(int64_t)sig * a.ld_x + s] = -1;
        a.x_val[(int64_t)sig * a.ld_x + s] = 0.f;
    }
    if (threadIdx.x == 0) {
        a.supp_len[sig] = tot;
        const bool bad = w.status[sig] & BMPL_SIG_NONFINITE;
        if (a.iters) a.iters[sig] = w.iters[sig];
        if (a.kkt) a.kkt[sig] = bad ? NAN : w.kkt[sig];
        if (a.lambda) a.lambda[sig] = w.lam[sig];
        if (a.objective) a.objective[sig] = bad ? NAN : w.obj[sig];
        if (a.status) a.status[sig] = w.status[sig];
    }
}

}  // namespace bmpl
