// Device code of the master problem (step 4 to 8 of Algorithm 1) for workgroups of NT threads.  Included by
// pursuit.hip (NT = 256) and pursuit_wave.hip (NT = 64), each of which declares NT in the namespace below first.
#pragma once

namespace bmpl {
namespace {

constexpr int NB = 16;      // new atoms per Gram pass
constexpr int CH = 64;      // k per Gram staging chunk (direct Gram rows)
constexpr int JADD = 32;    // most violators added to S per active-set step (the largest ones)
constexpr int JADD0 = 8;    // the width a signal starts with
constexpr int LAZY_MIN = 32;   // new slots in one pass above which the Gram matrix is kept lazily
// Exclusion flag of a slot left out of S for the rest of one pass (cleared at the write-back): an
// atom admitted alone whose sign-fixed coefficient came out with the wrong sign.  Alone, its exact
// coefficient is (|g_u| - lambda) / pivot^2 > 0, so the wrong sign means |g_u| exceeds lambda by
// less than the rounding of x*; it would be dropped with no step and admitted again at once.
constexpr unsigned char EX_PASS = 2;
constexpr int JB = SOLVE_JB;   // atoms per block factor append

__device__ inline double block_sum(double v, double* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (NT == 64) return v;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// block_sum for a caller that has passed a barrier since the last read of red (saves the first one).
__device__ inline double block_sum_fenced(double v, double* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_sum(v);
    if (NT == 64) { __syncthreads(); return v; }
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

__device__ inline double block_max(double v, double* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_max(v);
    __syncthreads();
    if (NT == 64) return v;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// e4m3 copy of residual row `sig` (already written to R by this workgroup) with its power-of-two
// scale, for the e4m3 ranking product.
__device__ inline void write_residual_fp8(const Workspace& w, int sig, double* red)
{
    const float* R = w.R + (int64_t)sig * w.kpad;
    double mx = 0.0;
    for (int r = threadIdx.x; r < w.kpad; r += NT) mx = fmax(mx, (double)fabsf(R[r]));
    const float s = fp8_pow2_scale((float)block_max(mx, red));   // the barriers also publish R
    const float inv = 1.0f / s;
    uint8_t* R8 = w.R8 + (int64_t)sig * w.kpad;
    for (int r = threadIdx.x; r < w.kpad; r += NT) R8[r] = fp8_e4m3(R[r] * inv);
    if (threadIdx.x == 0) w.rscale8[sig] = s;
}

// (alpha, position) minimum, ties to the smaller position.
__device__ inline void block_argmin(double& a, int& q, double* red, int* redi)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto take = [&](double oa, int oq) {
        if (oa < a || (oa == a && (unsigned)oq < (unsigned)q)) { a = oa; q = oq; }
    };
    take(lane_move<DPP_XOR1>(a), lane_move<DPP_XOR1>(q));
    take(lane_move<DPP_XOR2>(a), lane_move<DPP_XOR2>(q));
    take(lane_move<DPP_HALF_MIRROR>(a), lane_move<DPP_HALF_MIRROR>(q));
    take(lane_move<DPP_MIRROR>(a), lane_move<DPP_MIRROR>(q));
    take(lane_move<-1>(a), lane_move<-1>(q));
    {
        const double a0 = read_lane(a, 0), a1 = read_lane(a, 32);
        const int q0 = __builtin_amdgcn_readlane(q, 0), q1 = __builtin_amdgcn_readlane(q, 32);
        a = a0; q = q0;
        take(a1, q1);
    }
    __syncthreads();
    if (lane == 0) { red[wave] = a; redi[wave] = q; }
    __syncthreads();
    a = red[0];
    q = redi[0];
    for (int w = 1; w < NT / 64; ++w)
        if (red[w] < a || (red[w] == a && (unsigned)redi[w] < (unsigned)q)) { a = red[w]; q = redi[w]; }
}

// A block of `sz` doubles from the arena (one thread calls it), or null when no chunk has room.  The
// offset `top` only grows (one fetch-and-add per request, so many workgroups allocate at once without
// retry loops); a range that would straddle the end of a chunk is abandoned and the request is made
// again, which lands past that end.  The chunk list is constant while kernels run.
__device__ double* arena_alloc(Arena* A, unsigned long long sz)
{
    const int nc = A->nchunks;
    for (int attempt = 0; attempt < 4; ++attempt) {
        const unsigned long long off = atomicAdd(&A->top, sz);
        int c = 0;
        while (c < nc && off >= A->start[c] + A->size[c]) ++c;
        if (c == nc) return nullptr;
        if (off + sz <= A->start[c] + A->size[c]) return A->base[c] + (off - A->start[c]);
    }
    return nullptr;
}

// The factor when it is held in LDS, addressed as LDS: the compiler then reads it with LDS
// instructions instead of generic (flat) ones, which wait on both memory counters.
typedef __attribute__((address_space(3))) double lds_double;
__device__ __forceinline__ lds_double* to_lds(double* p) { return (lds_double*)p; }
__device__ __forceinline__ const lds_double* to_lds(const double* p) { return (const lds_double*)p; }
// A factor known to be in global memory, addressed as global: loads then take a scalar base and a
// 32-bit lane offset instead of a 64-bit address per load.  p must be the same in every thread.
typedef __attribute__((address_space(1))) const double global_cdouble;
typedef __attribute__((address_space(1))) double global_double;
__device__ __forceinline__ global_cdouble* to_global(const double* p)
{
    // the same pointer in every thread: read it from the first lane so it stays in scalar registers
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (global_cdouble*)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ global_double* to_global(double* p)
{
    return (global_double*)const_cast<global_cdouble*>(to_global(static_cast<const double*>(p)));
}
__device__ __forceinline__ bool is_lds(const double* p)
{
    return __builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)(p));
}

// Per-signal working view inside the solve kernel.  G is global (row-major,
// stride K); the rest points into LDS or into the global homes.
struct Sig {
    int K;
    bool r_lds;           // R lives in LDS (latency-optimised loops) or in global memory (coalesced loops)
    double* G;            // G_II by slot
    double* R;            // Rinv, packed lower row-major by support position
    double* x;            // coefficient by slot
    double* c;            // a_u^T b by slot
    signed char* th;      // sign by slot, 0 = not in S
    unsigned char* ex;    // slot excluded from S
    int* so;              // slot of each support position
};

// z[i] = sum_{k <= i} R(i, k) w[k] for i < s with the factor in global memory: one row per wave at a
// time, lanes across the row (coalesced, eight loads in flight: clamped indices, so no load is guarded
// by a branch that would wait for it), a wave reduction per row.
__device__ __forceinline__ void rows_matvec_global(const double* R, const double* w, double* z, int s)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = wave; i < s; i += NT / 64) {
        const double* Ri = R + tri(i);
        double a0 = 0.0, a1 = 0.0;
        for (int k0 = lane; k0 <= i; k0 += 512) {
            double r[8], wv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + 64 * e <= i ? k0 + 64 * e : i;
                r[e] = Ri[k];
                wv[e] = w[k];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                (e & 1 ? a1 : a0) += k0 + 64 * e <= i ? r[e] * wv[e] : 0.0;
        }
        const double acc = wave_sum(a0 + a1);
        if (lane == 0) z[i] = acc;
    }
}

// Lanes per row (or column) of an LDS-resident factor with s support positions: a short support
// leaves most threads idle, so P consecutive lanes share a row and the serial chain is s / P long.
__device__ inline int split_lanes(int s) { return s <= 64 ? 4 : (s <= 128 ? 2 : 1); }

// z[i] = sum_{k <= i} R(i, k) v[k] for i < s (packed lower factor in LDS), split_lanes(s) lanes per
// row combined by shuffles inside the group.  Returns this lane's share of sum_i z_i^2.
template <class VP>
__device__ __forceinline__ double rows_matvec_lds_t(const lds_double* R, VP v, double* z, int s)
{
    const int P = split_lanes(s);
    const int sub = threadIdx.x & (P - 1);
    double part = 0.0;
    for (int i = threadIdx.x / P; i < s; i += NT / P) {   // the P lanes of a group share i
        const lds_double* Ri = R + tri(i);
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        int k = sub;
        for (; k + 3 * P <= i; k += 4 * P) {
            a0 += Ri[k] * v[k];
            a1 += Ri[k + P] * v[k + P];
            a2 += Ri[k + 2 * P] * v[k + 2 * P];
            a3 += Ri[k + 3 * P] * v[k + 3 * P];
        }
        for (; k <= i; k += P) a0 += Ri[k] * v[k];
        const double acc = group_sum((a0 + a1) + (a2 + a3), P);
        if (sub == 0) {
            z[i] = acc;
            part += acc * acc;
        }
    }
    return part;
}

__device__ __forceinline__ double rows_matvec_lds(const double* Rg, const double* v, double* z, int s)
{
    // the vector too is addressed as LDS when it lives there (the usual case)
    if (__builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)(v)))
        return rows_matvec_lds_t(to_lds(Rg), to_lds(v), z, s);
    return rows_matvec_lds_t(to_lds(Rg), v, z, s);
}

// out[k] = (sum_{i = k}^{s-1} v[i] R(i, k)) / div for k < s (packed lower factor in LDS),
// split_lanes(s) lanes per column.
template <class VP, class OP>
__device__ __forceinline__ void cols_matvec_lds_t(const lds_double* R, VP v, OP out, int s, double div)
{
    const int P = split_lanes(s);
    const int sub = threadIdx.x & (P - 1);
    for (int k = threadIdx.x / P; k < s; k += NT / P) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        int i = k + sub;
        for (; i + 3 * P < s; i += 4 * P) {
            a0 += v[i] * R[tri(i) + k];
            a1 += v[i + P] * R[tri(i + P) + k];
            a2 += v[i + 2 * P] * R[tri(i + 2 * P) + k];
            a3 += v[i + 3 * P] * R[tri(i + 3 * P) + k];
        }
        for (; i < s; i += P) a0 += v[i] * R[tri(i) + k];
        const double acc = group_sum((a0 + a1) + (a2 + a3), P);
        if (sub == 0) out[k] = acc / div;
    }
}

// out[k] = (sum_{i >= k} v[i] R(i, k)) / div for k < s (the factor in LDS), split_lanes(s) lanes per
// column; the vector and the output are addressed as LDS too when both live there.
__device__ __forceinline__ void cols_matvec_lds(const double* R, const double* v, double* out, int s, double div)
{
    if (__builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)(v)) &&
        __builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)(out)))
        cols_matvec_lds_t(to_lds(R), to_lds(v), to_lds(out), s, div);
    else
        cols_matvec_lds_t(to_lds(R), v, out, s, div);
}

// sum_{i = k}^{s-1} v[i] R(i, k) over column k of a packed lower factor.
__device__ __forceinline__ double col_dot(const Sig& f, const double* v, int k, int s)
{
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    if (f.r_lds) {
        const lds_double* R = to_lds(f.R);
        int i = k;
        int o = (int)(tri(k) + k);           // offset of R(i, k); the next row adds i + 1
        for (; i + 4 <= s; i += 4) {
            const int o1 = o + i + 1, o2 = o1 + i + 2, o3 = o2 + i + 3;
            a0 += v[i] * R[o];
            a1 += v[i + 1] * R[o1];
            a2 += v[i + 2] * R[o2];
            a3 += v[i + 3] * R[o3];
            o = o3 + i + 4;
        }
        for (; i < s; ++i) {
            a0 += v[i] * R[o];
            o += i + 1;
        }
    } else {
        // global factor: rows in lockstep across the wave so loads of one row coalesce; eight rows'
        // loads in flight (rows above k read row k instead and count zero, so no load is guarded)
        int i = k & ~63;
        for (; i + 8 <= s; i += 8) {
            double r[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = f.R[tri(i + e >= k ? i + e : k) + k];
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = i + e >= k ? r[e] : 0.0;
            a0 += v[i] * r[0] + v[i + 4] * r[4];
            a1 += v[i + 1] * r[1] + v[i + 5] * r[5];
            a2 += v[i + 2] * r[2] + v[i + 6] * r[6];
            a3 += v[i + 3] * r[3] + v[i + 7] * r[7];
        }
        for (; i < s; ++i)
            if (i >= k) a0 += v[i] * f.R[tri(i) + k];
    }
    return (a0 + a1) + (a2 + a3);
}

// Rinv^T (Rinv w) in one pass over a factor in global memory with s <= 1024 positions:
// z_i = sum_{k <= i} R(i, k) w[k] and out_k = sum_i z_i R(i, k).  The columns are split over
// the waves (wave v owns the 64-column chunks v, v + 4, v + 8, v + 12, lane l column l of each), the
// rows taken in batches: a wave loads its chunks of the batch's rows (chunks past a row's diagonal
// are skipped by a test on the row index, a scalar branch that leaves the loads in flight; the chunk
// that holds the diagonal is read whole and masked, so every load of the wave shares one lane
// offset: it reads at most 63 entries past the factor's last one, which lie inside the signal's slot
// block, where the per-slot vectors follow the factor), forms its partial dot products, and the four
// waves' partials meet in LDS (double-buffered, one barrier per batch, added in wave order) to give
// z_i, which each lane folds into its columns' sums while the rows are still in registers.  A row
// below 512 has at most two chunks per wave, so batches there take 8 rows (4 beyond): up to sixteen
// loads per lane in flight in every batch.  One read of the factor, instead of a row pass
// and a column pass that waits for its loads row by row.  z_i goes to z[i].  Ends with a barrier.  (For the
// sign-fixed minimiser alone, after a pruning; an append's comes with its pass, chol_append_fold.)
constexpr int FOLD_MAX = 1024;

// Rows [i_begin, i_end) of the one-pass product, RB at a time, each lane's chunks j < NJ.
template <int RB, int NJ>
__device__ inline void fold_rows(global_cdouble* R, int i_begin, int i_end, const double (&g)[4], double (&acc)[4],
                                 int& buf, double* z, double (*part)[NT / 64][8])
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i0 = i_begin; i0 < i_end; i0 += RB) {
        double r[RB][NJ];
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int i = i0 + q < i_end ? i0 + q : i_end - 1;   // the same on every lane
            global_cdouble* Ri = R + tri(i);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int c0 = 64 * (wave + 4 * j);
                r[q][j] = c0 <= i ? Ri[c0 + lane] : 0.0;       // whole chunk, masked below
            }
        }
#pragma unroll
        for (int h = 0; h < (RB + 7) / 8; ++h) {
            double pq[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 8 * h; q < RB && q < 8 * h + 8; ++q) {
                double a = 0.0;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int k = 64 * (wave + 4 * j) + lane;
                    r[q][j] = k <= i0 + q && i0 + q < i_end ? r[q][j] : 0.0;
                    a += r[q][j] * g[j];
                }
                pq[q - 8 * h] = a;
            }
            const double mine = wave_sum8(pq);   // lane l holds the wave's sum for row wave_sum8_index(l)
            if (lane < 8 && 8 * h + wave_sum8_index(lane) < RB) part[buf][wave][8 * h + wave_sum8_index(lane)] = mine;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            double zi = part[buf][0][q];
#pragma unroll
            for (int w = 1; w < NT / 64; ++w) zi += part[buf][w][q];
            if (threadIdx.x == 0 && i0 + q < i_end) z[i0 + q] = zi;
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[j] += zi * r[q][j];
        }
        buf ^= 1;
    }
}

__device__ __noinline__ void fold_pass_global(const double* R, const double* w, int s, double* out, double* z)
{
    __shared__ double part_lds[2][NT / 64][8];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    s = __builtin_amdgcn_readfirstlane(s);      // the same in every thread: row indices stay scalar
    const int last = s > 0 ? s - 1 : 0;
    double g[4], acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = 64 * (wave + 4 * j) + lane;
        g[j] = w[k < s ? k : last];
        acc[j] = 0.0;
    }
    int buf = 0;
    global_cdouble* Rg = to_global(R);
    fold_rows<8, 2>(Rg, 0, s < 512 ? s : 512, g, acc, buf, z, part_lds);
    fold_rows<4, 4>(Rg, 512, s, g, acc, buf, z, part_lds);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = 64 * (wave + 4 * j) + lane;
        if (k < s) out[k] = acc[j];
    }
    __syncthreads();
}

// x over the lower half of the wave added to x over the upper half in lanes 0..31, the same of y in lanes 32..63.
__device__ __forceinline__ double fold_half(double x, double y)
{
    const uint64_t bx = (uint64_t)__double_as_longlong(x), by = (uint64_t)__double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)bx, (uint32_t)by, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(bx >> 32), (uint32_t)(by >> 32), false, false);
    return __longlong_as_double((int64_t)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((int64_t)(((uint64_t)hi[1] << 32) | lo[1]));
}

// The same between the two rows of 16 lanes of each half: x in the even rows, y in the odd ones.
__device__ __forceinline__ double fold_rows16(double x, double y)
{
    const uint64_t bx = (uint64_t)__double_as_longlong(x), by = (uint64_t)__double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)bx, (uint32_t)by, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(bx >> 32), (uint32_t)(by >> 32), false, false);
    return __longlong_as_double((int64_t)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((int64_t)(((uint64_t)hi[1] << 32) | lo[1]));
}

constexpr int DPP_ROR8 = 0x128;   // row_ror:8, lane ^ 8 within a row of 16

// Eight values per lane summed over the lanes with the same low three bits: lane l gets the sum for value l >> 3.
__device__ __forceinline__ double fold_eight(const double (&a)[8])
{
    const bool b3 = (threadIdx.x >> 3) & 1;
    double u[4], w[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = fold_half(a[i], a[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) w[i] = fold_rows16(u[i], u[i + 2]);
    return (b3 ? w[1] : w[0]) + lane_move<DPP_ROR8>(b3 ? w[0] : w[1]);
}

// The sum over the low three lane bits (every lane of a group of eight gets it).
__device__ __forceinline__ double sum_low8(double t)
{
    t += lane_move<DPP_HALF_MIRROR>(t);
    t += lane_move<DPP_XOR2>(t);
    return t + lane_move<DPP_XOR1>(t);
}

typedef uint32_t uint2_t __attribute__((ext_vector_type(2)));

// Rows of a packed factor in global memory, one buffer per row: a load past the row's diagonal returns zero and a
// store past it is dropped, by the buffer's bound, so neither needs an address or a mask per lane.
struct RowBuffers {
    uint64_t base;
    __device__ __forceinline__ explicit RowBuffers(const double* R)
    {
        const uint64_t p = reinterpret_cast<uint64_t>(R);
        base = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    }
    // row i (the same on every lane); empty: no entry
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t row(int i, bool empty) const
    {
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base + 4ull * (uint32_t)(i * (i + 1))), 0,
                                                 empty ? 0 : 8 * (i + 1), 0x00027000);
    }
};
__device__ __forceinline__ double row_load(__amdgpu_buffer_rsrc_t r, int c8)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, c8, 0, 0));
}
__device__ __forceinline__ void row_store(__amdgpu_buffer_rsrc_t r, int c8, double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2_t, v), r, c8, 0, 0);
}

// chol_append_fold: J <= 8 single appends to a factor in global memory from one pass over it.  One append at a time,
// each over all rows, was a chain of batches (load, sum over the wave, barrier): 50 us an atom on supports around
// 300 to 480, half of the ragged batch's time (300 signals of 512 x 4096, supports up to 480).  The rows before s0 are
// the same for all J atoms: they are read once, give each atom's z_i and are folded into each atom's column sums.
// The new rows, which later atoms of the list also need, stay in registers: a lane keeps the sums of its columns,
// which become the row's entries, so atom e takes one more round over the e rows before it.
// One pass for up to eight atoms takes 65 us there (9 us an atom), and its arithmetic bounds it: three quarters of the
// instructions are sums over lanes and broadcasts, not the products.  With the columns split over the waves (a sum over
// the waves and a barrier per eight rows, as beyond 512 columns) it took 82 us; prefetching rows, or skipping columns a row does not have,
// each gave a tenth.
// Excluded atoms (no pivot) leave a zero row here and take no support position.
// xs (J <= 7): the eighth right-hand side is w = c_S - lambda theta_S, whose z (vzc) and sums (vx) are the
// sign-fixed minimiser's (sign_fixed_solve) on the s0 positions before.
struct FoldLds {
    static constexpr int C = 2 * NT;              // columns of fold_rows_wave
    double part[2][NT / 64][64];
    double gl[8][8];                              // Gram entries of the list
    double z[C];                                  // fold_rows_wave: the eighth right-hand side's z
    double zz[NT / 64][8];
    union {
        double g[8][C];                           // fold_rows_wave: the right-hand sides, then the waves' sums
        double zs[8 * C];                         // fold_rows_split: the eighth right-hand side's z, up to FOLD_MAX
    };
};
static_assert(FOLD_MAX <= 8 * FoldLds::C, "fold_rows_split's z");

// The rows before s0, s0 > 256 NJ / 2 columns split over the waves (wave v, lane l: columns 64 (v + 4 j) + l): eight
// rows at a time give each right-hand side's z_i by a sum over the wave and one over the waves (a barrier).
// acc: this lane's columns' sums; zz: sum z_i^2 of right-hand side l & 7 (every lane with those low bits).
template <int NJ>
__device__ __forceinline__ void fold_rows_split(const RowBuffers& rows, int s0, const double (&g)[8][NJ],
                                                double (&acc)[8][NJ], double& zz, int& buf, FoldLds& w)
{
    constexpr int NR = 8, NW = NT / 64, RB = 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double zzl = 0.0;
    // rows [i0, i1) with the first JL of each lane's columns
    auto pass = [&](auto jl, int i0, int i1) {
        constexpr int JL = decltype(jl)::value;
        for (int i = i0; i < i1; i += RB) {
            double r[RB][JL];
#pragma unroll
            for (int q = 0; q < RB; ++q) {
                const auto b = rows.row(i + q, i + q >= s0);
#pragma unroll
                for (int j = 0; j < JL; ++j) r[q][j] = row_load(b, 8 * (64 * (wave + NW * j) + lane));
            }
            // lane l: the products of row l >> 3 with right-hand side l & 7
            double t[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                double p8[8];
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    double d = 0.0;
#pragma unroll
                    for (int j = 0; j < JL; ++j) d += r[q][j] * g[e][j];
                    p8[q] = d;
                }
                t[e] = fold_eight(p8);
                if (e & 1) __builtin_amdgcn_sched_barrier(0);   // two right-hand sides' products at a time
            }
            const bool b0 = lane & 1, b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1;
            double t4[4], t2[2];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                t4[q] = (b2 ? t[q + 4] : t[q]) + lane_move<DPP_HALF_MIRROR>(b2 ? t[q] : t[q + 4]);
#pragma unroll
            for (int q = 0; q < 2; ++q) t2[q] = (b1 ? t4[q + 2] : t4[q]) + lane_move<DPP_XOR2>(b1 ? t4[q] : t4[q + 2]);
            w.part[buf][wave][lane] = (b0 ? t2[1] : t2[0]) + lane_move<DPP_XOR1>(b0 ? t2[0] : t2[1]);
            __syncthreads();
            double z = w.part[buf][0][lane];
#pragma unroll
            for (int v2 = 1; v2 < NW; ++v2) z += w.part[buf][v2][lane];
            buf ^= 1;
            zzl += z * z;                         // zero past s0
            if (wave == 0 && (lane & 7) == 7) w.zs[i + (lane >> 3)] = z;
#pragma unroll
            for (int e = 0; e < NR; ++e) {
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    const double zi = read_lane(z, 8 * q + e);
#pragma unroll
                    for (int j = 0; j < JL; ++j) acc[e][j] += zi * r[q][j];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    pass(std::integral_constant<int, NJ / 2>{}, 0, min(s0, NT * (NJ / 2)));
    if (s0 > NT * (NJ / 2)) pass(std::integral_constant<int, NJ>{}, NT * (NJ / 2), s0);
    zzl += lane_move<DPP_ROR8>(zzl);
    zzl = fold_rows16(zzl, zzl);
    zz = fold_half(zzl, zzl);
}

// The same for s0 <= 512 with the rows split over the waves: a wave takes whole rows (lane l: columns 64 c + l), so
// a row's sum needs no other wave, no barrier, and a quarter of the reductions, and the load of the next rows
// runs under these rows' arithmetic; the waves' column sums meet in LDS at the end.  The arithmetic, not the bytes,
// takes the time.  w.g holds the right-hand sides; the right-hand sides' entries of this lane's columns of the
// column split are left in g.
__device__ __forceinline__ void fold_rows_wave(const RowBuffers& rows, int s0, double (&g)[8][2], double (&acc)[8][2],
                                               double& zz, FoldLds& w)
{
    constexpr int NR = 8, NW = NT / 64, NC = FoldLds::C / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
    double sum[NR][NC];
#pragma unroll
    for (int e = 0; e < NR; ++e)
#pragma unroll
        for (int c = 0; c < NC; ++c) sum[e][c] = 0.0;
    double zs = 0.0;                              // sum of z^2 of this lane's right-hand side
    // rows [i0, i1), RB per wave at a time, with the first CL chunks of columns
    auto pass = [&](auto cl, auto rb, int i0, int i1) {
        constexpr int CL = decltype(cl)::value, RB = decltype(rb)::value;
        auto load = [&](int i, double (&r)[RB][CL]) {
#pragma unroll
            for (int q = 0; q < RB; ++q) {
                const auto b = rows.row(i + q, i + q >= i1);
#pragma unroll
                for (int c = 0; c < CL; ++c) r[q][c] = row_load(b, 8 * (64 * c + lane));
            }
        };
        double zl = 0.0;
        auto batch = [&](int i, const double (&r)[RB][CL]) {
            double t[NR];
#pragma unroll
            for (int e = 0; e < NR; ++e) {
                double d[RB];
#pragma unroll
                for (int q = 0; q < RB; ++q) d[q] = 0.0;
#pragma unroll
                for (int c = 0; c < CL; ++c) {
                    const double ge = w.g[e][64 * c + lane];
#pragma unroll
                    for (int q = 0; q < RB; ++q) d[q] += r[q][c] * ge;
                }
                if constexpr (RB == 4)            // row 2 b5 + b4
                    t[e] = fold_rows16(fold_half(d[0], d[2]), fold_half(d[1], d[3]));
                else                              // row b5
                    t[e] = fold_half(d[0], d[1]);
                if (e & 1) __builtin_amdgcn_sched_barrier(0);
            }
            // the right-hand sides over the next three lane bits, then the sum over the rest
            double u[4], v[2], z;
            if constexpr (RB == 4) {              // right-hand side 4 b3 + 2 b2 + b1
#pragma unroll
                for (int k = 0; k < 4; ++k) u[k] = (b3 ? t[k + 4] : t[k]) + lane_move<DPP_ROR8>(b3 ? t[k] : t[k + 4]);
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    v[k] = (b2 ? u[k + 2] : u[k]) + lane_move<DPP_HALF_MIRROR>(b2 ? u[k] : u[k + 2]);
                z = (b1 ? v[1] : v[0]) + lane_move<DPP_XOR2>(b1 ? v[0] : v[1]);
                z += lane_move<DPP_XOR1>(z);
            } else {                              // right-hand side 4 b4 + 2 b3 + b2
#pragma unroll
                for (int k = 0; k < 4; ++k) u[k] = fold_rows16(t[k], t[k + 4]);
#pragma unroll
                for (int k = 0; k < 2; ++k) v[k] = (b3 ? u[k + 2] : u[k]) + lane_move<DPP_ROR8>(b3 ? u[k] : u[k + 2]);
                z = (b2 ? v[1] : v[0]) + lane_move<DPP_HALF_MIRROR>(b2 ? v[0] : v[1]);
                z += lane_move<DPP_XOR2>(z);
                z += lane_move<DPP_XOR1>(z);
            }
            zl += z * z;                          // zero past i1
            const int rhs = RB == 4 ? (lane >> 1) & 7 : (lane >> 2) & 7;
            if (rhs == 7) w.z[i + (RB == 4 ? lane >> 4 : lane >> 5)] = z;
#pragma unroll
            for (int e = 0; e < NR; ++e) {
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    const double zi = read_lane(z, RB == 4 ? 16 * q + 2 * e : 32 * q + 4 * e);
#pragma unroll
                    for (int c = 0; c < CL; ++c) sum[e][c] += zi * r[q][c];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        double ra[RB][CL], rb_[RB][CL];           // the next rows are in flight during these rows' arithmetic
        constexpr int STEP = RB * NW;
        int i = i0 + RB * wave;
        load(i, ra);
        for (; i < i1; i += 2 * STEP) {
            load(i + STEP, rb_);
            batch(i, ra);
            if (i + STEP >= i1) break;
            load(i + 2 * STEP, ra);
            batch(i + STEP, rb_);
        }
        // rows over the lanes: right-hand side e in lane 2 e (4 e)
        if constexpr (RB == 4) zl = fold_rows16(zl, zl);
        zl = fold_half(zl, zl);
        zs += __shfl(zl, RB == 4 ? 2 * (lane & 7) : 4 * (lane & 7));
    };
    pass(std::integral_constant<int, NC / 2>{}, std::integral_constant<int, 4>{}, 0, min(s0, NT));
    if (s0 > NT) pass(std::integral_constant<int, NC>{}, std::integral_constant<int, 2>{}, NT, s0);
    if (lane < 8) w.zz[wave][lane] = zs;
#pragma unroll
    for (int e = 0; e < NR; ++e)
#pragma unroll
        for (int j = 0; j < 2; ++j) g[e][j] = w.g[e][64 * (wave + NW * j) + lane];
    __syncthreads();                              // every wave is done with w.g: its memory takes the sums now
    zz = w.zz[0][lane & 7];
#pragma unroll
    for (int v = 1; v < NW; ++v) zz += w.zz[v][lane & 7];
#pragma unroll
    for (int e = 0; e < NR; ++e) {
        double(*m)[FoldLds::C] = &w.g[4 * (e & 1)];
#pragma unroll
        for (int c = 0; c < NC; ++c) m[wave][64 * c + lane] = sum[e][c];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = 64 * (wave + NW * j) + lane;
            acc[e][j] = m[0][k];
#pragma unroll
            for (int v = 1; v < NW; ++v) acc[e][j] += m[v][k];
        }
    }
}

template <int NJ>
__device__ __forceinline__ void chol_append_fold(Sig& v, int& nS, const int* list, int J, const double* vg, bool xs,
                                                 double lam, double* vzc, double* vx, FoldLds& w)
{
    constexpr int NR = 8, NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s0 = __builtin_amdgcn_readfirstlane(nS);
    J = __builtin_amdgcn_readfirstlane(J);
    global_cdouble* G = to_global((const double*)v.G);
    int slot[NR];                                 // past J the last atom again: computed, never used
#pragma unroll
    for (int e = 0; e < NR; ++e) slot[e] = __builtin_amdgcn_readfirstlane(list[e < J ? e : J - 1]);
    if (tid < NR * NR) {
        const int e = tid / NR, f = tid % NR;
        w.gl[e][f] = G[(int64_t)list[e < J ? e : J - 1] * v.K + list[f < J ? f : J - 1]];
    }
    double g[NR][NJ], acc[NR][NJ];
    double zzl = 0.0;
    int buf = 0;
    {
        int sk[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int k = 64 * (wave + NW * j) + lane;
            sk[j] = s0 > 0 ? v.so[k < s0 ? k : s0 - 1] : slot[0];
        }
#pragma unroll
        for (int e = 0; e < NR; ++e)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                g[e][j] = G[(int64_t)slot[e] * v.K + sk[j]];
                acc[e][j] = 0.0;
            }
        if (xs)
#pragma unroll
            for (int j = 0; j < NJ; ++j) g[NR - 1][j] = v.c[sk[j]] - lam * (double)v.th[sk[j]];
    }
    const RowBuffers rows(v.R);
    if (s0 > 0) {
        if constexpr (NJ == 2) {
#pragma unroll
            for (int e = 0; e < NR; ++e)
#pragma unroll
                for (int j = 0; j < NJ; ++j) w.g[e][64 * (wave + NW * j) + lane] = g[e][j];
            __syncthreads();
            fold_rows_wave(rows, s0, g, acc, zzl, w);
        } else {
            fold_rows_split<NJ>(rows, s0, g, acc, zzl, buf, w);
        }
    }
    __syncthreads();   // w.gl (when there were no rows), and the readers of w.part are done
    int s = s0;
#pragma unroll
    for (int e = 0; e < NR; ++e) {
        if (e >= J) break;                        // the same in every thread
        double zz = read_lane(zzl, e);
        if (e > 0) {
            // this atom's products with the new rows 0 .. e - 1 (zero rows for the excluded atoms)
            double pq[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                double a = 0.0;
                if (t < e)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) a += acc[t < NR ? t : 0][j] * g[e][j];
                pq[t] = a;
            }
            w.part[buf][wave][lane] = sum_low8(fold_eight(pq));
            __syncthreads();
            double z = w.part[buf][0][lane];
#pragma unroll
            for (int v2 = 1; v2 < NW; ++v2) z += w.part[buf][v2][lane];
            buf ^= 1;
#pragma unroll
            for (int t = 0; t < e; ++t) {
                const double zi = read_lane(z, 8 * t);
                zz += zi * zi;
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[e][j] += zi * acc[t][j];
            }
        }
        const double gjj = w.gl[e][e];
        const double dd = gjj - zz;
        const bool ok = dd > 1e-11 * gjj;
        const double d = sqrt(dd);
        const auto out = rows.row(s, !ok);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int k = 64 * (wave + NW * j) + lane;
            double o = 0.0;
            if (ok) o = k < s ? acc[e][j] / -d : (k == s ? 1.0 / d : 0.0);
            acc[e][j] = o;
            row_store(out, 8 * k, o);
#pragma unroll
            for (int f = e + 1; f < NR; ++f) g[f][j] = ok && k == s ? w.gl[f][e] : g[f][j];
        }
        if (tid == 0) {
            if (ok) {
                v.so[s] = slot[e];
                v.th[slot[e]] = vg[slot[e]] > 0.0 ? 1 : -1;
            } else {
                v.ex[slot[e]] = 1; v.th[slot[e]] = 0; v.x[slot[e]] = 0.0;
            }
        }
        s += ok ? 1 : 0;
    }
    if (xs) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int k = 64 * (wave + NW * j) + lane;
            if (k < s0) vx[k] = acc[NR - 1][j];
        }
        const double* wz = NJ == 2 ? w.z : w.zs;
        for (int k = tid; k < s0; k += NT) vzc[k] = wz[k];
    }
    nS = s;
    __syncthreads();
}

// Append slot j with sign th at support position s = nS (a Cholesky row append
// held as the inverse factor).  Returns false and excludes j if its Schur
// complement pivot vanishes, i.e. a_j is numerically in the span of A_S.
__device__ __forceinline__ bool chol_append(const Sig& v, int& nS, int j, signed char th, double* vw, double* vz, double* red,
                            uint64_t* cnt)
{
    const int s = nS;
    const int tid = threadIdx.x;
    const uint64_t t_in = cnt ? wall_clock64() : 0;
    if (cnt && tid == 0) atomicAdd(reinterpret_cast<unsigned long long*>(cnt), 1ull);
    const double* Gj = v.G + (int64_t)j * v.K;
    __shared__ double s_gjj;
    // w = G(S, j): four positions per thread at once, slot numbers first and then the gathers (clamped
    // indices: a load behind a per-thread test would be waited for before the next one is issued)
    for (int k0 = tid; k0 < s; k0 += 4 * NT) {
        int sk[4];
        double gv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = k0 + NT * e;
            sk[e] = v.so[k < s ? k : s - 1];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[e] = Gj[sk[e]];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k0 + NT * e < s) vw[k0 + NT * e] = gv[e];
    }
    if (tid == 0) s_gjj = Gj[j];
    __syncthreads();
    double* Rs = v.R + tri(s);
    const double gjj = s_gjj;
    double part = 0.0;
    if (v.r_lds) {
        part = rows_matvec_lds(v.R, vw, vz, s);    // z = Rinv w
    } else {
        rows_matvec_global(v.R, vw, vz, s);
        __syncthreads();
        for (int i = tid; i < s; i += NT) part += vz[i] * vz[i];
    }
    const double dd = gjj - block_sum_fenced(part, red);   // the barrier after the gather fences red
    if (!(dd > 1e-11 * gjj)) {
        if (tid == 0) { v.ex[j] = 1; v.th[j] = 0; v.x[j] = 0.0; }
        __syncthreads();
        if (cnt && tid == 0)   // cnt[-2]: ticks spent in appends (phase slot 4)
            atomicAdd(reinterpret_cast<unsigned long long*>(cnt - 2), (unsigned long long)(wall_clock64() - t_in));
        return false;
    }
    const double d = sqrt(dd);
    if (v.r_lds)                             // new row: -(z^T Rinv)_k / d
        cols_matvec_lds(v.R, vz, Rs, s, -d);
    else
        for (int k = tid; k < s; k += NT) Rs[k] = -col_dot(v, vz, k, s) / d;
    if (tid == 0) {
        Rs[s] = 1.0 / d;
        v.so[s] = j;
        v.th[j] = th;
    }
    nS = s + 1;
    __syncthreads();
    if (cnt && tid == 0)   // cnt[-2]: ticks spent in appends (phase slot 4)
        atomicAdd(reinterpret_cast<unsigned long long*>(cnt - 2), (unsigned long long)(wall_clock64() - t_in));
    return true;
}

// J <= NR appends to a factor in LDS (s0 + J <= NT positions) as one block: with W = G(S, list), Z = Rinv W and
// C = G(list, list) - Z^T Z, the rows are [-L^-1 Z^T Rinv, L^-1] with C = L L^T, eliminated in list order with
// the single append's pivot rule.  A single append is a chain of two products, a sum over the workgroup and four
// barriers: its latency, not its arithmetic, took the time (one signal of 1000 x 5001, |S| to 40: 367 us per solve
// with single appends, 325 with blocks).
// The waves split the right-hand sides.  A lane takes a row (Z) or a column (Z^T Rinv) and walks along it; the
// right-hand side's entry, which all lanes multiply by, comes from the lane that holds it.  Z, then Z^T Rinv
// use the new rows' memory; the 8 x 8 elimination runs in every wave, lane 8 e + f with entry (e, f).
// xs (J < NR): the last right-hand side is c_S - lambda theta_S, as in chol_append_fold.
template <int NR>
__device__ __forceinline__ void chol_append_lds(Sig& v, int& nS, const int* list, int J, const double* vg, bool xs,
                                                double lam, double* vzc, double* vx)
{
    constexpr int NW = NT / 64, H = NR > NW ? NR / NW : 1, NC = NT / 64;
    __shared__ double s_c[64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s0 = __builtin_amdgcn_readfirstlane(nS);
    J = __builtin_amdgcn_readfirstlane(J);
    lds_double* R = to_lds(v.R);
    global_cdouble* G = to_global((const double*)v.G);
    const int e8 = lane >> 3, f8 = lane & 7;
    const double gl = G[(int64_t)list[min(e8, J - 1)] * v.K + list[min(f8, J - 1)]];
    double acc[H][NC];
    const bool busy = H * wave < J || (xs && H * wave < NR && H * wave + H >= NR);   // the same in every lane
    if (busy && s0 > 0) {
        double g[H][NC], z[H][NC];
        int sk[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) sk[c] = v.so[min(64 * c + lane, s0 - 1)];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int slot = __builtin_amdgcn_readfirstlane(list[min(H * wave + h, J - 1)]);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                g[h][c] = G[(int64_t)slot * v.K + sk[c]];
                z[h][c] = 0.0;
                acc[h][c] = 0.0;
            }
        }
        if (xs && H * wave + H >= NR)
#pragma unroll
            for (int c = 0; c < NC; ++c) g[H - 1][c] = v.c[sk[c]] - lam * (double)v.th[sk[c]];
        // z of row 64 rc + lane (rows past s0 read row s0 - 1 and are zeroed)
#pragma unroll
        for (int rc = 0; rc < NC; ++rc) {
            if (64 * rc >= s0) break;
            const int i = min(64 * rc + lane, s0 - 1), base = (int)tri(i);
#pragma unroll
            for (int kc = 0; kc <= rc; ++kc) {
                const int top = min(64, s0 - 64 * kc);
#pragma unroll 4
                for (int k = 0; k < top; ++k) {
                    double r = R[base + 64 * kc + k];
                    if (kc == rc) r = 64 * kc + k <= i ? r : 0.0;
#pragma unroll
                    for (int h = 0; h < H; ++h) z[h][rc] += r * read_lane(g[h][kc], k);
                }
            }
            const bool in = 64 * rc + lane < s0;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                z[h][rc] = in ? z[h][rc] : 0.0;
                const int e = H * wave + h;
                if (xs && e == NR - 1) {
                    if (in) vzc[64 * rc + lane] = z[h][rc];
                } else if (e < J && in) {
                    R[(int)tri(s0 + e) + 64 * rc + lane] = z[h][rc];
                }
            }
        }
        // column 64 cc + lane of Z^T Rinv
#pragma unroll
        for (int cc = 0; cc < NC; ++cc) {
            if (64 * cc >= s0) break;
            const int k = min(64 * cc + lane, s0 - 1);
#pragma unroll
            for (int ic = cc; ic < NC; ++ic) {
                const int top = min(64, s0 - 64 * ic);
#pragma unroll 4
                for (int ii = 0; ii < top; ++ii) {
                    const int i = 64 * ic + ii;
                    double r = R[(int)tri(i) + k];
                    if (ic == cc) r = k <= i ? r : 0.0;
#pragma unroll
                    for (int h = 0; h < H; ++h) acc[h][cc] += r * read_lane(z[h][ic], ii);
                }
            }
            if (xs && H * wave + H >= NR && 64 * cc + lane < s0) vx[64 * cc + lane] = acc[H - 1][cc];
        }
    }
    __syncthreads();
    // C, entry (e, f) by NW lanes
    double c;
    {
        const int pe = (tid / NW) >> 3, pf = (tid / NW) & 7;
        double sum = 0.0;
        if (pe < J && pf < J) {
            const int be = (int)tri(s0 + pe), bf = (int)tri(s0 + pf);
            for (int i = tid & (NW - 1); i < s0; i += NW) sum += R[be + i] * R[bf + i];
        }
        sum = group_sum(sum, NW);
        if (NW == 1) {
            c = gl - sum;
        } else {
            if ((tid & (NW - 1)) == 0) s_c[tid / NW] = sum;
        }
        __syncthreads();
        if (NW > 1) c = gl - s_c[lane];
    }
    if (busy && s0 > 0)
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int cc = 0; cc < NC; ++cc)
                if (H * wave + h < J && 64 * cc + lane < s0)
                    R[(int)tri(s0 + H * wave + h) + 64 * cc + lane] = acc[h][cc];
    // elimination: C = L L^T, li = L^-1 over the accepted atoms
    double mi = e8 == f8 ? 1.0 : 0.0;
    unsigned okm = 0;
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        if (t >= J) break;
        const double d = read_lane(c, 9 * t);
        if (!(d > 1e-11 * read_lane(gl, 9 * t))) continue;   // in the span: left out
        okm |= 1u << t;
        const double m = e8 > t ? __shfl(c, 8 * e8 + t) / d : 0.0;
        const double ct = __shfl(c, 8 * t + f8), mt = __shfl(mi, 8 * t + f8);
        c -= m * ct;
        mi -= m * mt;
    }
    const double piv = __shfl(c, 9 * e8);
    const bool ok_ef = ((okm >> e8) & 1) && ((okm >> f8) & 1) && f8 <= e8;
    const double li = ok_ef ? mi / sqrt(piv) : 0.0;
    __syncthreads();                              // the rows of Z^T Rinv are complete
    for (int k = tid; k < s0; k += NT) {
        double a[NR];
#pragma unroll
        for (int f = 0; f < NR; ++f) a[f] = R[(int)tri(s0 + min(f, J - 1)) + k];
        int s = s0;
#pragma unroll
        for (int e = 0; e < NR; ++e) {
            if (e >= J) break;
            if (!((okm >> e) & 1)) continue;
            double o = 0.0;
#pragma unroll
            for (int f = 0; f <= e; ++f) o -= read_lane(li, 8 * e + f) * a[f];
            R[(int)tri(s) + k] = o;
            ++s;
        }
    }
    if (wave == 0) {
        const int pe = s0 + __popc(okm & ((1u << e8) - 1u)), pf = s0 + __popc(okm & ((1u << f8) - 1u));
        if (ok_ef) R[(int)tri(pe) + pf] = li;
        if (f8 == 0 && e8 < J) {
            const int slot = list[e8];
            if ((okm >> e8) & 1) {
                v.so[pe] = slot;
                v.th[slot] = vg[slot] > 0.0 ? 1 : -1;
            } else {
                v.ex[slot] = 1; v.th[slot] = 0; v.x[slot] = 0.0;
            }
        }
    }
    nS = s0 + __popc(okm);
    __syncthreads();
}

// Append the slots list[0..J) (J <= JB), in list order, at support positions nS, nS + 1, ...
// as one block.  With s0 = nS, W = G(S, list) and Z = Rinv W (s0 x J), the Schur complement
// C = G(list, list) - Z^T Z is factored in list order with the single-append pivot rule (an atom
// whose pivot C_ee - |l_e|^2 falls to 1e-11 g_ee or below is excluded, as chol_append would), and
// the accepted atoms A get the inverse-factor rows [-L22^{-1} Z_A^T Rinv, L22^{-1}].  The same
// factor as J single appends in exact arithmetic, for two passes over Rinv instead of 2J.
// Signs come from vg (sign of the gradient) or, with vg == nullptr, from the slots' current theta.
// zs: LDS scratch of (s0 + 1) * JB doubles.
__device__ __forceinline__ void chol_append_block(Sig& v, int& nS, const int* list, int J, const double* vg, double* zs,
                                  uint64_t* cnt)
{
    __shared__ double s_C[JB * JB];     // Schur complement (lower), then L22^{-1}
    __shared__ double s_L[JB * JB];     // L22, rows in accepted order
    __shared__ int s_acc[JB];
    __shared__ int s_na;
    const int s0 = nS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t t_in = cnt ? wall_clock64() : 0;
    if (cnt && tid == 0) atomicAdd(reinterpret_cast<unsigned long long*>(cnt), (unsigned long long)J);

    // 1. W = G(S, list): row k = support position, JB columns, zero past J
    for (int t = tid; t < s0 * JB; t += NT) {
        const int k = t / JB, e = t - k * JB;
        zs[t] = e < J ? v.G[(int64_t)list[e] * v.K + v.so[k]] : 0.0;
    }
    __syncthreads();
    // 2. Z = Rinv W in place.  Rows from the bottom, one per wave per round; row i needs the W rows
    //    at or below it, so a round's rows are written only after every wave has read them.
    for (int top = s0 - 1; top >= 0; top -= NT / 64) {
        const int i = top - wave;
        double acc[JB];
#pragma unroll
        for (int e = 0; e < JB; ++e) acc[e] = 0.0;
        if (i >= 0) {
            const double* Ri = v.R + tri(i);
            for (int k = lane; k <= i; k += 512) {   // eight loads in flight per lane, the row's tail too
                double r[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) r[q] = Ri[k + 64 * q <= i ? k + 64 * q : i];   // clamped, unguarded
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if (k + 64 * q > i) break;
                    const double* wk = zs + (k + 64 * q) * JB;
#pragma unroll
                    for (int e = 0; e < JB; ++e) acc[e] += r[q] * wk[e];
                }
            }
        }
        static_assert(JB == 8, "the eight-way wave sum");
        const double val = wave_sum8(acc);   // uniform per wave: every lane takes part
        __syncthreads();
        if (i >= 0 && lane < JB) zs[i * JB + wave_sum8_index(lane)] = val;
    }
    __syncthreads();
    // 3. C = G(list, list) - Z^T Z, lower triangle
    for (int t = tid; t < J * J; t += NT) {
        const int e = t / J, f = t - e * J;
        if (f > e) continue;
        double sum = 0.0;
        for (int i = 0; i < s0; ++i) sum += zs[i * JB + e] * zs[i * JB + f];
        s_C[e * JB + f] = v.G[(int64_t)list[e] * v.K + list[f]] - sum;
    }
    __syncthreads();
    // 4. Cholesky of C in list order with exclusion, then L22^{-1} into s_C (one thread, J <= JB)
    if (tid == 0) {
        int na = 0;
        for (int e = 0; e < J; ++e) {
            double dd = s_C[e * JB + e];
            for (int b = 0; b < na; ++b) {
                double x = s_C[e * JB + s_acc[b]];          // C(e, A_b), A_b < e
                for (int c = 0; c < b; ++c) x -= s_L[na * JB + c] * s_L[b * JB + c];
                x /= s_L[b * JB + b];
                s_L[na * JB + b] = x;
                dd -= x * x;
            }
            const int u = list[e];
            const double gjj = v.G[(int64_t)u * v.K + u];
            if (dd > 1e-11 * gjj) {
                s_L[na * JB + na] = sqrt(dd);
                s_acc[na++] = e;
            } else {
                v.ex[u] = 1; v.th[u] = 0; v.x[u] = 0.0;
            }
        }
        for (int a2 = 0; a2 < na; ++a2) {
            const double dinv = 1.0 / s_L[a2 * JB + a2];
            for (int b = 0; b < a2; ++b) {
                double x = 0.0;
                for (int c = b; c < a2; ++c) x += s_L[a2 * JB + c] * s_C[c * JB + b];
                s_C[a2 * JB + b] = -x * dinv;
            }
            s_C[a2 * JB + a2] = dinv;
        }
        s_na = na;
    }
    __syncthreads();
    const int na = s_na;
    if (na < J) {   // keep only the accepted columns of Z, in accepted order
        for (int i = tid; i < s0; i += NT) {
            double* zi = zs + i * JB;
            for (int b = 0; b < na; ++b) zi[b] = zi[s_acc[b]];
        }
        __syncthreads();
    }
    // 5. New rows: R(s0 + a, k) = -sum_{b <= a} L22^{-1}(a, b) M(b, k), M(b, k) = sum_{i >= k} Z(i, b) R(i, k).
    //    Threads own columns k; a wave's lanes walk the rows in lockstep so reads of one row coalesce.
    for (int kb = 0; kb < s0; kb += NT) {
        const int k = kb + tid;
        double acc[JB];
#pragma unroll
        for (int b = 0; b < JB; ++b) acc[b] = 0.0;
        int i = kb + wave * 64;
        for (; i + 8 <= s0; i += 8) {              // eight rows' loads in flight
            double r[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {   // clamped to row >= column and column < s0: always inside the factor
                const int kk = k < s0 ? k : s0 - 1;
                r[q] = v.R[tri(i + q >= kk ? i + q : kk) + kk];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) r[q] = i + q >= k ? r[q] : 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double* zi = zs + (i + q) * JB;
#pragma unroll
                for (int b = 0; b < JB; ++b) acc[b] += r[q] * zi[b];
            }
        }
        for (; i < s0; ++i) {
            if (i >= k) {
                const double r = v.R[tri(i) + k];
                const double* zi = zs + i * JB;
#pragma unroll
                for (int b = 0; b < JB; ++b) acc[b] += r * zi[b];
            }
        }
        if (k < s0) {
#pragma unroll
            for (int a2 = 0; a2 < JB; ++a2) {
                if (a2 >= na) break;
                double val = 0.0;
#pragma unroll
                for (int b = 0; b <= a2; ++b) val += s_C[a2 * JB + b] * acc[b];
                v.R[tri(s0 + a2) + k] = -val;
            }
        }
    }
    for (int t = tid; t < na * JB; t += NT) {
        const int a2 = t / JB, b = t - a2 * JB;
        if (b <= a2) v.R[tri(s0 + a2) + s0 + b] = s_C[a2 * JB + b];
    }
    if (tid < na) {
        const int u = list[s_acc[tid]];
        v.so[s0 + tid] = u;
        v.th[u] = vg ? (vg[u] > 0.0 ? 1 : -1) : v.th[u];
    }
    nS = s0 + na;
    __syncthreads();
    if (cnt && tid == 0)   // cnt[-2]: ticks spent in appends (phase slot 4)
        atomicAdd(reinterpret_cast<unsigned long long*>(cnt - 2), (unsigned long long)(wall_clock64() - t_in));
}

// Append the slots list[0..nv) in order, in blocks of JB, stopping at nmax support positions
// (the remaining slots are excluded).
__device__ __forceinline__ void append_list(Sig& v, int& nS, const int* list, int nv, const double* vg, int nmax, double* zs,
                            uint64_t* cnt)
{
    for (int e = 0; e < nv;) {
        if (nS >= nmax) {
            for (int t = threadIdx.x; t < nv - e; t += NT) v.ex[list[e + t]] = 1;
            __syncthreads();
            return;
        }
        int J = nv - e < JB ? nv - e : JB;
        J = J < nmax - nS ? J : nmax - nS;
        chol_append_block(v, nS, list + e, J, vg, zs, cnt);
        e += J;
    }
}

// Remove support position q from the inverse factor in O(|S|^2).  Moving column q of Rinv to the end
// only relabels G's order; Givens rotations of consecutive rows j, j + 1 (j = q .. s-2), each chosen to
// clear row j's entry in the moved column, then restore triangularity.  Rotations act on the left of
// Rinv, so Rinv^T Rinv = G^{-1} is unchanged for the remaining positions, and the leading
// (s-1) x (s-1) block is the new inverse factor (rows may change sign, which no product of the solver
// sees).  One barrier per row: row j's new values land where no later step reads, and the next step's
// writes (row j + 1) wait until every thread has read the old row j + 1.  The moved column's running
// entries live in `cbuf` (s doubles of scratch, each entry owned by one thread), so the downdate needs
// no per-thread arrays whatever |S| is.  The caller shifts the support order.
//
// zc (or null): the cached z = Rinv w of the sign-fixed solve (by position).  Rotating rows rotates z's
// entries the same way (the moved column's w entry moves with it, so every row's product with w is
// unchanged); thread 0 carries them along, and zc[s-1] receives the last (removed) row's value.  On
// return cbuf[0..s-2] holds that last row's entries.
//
// Up to DROP_COLS * 256 positions, each thread keeps its columns' running entries in registers and
// loads the next row's entries one iteration ahead, so the global factor's load latency overlaps the
// barrier; the next row is only read, never written, during an iteration, and the barrier per row keeps
// every read of a row before the iteration that writes it.  (The kernel capped at 128 registers uses a
// narrower register window: four columns, |S| <= 1024.)
template <int DROP_COLS, class RP>
__device__ __forceinline__ void chol_drop_t(RP R, int s, int q, double* cbuf, double* zc)
{
    const int tid = threadIdx.x;
    if (s <= DROP_COLS * NT) {
        // Loads take clamped, always valid indices and the unused values are zeroed after them: a
        // guarded load compiles to a branch whose end waits for the data, so a thread's loads would run
        // one after another.
        double cv[DROP_COLS], nx[DROP_COLS];
        const bool has_next = q + 1 < s;
#pragma unroll
        for (int t = 0; t < DROP_COLS; ++t) {
            const int c = tid + NT * t;
            const int cq = c < q ? c : q;
            cv[t] = R[tri(q) + cq];
            if (has_next) nx[t] = R[tri(q + 1) + (c < q ? c : q + 1)];
        }
#pragma unroll
        for (int t = 0; t < DROP_COLS; ++t) {
            const int c = tid + NT * t;
            cv[t] = c < q ? cv[t] : 0.0;
            nx[t] = (has_next && c <= q) ? nx[t] : 0.0;
        }
        double last = R[tri(q) + q];
        double b = q + 1 < s ? R[tri(q + 1) + q] : 0.0;
        double zcar = (zc && tid == 0) ? zc[q] : 0.0;
        // every thread has its R(q, q) before the owner of column q rewrites row q in the first rotation
        __syncthreads();
        for (int j = q; j < s - 1; ++j) {
            // prefetch row j + 2 (the next iteration's row), columns shifted past the moved one
            double nn[DROP_COLS];
            const bool more = j + 2 < s;   // the same for every thread
            const RP r2 = R + tri(j + 2);
            double bn = 0.0;
            if (more) {
#pragma unroll
                for (int t = 0; t < DROP_COLS; ++t) {
                    const int c = tid + NT * t;
                    const int cc = c <= j + 1 ? c : j + 1;
                    nn[t] = r2[cc < q ? cc : cc + 1];
                }
                bn = r2[q];
#pragma unroll
                for (int t = 0; t < DROP_COLS; ++t) nn[t] = tid + NT * t <= j + 1 ? nn[t] : 0.0;
            } else {
#pragma unroll
                for (int t = 0; t < DROP_COLS; ++t) nn[t] = 0.0;
            }
            const double r = hypot(last, b);
            const double cs = r > 0.0 ? b / r : 1.0;
            const double sn = r > 0.0 ? -last / r : 0.0;
            RP out = R + tri(j);
#pragma unroll
            for (int t = 0; t < DROP_COLS; ++t) {
                const int c = tid + NT * t;
                if (c <= j) {                    // columns past j stay zero in the moved column
                    out[c] = cs * cv[t] + sn * nx[t];
                    cv[t] = -sn * cv[t] + cs * nx[t];
                }
                nx[t] = nn[t];
            }
            if (zc && tid == 0) {
                const double zn = zc[j + 1];
                zc[j] = cs * zcar + sn * zn;
                zcar = -sn * zcar + cs * zn;
            }
            last = r;
            b = bn;
            __syncthreads();
        }
#pragma unroll
        for (int t = 0; t < DROP_COLS; ++t) {
            const int c = tid + NT * t;
            if (c < s) cbuf[c] = cv[t];
        }
        if (zc && tid == 0) zc[s - 1] = zcar;
        __syncthreads();
        return;
    }
    for (int c = tid; c < s; c += NT) cbuf[c] = c < q ? R[tri(q) + c] : 0.0;
    double last = R[tri(q) + q];
    double zcar = (zc && tid == 0) ? zc[q] : 0.0;
    __syncthreads();
    for (int j = q; j < s - 1; ++j) {
        const RP nx = R + tri(j + 1);
        const double b = nx[q];
        const double r = hypot(last, b);
        const double cs = r > 0.0 ? b / r : 1.0;
        const double sn = r > 0.0 ? -last / r : 0.0;
        RP out = R + tri(j);
        for (int c = tid; c <= j; c += NT) {     // columns past j stay zero in the moved column
            const double nxt = nx[c < q ? c : c + 1];
            const double cv = cbuf[c];
            out[c] = cs * cv + sn * nxt;
            cbuf[c] = -sn * cv + cs * nxt;
        }
        if (zc && tid == 0) {
            const double zn = zc[j + 1];
            zc[j] = cs * zcar + sn * zn;
            zcar = -sn * zcar + cs * zn;
        }
        last = r;
        __syncthreads();
    }
    if (zc && tid == 0) zc[s - 1] = zcar;
    __syncthreads();
}

template <int DROP_COLS>
__device__ __forceinline__ void chol_drop(const Sig& v, int s, int q, double* cbuf, double* zc)
{
    if (v.r_lds) chol_drop_t<DROP_COLS>(to_lds(v.R), s, q, cbuf, zc);
    else chol_drop_t<DROP_COLS>(to_global(v.R), s, q, cbuf, zc);
}

// The fold kernel's appends and drops beyond FOLD_MAX positions, out of line: inlined, they cost its hot loops registers.
__device__ __noinline__ int chol_append_far(Sig v, int nS, int j, signed char th, double* vw, double* vz, double* red,
                                            uint64_t* cnt)
{
    chol_append(v, nS, j, th, vw, vz, red, cnt);
    return nS;
}
__device__ __noinline__ void chol_drop_far(Sig v, int s, int q, double* cbuf, double* zc)
{
    chol_drop<4>(v, s, q, cbuf, zc);
}

// chol_drop for a factor in global memory (s <= 4 NT): the same rotations, eight rows per barrier.  The rotation of
// row j + 1 into row j needs b_j = R(j + 1, q) and the length of (R(q, q), b_q, .., b_{j-1}), both known before any
// row is touched: a wave takes 64 rows' lengths from a prefix sum of b^2, one lane per row (the chain of hypot and
// two divisions per row took as long as the row's memory access), and every column is then independent.  A thread
// reads columns of the next eight rows while it rotates these; a barrier between the arrival of eight rows and
// the first store into them keeps a wave from overwriting an entry that its neighbour, one column on, still reads
// (entry c of a row moves from column c + 1 for c >= q).  A row costs about 0.1 us (three reads of lane values and
// eight products per two columns); one barrier, one hypot and two divisions per row took 0.8 us: 99 us a drop on
// the ragged batch's supports, 21 us this way.
template <int DC>
__device__ __forceinline__ void chol_drop_rows(const Sig& v, int s, int q, double* cbuf, double* zc)
{
    constexpr int RB = 8;
    const int tid = threadIdx.x, lane = tid & 63;
    s = __builtin_amdgcn_readfirstlane(s);
    q = __builtin_amdgcn_readfirstlane(q);
    const RowBuffers rows(v.R);
    global_cdouble* R = to_global((const double*)v.R);
    double cv[DC];
    int src8[DC];                              // byte offset of this thread's source columns in a row
    {
        const auto rq = rows.row(q, false);
#pragma unroll
        for (int t = 0; t < DC; ++t) {
            const int c = tid + NT * t;
            src8[t] = 8 * (c < q ? c : c + 1);
            cv[t] = row_load(rq, 8 * c);
        }
#pragma unroll
        for (int t = 0; t < DC; ++t) cv[t] = tid + NT * t < q ? cv[t] : 0.0;
    }
    double last = R[tri(q) + q];               // signed; a length from the first rotation on
    double len2 = last * last;
    double zcar = zc ? zc[q] : 0.0;
    auto load = [&](int r0, double (&x)[RB][DC]) {   // rows r0 .. r0 + RB - 1, column q moved out, zero past the end
#pragma unroll
        for (int e = 0; e < RB; ++e) {
            const auto b = rows.row(r0 + e, r0 + e >= s);
#pragma unroll
            for (int t = 0; t < DC; ++t) x[e][t] = row_load(b, src8[t]);
        }
    };
    auto diag = [&](int j0) {                  // lane l: b of row j0 + l + 1
        const int r = j0 + lane + 1 < s ? j0 + lane + 1 : s - 1;
        return R[tri(r) + q];
    };
    double csl = 0.0, snl = 0.0, zl = 0.0, zout = 0.0;
    double bl = diag(q);
    auto rotate = [&](int j0, int l0, const double (&x)[RB][DC]) {   // rows j0 .. j0 + RB - 1, coefficients from lane l0
#pragma unroll
        for (int e = 0; e < RB; ++e)
#pragma unroll
            for (int t = 0; t < DC; ++t) asm volatile("" ::"v"(x[e][t]));   // arrived before the barrier
        __syncthreads();                       // every wave holds its entries of rows j0 + 1 .. j0 + RB
#pragma unroll
        for (int e = 0; e < RB; ++e) {
            const double cs = read_lane(csl, l0 + e), sn = read_lane(snl, l0 + e), zx = read_lane(zl, l0 + e);
            const auto b = rows.row(j0 + e, j0 + e >= s - 1);
#pragma unroll
            for (int t = 0; t < DC; ++t) {
                row_store(b, 8 * (tid + NT * t), cs * cv[t] + sn * x[e][t]);
                cv[t] = -sn * cv[t] + cs * x[e][t];   // columns past j: zero and zero
            }
            const double zj = cs * zcar + sn * zx;
            zcar = -sn * zcar + cs * zx;
            zout = lane == l0 + e ? zj : zout;
        }
    };
    double xa[RB][DC], xb[RB][DC];
    load(q + 1, xa);
    for (int j0 = q; j0 < s - 1; j0 += 64) {
        // coefficients of rows j0 .. j0 + 63; rows past s - 2 leave the carried column as it is
        const bool in = j0 + lane < s - 1;
        const double b = in ? bl : 0.0;
        zl = zc && in ? zc[j0 + lane + 1] : 0.0;
        double sum = b * b;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double up = __shfl_up(sum, o);
            sum += lane >= o ? up : 0.0;
        }
        sum += len2;
        const double r = sqrt(sum);
        const double prev = __shfl_up(r, 1);
        const double lst = lane == 0 ? last : prev;
        csl = in ? (r > 0.0 ? b / r : 1.0) : 0.0;
        snl = in ? (r > 0.0 ? -lst / r : 0.0) : -1.0;
        len2 = read_lane(sum, 63);
        last = read_lane(r, 63);
        bl = diag(j0 + 64);
        for (int l0 = 0; l0 < 64 && j0 + l0 < s - 1; l0 += 2 * RB) {
            load(j0 + l0 + RB + 1, xb);
            rotate(j0 + l0, l0, xa);
            load(j0 + l0 + 2 * RB + 1, xa);
            rotate(j0 + l0 + RB, l0 + RB, xb);
        }
        if (zc && tid < 64 && in) zc[j0 + lane] = zout;
    }
#pragma unroll
    for (int t = 0; t < DC; ++t) {
        const int c = tid + NT * t;
        if (c < s) cbuf[c] = cv[t];
    }
    __syncthreads();                           // every wave has read its zc entries and its rows
    if (zc && tid == 0) zc[s - 1] = zcar;
    __syncthreads();
}

// The sign-fixed minimiser after support positions s0..s1-1 were appended to the factor, from the cached
// z = Rinv w and x* = Rinv^T z of the positions before: the new factor is Rinv with rows s0..s1-1 added
// (its earlier rows unchanged), and w only gains the entries of the new positions (a member's sign does
// not change while it stays in S), so z gains the new rows' products with w and x* gains those rows'
// contributions: O((s1 - s0) s1) work instead of two passes over the factor.  vw: scratch.
template <class RP>
__device__ __forceinline__ void xstar_after_append_t(const RP R, const Sig& v, int s0, int s1, double lam, double* vw, double* vzc, double* vx)
{
    const int tid = threadIdx.x;
    for (int k = tid; k < s1; k += NT) {
        const int u = v.so[k];
        vw[k] = v.c[u] - lam * (double)v.th[u];
    }
    __syncthreads();
    // z of the new rows, a wave per row, four entries per lane in flight (clamped indices)
    const int lane = tid & 63, wave = tid >> 6;
    for (int p = s0 + wave; p < s1; p += NT / 64) {
        const RP Rp = R + tri(p);
        double part = 0.0;
        for (int k0 = lane; k0 <= p; k0 += 4 * 64) {
            double r[4], x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + 64 * e <= p ? k0 + 64 * e : p;
                r[e] = Rp[k];
                x[e] = vw[k];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) part += k0 + 64 * e <= p ? r[e] * x[e] : 0.0;
        }
        part = wave_sum(part);
        if (lane == 0) vzc[p] = part;
    }
    __syncthreads();
    for (int k = tid; k < s1; k += NT) {
        double acc = k < s0 ? vx[k] : 0.0;
        for (int p0 = k > s0 ? k : s0; p0 < s1; p0 += 8) {   // eight rows in flight
            double r[8], z[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int p = p0 + e < s1 ? p0 + e : s1 - 1;
                r[e] = R[tri(p) + k];
                z[e] = vzc[p];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += p0 + e < s1 ? r[e] * z[e] : 0.0;
        }
        vx[k] = acc;
    }
    __syncthreads();
}

__device__ __forceinline__ void xstar_after_append(const Sig& v, int s0, int s1, double lam, double* vw, double* vzc,
                                                   double* vx)
{
    if (v.r_lds) xstar_after_append_t(to_lds((const double*)v.R), v, s0, s1, lam, vw, vzc, vx);
    else xstar_after_append_t(to_global((const double*)v.R), v, s0, s1, lam, vw, vzc, vx);
}

// x_S = Rinv^T Rinv (c_S - lambda theta_S) into vx[0..nS).
template <bool FOLD>
__device__ __forceinline__ void sign_fixed_solve(const Sig& v, int nS, double lam, double* vw, double* vz, double* vx)
{
    const int tid = threadIdx.x;
    for (int k = tid; k < nS; k += NT) {
        const int u = v.so[k];
        vw[k] = v.c[u] - lam * (double)v.th[u];
    }
    __syncthreads();
    if (FOLD && !v.r_lds && nS <= FOLD_MAX) {   // one pass over a global factor
        fold_pass_global(v.R, vw, nS, vx, vz);
        return;
    }
    if (v.r_lds) {
        rows_matvec_lds(v.R, vw, vz, nS);
    } else {
        rows_matvec_global(v.R, vw, vz, nS);
    }
    __syncthreads();
    if (v.r_lds)
        cols_matvec_lds(v.R, vz, vx, nS, 1.0);
    else
        for (int k = tid; k < nS; k += NT) vx[k] = col_dot(v, vz, k, nS);
    __syncthreads();
}

// g_u = c_u - G_uS x_S for the slots u < nI (all of them, or only those outside S
// that may still enter it).  A row of 16 lanes takes two slots at a time and splits their support
// entries (G is global, so a slot costs one round trip with its loads in flight rather than a chain of
// |S| / 8), then sums each row by DPP moves inside the row.  (Reading the rows contiguously over all
// slots of I against x by slot was measured slower on large active sets: |I| / |S| times the entries.)
// DEPTH support entries per lane and slot are in flight at once (8 in the kernel without a register cap).
template <int DEPTH>
__device__ __forceinline__ void grad_slots(const Sig& v, int nI, int nS, double* vg, bool outside_only)
{
    constexpr int GL = 16, NG = NT / GL;
    const int sub = threadIdx.x & (GL - 1), grp = threadIdx.x / GL;
    for (int u0 = grp; u0 < nI; u0 += 2 * NG) {
        const int u1 = u0 + NG;
        const bool d0 = !(outside_only && (v.th[u0] != 0 || v.ex[u0]));
        const bool d1 = u1 < nI && !(outside_only && (v.th[u1] != 0 || v.ex[u1]));
        if (!d0 && !d1) continue;       // the same decision for the whole row of lanes
        const double* G0 = v.G + (int64_t)u0 * v.K;
        const double* G1 = v.G + (int64_t)(d1 ? u1 : u0) * v.K;
        double a0 = 0.0, a1 = 0.0;
        for (int k0 = sub; k0 < nS; k0 += GL * DEPTH) {
            double g0[DEPTH], g1[DEPTH], xv[DEPTH];
            // clamped positions: every load is issued (a guarded one would wait at its branch's end);
            // positions past nS count zero through xv
#pragma unroll
            for (int e = 0; e < DEPTH; ++e) {
                const int k = k0 + GL * e;
                const int sk = v.so[k < nS ? k : nS - 1];
                g0[e] = G0[sk];
                g1[e] = G1[sk];
                xv[e] = v.x[sk];
            }
#pragma unroll
            for (int e = 0; e < DEPTH; ++e) {
                const bool in = k0 + GL * e < nS;
                g0[e] = in && d0 ? g0[e] : 0.0;
                g1[e] = in && d1 ? g1[e] : 0.0;
                xv[e] = in ? xv[e] : 0.0;
            }
#pragma unroll
            for (int e = 0; e < DEPTH; ++e) {
                a0 += g0[e] * xv[e];
                a1 += g1[e] * xv[e];
            }
        }
        a0 = row16_sum(a0);
        a1 = row16_sum(a1);
        if (sub == 0) {
            if (d0) vg[u0] = v.c[u0] - a0;
            if (d1) vg[u1] = v.c[u1] - a1;
        }
    }
    __syncthreads();
}

// Element i of a global array that a generic pointer (the same in every thread) points into.
template <class T>
__device__ __forceinline__ T gld(const T* p, int64_t i)
{
    typedef __attribute__((address_space(1))) const T gT;
    return reinterpret_cast<gT*>(const_cast<gT*>(reinterpret_cast<gT*>(to_global(reinterpret_cast<const double*>(p)))))[i];
}
template <class T>
__device__ __forceinline__ void gst(T* p, int64_t i, T x)
{
    typedef __attribute__((address_space(1))) T gT;
    reinterpret_cast<gT*>(to_global(reinterpret_cast<double*>(p)))[i] = x;
}

// grad_slots for the fold kernel with the per-slot vectors in global memory (|S| <= GF_MS NT,
// |I| <= GF_MU NT): the same gradients, organised around the dependent gather G(u, so[k]).  Every
// thread reads the slot and coefficient of its support positions (tid + NT m) once; the slots that
// need a gradient are listed in slot order (list: nI ints of global scratch, written through wave
// ballots); the list is taken GF_B slots at a time: one round trip gathers every thread's entries of
// those rows (the next batch's slot numbers already in flight), the partial sums meet in LDS
// (double-buffered, added in wave order) and thread i writes slot i's gradient.  grad_slots takes a
// slot's support entries 16 lanes at a time, a slot-number load and then the gathers for every 64
// entries, so its round trips grow with |S|.  Ends with a barrier.
constexpr int GF_MS = 4, GF_MU = 8, GF_B = 4;

__device__ __forceinline__ void grad_fold(const Sig& v, int nI, int nS, double* vg, bool outside_only, int* list)
{
    __shared__ double part[2][NT / 64][GF_B];
    __shared__ int wcnt[NT / 64][GF_MU];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    nI = __builtin_amdgcn_readfirstlane(nI);
    nS = __builtin_amdgcn_readfirstlane(nS);
    if (nI == 0) {
        __syncthreads();
        return;
    }
    global_cdouble* G = to_global(v.G);
    const int64_t K = v.K;
    // this thread's support positions: slot and coefficient (zero past nS)
    int sk[GF_MS];
    double xs[GF_MS];
#pragma unroll
    for (int m = 0; m < GF_MS; ++m) {
        const int k = tid + NT * m;
        sk[m] = nS > 0 ? gld(v.so, k < nS ? k : nS - 1) : 0;
    }
#pragma unroll
    for (int m = 0; m < GF_MS; ++m) xs[m] = gld(v.x, sk[m]);
#pragma unroll
    for (int m = 0; m < GF_MS; ++m) xs[m] = tid + NT * m < nS ? xs[m] : 0.0;
    // the slots that need a gradient, listed in the order (m, wave, lane) = slot order
    unsigned need = 0;
#pragma unroll
    for (int m = 0; m < GF_MU; ++m) {
        const int u = tid + NT * m;
        const int uc = u < nI ? u : nI - 1;
        const signed char th = gld(v.th, uc);
        const unsigned char ex = gld(v.ex, uc);
        need |= (u < nI && (!outside_only || (th == 0 && !ex))) ? 1u << m : 0u;
    }
    unsigned long long bal[GF_MU];
#pragma unroll
    for (int m = 0; m < GF_MU; ++m) bal[m] = __ballot((need >> m) & 1);
    if (lane == 0) {
#pragma unroll
        for (int m = 0; m < GF_MU; ++m) wcnt[wave][m] = __popcll(bal[m]);
    }
    __syncthreads();
    int ncand = 0;
#pragma unroll
    for (int m = 0; m < GF_MU; ++m) {
        int off = ncand;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) {
            off += w < wave ? wcnt[w][m] : 0;
            ncand += wcnt[w][m];
        }
        if ((need >> m) & 1) {
            const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(bal[m] >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((unsigned)bal[m], 0));
            gst(list, off + rank, tid + NT * m);
        }
    }
    ncand = __builtin_amdgcn_readfirstlane(ncand);
    __syncthreads();
    int nx[GF_B];
#pragma unroll
    for (int i = 0; i < GF_B; ++i) nx[i] = gld(list, i < ncand ? i : ncand - 1);
    int buf = 0;
    for (int b = 0; b < ncand; b += GF_B) {
        int us[GF_B];
#pragma unroll
        for (int i = 0; i < GF_B; ++i) us[i] = __builtin_amdgcn_readfirstlane(nx[i]);
#pragma unroll
        for (int i = 0; i < GF_B; ++i) {
            const int e = b + GF_B + i;
            nx[i] = gld(list, e < ncand ? e : ncand - 1);
        }
        double cu[GF_B], gv[GF_B][GF_MS];
#pragma unroll
        for (int i = 0; i < GF_B; ++i) {
            cu[i] = gld(v.c, us[i]);
            global_cdouble* Gu = G + us[i] * K;
#pragma unroll
            for (int m = 0; m < GF_MS; ++m) gv[i][m] = Gu[sk[m]];
        }
        double pq[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < GF_B; ++i) {
            double acc = 0.0;
#pragma unroll
            for (int m = 0; m < GF_MS; ++m) acc += gv[i][m] * xs[m];
            pq[i] = acc;
        }
        const double mine = wave_sum8(pq);       // lane l holds the wave's sum for slot wave_sum8_index(l)
        if (lane < 8 && wave_sum8_index(lane) < GF_B) part[buf][wave][wave_sum8_index(lane)] = mine;
        __syncthreads();
        if (tid < GF_B && b + tid < ncand) {
            int u = us[0];
            double c = cu[0];
#pragma unroll
            for (int i = 1; i < GF_B; ++i) {
                u = tid == i ? us[i] : u;
                c = tid == i ? cu[i] : c;
            }
            double sum = part[buf][0][tid];
#pragma unroll
            for (int w = 1; w < NT / 64; ++w) sum += part[buf][w][tid];
            gst(vg, u, c - sum);
        }
        buf ^= 1;
    }
    __syncthreads();
}

// Gram rows G(q, u) of the new slots q against every slot u, and c_q = a_q^T b,
// as n-long float64 dot products (used when no Gram table is available).  The
// new atoms are staged through LDS in chunks (s_new: CH x NB doubles of the launch's dynamic
// LDS, present only when there is no table); each thread owns one slot u.
static_assert(CH * NB * 8 == GRAM_STAGE_BYTES, "direct Gram staging size");
__device__ __forceinline__ void gram_rows_direct(const SolveArgs& a, Sig& s, const int* g_atom, const float* bw, int nI0,
                                 int nnew, int nI, double* s_new)
{
    const int tid = threadIdx.x;
    const int kpad = a.w.kpad;
    const int K = s.K;
    for (int g0 = 0; g0 < nnew; g0 += NB) {
        const int nb = nnew - g0 < NB ? nnew - g0 : NB;
        for (int ub = 0; ub <= nI; ub += NT) {
            const int u = ub + tid;
            const bool live = u <= nI;
            const float* col = (u < nI) ? a.At + (int64_t)g_atom[u] * a.lda : bw;
            double acc[NB];
#pragma unroll
            for (int t = 0; t < NB; ++t) acc[t] = 0.0;
            for (int kc = 0; kc < kpad; kc += CH) {
                __syncthreads();
                for (int e = tid; e < nb * CH; e += NT) {
                    const int t = e / CH, kk = e % CH;
                    const int atom = g_atom[nI0 + g0 + t];
                    s_new[kk * NB + t] = (kc + kk < kpad) ? (double)a.At[(int64_t)atom * a.lda + kc + kk] : 0.0;
                }
                __syncthreads();
                if (live) {
                    const int kend = (kpad - kc) < CH ? (kpad - kc) : CH;
                    for (int kk = 0; kk < kend; kk += 4) {
                        const float4 f = *reinterpret_cast<const float4*>(col + kc + kk);
                        const double fv[4] = {(double)f.x, (double)f.y, (double)f.z, (double)f.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const double* sn = s_new + (kk + e) * NB;
#pragma unroll
                            for (int t = 0; t < NB; ++t)
                                if (t < nb) acc[t] += fv[e] * sn[t];
                        }
                    }
                }
            }
            if (live) {
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    if (t >= nb) break;
                    const int q = nI0 + g0 + t;
                    if (u == nI) {
                        s.c[q] = acc[t];
                    } else {
                        s.G[(int64_t)q * K + u] = acc[t];
                        s.G[(int64_t)u * K + q] = acc[t];
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Master problem on I for every running signal, then its residual and objective.
//
// Working set: the inverse factor Rinv and the per-slot vectors live in LDS
// when they fit (copied in at entry, written back at exit), otherwise they are
// used in place in global memory.  G_II (row-major, stride K) stays global.
// The kernels of pursuit.h share the body.  Appends: chol_append_lds with a factor in LDS, chol_append_fold with one
// in global memory, chol_append_block (BLOCK) with one in global memory and a scratch in LDS.
// ---------------------------------------------------------------------------
// Residual xi = b - A_S x_S (float64 accumulation, stored float32) and the objective
// lambda ||x||_1 + 1/2 ||xi||^2 of a signal that was just solved (step 7 of Algorithm 1), with the
// norms and reduced-precision copies the next product and its screening band use.  Run by the solve
// workgroup after its write-back: sx / satom hold the support's values and atoms (LDS), xl1 = ||x||_1.
// Four rows per thread, eight atoms' loads in flight, straight from the atom-major dictionary; a
// workgroup that finishes its master problem early computes its residual while others still solve.
__device__ __forceinline__ void residual_tail(const Workspace& w, int sig, const float* At, int64_t lda, const float* Bw,
                              const double* sx, const int* satom, int nS, double xl1, double* red)
{
    const int tid = threadIdx.x;
    const float* bw = Bw + (int64_t)sig * w.kpad;
    float* Rres = w.R + (int64_t)sig * w.kpad;
    double rr = 0.0, dr = 0.0;
    // rows 4 q .. 4 q + 3 per step (kpad and lda are multiples of 4)
    const int n4 = w.kpad / 4;
    const int64_t lda4 = lda / 4;
    const float4* At4 = reinterpret_cast<const float4*>(At);
    constexpr int CH = 8;
    for (int q = tid; q < n4; q += NT) {
        const float4 bv = reinterpret_cast<const float4*>(bw)[q];
        double acc[4] = {(double)bv.x, (double)bv.y, (double)bv.z, (double)bv.w};
        for (int k = 0; k < nS; k += CH) {        // past nS the last atom again, times zero
            float4 f[CH];
#pragma unroll
            for (int e = 0; e < CH; ++e) f[e] = At4[(int64_t)satom[k + e < nS ? k + e : nS - 1] * lda4 + q];
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                const double xv = k + e < nS ? sx[k + e] : 0.0;
                acc[0] -= (double)f[e].x * xv;
                acc[1] -= (double)f[e].y * xv;
                acc[2] -= (double)f[e].z * xv;
                acc[3] -= (double)f[e].w * xv;
            }
        }
        float4 out;
        float* o = reinterpret_cast<float*>(&out);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 4 * q + e;
            if (r >= w.n) acc[e] = 0.0;
            o[e] = (float)acc[e];
            if (w.R16) {
                const uint16_t h = bf16_round(o[e]);
                w.R16[(int64_t)sig * w.kpad + r] = h;
                const double d = (double)bf16_value(h) - (double)o[e];
                dr += d * d;
            }
            rr += acc[e] * acc[e];
        }
        reinterpret_cast<float4*>(Rres)[q] = out;
    }
    const double rn = block_sum(rr, red);
    const double rd = w.R16 ? block_sum(dr, red) : 0.0;
    if (tid == 0) {
        w.obj_prev[sig] = w.obj[sig];
        w.obj[sig] = 0.5 * rn + w.lam[sig] * xl1;
        w.rr2[sig] = rn;
        if (w.rnorm) w.rnorm[sig] = sqrt(rn);
        if (w.dxnorm) w.dxnorm[sig] = sqrt(rd);
    }
    if (w.R8) write_residual_fp8(w, sig, red);
}

// VEC: the vectors' memory, 1 LDS, 2 global, 0 by a.vec_lds.
template <bool BLOCK, bool FOLD, int VEC>
__device__ __forceinline__ void solve_body(const SolveArgs& a)
{
    // As a constant it lets the compiler address the vectors as what they are; a pointer to either memory takes flat
    // instructions, which wait on both counters and compute 64-bit addresses.
    const bool vec_lds = VEC == 0 ? a.vec_lds != 0 : VEC == 1;
    extern __shared__ double s_dyn[];
    __shared__ double red[4];
    __shared__ int redi[4];
    __shared__ int s_list[NT];
    __shared__ int s_cnt;

    const int n_act = *a.n_act_dev;
    const int row = blockIdx.x;
    if (row >= n_act) return;
    const Workspace& w = a.w;
    const int sig = a.act[row];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nnew = w.nsel[sig];
    if (nnew <= 0) return;
    const int nI0 = w.nI[sig];
    int nS = w.nS[sig];
    const double lam = w.lam[sig];
    int nI = nI0 + nnew;
    if (vec_lds && nI > a.kv) {
        // the launch was sized for a smaller |I| (a host-side bound that does not hold): stop the signal
        // at its current iterate, reported inexact, rather than overrun the LDS vectors
        if (tid == 0) w.status[sig] |= BMPL_SIG_INEXACT | ST_HALT;
        return;
    }

    // The signal's slot block (grown by grow_kernel before this launch); a block that could not grow
    // (no arena room) leaves the signal untouched: the host adds room and the next outer iteration
    // selects the same atoms again.
    const int K = w.cap[sig];
    if (nI > K) return;
    double* base = (double*)to_global(w.blk[sig]);   // global for the compiler too
    const SlotBlock hb = slot_block(base, K, w.n);
    const int max_steps = a.max_steps_per_slot * K + 256;
    uint64_t tick = a.phase ? wall_clock64() : 0;

    // global homes of this signal's state
    int* g_atom = hb.atom;
    double* g_x = hb.x;
    double* g_c = hb.c;
    signed char* g_th = hb.theta;
    unsigned char* g_ex = hb.excl;
    int* g_so = hb.sord;
    double* g_R = hb.Rinv;

    Sig s;
    s.K = K;
    // The LDS factor holds up to a.kl support positions; a signal whose support outgrows it moves its
    // factor to the global home and continues there (spill_factor below).
    s.r_lds = !FOLD && a.rinv_lds != 0 && nS <= a.kl;
    s.G = hb.G;
    char* lp = reinterpret_cast<char*>(s_dyn);
    if (a.rinv_lds) {
        s.R = s.r_lds ? reinterpret_cast<double*>(lp) : g_R;
        lp += sizeof(double) * tri(a.kl);
    } else {
        s.R = g_R;
    }
    double *vw, *vz, *vx, *vg;
    double* vzc;   // cached z = Rinv w of the sign-fixed solve, by position (x* is in vx)
    int* vatom;
    const int KV = a.kv;                      // LDS vectors by slot: KV >= |I| during this launch
    const int KP = a.kp;                      // by support position: |S| <= min(|I|, n) <= KP
    if (vec_lds) {
        double* d = reinterpret_cast<double*>(lp);
        s.x = d; s.c = d + KV; vg = d + 2 * KV;
        vw = d + 3 * KV; vz = vw + KP; vx = vz + KP; vzc = vx + KP;
        int* ip = reinterpret_cast<int*>(vzc + KP);
        s.so = ip; vatom = ip + KP;
        s.th = reinterpret_cast<signed char*>(vatom + KV);
        s.ex = reinterpret_cast<unsigned char*>(s.th + KV);
    } else {
        double* d = hb.vs;
        s.x = g_x; s.c = g_c; s.th = g_th; s.ex = g_ex; s.so = g_so;
        vw = d; vz = d + K; vx = d + 2 * K; vg = d + 3 * K;
        vatom = reinterpret_cast<int*>(d + 4 * K);
        vzc = d + 5 * K;
    }
    // the gradients' slot list (grad_fold), in the unused end of the global vector scratch
    int* glist = vec_lds ? nullptr : reinterpret_cast<int*>(hb.vs + 6 * (int64_t)K);
    // block-append scratch after the vectors (K rows of JB doubles), when the launch provided it
    double* zs = (BLOCK && a.zs_lds) ? reinterpret_cast<double*>(lp + (vec_lds ? vec_area_bytes(KV, KP) : 0)) : nullptr;
    // direct Gram staging (no table) after the vectors and the block scratch
    double* snew = a.Q ? nullptr
                       : reinterpret_cast<double*>(lp + (vec_lds ? vec_area_bytes(KV, KP) : 0) +
                                                   (a.zs_lds ? block_scratch_bytes(KP) : 0));

    // 1. Load the state, register the new slots.
    if (vec_lds) {
        for (int u = tid; u < nI0; u += NT) {
            s.x[u] = g_x[u]; s.c[u] = g_c[u]; s.th[u] = g_th[u]; s.ex[u] = g_ex[u];
        }
        for (int k = tid; k < nS; k += NT) s.so[k] = g_so[k];
    }
    if (s.r_lds) {   // eight loads in flight per thread
        const int64_t T = tri(nS);
        for (int64_t e0 = tid; e0 < T; e0 += 8 * NT) {
            double r[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) r[q] = g_R[e0 + q * NT < T ? e0 + q * NT : T - 1];   // clamped
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (e0 + q * NT < T) s.R[e0 + q * NT] = r[q];
        }
    }
    for (int u = tid; u < nI0; u += NT) vatom[u] = g_atom[u];
    for (int t = tid; t < nnew; t += NT) {
        const int q = nI0 + t;
        const int atom = w.sel[(int64_t)sig * w.selcap + t];
        g_atom[q] = atom;
        vatom[q] = atom;
        s.x[q] = 0.0;
        s.th[q] = 0;
        s.ex[q] = 0;
        atomicOr(&w.inI[(int64_t)sig * w.words + (atom >> 5)], 1u << (atom & 31));
    }
    __syncthreads();

    // Optional per-phase wall-clock ticks (kernel timing mode): load, Gram, active set,
    // certificate, (appends), write-back; the residual's ticks go to slot 14.
    auto phase_mark = [&](int ph) {
        if (a.phase && tid == 0) {
            const uint64_t now = wall_clock64();
            atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + ph), (unsigned long long)(now - tick));
            tick = now;
        }
    };
    phase_mark(0);
    // time spent in one call of a step of the active-set loop, summed into phase slot `slot`
    auto sub_ticks = [&](int slot, uint64_t t0) {
        if (a.phase && tid == 0)
            atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + slot), (unsigned long long)(wall_clock64() - t0));
    };

    // 2. Gram rows of the new slots and c = A_J^T b, in float64.  With many new slots (a warm start)
    //    the Gram matrix is kept lazily from then on: a new slot's row only against the support
    //    members and itself, and a slot's whole column when it enters S (gather_cols below), which is
    //    every entry the solver reads.  Most proposed slots never enter S.
    const float* bw = a.Bw + (int64_t)sig * w.kpad;
    const bool lazy = a.Q && (w.glazy[sig] != 0 || nnew > LAZY_MIN);
    if (a.Q && lazy) {
        if (tid == 0) w.glazy[sig] = 1;
        const int span = nS + 1;                  // support positions, then the diagonal
        const int tot = nnew * span;
        for (int e0 = tid; e0 < tot; e0 += 4 * NT) {
            double val[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {   // clamped entry index: all four reads issued together
                const int e = e0 + r * NT < tot ? e0 + r * NT : tot - 1;
                const int t = e / span, k = e - t * span;
                const int u = k < nS ? s.so[k] : nI0 + t;
                val[r] = a.Q[(int64_t)vatom[nI0 + t] * a.ldq + vatom[u]];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = e0 + r * NT;
                if (e < tot) {
                    const int t = e / span, k = e - t * span;
                    const int q = nI0 + t;
                    const int u = k < nS ? s.so[k] : q;
                    s.G[(int64_t)q * K + u] = val[r];
                    s.G[(int64_t)u * K + q] = val[r];
                }
            }
        }
    } else if (a.Q) {
        // four table reads per thread in flight before the symmetric stores
        const int tot = nnew * nI;
        for (int e0 = tid; e0 < tot; e0 += 4 * NT) {
            double val[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {   // clamped entry index: all four reads issued together
                const int e = e0 + r * NT < tot ? e0 + r * NT : tot - 1;
                const int t = e / nI, u = e - t * nI;
                val[r] = a.Q[(int64_t)vatom[nI0 + t] * a.ldq + vatom[u]];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = e0 + r * NT;
                if (e < tot) {
                    const int t = e / nI, u = e - t * nI;
                    const int q = nI0 + t;
                    s.G[(int64_t)q * K + u] = val[r];
                    s.G[(int64_t)u * K + q] = val[r];
                }
            }
        }
    }
    if (a.Q) {
        // c_q = a_q^T b: two new atoms per wave at a time, float4 loads, all issued before the sums
        constexpr int NA = 2;
        for (int t = NA * wave; t < nnew; t += NA * (NT / 64)) {
            const float4* aj[NA];
#pragma unroll
            for (int h = 0; h < NA; ++h)          // (past nnew the last atom again)
                aj[h] = reinterpret_cast<const float4*>(a.At + (int64_t)vatom[nI0 + min(t + h, nnew - 1)] * a.lda);
            const float4* b4 = reinterpret_cast<const float4*>(bw);
            double acc[NA] = {};
            const int n4 = w.kpad / 4;
            for (int k0 = lane; k0 < n4; k0 += 64 * 4) {
                float4 fa[NA][4], fb[4];
                // inside the vectors for the whole wave: no branch, so the loads are in flight together
                if (k0 - lane + 64 * 4 <= n4) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
#pragma unroll
                        for (int h = 0; h < NA; ++h) fa[h][e] = aj[h][k0 + 64 * e];
                        fb[e] = b4[k0 + 64 * e];
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {   // clamped, and zero past the end through b
                        const int k = min(k0 + 64 * e, n4 - 1);
#pragma unroll
                        for (int h = 0; h < NA; ++h) fa[h][e] = aj[h][k];
                        fb[e] = b4[k];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (k0 + 64 * e >= n4) fb[e] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int h = 0; h < NA; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[h] += (double)fa[h][e].x * fb[e].x + (double)fa[h][e].y * fb[e].y +
                                  (double)fa[h][e].z * fb[e].z + (double)fa[h][e].w * fb[e].w;
            }
#pragma unroll
            for (int h = 0; h < NA; ++h) {
                acc[h] = wave_sum(acc[h]);
                if (lane == 0 && t + h < nnew) s.c[nI0 + t + h] = acc[h];
            }
        }
    } else {
        gram_rows_direct(a, s, g_atom, bw, nI0, nnew, nI, snew);
    }
    __syncthreads();

    phase_mark(1);

    // 3. Sign-fixed active-set iterations (twice with subspace exploratory matching: on I u J_omega,
    //    then, after the pruning below, on I_t).
    int steps = 0;
    bool inexact = false;
    bool explored = false;
    bool resolve = false;   // after the pruning: solve on I_t even if no slot outside S violates
    // Violators admitted per step, adapted to the dictionary and carried from one outer iteration to
    // the next: doubled (up to JADD) after a step whose move to the sign-fixed minimiser dropped nothing;
    // on a small support (|S| < 128) halved after one that dropped at least a quarter as many atoms as it
    // admitted (correlated atoms that enter and leave together); otherwise trimmed by an eighth (by one
    // below 8): a large, nearly saturated support sees drops at almost every step, and each admission
    // saved there is a pass over a factor of hundreds of rows.
    int jadd = w.jadd[sig];
    jadd = jadd >= 1 && jadd <= JADD ? jadd : JADD0;
    // the sign-fixed minimiser x* (vx) and z = Rinv w (vzc) are computed in full once, then kept current
    // through appends (xstar_after_append) and drops (rotated z, and x* from the removed row)
    bool xs_ok = false;
    // the last pass of the loop computes the gradient on all of I for the certificate (one call site of
    // the gradient routine: each inlined copy costs the kernel registers)
    bool cert = false;
active_set:
    for (;;) {
        const uint64_t tg = a.phase ? wall_clock64() : 0;
        if (FOLD && VEC == 2 && nI <= GF_MU * NT && nS <= GF_MS * NT) grad_fold(s, nI, nS, vg, !cert, glist);
        else grad_slots<FOLD ? 16 : (BLOCK ? 8 : 4)>(s, nI, nS, vg, !cert);
        sub_ticks(11, tg);
        if (cert) break;
        const uint64_t tv = a.phase ? wall_clock64() : 0;
        if (wave == 0) {    // violators outside S, in slot order
            int base = 0;
            for (int u0 = 0; u0 < nI && base < NT; u0 += 64) {
                const int u = u0 + lane;
                bool viol = false;
                if (u < nI && s.th[u] == 0 && !s.ex[u])
                    viol = fabs(vg[u]) > lam * (1.0 + 1e-12) && fabs(vg[u]) > 0.0;
                const unsigned long long bal = __ballot(viol);
                const int pre = __popcll(bal & ((1ull << lane) - 1ull));
                if (viol && base + pre < NT) s_list[base + pre] = u;
                base += __popcll(bal);
            }
            if (lane == 0) s_cnt = base < NT ? base : NT;
        }
        __syncthreads();
        int nv = s_cnt;
        if (nv == 0 && !resolve) {
            cert = true;
            continue;
        }
        resolve = false;
        if (nv > jadd) {
            // keep the jadd largest violations (ties to the lower slot), in slot order: adding a few at a
            // time keeps sign changes, and with them drops, rare when many atoms of I violate at once
            int u = -1, rank = 0;
            double gu = 0.0;
            if (tid < nv) {
                u = s_list[tid];
                gu = fabs(vg[u]);
                for (int e = 0; e < nv; ++e) {
                    const int o = s_list[e];
                    const double go = fabs(vg[o]);
                    rank += (go > gu) || (go == gu && o < u);
                }
            }
            __syncthreads();
            const bool keep = tid < nv && rank < jadd;
            // compact the kept slots in slot order (s_list is in slot order)
            const unsigned long long bal = __ballot(keep);
            if (lane == 0) redi[wave] = __popcll(bal);
            __syncthreads();
            int before = 0;
            for (int w2 = 0; w2 < wave; ++w2) before += redi[w2];
            if (keep) s_list[before + __popcll(bal & ((1ull << lane) - 1ull))] = u;
            __syncthreads();
            nv = jadd;
        }
        sub_ticks(12, tv);
        if (lazy && nv > 0) {
            // lazy Gram: the columns of the slots about to enter S, against every slot of I
            const int tot = nv * nI;
            for (int e0 = tid; e0 < tot; e0 += 4 * NT) {
                double val[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {   // clamped entry index: all four reads issued together
                    const int e = e0 + r * NT < tot ? e0 + r * NT : tot - 1;
                    const int t = e / nI, u2 = e - t * nI;
                    val[r] = a.Q[(int64_t)g_atom[s_list[t]] * a.ldq + g_atom[u2]];
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = e0 + r * NT;
                    if (e < tot) {
                        const int t = e / nI, u2 = e - t * nI;
                        const int j = s_list[t];
                        s.G[(int64_t)j * K + u2] = val[r];
                        s.G[(int64_t)u2 * K + j] = val[r];
                    }
                }
            }
            __syncthreads();
        }
        if (s.r_lds && nS + nv > a.kl) {
            // the support outgrows the LDS factor: move it to the global home and continue there
            for (int64_t e = tid; e < tri(nS); e += NT) g_R[e] = s.R[e];
            __syncthreads();
            s.R = g_R;
            s.r_lds = false;
        }
        const int nS_before = nS;
        if (nv == 0) {
            // nothing to append: the pruned problem on I_t is solved from u restricted to it
        } else if (zs) {
            append_list(s, nS, s_list, nv, vg, w.n, zs, a.phase ? a.phase + 6 : nullptr);
        } else {
            int e = 0;
            if (FOLD && !s.r_lds) {
                __shared__ FoldLds w_fold;
                const uint64_t t_in = a.phase ? wall_clock64() : 0;
                const int e0 = e, top = min(w.n, FOLD_MAX);
                while (nS < top) {
                    // the minimiser of the support before comes with the first pass when it isn't known yet
                    const bool xs = !xs_ok && nS > 0;
                    const int J = min(min(nv - e, xs ? 7 : 8), top - nS);
                    if (J < 1) break;
                    if (nS + J <= 2 * NT) chol_append_fold<2>(s, nS, s_list + e, J, vg, xs, lam, vzc, vx, w_fold);
                    else chol_append_fold<4>(s, nS, s_list + e, J, vg, xs, lam, vzc, vx, w_fold);
                    e += J;
                    xs_ok = xs_ok || xs;
                }
                if (a.phase && tid == 0) {
                    atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + 6), (unsigned long long)(e - e0));
                    atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + 4), (unsigned long long)(wall_clock64() - t_in));
                }
            }
            if (!FOLD && !BLOCK && NT > 64 && s.r_lds) {
                const uint64_t t_in = a.phase ? wall_clock64() : 0;
                while (nS < w.n) {
                    // the minimiser of the support before comes with the first block when it isn't known yet
                    const bool xs = !xs_ok && nS > 0;
                    const int J = min(min(nv - e, xs ? 7 : 8), w.n - nS);
                    if (J < 1) break;
                    chol_append_lds<8>(s, nS, s_list + e, J, vg, xs, lam, vzc, vx);
                    e += J;
                    xs_ok = xs_ok || xs;
                }
                if (a.phase && tid == 0) {
                    atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + 6), (unsigned long long)e);
                    atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + 4), (unsigned long long)(wall_clock64() - t_in));
                }
            }
            for (; e < nv; ++e) {
                const int u = s_list[e];
                const signed char th = vg[u] > 0.0 ? 1 : -1;
                if (nS >= w.n) {
                    if (tid == 0) s.ex[u] = 1;
                    __syncthreads();
                    continue;
                }
                if (FOLD) nS = chol_append_far(s, nS, u, th, vw, vz, red, a.phase ? a.phase + 6 : nullptr);
                else chol_append(s, nS, u, th, vw, vz, red, a.phase ? a.phase + 6 : nullptr);
            }
        }
        if (xs_ok && nS > nS_before) {
            const uint64_t tsf = a.phase ? wall_clock64() : 0;
            xstar_after_append(s, nS_before, nS, lam, vw, vzc, vx);
            sub_ticks(10, tsf);
        }
        const int added = nS - nS_before;
        // move toward the sign-fixed minimiser, dropping at zero crossings
        int dropped = 0;
        for (;;) {
            if (++steps > max_steps) { inexact = true; break; }
            if (!xs_ok) {
                const uint64_t tsf = a.phase ? wall_clock64() : 0;
                sign_fixed_solve<FOLD>(s, nS, lam, vw, vzc, vx);
                sub_ticks(10, tsf);
                xs_ok = true;
            }
            if (a.phase && tid == 0) atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + 8), 1ull);
            const uint64_t tr = a.phase ? wall_clock64() : 0;
            double alpha = 1.0;
            int q = -1;
            for (int k = tid; k < nS; k += NT) {
                const int u = s.so[k];
                const double xo = s.x[u], xn = vx[k], th = (double)s.th[u];
                if (xn * th <= 0.0) {
                    const double ak = (xo == 0.0) ? 0.0 : fmax(xo / (xo - xn), 0.0);
                    if (ak < alpha || (ak == alpha && (q < 0 || k < q))) { alpha = ak; q = k; }
                }
            }
            block_argmin(alpha, q, red, redi);
            for (int k = tid; k < nS; k += NT) {
                const int u = s.so[k];
                const double xo = s.x[u];
                s.x[u] = xo + alpha * (vx[k] - xo);
            }
            __syncthreads();
            sub_ticks(13, tr);
            if (q < 0) break;
            // the atom admitted alone blocks at alpha = 0: a numerically void admission (EX_PASS)
            const bool void_admit = alpha == 0.0 && dropped == 0 && nS == nS_before + 1 && q == nS_before;
            ++dropped;
            // drop position q: downdate the factor (or truncate it and append the later positions again)
            if (a.phase && tid == 0) atomicAdd(reinterpret_cast<unsigned long long*>(a.phase + 7), 1ull);
            const int ns_old = nS;
            for (int k = tid; k < ns_old; k += NT) vatom[k] = s.so[k];
            __syncthreads();
            if (tid == 0) {
                const int u = vatom[q];
                s.x[u] = 0.0;
                s.th[u] = 0;
                if (void_admit) s.ex[u] = EX_PASS;
            }
            __syncthreads();
            // downdate the factor in place (vw is free scratch here); support positions past q move down
            const uint64_t td = a.phase ? wall_clock64() : 0;
            if (FOLD && ns_old <= 2 * NT) chol_drop_rows<2>(s, ns_old, q, vw, vzc);
            else if (FOLD && ns_old <= 4 * NT) chol_drop_rows<4>(s, ns_old, q, vw, vzc);
            else if (FOLD) chol_drop_far(s, ns_old, q, vw, vzc);
            else chol_drop<BLOCK ? 8 : 4>(s, ns_old, q, vw, vzc);
            // x* on S \ q: with the removed row b (vw) and its z entry zl, x*_new[k] = x*[k'] - b_k zl
            // (k' the position before the shift)
            {
                const double zl = vzc[ns_old - 1];
                for (int k = tid; k < ns_old - 1; k += NT) vz[k] = vx[k < q ? k : k + 1] - vw[k] * zl;
                double* t = vx; vx = vz; vz = t;
            }
            sub_ticks(9, td);
            for (int k = q + 1 + tid; k < ns_old; k += NT) s.so[k - 1] = vatom[k];
            nS = ns_old - 1;
            __syncthreads();
        }
        if (inexact) {
            cert = true;
            continue;
        }
        if (dropped == 0) jadd = jadd < JADD / 2 ? 2 * jadd : JADD;
        else if (nS < 128 && 4 * dropped >= added) jadd = jadd > 1 ? jadd / 2 : 1;
        else jadd = jadd > 8 ? jadd * 7 / 8 : (jadd > 1 ? jadd - 1 : 1);
    }
    if (a.smpl_keep > 0 && !explored && !inexact && nnew > a.smpl_keep && nnew <= NT && a.Q) {
        // Subspace exploratory matching (Algorithm 2): keep the smpl_keep new atoms with the largest |u_j|
        // (ties to the lower atom index); the others leave S (downdates) and I, the kept slots move down
        // to nI0.., and the master problem continues on I_t from u restricted to it.
        explored = true;
        int* s_keep = reinterpret_cast<int*>(vx);     // [nnew] (vx and vg are free once the step ends)
        int* s_newpos = reinterpret_cast<int*>(vg);   // [nnew]
        if (tid < nnew) {
            const int u = nI0 + tid;
            const double xu = fabs(s.x[u]);
            const int au = g_atom[u];
            int rank = 0;
            for (int e = 0; e < nnew; ++e) {
                const double xe = fabs(s.x[nI0 + e]);
                const int ae = g_atom[nI0 + e];
                rank += (xe > xu) || (xe == xu && ae < au);
            }
            s_keep[tid] = rank < a.smpl_keep ? 1 : 0;
        }
        __syncthreads();
        if (tid == 0) {                         // new positions of the kept slots, in slot order
            int pos = nI0;
            for (int e = 0; e < nnew; ++e) s_newpos[e] = s_keep[e] ? pos++ : -1;
        }
        __syncthreads();
        // discarded atoms in S leave it, from the last support position down
        for (int k = nS - 1; k >= 0; --k) {
            const int u = s.so[k];
            if (u < nI0 || s_keep[u - nI0]) continue;
            for (int q = tid; q < nS; q += NT) vatom[q] = s.so[q];   // vatom is scratch after the Gram phase
            __syncthreads();
            if (FOLD) chol_drop_far(s, nS, k, vw, nullptr);
            else chol_drop<BLOCK ? 8 : 4>(s, nS, k, vw, nullptr);
            for (int q = k + 1 + tid; q < nS; q += NT) s.so[q - 1] = vatom[q];
            --nS;
            __syncthreads();
        }
        if (!inexact) {
            // move the kept slots' state down; a slot only moves to a lower position, in increasing
            // order, so every destination has been read already
            for (int e = 0; e < nnew; ++e) {
                const int np = s_newpos[e], u = nI0 + e;
                if (tid == 0) {
                    if (np < 0) {
                        const int atom = g_atom[u];
                        atomicAnd(&w.inI[(int64_t)sig * w.words + (atom >> 5)], ~(1u << (atom & 31)));
                    } else if (np != u) {
                        s.x[np] = s.x[u]; s.c[np] = s.c[u]; s.th[np] = s.th[u]; s.ex[np] = s.ex[u];
                        g_atom[np] = g_atom[u];
                    }
                }
                __syncthreads();
            }
            for (int k = tid; k < nS; k += NT) {
                const int u = s.so[k];
                if (u >= nI0) s.so[k] = s_newpos[u - nI0];
            }
            int kept = 0;
            for (int e = 0; e < nnew; ++e) kept += s_keep[e];
            nI = nI0 + kept;
            __syncthreads();
            // Gram rows of the moved slots again, from the table
            for (int e = tid; e < kept * nI; e += NT) {
                const int t = e / nI, u = e - t * nI;
                const int q = nI0 + t;
                const double val = a.Q[(int64_t)g_atom[q] * a.ldq + g_atom[u]];
                s.G[(int64_t)q * K + u] = val;
                s.G[(int64_t)u * K + q] = val;
            }
            __syncthreads();
            resolve = true;
            xs_ok = false;
            cert = false;
            goto active_set;
        }
    }

    phase_mark(2);

    // 4. Certificate on I (float64), from the gradient on all of I the loop's last pass left in vg.
    double e = 0.0;
    for (int u = tid; u < nI; u += NT) {
        const double gu = vg[u];
        const int th = s.th[u];
        const double d = th != 0 ? fabs(gu - lam * th) : fabs(gu) - lam;
        e = fmax(e, d);
    }
    const double kon = block_max(e, red);
    phase_mark(3);


    // 5. Write the state back (slots left out for this pass only may enter S again).
    if (vec_lds) {
        for (int u = tid; u < nI; u += NT) {
            g_x[u] = s.x[u]; g_c[u] = s.c[u]; g_th[u] = s.th[u]; g_ex[u] = s.ex[u] == EX_PASS ? 0 : s.ex[u];
        }
        for (int k = tid; k < nS; k += NT) g_so[k] = s.so[k];
    } else {
        for (int u = tid; u < nI; u += NT)
            if (g_ex[u] == EX_PASS) g_ex[u] = 0;
    }
    if (s.r_lds)
        for (int64_t i = tid; i < tri(nS); i += NT) g_R[i] = s.R[i];
    if (tid == 0) {
        w.nI[sig] = nI;
        w.nS[sig] = nS;
        w.iters[sig] += 1;
        w.kkt_on[sig] = kon > 0.0 ? kon : 0.0;
        w.jadd[sig] = jadd;
        if (inexact) w.status[sig] |= BMPL_SIG_INEXACT;
    }
    phase_mark(5);
    const uint64_t t_res = a.phase ? wall_clock64() : 0;

    // 6. Residual and objective (step 7), from the support's values and atoms gathered into vw / vz
    //    (free after the certificate).
    {
        double* sx = vw;
        int* satom = reinterpret_cast<int*>(vz);
        double l1 = 0.0;
        for (int k = tid; k < nS; k += NT) {
            const int u = s.so[k];
            const double xv = s.x[u];
            sx[k] = xv;
            satom[k] = g_atom[u];
            l1 += fabs(xv);
        }
        const double xl1 = block_sum(l1, red);    // also orders the writes above
        residual_tail(w, sig, a.At, a.lda, a.Bw, sx, satom, nS, xl1, red);
    }
    sub_ticks(14, t_res);
}

}  // namespace
}  // namespace bmpl
