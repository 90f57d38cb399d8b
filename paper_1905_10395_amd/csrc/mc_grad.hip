// Per-worker gradient and loss of low-rank matrix completion on a batch of
// observed entries (the problem family of the motivating example and of the
// supplement's "Low-Rank Matrix Completion Experiments" in arXiv 1905.10395,
// in rectangular, partially observed form).
//
//   e_k = <U[a_k], V[b_k]> - M_k ;  loss = c * sum_k e_k^2
//   dU[a] = 2c * sum_{k: a_k = a} e_k V[b_k] ;  dV[b] = 2c * sum_{k: b_k = b} e_k U[a_k]
//
// Worker row of x and of g: [U (m x r) | V (n x r)], row-major factors.
#include <cmath>
#include <type_traits>

#include "common.h"

namespace lsgd {

constexpr int kMcThreads = 256;
constexpr int kMcEntriesPerBlock = 256;

// sums: n doubles per row to clear too, or NULL
__global__ __launch_bounds__(256) void fill_zero_kernel(float* __restrict__ g, int64_t ld, double* __restrict__ sums, int n)
{
    if (sums && blockIdx.x == 0 && threadIdx.x < n) sums[blockIdx.y * n + threadIdx.x] = 0.0;
    float* row = g + (int64_t)blockIdx.y * ld;
    const int64_t n4 = ld >> 2;
    float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n4; c += (int64_t)gridDim.x * blockDim.x)
        reinterpret_cast<float4*>(row)[c] = z;
    if (blockIdx.x == 0 && threadIdx.x < (ld & 3)) row[(n4 << 2) + threadIdx.x] = 0.f;
}
__global__ __launch_bounds__(256) void fill_zero_scalar_kernel(float* __restrict__ g, int64_t ld, double* __restrict__ sums, int n)
{
    if (sums && blockIdx.x == 0 && threadIdx.x < n) sums[blockIdx.y * n + threadIdx.x] = 0.0;
    float* row = g + (int64_t)blockIdx.y * ld;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < ld; c += (int64_t)gridDim.x * blockDim.x)
        row[c] = 0.f;
}

// (a, b, M) of observed entry s, from the 16-byte records when the caller supplied them
__device__ __forceinline__ void fetch_entry(const lsgd_mc_entry* __restrict__ entries, const int32_t* __restrict__ rows,
                                            const int32_t* __restrict__ cols, const float* __restrict__ vals, int64_t s,
                                            int& a, int& b, float& v)
{
    if (entries) {
        const int4 e = reinterpret_cast<const int4*>(entries)[s];
        a = e.x; b = e.y; v = __int_as_float(e.z);
    } else {
        a = rows[s]; b = cols[s]; v = vals[s];
    }
}

// Sum over the LPE adjacent lanes of a lane group, result in every lane of the group.  Steps inside a
// row of 16 lanes are data-parallel-primitive adds (swap neighbours, swap pairs, mirror 8, mirror 16:
// after the first two steps every lane of a quad holds the quad's sum, and a mirror maps each quad onto
// a different one); wider groups finish with lane shuffles.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int LPE>
__device__ __forceinline__ float group_sum(float v)
{
    if (LPE >= 2) v = dpp_add<0xB1>(v);       // quad_perm [1,0,3,2]
    if (LPE >= 4) v = dpp_add<0x4E>(v);       // quad_perm [2,3,0,1]
    if (LPE >= 8) v = dpp_add<0x141>(v);      // row_half_mirror
    if (LPE >= 16) v = dpp_add<0x140>(v);     // row_mirror
    if (LPE >= 32) v += __shfl_xor(v, 16, 64);
    if (LPE >= 64) v += __shfl_xor(v, 32, 64);
    return v;
}

// Inclusive sum over the lanes of a wavefront, by data-parallel-primitive adds (lane shuffles take an LDS round each).
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
__device__ __forceinline__ int wave_scan(int v)
{
    v = dpp_add<0x111, 0xF>(v);               // row_shr:1, 2, 4, 8
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);               // lane 15 of a row to the row behind it
    return dpp_add<0x143, 0xC>(v);            // lane 31 to the upper half
}
// Sum of the first n of up to 16 values in LDS (the same in every lane).
__device__ __forceinline__ int sum_first(const int* v, int of, int n)
{
    const int lane = threadIdx.x & (kWave - 1);
    return __builtin_amdgcn_readlane(wave_scan(lane < (n < of ? n : of) ? v[lane] : 0), 15);
}

// General path: S lanes cooperate on one entry (S = power of two >= min(r, 64)),
// residual by a sum over the lanes, gradient rows accumulated with hardware fp32
// atomics into the zero-filled g.  Any r, m, n.  GRAD = false evaluates the
// squared residuals only (g may be NULL).  Two loops:
//   FLY   small batches are bound by the chain index -> entry -> factor rows ->
//         residual of an entry, so a lane group has up to eight entries in flight,
//         and wide groups come in larger workgroups (256 entries each): 4 workers x
//         3000 entries of 100 x 100, rank 5, 13.9 -> 4 us; 4 x 256, rank 50, whole
//         gradient call 39 -> 18 us.
//   !FLY  one entry at a time, for batches that fill the chip: these are bound by the
//         atomics, and bursts of eight only queue up behind each other where rows are
//         hot (4 workers x 62000 entries, rank 5: 100 x 20000 145 -> 83 us, 3000 x
//         4001 47 -> 41).
// Sums are no less exact than the binned path's: squared residuals are added in double,
// per lane and over the workgroup, products of a residual keep what their rounding
// drops (a lane of the binned path fuses several columns), and a term of the gradient
// is rounded once.  Relative error of gradient / losses, 8 workers x 256 entries on
// 1000 x 800, rank 8: 5.6e-8 / 1.6e-8, binned 5.8e-8 / 1.8e-8, with all of it in
// 32 bits 6.2e-8 / 3.9e-8, at the same time per call.
//   FEW   FLY where workgroups of 256 entries would leave compute units idle: a lane group goes through its entries one
//         after the other once they are there, so it takes two, and there are as many more workgroups (mc_few).  Whole
//         steps, 4 workers x 3000 entries of 100 x 100, rank 5, 12.8 -> 11.5 us, 4 x 256 of 1000 x 800 11.9 -> 9.9, rank 50,
//         2 x 400 of 300 x 200, 21.0 -> 10.9, rank 12, 8 x 5000 of 600 x 900 (160 workgroups of 256) 17.9 -> 16.5.
constexpr int mc_atomic_threads(int S, bool FLY) { return !FLY || S <= 8 ? 256 : S == 16 ? 512 : 1024; }
constexpr int mc_few_entries(int S) { return 2 * mc_atomic_threads(S, true) / S; }

template <int S, bool GRAD, bool FLY, bool FEW = false>
__global__ __launch_bounds__(mc_atomic_threads(S, FLY)) void mc_grad_atomic_kernel(
    const float* __restrict__ x, float* __restrict__ g, int64_t ld, int m, int n, int r,
    const int32_t* __restrict__ rows, const int32_t* __restrict__ cols, const float* __restrict__ vals,
    const int32_t* __restrict__ batch_idx, int64_t nb, float two_c, float* __restrict__ partials, double* __restrict__ partials64, int nblk,
    const lsgd_mc_entry* __restrict__ entries)
{
    constexpr int kThreads = mc_atomic_threads(S, FLY);
    const int w = blockIdx.y;
    const float* U = x + (int64_t)w * ld;
    const float* V = U + (int64_t)m * r;
    float* gU = GRAD ? g + (int64_t)w * ld : nullptr;
    float* gV = GRAD ? gU + (int64_t)m * r : nullptr;
    const int sub = threadIdx.x / S, q0 = threadIdx.x % S;
    constexpr int kSubs = kThreads / S;
    constexpr int kPer = FEW ? mc_few_entries(S) : kMcEntriesPerBlock;
    const int64_t k0 = (int64_t)blockIdx.x * kPer;
    const int64_t k1 = (k0 + kPer < nb) ? k0 + kPer : nb;
    double sq = 0.0;
    auto residual = [&](float dot, float low, float v) {
        low = fabsf(low) < INFINITY ? low : 0.f;         // (nothing, where the product is infinite)
        return (group_sum<S>(dot) - v) + group_sum<S>(low);
    };
    if constexpr (!FLY) {
        for (int64_t k = k0 + sub; k < k1; k += kSubs) {
            const int64_t s = batch_idx ? (int64_t)batch_idx[(int64_t)w * nb + k] : k;
            int a, b;
            float mv;
            fetch_entry(entries, rows, cols, vals, s, a, b, mv);
            const float* ua = U + (int64_t)a * r;
            const float* vb = V + (int64_t)b * r;
            float dot = 0.f, low = 0.f;
            for (int q = q0; q < r; q += S) {
                const float p = ua[q] * vb[q];
                if (q == q0) { dot = p; low = fmaf(ua[q], vb[q], -p); }
                else dot = fmaf(ua[q], vb[q], dot);
            }
            const float e = residual(dot, low, mv);
            if (q0 == 0) sq += (double)e * (double)e;
            if (GRAD) {
                const double f = (double)two_c * (double)e;
                for (int q = q0; q < r; q += S) {
                    unsafeAtomicAdd(gU + (int64_t)a * r + q, (float)(f * (double)vb[q]));
                    unsafeAtomicAdd(gV + (int64_t)b * r + q, (float)(f * (double)ua[q]));
                }
            }
        }
    } else {
        constexpr int kFly = FEW ? 2 : S < 8 ? S : 8;    // entries of a lane group in flight
        for (int64_t kb = k0 + sub; kb < k1; kb += (int64_t)kSubs * kFly) {
            int a[kFly], b[kFly];
            float mv[kFly], ua[kFly], vb[kFly];
            bool live[kFly];
#pragma unroll
            for (int u = 0; u < kFly; ++u) {
                const int64_t k = kb + (int64_t)u * kSubs;
                live[u] = k < k1;
                const int64_t kc = live[u] ? k : kb;     // past the end: the first entry again, its results dropped
                const int64_t s = batch_idx ? (int64_t)batch_idx[(int64_t)w * nb + kc] : kc;
                fetch_entry(entries, rows, cols, vals, s, a[u], b[u], mv[u]);
            }
#pragma unroll
            for (int u = 0; u < kFly; ++u) {
                ua[u] = q0 < r ? U[(int64_t)a[u] * r + q0] : 0.f;
                vb[u] = q0 < r ? V[(int64_t)b[u] * r + q0] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kFly; ++u) {
                const float* uu = U + (int64_t)a[u] * r;
                const float* vv = V + (int64_t)b[u] * r;
                float dot = ua[u] * vb[u];
                const float low = fmaf(ua[u], vb[u], -dot);      // what the product's rounding dropped
                for (int q = q0 + S; q < r; q += S) dot = fmaf(uu[q], vv[q], dot);
                const float e = residual(dot, low, mv[u]);
                if (!live[u]) continue;
                if (q0 == 0) sq += (double)e * (double)e;
                if (GRAD) {
                    const double f = (double)two_c * (double)e;
                    if (q0 < r) {
                        unsafeAtomicAdd(gU + (int64_t)a[u] * r + q0, (float)(f * (double)vb[u]));
                        unsafeAtomicAdd(gV + (int64_t)b[u] * r + q0, (float)(f * (double)ua[u]));
                    }
                    for (int q = q0 + S; q < r; q += S) {
                        unsafeAtomicAdd(gU + (int64_t)a[u] * r + q, (float)(f * (double)vv[q]));
                        unsafeAtomicAdd(gV + (int64_t)b[u] * r + q, (float)(f * (double)uu[q]));
                    }
                }
            }
        }
    }
    // block sum of squared residuals in a fixed order (one lane of a group holds its sum); FEW: several blocks then add theirs to
    // one slot, in the order in which they come
#pragma unroll
    for (int d = S; d < kWave; d <<= 1) sq += __shfl_xor(sq, d, kWave);
    __shared__ double red[kThreads / kWave];
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kThreads / kWave; ++q) red[0] += red[q];
        if (FEW) unsafeAtomicAdd(partials64 + (int64_t)w * nblk + blockIdx.x % (unsigned)nblk, red[0]);   // (nblk: slots)
        else if (partials64) partials64[(int64_t)w * nblk + blockIdx.x] = red[0];
        else partials[(int64_t)w * nblk + blockIdx.x] = (float)red[0];
    }
}

// The general path where a factor has few values: its gradient (LU: of U, LV: of V) is added up in LDS, and only the
// workgroup's sums go to g.  Entries that meet in a few rows queue up at the memory side otherwise, 40 ns each.  As above,
// with entries in flight.  Atomics on g / in LDS, us: 93 x 3965, rank 2, 4 workers x 40409 entries 99 to 155 / 20 (as g
// lies in memory); 87 x 362, rank 1, 8 x 27762 69 / 13; 80 x 8283, rank 8, 5 x 60721 95 / 39; 280 x 3930, rank 16,
// 16 x 55831 132 / 98; 420 drawn gradient calls with a side of up to 38000 values, as the rule sends them, 0.89 of the
// time, those of 50 us and more 0.63.
constexpr int kLdsThreads = 1024;

template <int S, bool LU, bool LV>
__global__ __launch_bounds__(kLdsThreads) void mc_grad_lds_kernel(
    const float* __restrict__ x, float* __restrict__ g, int64_t ld, int m, int n, int r,
    const int32_t* __restrict__ rows, const int32_t* __restrict__ cols, const float* __restrict__ vals,
    const int32_t* __restrict__ batch_idx, int64_t nb, int64_t per, float two_c, float* __restrict__ partials, double* __restrict__ partials64,
    const lsgd_mc_entry* __restrict__ entries)
{
    constexpr int kSubs = kLdsThreads / S, kFly = S <= 2 ? 2 : S < 8 ? 4 : 8;
    extern __shared__ float acc[];                       // [LU ? m r : 0][LV ? n r : 0]
    const int w = blockIdx.y, t = threadIdx.x;
    const int64_t nu = (int64_t)m * r;
    const int held = (LU ? (int)nu : 0) + (LV ? n * r : 0);           // fits LDS
    float* const accV = acc + (LU ? nu : 0);
    const float* U = x + (int64_t)w * ld;
    const float* V = U + nu;
    float* gU = g + (int64_t)w * ld;
    float* gV = gU + nu;
    for (int i = t; i < held; i += kLdsThreads) acc[i] = 0.f;
    __syncthreads();
    const int sub = t / S, q0 = t % S;
    const int64_t k0 = (int64_t)blockIdx.x * per, k1 = k0 + per < nb ? k0 + per : nb;
    double sq = 0.0;
    auto add = [&](int a, int b, int q, double f, float uq, float vq) {
        const float du = (float)(f * (double)vq), dv = (float)(f * (double)uq);
        if (LU) unsafeAtomicAdd(acc + a * r + q, du); else unsafeAtomicAdd(gU + (int64_t)a * r + q, du);
        if (LV) unsafeAtomicAdd(accV + b * r + q, dv); else unsafeAtomicAdd(gV + (int64_t)b * r + q, dv);
    };
    for (int64_t kb = k0 + sub; kb < k1; kb += (int64_t)kSubs * kFly) {
        int a[kFly], b[kFly];
        float mv[kFly], ua[kFly], vb[kFly];
        bool live[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const int64_t k = kb + (int64_t)u * kSubs;
            live[u] = k < k1;
            const int64_t kc = live[u] ? k : kb;         // past the end: the first entry again, its results dropped
            const int64_t s = batch_idx ? (int64_t)batch_idx[(int64_t)w * nb + kc] : kc;
            fetch_entry(entries, rows, cols, vals, s, a[u], b[u], mv[u]);
        }
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            ua[u] = q0 < r ? U[(int64_t)a[u] * r + q0] : 0.f;
            vb[u] = q0 < r ? V[(int64_t)b[u] * r + q0] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const float* uu = U + (int64_t)a[u] * r;
            const float* vv = V + (int64_t)b[u] * r;
            float dot = ua[u] * vb[u];
            float low = fmaf(ua[u], vb[u], -dot);        // what the product's rounding dropped
            for (int q = q0 + S; q < r; q += S) dot = fmaf(uu[q], vv[q], dot);
            low = fabsf(low) < INFINITY ? low : 0.f;
            const float e = (group_sum<S>(dot) - mv[u]) + group_sum<S>(low);
            if (!live[u]) continue;
            if (q0 == 0) sq += (double)e * (double)e;
            const double f = (double)two_c * (double)e;
            if (q0 < r) add(a[u], b[u], q0, f, ua[u], vb[u]);
            for (int q = q0 + S; q < r; q += S) add(a[u], b[u], q, f, uu[q], vv[q]);
        }
    }
#pragma unroll
    for (int d = S; d < kWave; d <<= 1) sq += __shfl_xor(sq, d, kWave);
    __shared__ double red[kLdsThreads / kWave];
    if (t % kWave == 0) red[t / kWave] = sq;
    __syncthreads();
    float* const to = LU ? gU : gV;
    for (int i = t; i < held; i += kLdsThreads)
        if (acc[i] != 0.f) unsafeAtomicAdd(to + i, acc[i]);
    if (t == 0) {
        for (int q = 1; q < kLdsThreads / kWave; ++q) red[0] += red[q];
        if (partials64) partials64[(int64_t)w * gridDim.x + blockIdx.x] = red[0];
        else partials[(int64_t)w * gridDim.x + blockIdx.x] = (float)red[0];
    }
}

// Objective only, rank a multiple of 4 and 16-byte aligned rows: LPE lanes share an entry with one float4
// of each factor row per lane, and four entries per lane group are in flight (index, record and both rows
// of each are fetched before the first product), since nothing but gathers happens here.
template <int LPE>
__global__ __launch_bounds__(kMcThreads) void mc_loss_vec_kernel(
    const float* __restrict__ x, int64_t ld, int m, int n, int r,
    const int32_t* __restrict__ rows, const int32_t* __restrict__ cols, const float* __restrict__ vals,
    const int32_t* __restrict__ batch_idx, int64_t nb, float* __restrict__ partials, int nblk,
    const lsgd_mc_entry* __restrict__ entries)
{
    constexpr int kSubs = kMcThreads / LPE, kFly = 4;
    const int w = blockIdx.y;
    const float* U = x + (int64_t)w * ld;
    const float* V = U + (int64_t)m * r;
    const int sub = threadIdx.x / LPE, q0 = threadIdx.x % LPE;
    const bool lane_on = q0 < (r >> 2);
    const int64_t k0 = (int64_t)blockIdx.x * kMcEntriesPerBlock;
    const int64_t k1 = (k0 + kMcEntriesPerBlock < nb) ? k0 + kMcEntriesPerBlock : nb;
    float sq = 0.f;
    for (int64_t kb = k0; kb < k1; kb += kSubs * kFly) {
        float4 ua[kFly], vb[kFly];
        float mv[kFly];
        bool live[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const int64_t k = kb + (int64_t)u * kSubs + sub;
            live[u] = k < k1;
            const int64_t kc = live[u] ? k : k1 - 1;           // a lane group past the end repeats the last entry
            const int64_t s = batch_idx ? (int64_t)batch_idx[(int64_t)w * nb + kc] : kc;
            int a, b;
            fetch_entry(entries, rows, cols, vals, s, a, b, mv[u]);
            ua[u] = vb[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (lane_on) {
                ua[u] = reinterpret_cast<const float4*>(U + (int64_t)a * r)[q0];
                vb[u] = reinterpret_cast<const float4*>(V + (int64_t)b * r)[q0];
            }
        }
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            float dot = ua[u].x * vb[u].x;
            dot = fmaf(ua[u].y, vb[u].y, dot);
            dot = fmaf(ua[u].z, vb[u].z, dot);
            dot = fmaf(ua[u].w, vb[u].w, dot);
#pragma unroll
            for (int d = 1; d < LPE; d <<= 1) dot += __shfl_xor(dot, d, LPE);
            const float e = dot - mv[u];
            if (q0 == 0 && live[u]) sq = fmaf(e, e, sq);
        }
    }
    __shared__ float red[kMcThreads];
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int d = kMcThreads / 2; d > 0; d >>= 1) {
        if (threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[(int64_t)w * nblk + blockIdx.x] = red[0];
}

// losses[w] = c * sum of the worker's partial sums, accumulated in fp64 in a fixed order.
template <class T>
__global__ __launch_bounds__(256) void mc_loss_finish_kernel(const T* __restrict__ partials, int nblk, float c,
                                                             float* __restrict__ losses)
{
    const int w = blockIdx.x;
    double acc = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) acc += (double)partials[(int64_t)w * nblk + i];
    __shared__ double red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
        if (threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) losses[w] = (float)((double)c * red[0]);
}

// ------------------------------------------------------------------------------------------
// Binned path (up to 64 column groups of 4, 2 or 1 in a row): no global floating-point atomics, and each
// factor row an entry touches is gathered once per side.
// Factor rows are grouped in bins of 128 consecutive rows (U bins, then V bins).
//   1. prepare kernel (1024 threads, E = 1024..4096 entries per workgroup): fetches each entry's
//      (a, b, M), ranks the workgroup's entries inside their U bin and V bin with LDS counters,
//      scans the counters, and writes every entry twice into the workgroup's own region of 2E
//      records: as (row of a inside its bin, b, M) grouped by U bin, and as (row of b inside its
//      bin, a, M) grouped by V bin, plus the table of where each bin starts in that region.  No
//      factor row is read here, and no pass over all workgroups is needed: a bin's records are
//      the union of one short segment per workgroup.
//   2. side kernel: one workgroup per (worker, bin), U and V bins alike, in one launch.  It
//      collects the bin's segments and sorts the records by row in LDS; a lane group takes its own
//      row from an LDS copy of the bin's rows, gathers the other factor's row for each record,
//      forms e = <U[a], V[b]> - M and adds e times the gathered row to its row's gradient.  Both
//      sides form e with the same lane partition and reduction tree, so they get the same bits.
//      U bins also sum e^2 (double per lane, fixed tree over the workgroup).
//   3. loss: c * the U bins' sums, added in bin order in double.
// Gradient rows are written once, scaled by 2c; rows without entries come out as zeros, so
// there is no separate zero fill.  The order of a row's records follows LDS rank order, so the
// last bits of a gradient row (fp32 sums) can differ between runs; the loss is summed in double,
// where a different order changes the rounded fp32 result only in freak cases.
// Workgroups of one worker are numbered so that they land on one die, or few (workgroup id modulo 8),
// which keeps the worker's factors, 5 MB at rank 32, in that die's L2.  This placement only
// affects speed, never results.
// ------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* global_ptr;
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
// a lane's part of a factor row: four, two or one of its columns, by the rank and the alignment of the rows
template <int VW> struct Cols;
template <> struct Cols<4> { using type = v4f; };
template <> struct Cols<2> { using type = v2f; };
template <> struct Cols<1> { using type = float; };
__device__ __forceinline__ float col_dot(v4f a, v4f b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }
__device__ __forceinline__ float col_dot(v2f a, v2f b) { return a.x * b.x + a.y * b.y; }
__device__ __forceinline__ float col_dot(float a, float b) { return a * b; }
__device__ __forceinline__ float col_dot_add(v4f a, v4f b, float c) { return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, fmaf(a.x, b.x, c)))); }
__device__ __forceinline__ float col_dot_add(v2f a, v2f b, float c) { return fmaf(a.y, b.y, fmaf(a.x, b.x, c)); }
__device__ __forceinline__ float col_dot_add(float a, float b, float c) { return fmaf(a, b, c); }

constexpr int kBinRows = 128;         // factor rows per bin (64, 128 or 256)
constexpr int kKeyShift = (kBinRows == 64) ? 26 : (kBinRows == 128) ? 25 : 24;   // record key: row in bin above, other row below
constexpr int kKeyMask = (1 << kKeyShift) - 1;
constexpr int kPrepThreads = 1024;    // threads per workgroup in the prepare kernel
constexpr int kMaxBins = 8192;        // LDS histogram capacity (U bins + V bins)
constexpr int kXcd = 8;

struct McBinned {
    int32_t* segs;   // [W][nblk][nbins+1] first record of each bin inside the workgroup's region
                     // (U bins fill [0, count), V bins [count, 2 count); entry nbins = 2 count)
    int2* rec;       // [W][nblk][2E] (row-in-bin << kKeyShift | other factor's row, M bits)
    int nbinsU, nbins, nblk, E;
    double* sums;    // [W][kLossSlots] squared residuals of the U bins, added up by atomics; or NULL: one sum per bin
};
constexpr int kLossSlots = 8;

// Maps a linear workgroup id to (worker, chunk), a die being id modulo 8.  per_die = 0: worker w lives on die w % 8, all
// dies work through workers 0 .. 7, then 8 .. 15.  Else a die takes a contiguous run of per_die chunks of all workers,
// so that no die is left without work when the number of workers is no multiple of eight (see mc_runs).
__device__ __forceinline__ bool xcd_map(int64_t id, int64_t per_die, int W, int nchunk, int& w, int& chunk)
{
    const int64_t t = id / kXcd;
    if (per_die > 0) {
        const int64_t lin = (id % kXcd) * per_die + t;
        w = (int)(lin / nchunk);
        chunk = (int)(lin % nchunk);
    } else {
        w = (int)(t / nchunk) * kXcd + (int)(id % kXcd);
        chunk = (int)(t % nchunk);
    }
    return w < W;
}

template <int EPT>
__global__ __launch_bounds__(kPrepThreads) void mc_prep_kernel(
    const int32_t* __restrict__ rows, const int32_t* __restrict__ cols, const float* __restrict__ vals,
    const int32_t* __restrict__ batch_idx, int64_t nb, McBinned S, const lsgd_mc_entry* __restrict__ entries)
{
    constexpr int E = EPT * kPrepThreads;
    const int w = blockIdx.y, blk = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    extern __shared__ int lhist[];                 // [nbins + 1]
    __shared__ int wsum[kPrepThreads / 64];
    for (int i = t; i <= S.nbins; i += kPrepThreads) lhist[i] = 0;
    if (S.sums && blk == 0 && t < kLossSlots) S.sums[w * kLossSlots + t] = 0.0;
    const int64_t k0 = (int64_t)blk * E;
    const int cnt_here = (int)((nb - k0 < E) ? nb - k0 : E);
    // every index chase of the workgroup is in flight at once
    int64_t src[EPT];
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const int i = u * kPrepThreads + t;
        src[u] = (i < cnt_here) ? (batch_idx ? (int64_t)batch_idx[(int64_t)w * nb + k0 + i] : k0 + i) : 0;
    }
    int a[EPT], b[EPT];
    float mv[EPT];
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        a[u] = b[u] = 0; mv[u] = 0.f;
        if (u * kPrepThreads + t < cnt_here) fetch_entry(entries, rows, cols, vals, src[u], a[u], b[u], mv[u]);
    }
    __syncthreads();
    int ru[EPT], rv[EPT];
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        if (u * kPrepThreads + t < cnt_here) {
            ru[u] = atomicAdd(&lhist[a[u] / kBinRows], 1);
            rv[u] = atomicAdd(&lhist[S.nbinsU + b[u] / kBinRows], 1);
        }
    }
    __syncthreads();
    // exclusive scan of the counters in place: thread t owns `per` consecutive bins
    const int per = (S.nbins + kPrepThreads - 1) / kPrepThreads;     // <= kMaxBins / 1024
    int loc[kMaxBins / kPrepThreads];
    int tot = 0;
    if (per == 1) {
        tot = t < S.nbins ? lhist[t] : 0;
    } else {
#pragma unroll
        for (int q = 0; q < kMaxBins / kPrepThreads; ++q) {
            const int i = t * per + q;
            loc[q] = (q < per && i < S.nbins) ? lhist[i] : 0;
            tot += loc[q];
        }
    }
    const int inc = wave_scan(tot);
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    int run = inc - tot + sum_first(wsum, kPrepThreads / 64, wv);
    if (per == 1) {
        if (t < S.nbins) lhist[t] = run;
    } else {
#pragma unroll
        for (int q = 0; q < kMaxBins / kPrepThreads; ++q) {
            const int i = t * per + q;
            if (q < per && i < S.nbins) { lhist[i] = run; run += loc[q]; }
        }
    }
    if (t == 0) lhist[S.nbins] = 2 * cnt_here;
    __syncthreads();
    int32_t* seg = S.segs + ((int64_t)w * S.nblk + blk) * (S.nbins + 1);
    for (int i = t; i <= S.nbins; i += kPrepThreads) seg[i] = lhist[i];
    // the records take their sorted places in LDS first, so that they leave as one contiguous run
    int2* stage = reinterpret_cast<int2*>(lhist + ((S.nbins + 2) & ~1));     // [2 E], 8-byte aligned behind the counters
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        if (u * kPrepThreads + t < cnt_here) {
            const int mb = __float_as_int(mv[u]);
            stage[lhist[a[u] / kBinRows] + ru[u]] = make_int2(((a[u] % kBinRows) << kKeyShift) | b[u], mb);
            stage[lhist[S.nbinsU + b[u] / kBinRows] + rv[u]] = make_int2(((b[u] % kBinRows) << kKeyShift) | a[u], mb);
        }
    }
    __syncthreads();
    int2* rec = S.rec + ((int64_t)w * S.nblk + blk) * (2 * E);
    for (int i = t; i < 2 * cnt_here; i += kPrepThreads) rec[i] = stage[i];
}

// One workgroup per (worker, bin).  The bin's records (one segment per prepare workgroup) are
// staged in LDS and counting-sorted by their row inside the bin (one integer LDS counter per row), so that
// each lane group owns whole rows: it walks the row's records, four gathers of the other factor's
// rows in flight, forms each record's residual against its own row, accumulates in registers and
// writes the gradient row once (scaled by 2c).  Rows without records are written as zeros.
// A workgroup is a chain of dependent steps (bounds, records, counts, places, gathers), 16 us of it at 20000^2, rank 32, four
// after each other on a compute unit, so what counts is the chain's length: own rows go straight to LDS while the bounds
// are on their way (a loop of load, wait and store took four latencies), scans are data-parallel-primitive adds.  Gradient
// of 16 workers x 65536 entries 82.3 -> 77.1 us, x 16384 59.8 -> 53.6, 8 x 16384 at 6001 x 3517, rank 10, 18.7 -> 17.6.  (Six
// workgroups per compute unit instead of five, at 80 registers: 76 to 77, other ranks up to 4 % slower.)
constexpr int kSideThreads = 256;
constexpr int kRedCap = 1024;                     // records staged per pass
constexpr int kSegCap = kSideThreads;             // segments collected at a time

// LPE lanes share a row, NV vectors each (vectors q0, q0 + LPE, ...).  EXACT: r == VW * LPE * NV, every lane holds NV of them.
template <int LPE, int NV, bool EXACT, int VW>
__global__ __launch_bounds__(kSideThreads) void mc_side_kernel(const float* __restrict__ x, float* __restrict__ g, int64_t ld,
                                                             int m, int n, int r, McBinned S, float two_c,
                                                             float* __restrict__ partials, int W, int64_t per_die)
{
    using V = typename Cols<VW>::type;
    constexpr int kSubs = kSideThreads / LPE;                          // lane groups per workgroup
    constexpr int RPG = (kBinRows + kSubs - 1) / kSubs;              // rows per lane group
    constexpr int PER = kRedCap / kSideThreads;                        // records per thread and pass
    int w, gbin;
    if (!xcd_map(blockIdx.x, per_die, W, S.nbins, w, gbin)) return;
    extern __shared__ __attribute__((aligned(16))) char tile_mem[];   // the bin's own rows [kBinRows][r]
    V* tile = reinterpret_cast<V*>(tile_mem);
    __shared__ int2 sorted[kRedCap];
    __shared__ int cnt[kBinRows], start[kBinRows + 1];
    __shared__ int segoff[kSegCap + 1], segbase[kSegCap], wtot[kSideThreads / 64];
    __shared__ double sqred[kSideThreads / 64];
    __shared__ int crowded;                                           // some segment does not fit its team's registers
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const bool uside = gbin < S.nbinsU;
    const int row0 = (uside ? gbin : gbin - S.nbinsU) * kBinRows;     // first factor row of the bin
    const int nrows = uside ? m : n;
    const float* xw = x + (int64_t)w * ld;
    const float* own = uside ? xw : xw + (int64_t)m * r;
    const float* other = uside ? xw + (int64_t)m * r : xw;            // U rows gather V rows and vice versa
    const int rv = r / VW;
    if (gbin == 0)                                                    // padding columns are zero
        for (int64_t c = (int64_t)(m + (int64_t)n) * r + t; c < ld; c += kSideThreads) g[(int64_t)w * ld + c] = 0.f;
    const int2* rec = S.rec + (int64_t)w * S.nblk * (2 * S.E);
    const int32_t* segs = S.segs + (int64_t)w * S.nblk * (S.nbins + 1) + gbin;
    const int sub = t / LPE, q0 = t % LPE;
    bool on[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) on[k] = EXACT || q0 + k * LPE < rv;
    V acc[RPG][NV];
#pragma unroll
    for (int i = 0; i < RPG; ++i)
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[i][k] = V(0.f);
    double sq = 0.0;

    // exclusive scan of the row counts (all threads; ends without a barrier)
    auto scan_rows = [&]() {
        if (kBinRows > 64 || t < 64) {
            const int cc = (t < kBinRows) ? cnt[t] : 0;
            int in2 = wave_scan(cc);
            if (kBinRows > 64) {
                if (lane == 63) wtot[wv] = in2;
                __syncthreads();
                for (int q = 0; q < wv; ++q) in2 += wtot[q];
            }
            if (t < kBinRows) start[t] = in2 - cc;
            if (t == kBinRows - 1) start[kBinRows] = in2;
        }
    };
    // rows of the other factor: at most kMaxBins * kBinRows rows of 128 values, so an offset has fewer than 32 bits
    const uint32_t row_bytes = 4u * (uint32_t)r;
    // the sorted records of one pass
    auto walk = [&]() {
#pragma unroll
        for (int i = 0; i < RPG; ++i) {
            const int row = sub + i * kSubs;
            if (row < kBinRows) {
                const int s0 = start[row], s1 = start[row + 1];
                if (s0 < s1) {
                    V mine_row[NV];
#pragma unroll
                    for (int k = 0; k < NV; ++k) mine_row[k] = on[k] ? tile[row * rv + q0 + k * LPE] : V(0.f);
                    float rowsq = 0.f;
                    for (int sidx = s0; sidx < s1; sidx += 4) {
                        // straight-line body: slots past the row's end repeat its last record with weight zero
                        int2 rc[4];
                        V ov[4][NV];
#pragma unroll
                        for (int u = 0; u < 4; ++u) rc[u] = sorted[(sidx + u < s1) ? sidx + u : s1 - 1];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint32_t off = __umul24((uint32_t)(rc[u].x & kKeyMask), row_bytes) + (uint32_t)(q0 * VW * 4);
#pragma unroll
                            for (int k = 0; k < NV; ++k)
                                ov[u][k] = on[k] ? *reinterpret_cast<const V*>(reinterpret_cast<const char*>(other) + off + (uint32_t)(k * LPE * VW * 4)) : V(0.f);
                        }
                        float d[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            float dot = col_dot(mine_row[0], ov[u][0]);
#pragma unroll
                            for (int k = 1; k < NV; ++k) dot = col_dot_add(mine_row[k], ov[u][k], dot);
                            d[u] = group_sum<LPE>(dot);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float e = (sidx + u < s1) ? d[u] - __int_as_float(rc[u].y) : 0.f;
#pragma unroll
                            for (int k = 0; k < NV; ++k) acc[i][k] += e * ov[u][k];
                            rowsq = fmaf(e, e, rowsq);
                        }
                    }
                    if (q0 == 0) sq += (double)rowsq;
                }
            }
        }
    };

    // The bin's own rows, which lie in one piece, to the tile.  No loop that loads, waits and stores: straight to LDS where
    // a lane's columns are 16 bytes, else a few loads at a time.
    auto own_rows = [&]() {
        const int live = (nrows - row0 < kBinRows ? nrows - row0 : kBinRows) * rv;
        const V* src = reinterpret_cast<const V*>(own + (int64_t)row0 * r);
        if constexpr (VW == 4) {
            const int wave0 = __builtin_amdgcn_readfirstlane(t & ~63);
            auto piece = [&](int at) {                                // 64 lanes from `at` on; past the end the last again
                __builtin_amdgcn_global_load_lds((global_ptr)(src + (at + lane < live ? at + lane : live - 1)), (lds_ptr)(tile + at), 16, 0, 0);
            };
            if constexpr (EXACT) {
#pragma unroll
                for (int i = 0; i < kBinRows * LPE * NV; i += kSideThreads)
                    if (LPE * NV * kBinRows >= kSideThreads || wave0 < LPE * NV * kBinRows) piece(i + wave0);
            } else {
                for (int i = wave0; i < kBinRows * rv; i += kSideThreads) piece(i);
            }
        } else {
            for (int i = t; i < live; i += 4 * kSideThreads) {
                V v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = src[i + u * kSideThreads < live ? i + u * kSideThreads : i];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i + u * kSideThreads < live) tile[i + u * kSideThreads] = v[u];
            }
        }
    };

    // A team of lanes per segment reads its bounds and its records, as many as the registers hold; no list of all records
    // in between.
    int team = kSideThreads;
    while (team > 1 && team * S.nblk > kSideThreads) team >>= 1;
    bool teams = team * S.nblk <= kSideThreads && (int64_t)S.nblk * S.E * kBinRows <= (int64_t)kRedCap * nrows;   // uniform; on average they fit
    int2 mine[PER];
    int len = 0;                                                      // records of this lane
    const int blk = t / team, l = t % team;
    const int32_t* sp = segs + (int64_t)(blk < S.nblk ? blk : 0) * (S.nbins + 1);
    const int s0 = sp[0], s1 = sp[1];
    __builtin_amdgcn_sched_barrier(0);                                // (the bounds first: loads return in order)
    own_rows();
    __builtin_amdgcn_sched_barrier(0);
    if (teams) {
        if (blk < S.nblk) {
            const int left = s1 - s0 - l;
            const int2* src = rec + (int64_t)blk * (2 * S.E) + s0 + l;
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (u * team < left) mine[u] = src[u * team];
            len = left > 0 ? (left + team - 1) / team : 0;
        }
    }
    if (t < kBinRows) cnt[t] = 0;
    if (t == 0) crowded = 0;
    __builtin_amdgcn_s_waitcnt(0x0F70);                               // vmcnt 0: the tile is there
    __syncthreads();
    if (teams) {
        if (len > PER) crowded = 1;
        int rank[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (u < len) rank[u] = atomicAdd(&cnt[(uint32_t)mine[u].x >> kKeyShift], 1);
        __syncthreads();
        teams = crowded == 0;
        if (teams) {
            scan_rows();
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (u < len) sorted[start[(uint32_t)mine[u].x >> kKeyShift] + rank[u]] = mine[u];
            __syncthreads();
            walk();
        }
    }
    // More records: all segments' are numbered through, kRedCap at a time.
    for (int blk0 = 0; blk0 < S.nblk && !teams; blk0 += kSegCap) {
        const int nseg = (S.nblk - blk0 < kSegCap) ? S.nblk - blk0 : kSegCap;
        // these segments: thread t takes segment t, counts are scanned into segoff
        int c = 0;
        if (t < nseg) {
            const int blk = blk0 + t;
            const int32_t* sp = segs + (int64_t)blk * (S.nbins + 1);
            const int s0 = sp[0];
            c = sp[1] - s0;
            segbase[t] = blk * (2 * S.E) + s0;
        }
        const int inc = wave_scan(c);
        if (lane == 63) wtot[wv] = inc;
        __syncthreads();
        const int before = sum_first(wtot, kSideThreads / 64, wv);
        segoff[t + 1] = before + inc;
        if (t == 0) segoff[0] = 0;
        __syncthreads();
        const int total = segoff[kSideThreads];

        for (int c0 = 0; c0 < total; c0 += kRedCap) {
            const int nrec = (total - c0 < kRedCap) ? total - c0 : kRedCap;
            if (t < kBinRows) cnt[t] = 0;
            __syncthreads();
            int rank[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = t + u * kSideThreads;
                if (i < nrec) {
                    // segment holding record c0 + i: the s with segoff[s] <= c0 + i < segoff[s + 1]
                    const int key = c0 + i;
                    int lo = 0, hi = nseg;
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (segoff[mid] <= key) lo = mid; else hi = mid;
                    }
                    mine[u] = rec[segbase[lo] + (key - segoff[lo])];
                    rank[u] = atomicAdd(&cnt[(uint32_t)mine[u].x >> kKeyShift], 1);
                }
            }
            __syncthreads();
            scan_rows();
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = t + u * kSideThreads;
                if (i < nrec) sorted[start[(uint32_t)mine[u].x >> kKeyShift] + rank[u]] = mine[u];
            }
            __syncthreads();
            walk();
            __syncthreads();
        }
    }
    float* out = g + (int64_t)w * ld + (uside ? (int64_t)0 : (int64_t)m * r) + (int64_t)row0 * r;
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
        const int row = sub + i * kSubs;
        if (row < kBinRows && row0 + row < nrows)
#pragma unroll
            for (int k = 0; k < NV; ++k)
                if (on[k]) reinterpret_cast<V*>(out + (int64_t)row * r)[q0 + k * LPE] = two_c * acc[i][k];
    }
    if (uside) {                                                      // sum of squared residuals of this U bin
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) sq += __shfl_xor(sq, d, 64);
        if (lane == 0) sqred[wv] = sq;
        __syncthreads();
        if (t == 0) {
            double tot = 0.0;
            for (int q = 0; q < kSideThreads / 64; ++q) tot += sqred[q];
            if (S.sums) unsafeAtomicAdd(S.sums + w * kLossSlots + gbin % kLossSlots, tot);
            else partials[(int64_t)w * S.nbinsU + gbin] = (float)tot;
        }
    }
}

__global__ __launch_bounds__(256) void mc_pack_kernel(const int32_t* __restrict__ rows, const int32_t* __restrict__ cols,
                                                      const float* __restrict__ vals, int64_t n, lsgd_mc_entry* __restrict__ out)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
        int4 e = make_int4(rows[k], cols[k], __float_as_int(vals[k]), 0);
        reinterpret_cast<int4*>(out)[k] = e;
    }
}

hipError_t launch_mc_pack(const int32_t* rows, const int32_t* cols, const float* vals, int64_t n, lsgd_mc_entry* out, hipStream_t s)
{
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(mc_pack_kernel, dim3((unsigned)blocks), dim3(256), 0, s, rows, cols, vals, n, out);
    return hipGetLastError();
}

static int64_t mc_entries(const lsgd_mc_batch& b) { return b.batch_idx ? b.B : b.n_obs; }

static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

static int mc_bins_u(const lsgd_mc_batch& b) { return (b.m + kBinRows - 1) / kBinRows; }
static int mc_bins(const lsgd_mc_batch& b) { return mc_bins_u(b) + (b.n + kBinRows - 1) / kBinRows; }
// entries per prepare workgroup: as many as keeps at least ~2 workgroups per compute unit busy,
// more when the segment table would otherwise outgrow its bound
static int mc_ept(int W, const lsgd_mc_batch& b)
{
    const int64_t nb = mc_entries(b);
    int ept = 4;
    while (ept > 1 && (int64_t)W * ((nb + (int64_t)ept * kPrepThreads - 1) / ((int64_t)ept * kPrepThreads)) < 512) ept >>= 1;
    while (ept < 4 && ((nb + (int64_t)ept * kPrepThreads - 1) / ((int64_t)ept * kPrepThreads)) * (mc_bins(b) + 1) > ((int64_t)1 << 22))
        ept <<= 1;
    return ept;
}
static int mc_prep_blocks(int W, const lsgd_mc_batch& b)
{
    const int64_t E = (int64_t)mc_ept(W, b) * kPrepThreads;
    return (int)((mc_entries(b) + E - 1) / E);
}
// Columns per lane in the side kernel by the rank alone.
static int mc_cols(int r) { return r % 4 == 0 ? 4 : r % 2 == 0 ? 2 : 1; }

// Time of one gradient call, us, from what bounds each route.  The constants are those that choose best over 2038 shapes,
// each timed on every route: 60 to 20000 rows a side, ranks 1 to 128, 100 to 66000 entries per worker, 1 to 32 workers.
struct McCost {
    double one, flight, binned; // atomics an entry at a time, atomics with entries in flight, binned
    double walk, stream;        // binned: the fullest bin's records, which one workgroup walks; all records and rows
};
// Requests of one worker that meet in the same 64 bytes, us.
static double mc_meet(const lsgd_mc_batch& b)
{
    const double r = b.r, lo = b.m < b.n ? b.m : b.n;
    return (double)mc_entries(b) / (lo * r > 16 ? lo * r / 16 : 1.0) * (0.0068 + 0.0045 * (r < 16 ? r : 16));
}
// Requests of 64 bytes, and where one side is narrow their queues at its few channels, us.
static double mc_queue(int W, const lsgd_mc_batch& b)
{
    const double r = b.r, lo = b.m < b.n ? b.m : b.n, hi = b.m < b.n ? b.n : b.m;
    const double pieces = b.r % 16 == 0 || 16 % b.r == 0 ? (r > 16 ? r / 16 : 1.0) : 1.0 + (r - 1) / 16;
    return 1e-3 * (double)W * (double)mc_entries(b) * (0.093 * pieces + 0.017 * log(hi / lo) / (1 + 0.14 * r));
}
static double dominant(double a, double b, double c = 0.0) { return sqrt(sqrt(a * a * a * a + b * b * b * b + c * c * c * c)); }
static McCost mc_cost(int W, const lsgd_mc_batch& b, int vw)
{
    const double nb = (double)mc_entries(b), thousands = 1e-3 * (double)W * nb, r = b.r;
    const double lo = b.m < b.n ? b.m : b.n, hi = b.m < b.n ? b.n : b.m;
    const double rows = (double)W * (lo + hi) * r * 4.0 / 5e6;          // one pass over all factor rows
    // Atomics: requests of 64 bytes and, where one side is narrow, their queues at its few channels; or the requests of
    // one worker that meet in the same 64 bytes; or the latency of the entries that a lane group takes one after the other:
    // eight of them.  (Batches of mc_few's range take two and less time, which the estimate does not know: of its constants
    // that is the one that was not fitted again.  Up to rank 32 they go this way all the same; above, most go binned: 150 drawn
    // ones of ranks 33 to 64 there 1.34 times as long as with two entries, 9.3 us against 10.5 to 17.)
    const double queue = mc_queue(W, b);
    const double meet = mc_meet(b);
    int group = 1;                                                      // lanes per entry
    while (group < b.r && group < kWave) group <<= 1;
    const double turns = ceil(r / group);
    McCost c;
    c.one = 5.7 + dominant(queue, meet, 1.3 * group * turns) + 1.1 * rows;
    c.flight = 5.7 + dominant(1.1 * queue, meet, 4.3 * (group > 32 ? group / 32 : 1) * turns) + 1.1 * rows;
    // Binned: one launch more; the records; and every factor row read and gradient row written, touched or not.
    int64_t lanes = 1;
    while (lanes * vw < b.r) lanes <<= 1;
    c.walk = nb * (lo > kBinRows ? kBinRows / lo : 1.0) * (0.0046 + 0.00044 * (double)lanes);
    const double records = thousands * (0.026 + 0.0027 * (double)lanes);
    c.stream = records + 2.0 * rows;
    c.binned = 12.0 + dominant(c.walk, records) + 2.0 * rows;
    return c;
}

// The route of a gradient call.  Between binned and atomics the usual one of the rank keeps the call (binned for multiples
// of four on aligned rows, 16 bytes per lane) unless the other's estimate is 7 % lower.  Over the shapes above the choice
// costs 0.6 % against the best route of each; 6 are more than 10 % slower than on the usual route (at most 1.28 times),
// all together 31 % faster.  Measured, us, one at a time / in flight / binned:
//   100 x 20000   rank 5    4 x 62000   84 / 144 / 605      9468 x 466      rank 2   16 x 62000  180 / 194 / 134
//   6001 x 3517   rank 10   8 x  4096   34 /  16 /  20      6001 x 3517     rank 10   8 x 16384   38 /  34 /  26
//   1000 x 800    rank 64   8 x   256   89 /  18 /  15      20000 x 20000   rank 32  16 x 32768  128 / 136 /  77
enum McRoute { kMcOne, kMcFlight, kMcBinned, kMcLds };
static McRoute mc_route(const McCost& c, int vw, bool binned_ok)
{
    const double atomics = c.flight < c.one ? c.flight : c.one;
    if (binned_ok && (vw == 4 ? c.binned < 1.07 * atomics : 1.07 * c.binned < atomics)) return kMcBinned;
    return c.flight < c.one ? kMcFlight : kMcOne;
}

// The same for gradients that are added up in LDS: of the side with fewer values, or of both.  A workgroup per compute unit,
// chunks per worker, each of at least as many entries as a workgroup of the other loops takes.  What bounds it: the
// LDS atomics of a workgroup (1.55 us per thousand values), or the requests of the other side and of the workgroups' sums;
// clearing and writing out what is held.  Fitted to 420 shapes that could go this way, ranks 1 to 64, 10 % rms error.
constexpr int64_t kLdsValues = 38000;
struct McLds {
    double narrow, both;        // us
    int64_t chunks, per;
};
static McLds mc_lds(int W, const lsgd_mc_batch& b)
{
    McLds c{1e30, 1e30, 0, 0};
    const int64_t nb = mc_entries(b), lo = b.m < b.n ? b.m : b.n, hi = b.m < b.n ? b.n : b.m;
    if (nb <= 0 || lo * b.r > kLdsValues) return c;
    const int64_t most = (nb + kMcEntriesPerBlock - 1) / kMcEntriesPerBlock;
    c.chunks = W < 256 ? 256 / W : 1;
    if (c.chunks > most) c.chunks = most;
    c.per = (nb + c.chunks - 1) / c.chunks;
    c.chunks = (nb + c.per - 1) / c.per;
    int group = 1;                                                      // lanes per entry
    while (group < b.r && group < kWave) group <<= 1;
    const int fly = group <= 2 ? 2 : group < 8 ? 4 : 8;
    const double per = (double)c.per, turns = ceil((double)b.r / group), slots = ceil(per * group / kLdsThreads), rounds = ceil(slots / fly);
    const double rows = (double)W * (double)(lo + hi) * b.r * 4.0 / 5e6, sums = 1e-3 * (double)c.chunks * W / 16.0;
    const double pieces = b.r % 16 == 0 || 16 % b.r == 0 ? (b.r > 16 ? b.r / 16.0 : 1.0) : 1.0 + (b.r - 1) / 16.0;
    const double held = (double)(lo * b.r);
    c.narrow = 8.0 + dominant(1.55e-3 * per * b.r, 0.07e-3 * (double)W * (double)nb * pieces + 0.015 * sums * held) + 0.069e-3 * held + 1.1 * rows;
    if ((lo + hi) * b.r <= kLdsValues)
        c.both = 8.8 + dominant(0.13 * rounds + 0.22 * slots * turns + 3.05e-3 * per * b.r, 0.036 * sums * (double)((lo + hi) * b.r)) + 1.1 * rows;
    return c;
}

// Whether dies take contiguous runs of bins (xcd_map).  With a worker per die and W no multiple of eight the busiest die
// has 8 ceil(W / 8) / W times the average; runs even that out, but spread a worker over dies, so that the fullest bin's
// records, if that is what the launch waits for, find less of the other factor in their die's L2 (up to 29 % longer).
// Over 1359 shapes of 1 to 28 workers 5 are more than 10 % slower than with a worker per die (at most 1.16 times), 14 than
// with runs (1.27).  Measured, us, worker per die / runs: 20000 x 20000, rank 64, 4 workers x 16384 entries 59 / 38,
// 9 workers 99 / 68; 3000 x 4001, rank 64, 12 x 2000 33 / 25; 466 x 9468, rank 32, 4 x 16384 52 / 64; 100 x 5000, rank 32,
// 9 x 16384 152 / 192.
static bool mc_runs(const McCost& c, int W)
{
    const double excess = (double)kXcd * ((W + kXcd - 1) / kXcd) / W - 1.0;
    return c.walk < 2.0 * excess * c.stream;
}

// ... as wide as the rank and the alignment of the rows allow
static int mc_cols(const float* x, const float* g, int64_t ld, int r)
{
    int vw = mc_cols(r);
    auto ok = [&](int v) {
        return (reinterpret_cast<uintptr_t>(x) & (4u * (unsigned)v - 1u)) == 0 && (reinterpret_cast<uintptr_t>(g) & (4u * (unsigned)v - 1u)) == 0 && ld % v == 0;
    };
    while (vw > 1 && !ok(vw)) vw >>= 1;
    return vw;
}
static bool mc_binned_ok(int W, const lsgd_mc_batch& b, int vw)
{
    const int64_t nb = mc_entries(b);
    if (!(b.r / vw <= 64 && nb > 0 && nb < ((int64_t)1 << 30) && mc_bins(b) <= kMaxBins && b.m < (1 << kKeyShift) && b.n < (1 << kKeyShift) &&
          (size_t)kBinRows * b.r * 4 <= 64 * 1024))
        return false;
    return (int64_t)mc_prep_blocks(W, b) * (mc_bins(b) + 1) <= ((int64_t)1 << 22);
}

size_t mc_partials(int W, const lsgd_mc_batch& b)
{
    int64_t nblk = (mc_entries(b) + kMcEntriesPerBlock - 1) / kMcEntriesPerBlock;   // general path: one per workgroup
    if (nblk < mc_bins_u(b)) nblk = mc_bins_u(b);                                  // binned path: one per U bin
    return (size_t)W * (size_t)(nblk > 0 ? nblk : 1);
}

// Entries in flight, two per lane group: workgroups per worker, which share a few double slots (where the sums of larger workgroups
// or of bins would lie; the order of their additions is open, so that losses can differ in the last bit between calls); none: 0.  Where workgroups of 256 entries are no more than compute units and it is the chain of a lane
// group's entries that the launch waits for, not requests that queue (5 x 12534 entries of 1911 x 919, rank 5, 16.7 / 18.6) or
// meet in the same lines (2 x 29762 of 223 x 2125, rank 12, 19.0 / 22.9).  180 drawn gradients and steps of this size 0.91 of the time.
struct McFew { int workgroups, slots; };
static McFew mc_few(int W, const lsgd_mc_batch& b)
{
    McFew f{0, 0};
    int group = 4;
    while (group < b.r && group < kWave) group <<= 1;
    const int64_t nb = mc_entries(b), blocks = (nb + kMcEntriesPerBlock - 1) / kMcEntriesPerBlock;
    const int64_t room = (int64_t)(mc_partials(W, b) / (size_t)W) / 2;                   // doubles per worker
    if (b.r <= 2 || nb <= 0 || (int64_t)W * blocks > 256 || room < 1 || W > kColumnMaxWorkers || mc_meet(b) > 5.0 ||
        1.1 * mc_queue(W, b) > (group > 32 ? 8.6 : 4.3))
        return f;
    f.workgroups = (int)((nb + mc_few_entries(group) - 1) / mc_few_entries(group));
    f.slots = (int)(room < kLossSlots ? room : kLossSlots);
    return f;
}

static size_t mc_binned_bytes(int W, const lsgd_mc_batch& b)
{
    const size_t slots = (size_t)mc_prep_blocks(W, b) * mc_ept(W, b) * kPrepThreads;
    return up256((size_t)W * mc_prep_blocks(W, b) * (mc_bins(b) + 1) * 4) + up256((size_t)W * 2 * slots * 8);
}

size_t mc_scratch_bytes(int W, const lsgd_mc_batch& b)
{
    const int vw = mc_cols(b.r);
    if (!mc_binned_ok(W, b, vw) || (b.r % 4 != 0 && mc_route(mc_cost(W, b, vw), vw, true) != kMcBinned)) return 0;
    return mc_binned_bytes(W, b);
}

// The route of a call whose rows allow vw columns per lane, with scratch_bytes of scratch; what else the launch needs of it.
struct McPath {
    McRoute route;
    McCost cost;
    McLds lds;                  // kMcLds: gradients held in LDS, of U, of V
    bool lu, lv;
};
static McPath mc_path(int W, const lsgd_mc_batch& b, int vw, size_t scratch_bytes)
{
    McPath p{};
    p.cost = mc_cost(W, b, vw);
    p.route = mc_route(p.cost, vw, mc_binned_ok(W, b, vw) && scratch_bytes >= mc_binned_bytes(W, b));
    p.lds = mc_lds(W, b);
    const double other = p.route == kMcBinned ? p.cost.binned : p.route == kMcFlight ? p.cost.flight : p.cost.one;
    // The usual route keeps the call unless the estimate is 13 % and 0.7 us lower: at 10 us all routes are launches.
    if (1.15 * (p.lds.narrow < p.lds.both ? p.lds.narrow : p.lds.both) + 0.7 < other) {
        const bool both = p.lds.both <= p.lds.narrow;
        p.route = kMcLds;
        p.lu = both || b.m <= b.n; p.lv = both || !p.lu;
    }
    return p;
}

// What mc_path says, for tests: route, factors held in LDS, where binned the prepare workgroups and their entries, and where
// lane groups take two entries each the workgroups per worker and the slots of their sums (mc_few).
void mc_describe_path(int W, const lsgd_mc_batch& b, int vw, size_t scratch_bytes, int out[7])
{
    const McPath p = mc_path(W, b, vw, scratch_bytes);
    out[0] = p.route; out[1] = p.lu; out[2] = p.lv;
    out[3] = p.route == kMcBinned ? mc_prep_blocks(W, b) : 0;
    out[4] = p.route == kMcBinned ? mc_ept(W, b) * kPrepThreads : 0;
    const McFew few = p.route == kMcFlight ? mc_few(W, b) : McFew{0, 0};
    out[5] = few.workgroups; out[6] = few.slots;
}

// The binned path's scratch is a condition only for ranks that are multiples of four; with others a workspace
// without room for it takes the general path.
size_t mc_scratch_required(int W, const lsgd_mc_batch& b) { return b.r % 4 == 0 ? mc_scratch_bytes(W, b) : 0; }

static void launch_prep(int W, const lsgd_mc_batch& b, int64_t nb, const McBinned& S, hipStream_t s)
{
    const dim3 pgrid((unsigned)S.nblk, (unsigned)W);
    const size_t plds = (size_t)((S.nbins + 2) & ~1) * 4 + (size_t)2 * S.E * 8;     // counters, then the staged records
    static bool big_lds = false;
    if (!big_lds) {                                   // 4096 entries per workgroup stage 64 KB of records
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&mc_prep_kernel<4>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)((kMaxBins + 2) * 4 + 2 * 4 * kPrepThreads * 8));
        big_lds = true;
    }
    if (S.E == kPrepThreads)
        hipLaunchKernelGGL((mc_prep_kernel<1>), pgrid, dim3(kPrepThreads), plds, s, b.rows, b.cols, b.vals, b.batch_idx, nb, S, b.entries);
    else if (S.E == 2 * kPrepThreads)
        hipLaunchKernelGGL((mc_prep_kernel<2>), pgrid, dim3(kPrepThreads), plds, s, b.rows, b.cols, b.vals, b.batch_idx, nb, S, b.entries);
    else
        hipLaunchKernelGGL((mc_prep_kernel<4>), pgrid, dim3(kPrepThreads), plds, s, b.rows, b.cols, b.vals, b.batch_idx, nb, S, b.entries);
}

template <int LPE, int NV, int VW>
static void launch_side(const float* x, float* g, int W, int64_t ld, const lsgd_mc_batch& b,
                        const McBinned& S, float* partials, bool runs, hipStream_t s)
{
    const int64_t run = ((int64_t)W * S.nbins + kXcd - 1) / kXcd, per_die = runs ? run : 0;
    const int64_t groups = per_die ? run * kXcd : (int64_t)((W + kXcd - 1) / kXcd) * kXcd * S.nbins;
    auto go = [&](auto exact) {
        hipLaunchKernelGGL((mc_side_kernel<LPE, NV, decltype(exact)::value, VW>), dim3((unsigned)groups), dim3(kSideThreads),
                           (size_t)kBinRows * b.r * 4, s, x, g, ld, b.m, b.n, b.r, S, 2.0f * b.c, partials, W, per_die);
    };
    if (b.r == VW * LPE * NV) go(std::true_type{});
    else go(std::false_type{});
}

template <int VW>
static void launch_side_lanes(const float* x, float* g, int W, int64_t ld, const lsgd_mc_batch& b, const McBinned& S, float* partials,
                              bool runs, hipStream_t s)
{
    const int rv = b.r / VW;
    // Two vectors per lane where that many lanes would mostly repeat each other's work on a record (its address, residual and
    // place in the row): from sixteen lanes, from eight with narrow vectors.  One / two, gradient call, us: 20000 x 20000, rank
    // 64, 8 workers x 32768 entries 85 / 79; 9468 x 5000, rank 50, 48 / 43; 20000 x 20000, rank 5, 16 x 65536 80 / 72; but rank
    // 32 there 90 / 92, rank 16 66 / 71.
    constexpr bool wide = VW == 4;
    if (rv <= 1) launch_side<1, 1, VW>(x, g, W, ld, b, S, partials, runs, s);
    else if (rv <= 2) launch_side<2, 1, VW>(x, g, W, ld, b, S, partials, runs, s);
    else if (rv <= 4) launch_side<4, 1, VW>(x, g, W, ld, b, S, partials, runs, s);
    else if (rv <= 8) launch_side<wide ? 8 : 4, wide ? 1 : 2, VW>(x, g, W, ld, b, S, partials, runs, s);
    else if (rv <= 16) launch_side<8, 2, VW>(x, g, W, ld, b, S, partials, runs, s);
    else if (rv <= 32) launch_side<16, 2, VW>(x, g, W, ld, b, S, partials, runs, s);
    else launch_side<32, 2, VW>(x, g, W, ld, b, S, partials, runs, s);
}

static void launch_fill_zero(float* g, int W, int64_t ld, hipStream_t s, double* sums = nullptr, int n = 0)
{
    const bool v4 = (reinterpret_cast<uintptr_t>(g) & 15u) == 0 && (ld % 4 == 0);
    int64_t blocks = ((v4 ? ld / 4 : ld) + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    if (v4) hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks, (unsigned)W), dim3(256), 0, s, g, ld, sums, n);
    else hipLaunchKernelGGL(fill_zero_scalar_kernel, dim3((unsigned)blocks, (unsigned)W), dim3(256), 0, s, g, ld, sums, n);
}

template <int S>
static void launch_lds_lanes(const float* x, float* g, int W, int64_t ld, const lsgd_mc_batch& b, int64_t nb, const McLds& c, bool lu, bool lv,
                             float* partials, double* sums64, hipStream_t s)
{
    const size_t lds = sizeof(float) * (size_t)((lu ? (int64_t)b.m * b.r : 0) + (lv ? (int64_t)b.n * b.r : 0));
    auto go = [&](auto u, auto v) {
        auto kernel = mc_grad_lds_kernel<S, decltype(u)::value, decltype(v)::value>;
        if (lds > 48 * 1024) {
            static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsValues * sizeof(float)));
            (void)once;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)c.chunks, (unsigned)W), dim3(kLdsThreads), lds, s, x, g, ld, b.m, b.n, b.r, b.rows, b.cols, b.vals,
                           b.batch_idx, nb, c.per, 2.0f * b.c, partials, sums64, b.entries);
    };
    if (lu && lv) go(std::true_type{}, std::true_type{});
    else if (lu) go(std::true_type{}, std::false_type{});
    else go(std::false_type{}, std::true_type{});
}

static void launch_lds(const float* x, float* g, int W, int64_t ld, const lsgd_mc_batch& b, int64_t nb, const McLds& c, bool lu, bool lv,
                       float* partials, double* sums64, hipStream_t s)
{
    if (b.r <= 1) launch_lds_lanes<1>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
    else if (b.r <= 2) launch_lds_lanes<2>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
    else if (b.r <= 4) launch_lds_lanes<4>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
    else if (b.r <= 8) launch_lds_lanes<8>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
    else if (b.r <= 16) launch_lds_lanes<16>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
    else if (b.r <= 32) launch_lds_lanes<32>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
    else launch_lds_lanes<64>(x, g, W, ld, b, nb, c, lu, lv, partials, sums64, s);
}

hipError_t launch_mc_grad_loss(const float* x, float* g, float* losses, int W, int64_t P, int64_t ld,
                               const lsgd_mc_batch& b, const DeviceState& st, hipStream_t s, LossParts* parts)
{
    const int64_t nb = mc_entries(b);
    // the partial sums are added up by a launch of their own, or left to a caller that says it can; few of them in one
    // order either way, so that a step and the calls it is made of find the same losses
    auto finish_loss = [&](int n, const double* sums64) {
        if (loss_parts_ok(W, n)) {
            LossParts p;
            p.sums = st.partials; p.sums64 = sums64; p.stride = n; p.n = n; p.c = (double)b.c; p.div = 1;
            if (!parts) return launch_loss_parts(p, W, losses, s);
            *parts = p;
        } else if (sums64) {
            hipLaunchKernelGGL((mc_loss_finish_kernel<double>), dim3((unsigned)W), dim3(256), 0, s, sums64, n, b.c, losses);
        } else {
            hipLaunchKernelGGL((mc_loss_finish_kernel<float>), dim3((unsigned)W), dim3(256), 0, s, st.partials, n, b.c, losses);
        }
        return hipGetLastError();
    };
    const int vw = mc_cols(x, g, ld, b.r);
    const McPath path = mc_path(W, b, vw, st.scratch_bytes);
    const McRoute route = path.route;
    if (route == kMcLds) {
        const McLds& lds = path.lds;
        double* sums64 = st.scratch_bytes >= sizeof(double) * (size_t)W * (size_t)lds.chunks ? reinterpret_cast<double*>(st.scratch) : nullptr;
        launch_fill_zero(g, W, ld, s);
        launch_lds(x, g, W, ld, b, nb, lds, path.lu, path.lv, st.partials, sums64, s);
        return finish_loss((int)lds.chunks, sums64);
    }
    if (route == kMcBinned) {
        McBinned S;
        S.nbinsU = mc_bins_u(b); S.nbins = mc_bins(b); S.nblk = mc_prep_blocks(W, b); S.E = mc_ept(W, b) * kPrepThreads;
        char* p = st.scratch;
        S.segs = reinterpret_cast<int32_t*>(p); p += up256((size_t)W * S.nblk * (S.nbins + 1) * 4);
        S.rec = reinterpret_cast<int2*>(p);
        // More sums than the next launch adds up itself: the bins of a worker share a few slots (which lie where the sums
        // would: more than kLossPartsMax sums of at most kColumnMaxWorkers workers are more than two floats per slot), in
        // double, so that their order does not show.  20000 x 20000, 16 workers, whole step: 5 us less.
        S.sums = W <= kColumnMaxWorkers && !loss_parts_ok(W, S.nbinsU) ? reinterpret_cast<double*>(st.partials) : nullptr;
        launch_prep(W, b, nb, S, s);
        if (vw == 4) launch_side_lanes<4>(x, g, W, ld, b, S, st.partials, mc_runs(path.cost, W), s);
        else if (vw == 2) launch_side_lanes<2>(x, g, W, ld, b, S, st.partials, mc_runs(path.cost, W), s);
        else launch_side_lanes<1>(x, g, W, ld, b, S, st.partials, mc_runs(path.cost, W), s);
        return S.sums ? finish_loss(kLossSlots, S.sums) : finish_loss(S.nbinsU, nullptr);
    }
    const McFew few = route == kMcFlight ? mc_few(W, b) : McFew{0, 0};
    const int nblk = few.workgroups ? few.workgroups : (int)((nb + kMcEntriesPerBlock - 1) / kMcEntriesPerBlock);
    // the block sums of squares stay in double where the binned path's scratch, idle now, has room for them (always for
    // ranks that are multiples of four and could have taken that path)
    double* sums64 = few.workgroups ? reinterpret_cast<double*>(st.partials)
                   : st.scratch_bytes >= sizeof(double) * (size_t)W * (size_t)nblk ? reinterpret_cast<double*>(st.scratch) : nullptr;
    launch_fill_zero(g, W, ld, s, few.workgroups ? sums64 : nullptr, few.slots);   // general path: whole rows (padding included), then atomics
    if (nblk > 0) {
        dim3 grid((unsigned)nblk, (unsigned)W);
        const float two_c = 2.0f * b.c;
#define LSGD_MC_LAUNCH_AS(S, FLY, FEW)                                                                          \
    hipLaunchKernelGGL((mc_grad_atomic_kernel<S, true, FLY, FEW>), grid, dim3(mc_atomic_threads(S, FLY)), 0, s, x, g, ld, b.m, b.n, b.r, \
                       b.rows, b.cols, b.vals, b.batch_idx, nb, two_c, st.partials, sums64, FEW ? few.slots : nblk, b.entries)
// (ranks 1 and 2 have short chains anyway: the estimate never gives them entries in flight)
#define LSGD_MC_LAUNCH(S) do { if (few.workgroups) LSGD_MC_LAUNCH_AS(S, (S > 2), (S > 2)); else if (route == kMcFlight) LSGD_MC_LAUNCH_AS(S, (S > 2), false); \
                               else LSGD_MC_LAUNCH_AS(S, false, false); } while (0)
        if (b.r <= 1) LSGD_MC_LAUNCH(1);
        else if (b.r <= 2) LSGD_MC_LAUNCH(2);
        else if (b.r <= 4) LSGD_MC_LAUNCH(4);
        else if (b.r <= 8) LSGD_MC_LAUNCH(8);
        else if (b.r <= 16) LSGD_MC_LAUNCH(16);
        else if (b.r <= 32) LSGD_MC_LAUNCH(32);
        else LSGD_MC_LAUNCH(64);
#undef LSGD_MC_LAUNCH
#undef LSGD_MC_LAUNCH_AS
    }
    return finish_loss(few.workgroups ? few.slots : nblk, sums64);
}

// Objective values only: the residual pass of the general path without its atomics, one partial sum per
// block of entries, then the same fixed-order finish.
hipError_t launch_mc_loss(const float* x, float* losses, int W, int64_t ld, const lsgd_mc_batch& b, const DeviceState& st,
                          hipStream_t s)
{
    const int64_t nb = mc_entries(b);
    const int nblk = (int)((nb + kMcEntriesPerBlock - 1) / kMcEntriesPerBlock);
    const bool vec = b.r % 4 == 0 && b.r <= 256 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0 && ld % 4 == 0;
    if (nblk > 0 && vec) {
        dim3 grid((unsigned)nblk, (unsigned)W);
#define LSGD_MC_LAUNCH(LPE)                                                                                      \
    hipLaunchKernelGGL((mc_loss_vec_kernel<LPE>), grid, dim3(kMcThreads), 0, s, x, ld, b.m, b.n, b.r, b.rows,   \
                       b.cols, b.vals, b.batch_idx, nb, st.partials, nblk, b.entries)
        const int r4 = b.r / 4;
        if (r4 <= 1) LSGD_MC_LAUNCH(1);
        else if (r4 <= 2) LSGD_MC_LAUNCH(2);
        else if (r4 <= 4) LSGD_MC_LAUNCH(4);
        else if (r4 <= 8) LSGD_MC_LAUNCH(8);
        else if (r4 <= 16) LSGD_MC_LAUNCH(16);
        else if (r4 <= 32) LSGD_MC_LAUNCH(32);
        else LSGD_MC_LAUNCH(64);
#undef LSGD_MC_LAUNCH
    } else if (nblk > 0) {
        dim3 grid((unsigned)nblk, (unsigned)W);
#define LSGD_MC_LAUNCH(S)                                                                                              \
    hipLaunchKernelGGL((mc_grad_atomic_kernel<S, false, true>), grid, dim3(mc_atomic_threads(S, true)), 0, s, x, (float*)nullptr, ld, b.m, b.n, \
                       b.r, b.rows, b.cols, b.vals, b.batch_idx, nb, 0.0f, st.partials, (double*)nullptr, nblk, b.entries)
        if (b.r <= 1) LSGD_MC_LAUNCH(1);
        else if (b.r <= 2) LSGD_MC_LAUNCH(2);
        else if (b.r <= 4) LSGD_MC_LAUNCH(4);
        else if (b.r <= 8) LSGD_MC_LAUNCH(8);
        else if (b.r <= 16) LSGD_MC_LAUNCH(16);
        else if (b.r <= 32) LSGD_MC_LAUNCH(32);
        else LSGD_MC_LAUNCH(64);
#undef LSGD_MC_LAUNCH
    }
    hipLaunchKernelGGL((mc_loss_finish_kernel<float>), dim3((unsigned)W), dim3(256), 0, s, st.partials, nblk, b.c, losses);
    return hipGetLastError();
}

} // namespace lsgd
