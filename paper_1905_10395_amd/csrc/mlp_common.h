// What the matrix-core kernels of the MLP path share: operand descriptions, the fused update's per-row view and
// the LDS transposing read.
#pragma once

#include "common.h"
#include "update_math.h"

namespace lsgd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// the same at any element boundary (the hardware takes unaligned vector accesses; the type tells the compiler)
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

enum { EPI_FWD = 0, EPI_DX = 1, EPI_DW = 2, EPI_DWU = 3, EPI_LOGITS = 4, EPI_HEAD = 5 };   // DWU: d-weight with the update applied in place of the store

struct GemmArgs {
    const uint16_t* A; int64_t sA; int64_t lda;   // [M][K], per-worker stride sA (elements)
    const uint16_t* B; int64_t sB; int64_t ldb;   // TRANS_B ? [K][N] : [N][K]
    int M, N, K;
    int updated;                                  // EPI_FWD: a fused update goes over all weights between two passes
    const float* A32; uint16_t* copy; int64_t sCopy; // EPI_FWD on fp32 inputs (in place of A, strides sA and lda): where their bf16 copy [M][K] goes, or NULL
    const float* bias; int64_t sBias;             // EPI_FWD: fp32 [N]
    const uint16_t* mask; int64_t sMask; int64_t ldmask; // EPI_DX: h_{k-1} [M][N]
    uint16_t* out; int64_t sOut; int64_t ldout;   // EPI_FWD: h [M][N]; EPI_DX: delta [M][N]
    uint16_t* outT; int64_t sOutT; int64_t ldoutT;// EPI_DX: delta^T [N][M]
    float* C; int64_t sC; int64_t ldc;            // EPI_DW, EPI_LOGITS: fp32 [M][N]
    // EPI_HEAD (out, outT: the output deltas [M][N] and [N][M], or NULL)
    const int32_t* y;                             // [M] per worker
    uint16_t* dx; uint16_t* dxT;                  // the d-input product [M][K] and [K][M] (strides of out), or NULL
    double* loss_parts; int64_t sLoss; float* losses; // loss sums of the row tiles (sLoss doubles between workers), or the losses when one tile holds the batch
    float* pad; int64_t pad_from, pad_to;         // columns [pad_from, pad_to) of rows of pad_to floats to clear, or NULL
    FusedUpdate fu; int64_t colC;                 // EPI_DWU: update state; column of C[0][0] in the parameter row
};

// Per-worker view of the fused update: coefficients (with the leader exemption resolved) and row pointers.
struct FusedRow {
    Coef c;
    float* x;
    float* m;
    uint16_t* xb;
    const float* zl;
    const float* zg;
};

__device__ __forceinline__ FusedRow fused_row(const FusedUpdate& u, int w, int64_t ld)
{
    FusedRow r;
    r.c.eta = u.eta; r.c.mu = u.mu; r.c.wd = u.wd; r.c.cL = u.lamL; r.c.cG = u.lamG;
    r.c.nesterov = (u.flags & LSGD_NESTEROV) != 0;
    r.c.grad_only = (u.flags & LSGD_MOMENTUM_GRAD_ONLY) != 0;
    const int j = u.group_of[w];
    if (u.flags & LSGD_LEADER_EXEMPT) {
        if (u.lamL != 0.0f && u.lead[j] == w) r.c.cL = 0.0f;
        if (u.lamG != 0.0f && u.glead[0] == w) r.c.cG = 0.0f;
    }
    r.x = u.x + (int64_t)w * ld;
    r.m = u.m ? u.m + (int64_t)w * ld : nullptr;
    r.xb = u.xb + (int64_t)w * ld;
    r.zl = (u.lamL != 0.0f) ? u.Z + (int64_t)j * ld : nullptr;
    r.zg = (u.lamG != 0.0f) ? u.Z + (int64_t)u.G * ld : nullptr;
    return r;
}

// N parameters at columns base + off[0..N) of the worker's row, gradient values gv: all loads first,
// then the arithmetic, then the stores (x, m, bf16 copy).
template <int N>
__device__ __forceinline__ void fused_apply(const FusedRow& r, int64_t base, const int (&off)[N], const float (&gv)[N])
{
    float* xp = r.x + base;
    float* mp = r.m ? r.m + base : nullptr;
    const float* lp = r.zl ? r.zl + base : nullptr;
    const float* gp = r.zg ? r.zg + base : nullptr;
    uint16_t* bp = r.xb + base;
    float xv[N], mv[N], zl[N], zg[N];
#pragma unroll
    for (int v = 0; v < N; ++v) xv[v] = xp[off[v]];
#pragma unroll
    for (int v = 0; v < N; ++v) mv[v] = mp ? mp[off[v]] : 0.f;
#pragma unroll
    for (int v = 0; v < N; ++v) zl[v] = lp ? lp[off[v]] : 0.f;
#pragma unroll
    for (int v = 0; v < N; ++v) zg[v] = gp ? gp[off[v]] : 0.f;
#pragma unroll
    for (int v = 0; v < N; ++v) {
        if (mp) update_vec<1, float>(xv[v], gv[v], mv[v], zl[v], zg[v], r.c);
        else update_vec<0, float>(xv[v], gv[v], mv[v], zl[v], zg[v], r.c);
    }
#pragma unroll
    for (int v = 0; v < N; ++v) {
        xp[off[v]] = xv[v];
        if (mp) mp[off[v]] = mv[v];
        bp[off[v]] = f32_to_bf16_rne(xv[v]);
    }
}

// R groups of four adjacent parameters (columns multiples of 4, rows 16-byte aligned) at element offsets
// `off` of the worker's row: the loads of one batch are issued as a block, so that they are in flight while the previous batch is updated and stored.
template <int R>
struct FusedBatch {
    int64_t off[R];
    f32x4 xv[R], mv[R], zl[R], zg[R];
};

template <int R>
__device__ __forceinline__ void fused_load4(const FusedRow& r, FusedBatch<R>& b)
{
    const f32x4 zero = (f32x4)(0.f);
#pragma unroll
    for (int q = 0; q < R; ++q) b.xv[q] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(r.x + b.off[q]));
#pragma unroll
    for (int q = 0; q < R; ++q) b.mv[q] = r.m ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(r.m + b.off[q])) : zero;
#pragma unroll
    for (int q = 0; q < R; ++q) b.zl[q] = r.zl ? *reinterpret_cast<const f32x4*>(r.zl + b.off[q]) : zero;
#pragma unroll
    for (int q = 0; q < R; ++q) b.zg[q] = r.zg ? *reinterpret_cast<const f32x4*>(r.zg + b.off[q]) : zero;
}

template <int R>
__device__ __forceinline__ void fused_store4(const FusedRow& r, FusedBatch<R>& b, const f32x4 (&gv)[R])
{
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (r.m) update_vec<1, f32x4>(b.xv[q], gv[q], b.mv[q], b.zl[q], b.zg[q], r.c);
        else update_vec<0, f32x4>(b.xv[q], gv[q], b.mv[q], b.zl[q], b.zg[q], r.c);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        __builtin_nontemporal_store(b.xv[q], reinterpret_cast<f32x4*>(r.x + b.off[q]));
        if (r.m) __builtin_nontemporal_store(b.mv[q], reinterpret_cast<f32x4*>(r.m + b.off[q]));
        const u32x2 o = {f32x2_to_bf16x2(b.xv[q].x, b.xv[q].y), f32x2_to_bf16x2(b.xv[q].z, b.xv[q].w)};
        *reinterpret_cast<u32x2*>(r.xb + b.off[q]) = o;
    }
}

// An operand given as [k][n] (n contiguous: the weights in the d-input product, the activations in the
// d-weight product) is staged in LDS as it lies in memory, 64 k-rows of BN + kPadN elements: the padding shifts
// consecutive rows by 64 bytes, i.e. a quarter of the banks, so that the four rows one transposing read touches
// cover all banks once.  The matrix cores want, per lane, eight consecutive k of one column n; the LDS
// transposing read delivers that: in every group of 16 lanes, lane i supplies the address of four consecutive
// elements, the 16 x 4 elements are taken as a 4 x 16 matrix (lanes 4r .. 4r+3 hold row r), and lane i receives
// column i.  With lanes 4r .. 4r+3 pointing at k-row r, columns n0 .. n0+15, lane i gets (k0 .. k0+3, n0 + i).
constexpr int kPadN = 32;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ s16x4 lds_read_tr(const uint16_t* p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
}

__device__ __forceinline__ void unpack8(const u32x4 v, float* f)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f[2 * q] = __uint_as_float(v[q] << 16);
        f[2 * q + 1] = __uint_as_float(v[q] & 0xFFFF0000u);
    }
}

// Sums over k of the rows of a [ROWS][K] operand as its tiles pass through LDS (rows of LD elements, BK of them live):
// THREADS / ROWS adjacent threads per row, eight partial sums each, so that the chains stay short.
template <int ROWS, int THREADS, int BK, int LD>
struct BiasSum {
    static constexpr int TPR = THREADS / ROWS, CHUNKS = BK / 8 / TPR;
    static_assert(TPR >= 1 && CHUNKS >= 1 && TPR * ROWS == THREADS && CHUNKS * TPR * 8 == BK, "tile shape");
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    static __device__ __forceinline__ int row(int tid) { return tid / TPR; }
    static __device__ __forceinline__ bool first(int tid) { return tid % TPR == 0; }
    __device__ __forceinline__ void add(const uint16_t* tile, int tid)
    {
        const uint16_t* p = tile + row(tid) * LD + (tid % TPR) * 8;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            float a[8];
            unpack8(*reinterpret_cast<const u32x4*>(p + c * TPR * 8), a);
#pragma unroll
            for (int q = 0; q < 8; ++q) s[q] += a[q];
        }
    }
    // valid in the first thread of a row
    __device__ __forceinline__ float row_sum() const
    {
        float v = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
#pragma unroll
        for (int d = 1; d < TPR; d <<= 1) v += __shfl_xor(v, d, 64);
        return v;
    }
};

// Bias gradient m of a layer: the M x N weights start at C, or at column colC of the parameter row, the biases follow.
template <int EPI>
__device__ __forceinline__ void store_bias_grad(const GemmArgs& g, int w, int m, float db)
{
    if (EPI == EPI_DWU) {
        const int off[1] = {0};
        const float gv[1] = {db};
        fused_apply<1>(fused_row(g.fu, w, g.sC), g.colC + (int64_t)g.M * g.N + m, off, gv);
    } else {
        g.C[(int64_t)w * g.sC + (int64_t)g.M * g.N + m] = db;
    }
}

// Forward and d-input products of 16-byte aligned operands (mlp_gemm_direct.hip): M a multiple of 128, N and K of 64;
// or, if it returns true, other sizes.  better_direct: whether it is the faster way for a product of more than two K steps.
bool better_direct(const GemmArgs& g, int W, int epi);
void launch_gemm_direct(const GemmArgs& g, int W, int epi, hipStream_t s);
bool launch_gemm_direct_any(const GemmArgs& g, int W, int epi, hipStream_t s);

// Matrix products of any shape and alignment (mlp_gemm_ragged.hip).
void launch_gemm_ragged(const GemmArgs& g, int W, int epi, hipStream_t s);
// Forward product of fp32 inputs g.A32, rounded to bf16 on their way; false (nothing launched) where a launch that converts
// them first is the better way.
bool launch_gemm_ragged_f32(const GemmArgs& g, int W, hipStream_t s);

// d-weight products (EPI_DW or EPI_DWU) of up to kGroupMax layers in one launch.
constexpr int kGroupMax = 6;
struct GemmGroup {
    GemmArgs g[kGroupMax];
    int n;
};
bool gemm_joins_group(const GemmArgs& g, int W, int epi);     // whether the product does not lose by it
void launch_gemm_group(const GemmGroup& q, int W, int epi, hipStream_t s);

} // namespace lsgd
