// Matrix products of the MLP path for any shape and alignment: batches that are no multiple of a tile, layer
// widths of any size (rows that start on any 2-byte boundary), the narrow classifier layer.
//
//   forward   out[m][n] = bf16(relu(<A[m,:], B[n,:]> + bias[n]))      A = h_{k-1}, B = W_k       (both [.][k])
//   logits    C[m][n]   = <A[m,:], B[n,:]> + bias[n]
//   head      the same for up to 64 classes, kept in LDS: softmax cross-entropy, its sum per row tile, output deltas, and
//             the classifier's d-input product where the caller asks for it
//   d-input   out[m][n] = bf16(sum_k A[m][k] B[k][n]) * [mask != 0]   A = delta_k, B = W_k       (B as [k][n])
//   d-weight  C[m][n]   = sum_k A[m][k] B[k][n]                       A = delta_k^T, B = h_{k-1}  (or the update)
//
// Loads are 16 bytes per lane at any 2-byte boundary.  Nothing outside an operand's rows is read: a row index past
// the end is clamped to the last row, a 16-byte piece past the end of a row is moved back to the row's last 16
// bytes and shifted into place (zeros behind it) on its way to LDS, so the K loop has no branches per lane.
//
// Tiles.  These shapes are small or have few rows per weight, so what counts is to have enough bytes in flight on
// enough compute units, not flops per LDS byte: BN = 64 columns (32 where tiles are few), 32 / 64 / 128 rows.  With 32 rows, and in the forward
// and d-input products with 64 (a whole small batch), the wavefronts split the contraction of one tile among them (K
// steps of 128, a quarter or a half each; 64 where the contraction is one step) instead of splitting the rows.  Few tiles
// with a long contraction take 32 x 32 tiles of sixteen wavefronts and K steps of 512, large forward batches 128 x 128
// tiles (launch_head, launch_epi).
//
// Sums.  One chain of v_mfma_f32_32x32x16_bf16 rounds its fp32 accumulator once per 16 products: measured 1.6e-7 of
// the result at K = 784 and 3.2e-7 at K = 3072 (normal operands), where a plain dot product spread over 64 lanes
// has 6e-8 and 8e-8.  Activations and back-propagated deltas are rounded to bf16 next, and the larger that error, the
// more of them land on the wrong side of a rounding boundary.  The forward and d-input products therefore carry a sum
// in double, to which the accumulators are added before they start again from zero: after every matrix instruction
// with 32-row tiles (1.6e-8 at any K), every two with 64 (2.7e-8), every eight with 128, where the vector units would
// become the limit (5.7e-8; 105 against 81 us without sums on 500 x 3072 x 1024, 16 workers).
//
// Measured (whole passes, against one-thread-per-output vector-ALU kernels that re-read an operand per output):
// gradients of 3072-1024-512-10, 16 workers, batch 32: 19.7 ms -> 0.10 ms; whole step of 784-300-100-10, 8 workers,
// batch 50: 1.26 -> 0.052 ms (4 to 9 us per product: launch and fill, not work).
#include <type_traits>

#include "mlp_common.h"

namespace lsgd {

namespace {

constexpr int kXcds = 8;

__device__ __forceinline__ u32x4 load16(const uint16_t* p) { return *reinterpret_cast<const u32x4_any*>(p); }
// weights: read by one tile row, or by a few workgroups of one die at a time, and not again in this launch
__device__ __forceinline__ u32x4 load16_once(const uint16_t* p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p)); }

// v moved down by s elements of 16 bits, zeros from above (s = 0 .. 8)
__device__ __forceinline__ u32x4 shift_in(u32x4 v, int s)
{
    uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
    if (s >= 4) { lo = hi; hi = 0; s -= 4; }
    if (s >= 4) { lo = 0; s = 0; }
    if (s > 0) { lo = (lo >> (16 * s)) | (hi << (64 - 16 * s)); hi >>= 16 * s; }
    return (u32x4){(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// rows shorter than 8 elements: element by element
__device__ __forceinline__ u32x4 load_short(const uint16_t* p, int n)
{
    uint32_t e[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) e[q] = q < n ? p[q] : 0;
    return (u32x4){e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
}

// the first n < 4 of four values
__device__ __forceinline__ void store_some(float* p, f32x4 v, int n)
{
#pragma unroll
    for (int e = 0; e < 3; ++e)
        if (e < n) p[e] = v[e];
}
__device__ __forceinline__ void store_some(uint16_t* p, u32x2 v, int n)
{
#pragma unroll
    for (int e = 0; e < 3; ++e)
        if (e < n) p[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
}

template <int R>
__device__ __forceinline__ void ragged_update(const FusedRow& r, const int64_t (&off)[R], const f32x4 (&gv)[R], const bool (&on)[R])
{
    const f32x4 zero = (f32x4)(0.f);
    f32x4 xv[R], mv[R], zl[R], zg[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        xv[q] = mv[q] = zl[q] = zg[q] = zero;
        if (on[q]) {
            xv[q] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(r.x + off[q]));
            if (r.m) mv[q] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(r.m + off[q]));
            if (r.zl) zl[q] = *reinterpret_cast<const f32x4_any*>(r.zl + off[q]);
            if (r.zg) zg[q] = *reinterpret_cast<const f32x4_any*>(r.zg + off[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (!on[q]) continue;
        if (r.m) update_vec<1, f32x4>(xv[q], gv[q], mv[q], zl[q], zg[q], r.c);
        else update_vec<0, f32x4>(xv[q], gv[q], mv[q], zl[q], zg[q], r.c);
        __builtin_nontemporal_store((f32x4_any)xv[q], reinterpret_cast<f32x4_any*>(r.x + off[q]));
        if (r.m) __builtin_nontemporal_store((f32x4_any)mv[q], reinterpret_cast<f32x4_any*>(r.m + off[q]));
        const u32x2 o = {f32x2_to_bf16x2(xv[q].x, xv[q].y), f32x2_to_bf16x2(xv[q].z, xv[q].w)};
        *reinterpret_cast<u32x2_any*>(r.xb + off[q]) = o;
    }
}

template <int BM, int BN, int WVM, int WVN, int WVK, int BK, int EPI>
struct RaggedShape {
    static constexpr int THREADS = 64 * WVM * WVN * WVK;
    static constexpr bool FORWARD = EPI == EPI_FWD || EPI == EPI_LOGITS || EPI == EPI_HEAD;
    static constexpr bool TRANS_B = !FORWARD;                           // B given as [k][n]
    static constexpr bool WIDE = FORWARD || (EPI == EPI_DX && (BK == 128 || BM == 128));   // (one K step: the chain is short)
    using Sum = typename std::conditional<WIDE, double, float>::type;
    static constexpr int EVERY = BM == 32 ? 1 : BM == 64 ? 2 : 8;       // matrix instructions between additions to the sum
    static constexpr int LDA = BK + 8;                                  // padded LDS row of a [.][k] operand
    static constexpr int LDN = BN + kPadN;                              // of a [k][n] operand
    static constexpr int A_TILE = BM * LDA;
    static constexpr int B_TILE = TRANS_B ? BK * LDN : BN * LDA;
    static constexpr int LDC = BN + 4;                                  // row of the result tile
    static constexpr size_t result_bytes = (size_t)WVK * BM * LDC * sizeof(Sum);
    // A contraction of one K step needs one buffer: three or four workgroups per compute unit instead of two where the
    // result is what costs (d-weight products of 3072-1024-512-10, 16 workers, batch 32: 54 -> 44 us).
    static constexpr size_t bytes(int buffers)
    {
        const size_t operands = (size_t)buffers * (A_TILE + B_TILE) * 2;
        return operands > result_bytes ? operands : result_bytes;
    }
    static constexpr size_t lds = bytes(2);
};

// A 16-byte piece of a row of A, or the eight fp32 values that become one.
struct F32Piece { f32x4 lo, hi; };
__device__ __forceinline__ u32x4 as_piece(const F32Piece& v)
{
    return (u32x4){f32x2_to_bf16x2(v.lo.x, v.lo.y), f32x2_to_bf16x2(v.lo.z, v.lo.w), f32x2_to_bf16x2(v.hi.x, v.hi.y), f32x2_to_bf16x2(v.hi.z, v.hi.w)};
}
__device__ __forceinline__ void load_piece(u32x4& v, const uint16_t* p) { v = load16(p); }
__device__ __forceinline__ void load_piece(F32Piece& v, const float* p)
{
    v.lo = *reinterpret_cast<const f32x4_any*>(p);
    v.hi = *reinterpret_cast<const f32x4_any*>(p + 4);
}

// Tile `id` of a product's tiles_m x tiles_n x W.  F32A: A in fp32, rows of at least 8 values.
template <int BM, int BN, int WVM, int WVN, int WVK, int BK, int EPI, bool F32A = false>
__device__ __forceinline__ void gemm_ragged_tile(const GemmArgs& g, int tiles_m, int tiles_n, int W, int64_t id)
{
    using S = RaggedShape<BM, BN, WVM, WVN, WVK, BK, EPI>;
    using Sum = typename S::Sum;
    constexpr bool TRANS_B = S::TRANS_B;
    constexpr int THREADS = S::THREADS, LDA = S::LDA, LDN = S::LDN, LDC = S::LDC;
    constexpr int TM = BM / WVM / 32, TN = BN / WVN / 32;               // 32x32 MFMA tiles per wavefront
    constexpr int KCH = BK / 8;                                         // 16-byte pieces of a [.][k] row
    constexpr int A_CHUNKS = BM * KCH / THREADS, B_CHUNKS = BN * BK / 8 / THREADS;
    constexpr int A_STEP = THREADS / KCH;                               // rows between a thread's pieces
    constexpr int KK = BK / 16 / WVK;                                   // MFMA steps of a wavefront per K step
    constexpr int NCH = BN / 8, B_STEP = THREADS / NCH;                 // [k][n]: pieces per row, rows between a thread's pieces

    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t* As = smem;                                                // [2][BM][LDA]
    uint16_t* Bs = smem + (g.K > BK ? 2 : 1) * S::A_TILE;               // [2][BN][LDA], or [2][BK][LDN] (one buffer each: one K step)

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wk = wid % WVK, wn = (wid / WVK) % WVN, wm = wid / (WVK * WVN);

    // Row tiles vary fastest, so that the tiles that share a weight tile, and the workgroups of a worker, which share
    // its activations, run on one die.  In the fused update the workers vary fastest instead: they share the leader
    // copies' tile.
    int w, tm, tn;
    if (EPI == EPI_DWU) {
        w = (int)(id % W);
        const int64_t tile = id / W;
        tn = (int)(tile % tiles_n); tm = (int)(tile / tiles_n);
    } else {
        tm = (int)(id % tiles_m);
        const int64_t r = id / tiles_m;
        tn = (int)(r % tiles_n); w = (int)(r / tiles_n);
    }
    const int m0 = tm * BM, n0 = tn * BN, M = g.M, N = g.N, K = g.K;
    using AElem = typename std::conditional<F32A, float, uint16_t>::type;
    using APiece = typename std::conditional<F32A, F32Piece, u32x4>::type;
    const AElem* A;
    if constexpr (F32A) A = g.A32 + (int64_t)w * g.sA;
    else A = g.A + (int64_t)w * g.sA;
    const uint16_t* B = g.B + (int64_t)w * g.sB;
    const bool short_k = !F32A && K < 8, short_n = TRANS_B && N < 8;             // uniform

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    Sum sum[S::WIDE ? TM : 1][S::WIDE ? TN : 1][16];
    if (S::WIDE) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[i][j][v] = 0;
    }
    auto promote = [&]() {
        if (!S::WIDE) return;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) { sum[i][j][v] += (Sum)acc[i][j][v]; acc[i][j][v] = 0.f; }
    };

    auto promote_pair = [&]() {                                          // after two K steps
        if (S::EVERY > KK) promote();
    };
    static_assert(S::EVERY <= KK || S::EVERY == 2 * KK || !S::WIDE, "sum cadence");

    // this thread's pieces: column piece kc of rows ra0 + c * A_STEP (a [k][n] operand: piece nc of rows kr0 + c * B_STEP)
    const int kc = (tid % KCH) * 8, ra0 = tid / KCH;
    const int nc = (tid % NCH) * 8, kr0 = tid / NCH;
    const AElem* arow[A_CHUNKS];
    const uint16_t* brow[B_CHUNKS];
#pragma unroll
    for (int c = 0; c < A_CHUNKS; ++c) {
        const int r = m0 + ra0 + c * A_STEP;
        arow[c] = A + (int64_t)(r < M ? r : M - 1) * g.lda;
    }
    if (!TRANS_B) {
#pragma unroll
        for (int c = 0; c < B_CHUNKS; ++c) {
            const int r = n0 + ra0 + c * A_STEP;
            brow[c] = B + (int64_t)(r < N ? r : N - 1) * g.ldb;
        }
    }
    const int bcol = n0 + nc, bcol_in = bcol < N - 8 ? bcol : N - 8;     // [k][n]: first column read
    const int bshift = bcol - bcol_in < 8 ? bcol - bcol_in : 8;
    const bool edge_n = n0 + BN > N;                                     // uniform

    auto load_global = [&](int kt, APiece* ra, u32x4* rb) {              // rows of at least 8 elements
        const int k = kt * BK + kc, kin = k < K - 8 ? k : K - 8;
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) load_piece(ra[c], arow[c] + kin);
#pragma unroll
        for (int c = 0; c < B_CHUNKS; ++c) {
            if (TRANS_B) {
                const int kr = kt * BK + kr0 + c * B_STEP;
                const uint16_t* p = B + (int64_t)(kr < K ? kr : K - 1) * g.ldb + bcol_in;
                rb[c] = EPI == EPI_DX ? load16_once(p) : load16(p);
            } else {
                rb[c] = load16_once(brow[c] + kin);
            }
        }
    };
    auto load_global_short = [&](int kt, u32x4* ra, u32x4* rb) {         // any length
        if constexpr (!F32A) {
        const int k = kt * BK + kc, n = K - k < 0 ? 0 : K - k;
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) ra[c] = load_short(arow[c] + k, n);
#pragma unroll
        for (int c = 0; c < B_CHUNKS; ++c) {
            if (TRANS_B) {
                const int kr = kt * BK + kr0 + c * B_STEP;
                rb[c] = load_short(B + (int64_t)(kr < K ? kr : K - 1) * g.ldb + bcol, kr < K && N > bcol ? N - bcol : 0);
            } else {
                rb[c] = load_short(brow[c] + k, n);
            }
        }
        }
    };
    auto store_lds = [&](int buf, int kt, u32x4* ra, u32x4* rb, bool shift) {
        uint16_t* as = As + buf * S::A_TILE;
        uint16_t* bs = Bs + buf * S::B_TILE;
        const bool tail = shift && (kt + 1) * BK > K;                    // uniform: the last K step, if it is not full
        if (tail) {
            const int k = kt * BK + kc, kin = k < K - 8 ? k : K - 8;
            const int s = k - kin < 8 ? k - kin : 8;
#pragma unroll
            for (int c = 0; c < A_CHUNKS; ++c) ra[c] = shift_in(ra[c], s);
            if (!TRANS_B) {
#pragma unroll
                for (int c = 0; c < B_CHUNKS; ++c) rb[c] = shift_in(rb[c], s);
            }
        }
        if (TRANS_B && (tail || (shift && edge_n))) {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) rb[c] = shift_in(rb[c], kt * BK + kr0 + c * B_STEP < K ? bshift : 8);
        }
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) *reinterpret_cast<u32x4*>(as + (ra0 + c * A_STEP) * LDA + kc) = ra[c];
        if (TRANS_B) {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) *reinterpret_cast<u32x4*>(bs + (kr0 + c * B_STEP) * LDN + nc) = rb[c];
        } else {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) *reinterpret_cast<u32x4*>(bs + (ra0 + c * A_STEP) * LDA + kc) = rb[c];
        }
    };
    // The first tile column of a product on fp32 inputs also leaves their bf16 copy (pieces that were moved back, and rows
    // past the end, write what is there already).
    uint16_t* const copy = F32A && g.copy && tn == 0 ? g.copy + (int64_t)w * g.sCopy : nullptr;      // uniform
    auto store_step = [&](int buf, int kt, APiece* pa, u32x4* rb) {
        if constexpr (F32A) {
            u32x4 ra[A_CHUNKS];
            const int k = kt * BK + kc, kin = k < K - 8 ? k : K - 8;
#pragma unroll
            for (int c = 0; c < A_CHUNKS; ++c) ra[c] = as_piece(pa[c]);
            if (copy) {
#pragma unroll
                for (int c = 0; c < A_CHUNKS; ++c) {
                    const int r = m0 + ra0 + c * A_STEP;
                    *reinterpret_cast<u32x4_any*>(copy + (int64_t)(r < M ? r : M - 1) * K + kin) = ra[c];
                }
            }
            store_lds(buf, kt, ra, rb, true);
        } else {
            store_lds(buf, kt, pa, rb, true);
        }
    };
    // the first tile column of a d-weight product also sums its rows of delta^T: the bias gradients
    constexpr bool BIAS = EPI == EPI_DW || EPI == EPI_DWU;
    const bool bias_rows = BIAS && tn == 0;                              // uniform
    BiasSum<BM, BIAS ? THREADS : BM, BK, LDA> bsum;
    auto compute = [&](int buf) {
        const uint16_t* as = As + buf * S::A_TILE;
        const uint16_t* bs = Bs + buf * S::B_TILE;
        if (BIAS && bias_rows) bsum.add(as, tid);
#pragma unroll
        for (int q = 0; q < KK; ++q) {
            const int kk = wk * KK + q;
            bf16x8 af[TM], bfr[TN];
            const int ch = kk * 2 + (lane >> 5);
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *reinterpret_cast<const bf16x8*>(as + ((wm * TM + i) * 32 + (lane & 31)) * LDA + ch * 8);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (TRANS_B) {
                    // lane (n = lane % 32, k-half = lane / 32): k = 16 kk + 8 (lane / 32) + 0..7 of column n
                    const int i = lane & 15;
                    const int col = (wn * TN + j) * 32 + (lane & 16) + 4 * (i & 3);
                    const int row = kk * 16 + 8 * (lane >> 5) + (i >> 2);
                    const s16x4 lo = lds_read_tr(bs + row * LDN + col);
                    const s16x4 hi = lds_read_tr(bs + (row + 4) * LDN + col);
                    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    bfr[j] = __builtin_bit_cast(bf16x8, v);
                } else {
                    bfr[j] = *reinterpret_cast<const bf16x8*>(bs + ((wn * TN + j) * 32 + (lane & 31)) * LDA + ch * 8);
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
            if (S::EVERY <= KK && (q + 1) % S::EVERY == 0) promote();
        }
    };

    // K loop: LDS holds steps kt (being multiplied) and kt + 1, registers the next two
    const int nk = (K + BK - 1) / BK;
    if (short_k || short_n) {                                            // rows of fewer than 8 elements: nothing in flight
        for (int kt = 0; kt < nk; ++kt) {
            u32x4 ra[A_CHUNKS], rb[B_CHUNKS];
            load_global_short(kt, ra, rb);
            store_lds(0, kt, ra, rb, false);
            __syncthreads();
            compute(0);
            promote_pair();
            __syncthreads();
        }
    } else {
        APiece ra[A_CHUNKS], qa[A_CHUNKS];
        u32x4 rb[B_CHUNKS], qb[B_CHUNKS];
        int kt = 0;
        load_global(0, ra, rb);
        if (nk > 4) {
            load_global(1, qa, qb);
            __builtin_amdgcn_sched_barrier(0);           // the two stages' loads in the order in which the loop waits for them
            store_step(0, 0, ra, rb);
            load_global(2, ra, rb);
            __syncthreads();
            // no conditional load in here: behind a branch around loads the compiler waits for all loads in flight
            for (; kt + 4 < nk; kt += 2) {
                store_step(1, kt + 1, qa, qb);
                load_global(kt + 3, qa, qb);
                compute(0);
                __syncthreads();
                store_step(0, kt + 2, ra, rb);
                load_global(kt + 4, ra, rb);
                compute(1);
                promote_pair();
                __syncthreads();
            }
        } else {
            if (nk > 1) load_global(1, qa, qb);
            store_step(0, 0, ra, rb);
            if (nk > 2) load_global(2, ra, rb);
            __syncthreads();
        }
        const int left = nk - kt;                                        // 1 .. 4 steps, the first already in buffer 0
        if (left > 1) store_step(1, kt + 1, qa, qb);
        if (left > 3) load_global(kt + 3, qa, qb);
        compute(0);
        __syncthreads();
        if (left > 1) {
            if (left > 2) store_step(0, kt + 2, ra, rb);
            compute(1);
            promote_pair();
            __syncthreads();
        }
        if (left > 2) {
            if (left > 3) store_step(1, kt + 3, qa, qb);
            compute(0);
            __syncthreads();
        }
        if (left > 3) {
            compute(1);
            __syncthreads();
        }
        promote_pair();
    }

    if (BIAS && bias_rows) {
        const float db = bsum.row_sum();
        const int m = m0 + bsum.row(tid);
        if (bsum.first(tid) && m < M) store_bias_grad<EPI>(g, w, m, db);
    }

    // The wavefronts' accumulators meet in LDS (lane: column lane % 32, rows (lane / 32) * 4 + 8 (v / 4) + v % 4 of
    // each 32x32 tile) and come back as four adjacent columns per thread.
    Sum* T = reinterpret_cast<Sum*>(smem);                              // [WVK][BM][LDC]
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = (wm * TM + i) * 32 + (lane >> 5) * 4 + 8 * (v >> 2) + (v & 3);
                T[(wk * BM + r) * LDC + (wn * TN + j) * 32 + (lane & 31)] = S::WIDE ? sum[S::WIDE ? i : 0][S::WIDE ? j : 0][v] : (Sum)acc[i][j][v];
            }
    __syncthreads();
    if constexpr (EPI == EPI_HEAD) {
        static_assert(BM == 32 && THREADS >= 256, "eight lanes per sample");
        __shared__ double row_loss[BM];
        __shared__ __attribute__((aligned(16))) uint16_t dl[BM][BN + 8];  // output deltas, zeros beyond M and N
        if (tid < 256) {
            const int r = tid >> 3, l = tid & 7, m = m0 + r;             // lane l of the sample's eight: classes l, l + 8, ...
            const int yb = m < M ? g.y[(int64_t)w * M + m] : -1;
            float z[BN / 8];
            float mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < BN / 8; ++j) {
                const int c = l + 8 * j;
                z[j] = -INFINITY;
                if (BN == 32 && 8 * j >= N) continue;                    // uniform: no such classes (here and below; with 64 columns the branches cost more)
                Sum v = T[r * LDC + c];
#pragma unroll
                for (int q = 1; q < WVK; ++q) v += T[(q * BM + r) * LDC + c];
                z[j] = c < N ? (float)(v + (Sum)g.bias[(int64_t)w * g.sBias + c]) : -INFINITY;
                mx = fmaxf(mx, z[j]);
            }
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
            float se = 0.f, zy = 0.f;
#pragma unroll
            for (int j = 0; j < BN / 8; ++j) {
                const int c = l + 8 * j;
                if (BN == 32 && 8 * j >= N) continue;
                if (c < N) se += expf(z[j] - mx);
                if (c < N && c == yb) zy = z[j];
            }
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) { se += __shfl_xor(se, d, 64); zy += __shfl_xor(zy, d, 64); }
            const float lse = mx + logf(se);
            if (l == 0) row_loss[r] = m < M ? (double)(lse - zy) : 0.0;
            if (g.out) {
                const float inv = 1.0f / (float)M;
#pragma unroll
                for (int j = 0; j < BN / 8; ++j) {
                    const int c = l + 8 * j;
                    uint16_t q = 0;
                    if (BN == 32 && 8 * j >= N) { dl[r][c] = 0; continue; }
                    if (m < M && c < N) {
                        q = f32_to_bf16_rne((expf(z[j] - lse) - (c == yb ? 1.f : 0.f)) * inv);
                        if (!g.dx) g.out[(int64_t)w * g.sOut + (int64_t)m * N + c] = q;
                        g.outT[(int64_t)w * g.sOut + (int64_t)c * M + m] = q;
                    }
                    dl[r][c] = q;
                }
            }
        }
        __syncthreads();
        if (g.dx) {
            // The d-input product of the classifier: its deltas are here.  A wavefront takes 32 columns at a time; lane
            // (n = lane % 32, k-half = lane / 32) reads eight rows of W at column n.
            bf16x8 af[BN / 16];
#pragma unroll
            for (int q = 0; q < BN / 16; ++q)
                af[q] = *reinterpret_cast<const bf16x8*>(&dl[lane & 31][q * 16 + 8 * (lane >> 5)]);
            uint16_t* const dx = g.dx + (int64_t)w * g.sOut + (int64_t)m0 * K;
            uint16_t* const dxT = g.dxT + (int64_t)w * g.sOut + m0;
            const uint16_t* const Am = A + (int64_t)m0 * g.lda;
            int half = lane >> 5, left = M - m0 < BM ? M - m0 : BM;
#pragma unroll 1
            for (int c0 = wid * 32; c0 < K; c0 += THREADS / 2) {
                asm("" : "+v"(half), "+v"(left));                        // or the loop carries a mask and an address per row
                const int n = c0 + (lane & 31), nin = n < K ? n : K - 1;
                uint16_t hv[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = half * 4 + 8 * (v >> 2) + (v & 3);
                    hv[v] = Am[(uint32_t)((r < left ? r : left - 1) * (int)g.lda + nin)];
                }
                f32x16 d;
#pragma unroll
                for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll
                for (int q = 0; q < BN / 16; ++q) {
                    if (BN == 32 && 16 * q >= N) break;
                    s16x8 b;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int c = q * 16 + 8 * half + e;             // past the last class: zero (a zero delta times infinity is not)
                        const uint16_t wv = B[(uint32_t)((c < N ? c : N - 1) * (int)g.ldb + nin)];
                        b[e] = c < N ? (short)wv : (short)0;
                    }
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[q], __builtin_bit_cast(bf16x8, b), d, 0, 0, 0);
                }
                if (n >= K) continue;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int r = half * 4 + 8 * p;
                    uint32_t o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        o[e] = hv[4 * p + e] == 0 ? 0u : (uint32_t)f32_to_bf16_rne(d[4 * p + e]);
                        if (r + e < left) dx[(uint32_t)((r + e) * K + n)] = (uint16_t)o[e];
                    }
                    const u32x2 t = {o[0] | o[1] << 16, o[2] | o[3] << 16};
                    uint16_t* const to = dxT + (int64_t)n * M + r;
                    if (r + 4 <= left) *reinterpret_cast<u32x2_any*>(to) = t;
                    else store_some(to, t, left - r);
                }
            }
        }
        if (tid == 0) {
            double t = 0.0;
            for (int r = 0; r < BM; ++r) t += row_loss[r];
            if (tiles_m == 1) g.losses[w] = (float)(t / (double)M);
            else g.loss_parts[(int64_t)w * g.sLoss + tm] = t;
        }
        if (g.pad && tm == 0)                                            // the padding columns of g are zero
            for (int64_t c = g.pad_from + tid; c < g.pad_to; c += THREADS) g.pad[(int64_t)w * g.pad_to + c] = 0.f;
        return;
    } else {
    constexpr int RPP = THREADS / (BN / 4) < BM ? THREADS / (BN / 4) : BM;   // rows per pass
    constexpr int PASSES = BM / RPP;
    if (THREADS / (BN / 4) > BM && tid >= BM * (BN / 4)) return;         // more threads than the tile has groups of four
    const int c4 = (tid % (BN / 4)) * 4, r0 = tid / (BN / 4), n = n0 + c4;
    const int nv = N - n < 4 ? N - n : 4;                               // columns of this thread (may be <= 0)
    typedef Sum sum4 __attribute__((ext_vector_type(4)));
    auto value = [&](int p) {
        sum4 v = *reinterpret_cast<const sum4*>(T + (r0 + RPP * p) * LDC + c4);
#pragma unroll
        for (int q = 1; q < WVK; ++q) v += *reinterpret_cast<const sum4*>(T + (q * BM + r0 + RPP * p) * LDC + c4);
        return v;
    };
    if constexpr (S::FORWARD) {
        sum4 b = (sum4)(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < nv) b[e] = g.bias[(int64_t)w * g.sBias + n + e];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int m = m0 + r0 + RPP * p;
            if (m >= M || nv <= 0) continue;
            const sum4 zs = value(p) + b;
            const f32x4 z = {(float)zs.x, (float)zs.y, (float)zs.z, (float)zs.w};
            if (EPI == EPI_LOGITS) {
                float* dst = g.C + (int64_t)w * g.sC + (int64_t)m * g.ldc + n;
                if (nv == 4) *reinterpret_cast<f32x4_any*>(dst) = z;
                else store_some(dst, z, nv);
            } else {
                uint16_t* dst = g.out + (int64_t)w * g.sOut + (int64_t)m * g.ldout + n;
                const u32x2 o = {f32x2_to_bf16x2(z.x > 0.f ? z.x : 0.f, z.y > 0.f ? z.y : 0.f),
                                 f32x2_to_bf16x2(z.z > 0.f ? z.z : 0.f, z.w > 0.f ? z.w : 0.f)};
                if (nv == 4) *reinterpret_cast<u32x2_any*>(dst) = o;
                else store_some(dst, o, nv);
            }
        }
        return;
    } else if constexpr (EPI == EPI_DX) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int m = m0 + r0 + RPP * p;
            sum4 v = value(p);
            if (m < M && nv > 0) {
                const uint16_t* mk = g.mask + (int64_t)w * g.sMask + (int64_t)m * g.ldmask + n;
                u32x2 h = {0u, 0u};
                if (nv == 4) h = *reinterpret_cast<const u32x2_any*>(mk);
                else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (e < nv) h[e >> 1] |= (uint32_t)mk[e] << (16 * (e & 1));
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (((h[e >> 1] >> (16 * (e & 1))) & 0xFFFFu) == 0) v[e] = 0;
                uint16_t* dst = g.out + (int64_t)w * g.sOut + (int64_t)m * g.ldout + n;
                const u32x2 o = {f32x2_to_bf16x2((float)v.x, (float)v.y), f32x2_to_bf16x2((float)v.z, (float)v.w)};
                if (nv == 4) *reinterpret_cast<u32x2_any*>(dst) = o;
                else store_some(dst, o, nv);
            }
            *reinterpret_cast<sum4*>(T + (r0 + RPP * p) * LDC + c4) = v;   // this thread's own elements of copy 0
        }
        __syncthreads();
        // the transposed copy: four samples of one column per thread
        constexpr int MQ = BM / 4, CPP = THREADS / MQ;            // threads per column, columns per pass
        const int mq = (tid % MQ) * 4, mm = m0 + mq;
        const int mv = M - mm < 4 ? M - mm : 4;
#pragma unroll
        for (int p = 0; p < BN / CPP; ++p) {
            const int col = tid / MQ + p * CPP;
            if (n0 + col >= N || mv <= 0) continue;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (float)T[(mq + e) * LDC + col];
            const u32x2 o = {f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3])};
            uint16_t* dst = g.outT + (int64_t)w * g.sOutT + (int64_t)(n0 + col) * g.ldoutT + mm;
            if (mv == 4) *reinterpret_cast<u32x2_any*>(dst) = o;
            else store_some(dst, o, mv);
        }
        return;
    } else if constexpr (EPI == EPI_DW) {
        float* C = g.C + (int64_t)w * g.sC;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int m = m0 + r0 + RPP * p;
            if (m >= M || nv <= 0) continue;
            const f32x4 v = value(p);
            float* dst = C + (int64_t)m * g.ldc + n;
            if (nv == 4) __builtin_nontemporal_store((f32x4_any)v, reinterpret_cast<f32x4_any*>(dst));
            else store_some(dst, v, nv);
        }
        return;
    } else {
    // EPI_DWU: the update in place of the store
    constexpr int R = PASSES < 4 ? PASSES : 4;                          // rows in flight per thread
    const FusedRow fr = fused_row(g.fu, w, g.sC);
#pragma unroll
    for (int p0 = 0; p0 < PASSES; p0 += R) {
        f32x4 gv[R];
        int64_t off[R];
        bool on[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int m = m0 + r0 + RPP * (p0 + q);
            gv[q] = value(p0 + q);
            off[q] = g.colC + (int64_t)m * g.ldc + n;
            on[q] = m < M && nv == 4;
            if (m < M && nv > 0 && nv < 4) {
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const int o1[1] = {0};
                    const float g1[1] = {gv[q][e]};
                    if (e < nv) fused_apply<1>(fr, off[q] + e, o1, g1);
                }
            }
        }
        ragged_update<R>(fr, off, gv, on);
    }
    }
    }
}

// A die (workgroup id modulo 8) takes a contiguous run of tiles.
template <int BM, int BN, int WVM, int WVN, int WVK, int BK, int EPI, bool F32A = false>
__global__ __launch_bounds__(64 * WVM * WVN * WVK, WVM * WVN * WVK == 4 ? 2 : 1) void gemm_ragged_kernel(GemmArgs g, int tiles_m, int tiles_n, int W, int64_t per_xcd)
{
    const int64_t id = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (id >= (int64_t)tiles_m * tiles_n * W) return;
    gemm_ragged_tile<BM, BN, WVM, WVN, WVK, BK, EPI, F32A>(g, tiles_m, tiles_n, W, id);
}

// Tiles of several products, of BM rows, or of 32 where a product has no more.  Every die takes a run of each product,
// the last product first (layer 1, mostly the largest: the short tiles of the classifier fill the end).  A launch of a
// few us per layer otherwise: 784-300-100-10, 8 workers, batch 50, 14 -> 7 us; with one run of all tiles per die, and
// so the short tiles on some dies only, 256-4096-10, 16 x 32, took 63 us for a gradient instead of 57.
template <int BM>
__host__ __device__ inline int64_t group_tiles(const GemmArgs& g, int W, int& tiles_m, int& tiles_n)
{
    tiles_m = g.M > 32 ? (g.M + BM - 1) / BM : 1;
    tiles_n = (g.N + 63) / 64;
    return (int64_t)tiles_m * tiles_n * W;
}

template <int BM, int EPI>
__global__ __launch_bounds__(256, 2) void gemm_group_kernel(GemmGroup q, int W)
{
    int64_t l = blockIdx.x / kXcds;
    for (int i = q.n - 1; i >= 0; --i) {                                 // uniform
        int tiles_m, tiles_n;
        const int64_t tiles = group_tiles<BM>(q.g[i], W, tiles_m, tiles_n), run = (tiles + kXcds - 1) / kXcds;
        if (l < run) {
            const int64_t id = (int64_t)(blockIdx.x % kXcds) * run + l;
            if (id >= tiles) return;
            if (q.g[i].M > 32) gemm_ragged_tile<BM, 64, 2, 2, 1, 64, EPI>(q.g[i], tiles_m, tiles_n, W, id);
            else gemm_ragged_tile<32, 64, 1, 2, 2, 64, EPI>(q.g[i], tiles_m, tiles_n, W, id);
            return;
        }
        l -= run;
    }
}

template <int BM, int EPI>
void launch_tiles(const GemmGroup& q, int W, hipStream_t s)
{
    using Big = RaggedShape<BM, 64, 2, 2, 1, 64, EPI>;
    using Small = RaggedShape<32, 64, 1, 2, 2, 64, EPI>;
    static_assert(Big::lds <= 64 * 1024 && Small::lds <= 64 * 1024, "no attribute set");
    int buffers = 1;
    for (int i = 0; i < q.n; ++i)
        if (q.g[i].K > 64) buffers = 2;
    const size_t big = Big::bytes(buffers), small = Small::bytes(buffers);
    int64_t runs = 0;
    int tm, tn;
    for (int i = 0; i < q.n; ++i) runs += (group_tiles<BM>(q.g[i], W, tm, tn) + kXcds - 1) / kXcds;
    hipLaunchKernelGGL((gemm_group_kernel<BM, EPI>), dim3((unsigned)(runs * kXcds)), dim3(256), big > small ? big : small, s, q, W);
}

// A gradient of one K step so large that three or four workgroups per compute unit, each writing its rows, are too many streams
// for the memory; from sixteen workers on.  Two / more, whole gradients, us, batch 32: 3072-2048-10, 16 workers, 128 / 139,
// 3072-1536-10 105 / 113, 3072-1024-10, 32 workers, 124 / 132; but 8 workers 3072-2048-10 85 / 81, 16 with 2048-1024-10 (134 MB) 76 / 70.
bool crowds(const GemmArgs& g, int W) { return W >= 16 && 4.0 * W * (double)g.M * g.N > 240e6; }

template <int BM, int BN, int WVM, int WVN, int WVK, int BK, int EPI, bool F32A = false>
void launch_tile(const GemmArgs& g, int W, hipStream_t s)
{
    using S = RaggedShape<BM, BN, WVM, WVN, WVK, BK, EPI>;
    auto kernel = gemm_ragged_kernel<BM, BN, WVM, WVN, WVK, BK, EPI, F32A>;
    static_assert(S::FORWARD || S::THREADS / (BN / 4) <= BM, "the other epilogues use every thread");
    if (S::lds > 64 * 1024) {
        static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::lds);
        (void)once;
    }
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const int64_t per_xcd = ((int64_t)tiles_m * tiles_n * W + kXcds - 1) / kXcds;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(per_xcd * kXcds)), dim3(S::THREADS), S::bytes(g.K > BK || (EPI == EPI_DW && crowds(g, W)) ? 2 : 1), s, g, tiles_m, tiles_n, W, per_xcd);
}

// Row tile: a batch of up to 32 / 64 fits one tile; larger ones take 128 rows, unless that leaves compute units
// without a workgroup.  When there are few tiles and a long contraction (the classifier layer, a narrow first
// layer), sixteen wavefronts split the contraction of a 32 x 32 tile, 64 KB of operands per K step: logits of
// 4096 -> 10, 8 workers, batch 256 25 -> 17 us, of 1024 -> 10, 16 workers, batch 128 11 -> 8 us; whole gradients of
// 256-73-377-10, 16 x 16, 36.7 -> 34.0 us, of 100-353-2, 15 x 128, 27.1 -> 25.0; at 256 units half the K step would be
// empty (256-256-10, 4 x 200, 12.4 -> 14.1).
void launch_head(const GemmArgs& g, int W, hipStream_t s)
{
    const int64_t tiles = (int64_t)W * ((g.M + 31) / 32);
    if (g.N <= 32 && g.K > 256 && tiles <= 512) launch_tile<32, 32, 1, 1, 16, 512, EPI_HEAD>(g, W, s);
    else if (g.N <= 32) launch_tile<32, 32, 1, 1, 4, 128, EPI_HEAD>(g, W, s);
    else launch_tile<32, 64, 1, 1, 4, 128, EPI_HEAD>(g, W, s);
}

// Whether a product has enough tiles of 64 columns and `rows` rows for every compute unit; whether it has so few, and so
// long a contraction, that sixteen wavefronts split one.
bool fills(const GemmArgs& g, int W, int rows) { return (int64_t)((g.N + 63) / 64) * W * ((g.M + rows - 1) / rows) >= 256; }
bool long_and_few(const GemmArgs& g, int W) { return g.K >= 1024 && (int64_t)((g.N + 63) / 64) * W * ((g.M + 31) / 32) <= 128; }

// Whether 32 rows go with 32 columns instead of 64.  What a workgroup of so few rows waits for is its own chain of K steps,
// most of it additions to the double sums, of which half as many columns have half; twice as many workgroups load A again.
// So while every narrow tile has a compute unit of its own, and where two or three rounds of them replace wide tiles that fill a
// second round badly; not where some units have two narrow tiles and would have had one wide one.  64 / 32 columns, us
// (the same bits): objective of 784-300-100-10, 8 workers, batch 50, 21.7 / 18.7, of 3072-1500-10, 12 x 16 (576 narrow tiles)
// 39.2 / 36.0; but with fp32 inputs of 2000-491-10, 20 x 32 (320 of them) 23.2 / 27.5, of 3072-1222-10, 10 x 64 (780) 46.5 / 55.0.
// 260 objectives and gradients: up to 256 narrow tiles 0.91 of the time; 257 to 448 1.03 forward, 0.98 d-input; 513 to 768 0.95,
// beyond 1.05.
template <int EPI>
bool narrow(const GemmArgs& g, int W)
{
    const int64_t tiles = (int64_t)((g.N + 31) / 32) * W * ((g.M + 31) / 32);
    return tiles <= (EPI == EPI_DX ? 320 : 256) || (tiles > 512 && tiles <= 768);
}

template <int EPI>
void launch_epi(const GemmArgs& g, int W, hipStream_t s)
{
    const bool fill64 = fills(g, W, 64), fill128 = fills(g, W, 128);
    if constexpr (EPI == EPI_DW || EPI == EPI_DWU) {
        if (g.M > 64 && fill128) launch_tile<128, 64, 2, 2, 1, 64, EPI>(g, W, s);
        else if (g.M > 32) launch_tile<64, 64, 2, 2, 1, 64, EPI>(g, W, s);
        else launch_tile<32, 64, 1, 2, 2, 64, EPI>(g, W, s);
    } else {
        // one K step (the classifier layer's d-input): a stream of results, many small workgroups
        if constexpr (EPI == EPI_DX) {
            if (g.K <= 64) {
                if (g.M > 32) launch_tile<64, 64, 2, 2, 1, 64, EPI>(g, W, s);
                else launch_tile<32, 64, 1, 2, 2, 64, EPI>(g, W, s);
                return;
            }
        }
        if constexpr (EPI == EPI_FWD || EPI == EPI_LOGITS) {
            if (long_and_few(g, W)) {
                launch_tile<32, 32, 1, 1, 16, 512, EPI>(g, W, s);
                return;
            }
        }
        if constexpr (EPI == EPI_FWD) {
            // large batches are bound by what reaches the compute units through L2: fewer bytes per product
            if (g.M > 128 && (int64_t)((g.N + 127) / 128) * ((g.M + 127) / 128) * W >= 256) {
                launch_tile<128, 128, 2, 4, 1, 64, EPI>(g, W, s);
                return;
            }
        }
        if (g.M > 64 && fill128) launch_tile<128, 64, 2, 2, 1, 64, EPI>(g, W, s);
        else if (g.M > 32 && fill64) launch_tile<64, 64, 1, 2, 2, 128, EPI>(g, W, s);
        else if (narrow<EPI>(g, W)) launch_tile<32, 32, 1, 1, 4, 128, EPI>(g, W, s);
        else launch_tile<32, 64, 1, 1, 4, 128, EPI>(g, W, s);
    }
}

template <int EPI>
void launch_group_epi(const GemmGroup& q, int W, hipStream_t s)
{
    int64_t tiles = 0;                                       // of 128 rows
    int widest = 0, tm, tn;
    for (int i = 0; i < q.n; ++i) {
        tiles += group_tiles<128>(q.g[i], W, tm, tn);
        if (q.g[i].M > widest) widest = q.g[i].M;
    }
    if (widest > 64 && tiles >= 256) launch_tiles<128, EPI>(q, W, s);
    else launch_tiles<64, EPI>(q, W, s);
}

} // namespace

// Large products are better off alone: the launch that a group saves is nothing to them, and with more than one K step its kernel is
// the slower one.  Alone / in a group with the classifier's, whole gradients, us, 16 workers, batch 100: 3072-2000-10 (393 MB of
// gradients) 174 / 191, 3072-1000-10 (197 MB) 99 / 104, but 3072-512-10 (100 MB) 65.5 / 64.7, 1000-2000-10 (128 MB) 97 / 96.
bool gemm_joins_group(const GemmArgs& g, int W, int epi)
{
    const double bytes = 4.0 * W * (double)g.M * g.N;
    return g.K > 64 ? bytes <= 150e6 : !(epi == EPI_DW && crowds(g, W));
}

void launch_gemm_group(const GemmGroup& q, int W, int epi, hipStream_t s)
{
    if (q.n == 1) launch_gemm_ragged(q.g[0], W, epi, s);
    else if (epi == EPI_DW) launch_group_epi<EPI_DW>(q, W, s);
    else launch_group_epi<EPI_DWU>(q, W, s);
}

// The 32-row tile converts as it goes: its products are small enough that a launch for the conversion counts and reading
// the inputs in fp32 once per tile of columns does not.  Objective of 617-132-10, 3 workers, batch 16, 14.2 -> 12.4 us, step of
// 784-300-100-10, 8 x 50, 51.9 -> 50.6; 47 drawn calls, part of them of this size, 0.966 of the time.  Where every 64 columns read
// more than 90 MB a second time in all, the launch is the cheaper way: gradients, launch of its own / as it goes, us, batch 32,
// 3072-4096-10, 16 workers (201 MB) 278 / 288, 8 (101 MB) 155.7 / 158.5; 3072-2048-10, 16 (101 MB) 148 / 150, 8 (50 MB) 86.9 / 86.6.
// It is the 64 columns that are counted, also where tiles have 32 and read twice as much (objectives, launch of its own / 32 / 64
// columns as it goes, 384 and 363 wide tiles: 3072-2048-10, 12 x 32 (75 MB by 64) 49.3 / 49.3 / 49.0; 3072-723-10, 32 x 32 (75 MB)
// 54.4 / 47.4 / 47.0; the other way 4096-2666-10, 8 x 32 (88 MB) 55.4 / 59.9 / 59.2): what the launch saves depends on how often
// an input is read, what it costs on how large the inputs are, and the volume is no more than their product.
// The larger tiles have no registers for fp32 pieces in flight.
bool launch_gemm_ragged_f32(const GemmArgs& g, int W, hipStream_t s)
{
    if (2.0 * W * (double)g.M * g.K * ((g.N + 63) / 64) > 90e6) return false;
    if (g.K < 8 || long_and_few(g, W) || (g.M > 32 && fills(g, W, 64)) || (g.M > 64 && fills(g, W, 128))) return false;
    if (narrow<EPI_FWD>(g, W)) launch_tile<32, 32, 1, 1, 4, 128, EPI_FWD, true>(g, W, s);
    else launch_tile<32, 64, 1, 1, 4, 128, EPI_FWD, true>(g, W, s);
    return true;
}

void launch_gemm_ragged(const GemmArgs& g, int W, int epi, hipStream_t s)
{
    switch (epi) {
    case EPI_FWD: launch_epi<EPI_FWD>(g, W, s); break;
    case EPI_LOGITS: launch_epi<EPI_LOGITS>(g, W, s); break;
    case EPI_HEAD: launch_head(g, W, s); break;
    case EPI_DX: launch_epi<EPI_DX>(g, W, s); break;
    case EPI_DW: launch_epi<EPI_DW>(g, W, s); break;
    case EPI_DWU: launch_epi<EPI_DWU>(g, W, s); break;
    }
}

} // namespace lsgd
