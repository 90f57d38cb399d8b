// Per-worker gradient and loss of a fully connected ReLU classifier with softmax
// cross-entropy, for all W workers of the population at once (each worker has
// its own weights).  This is the stochastic gradient g_t^{j,i} that a worker
// takes on its own minibatch in arXiv 1905.10395 (Section 2), for the MLP
// workload: bf16 matrix operands, fp32 accumulation, fp32 gradients.
//
//   forward   z_k = h_{k-1} W_k^T + b_k ; h_k = bf16(relu(z_k)) ; logits fp32
//   loss      mean_b (logsumexp(z_L) - z_L[y_b]) ; delta_L = bf16((softmax - onehot)/B)
//   backward  dW_k = delta_k^T h_{k-1} ; db_k = sum_b delta_k ;
//             delta_{k-1} = bf16((delta_k W_k) .* [h_{k-1} > 0])
//
// The three matrix products are dense contractions and run on the matrix
// cores (v_mfma_f32_32x32x16_bf16).  Shapes that are multiples of the tile sizes
// with 16-byte aligned rows: d-weight products, and forward and d-input products of one or two
// K steps, with large weights that are used once, or that fill the chip with 256 x 256 tiles, with
// the kernel in this file, other forward and d-input products with mlp_gemm_direct.hip, which also takes other sizes of aligned rows;
// the rest with the any-shape kernel (mlp_gemm_ragged.hip), the narrow classifier layer included.
//
// Operand layouts for the MFMA kernel.  A lane feeds the matrix core eight
// consecutive values along the contraction index:
//   forward : A = h_{k-1} [B][d_in]   B-operand = W_k [d_out][d_in]    both contiguous in d_in
//   d-input : A = delta_k [B][d_out]  B-operand = W_k [d_out][d_in]    contraction over d_out: rows of W
//   d-weight: A = delta_k^T [d_out][B] B-operand = h_{k-1} [B][d_in]   contraction over B: rows of h
// In the last two the B-operand is contiguous along the *output* column.  Its
// tile is staged in LDS as it lies in memory and the fragments are fetched
// with the LDS transposing read (see lds_read_tr).  delta_k is stored in both
// layouts by the kernel that produces it.
#include "mlp_common.h"

namespace lsgd {

constexpr int kBK = 64;          // contraction tile
constexpr int kLdk = kBK + 8;    // padded LDS row (bf16 elements): 144 B

// BM x BN output tile per workgroup, WVM x WVN wavefronts, each owning (BM/WVM) x (BN/WVN).
// 128x128 / 128x64 with 2x2 wavefronts run two workgroups per CU; 256x256 with 2x4 wavefronts
// (128x64 per wavefront, all 147 KB of LDS) moves half the bytes through LDS per flop.
template <int BM, int BN, int WVM, int WVN, bool TRANS_B, int EPI>
__global__ __launch_bounds__(64 * WVM * WVN, (WVM * WVN > 4) ? 1 : 2) void gemm_bf16_kernel(GemmArgs g)  // min. workgroups per CU
{
    constexpr int kGemmThreads = 64 * WVM * WVN;
    constexpr int WTM = BM / WVM, WTN = BN / WVN;
    constexpr int TM = WTM / 32, TN = WTN / 32;      // 32x32 MFMA tiles per wavefront
    constexpr int A_CHUNKS = BM * (kBK / 8) / kGemmThreads; // 16-byte chunks per thread
    constexpr int B_CHUNKS = BN * (kBK / 8) / kGemmThreads;
    constexpr int LDN = BN + kPadN;                  // row of a [k][n]-staged tile
    constexpr int B_TILE = TRANS_B ? kBK * LDN : BN * kLdk;   // elements of one B buffer
    constexpr int STAGES = (TM * TN > 4) ? 1 : 2;    // register stages of global prefetch (one beside 128 accumulator registers)

    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t* As = smem;                              // [2][BM][kLdk]
    uint16_t* Bs = smem + 2 * BM * kLdk;              // [2][BN][kLdk], or [2][kBK][LDN] for a [k][n] operand

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WVN, wn = wid % WVN;
    // Fused update: a die (workgroup id modulo 8) owns every eighth tile column, and visits its tiles
    // row by row with the workers varying fastest.  All workers' workgroups for one tile then run
    // together on one die, so the tile of the leader copies they share is fetched into that die's L2
    // once; a worker's delta^T tile is reused across the die's columns and its h tiles across rows.
    int w, tm, tn;
    if (EPI == EPI_DWU) {
        const int W = (int)gridDim.z, tiles_n = (int)gridDim.x;
        const int64_t id = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        if (tiles_n % 8 == 0) {
            const int xcd = (int)(id & 7);
            int64_t s = id >> 3;
            w = (int)(s % W); s /= W;
            const int per = tiles_n / 8;
            tn = (int)(s % per) * 8 + xcd;
            tm = (int)(s / per);
        } else {
            w = (int)(id % W);
            const int64_t tile = id / W;
            tn = (int)(tile % tiles_n); tm = (int)(tile / tiles_n);
        }
    } else {
        // The other products: a die takes a contiguous run of tiles, row tiles varying fastest, then columns, then
        // workers, so that a worker's activations stay in one die's L2 while its weights stream through (plain grid
        // order spreads every worker over all dies; gradients of 3072-1024-1024-10, 16 workers, batch 128: 148.5 -> 140.0
        // us, of 1024-2048-2048-10, 8 workers, batch 256: 167.1 -> 163.3; the whole fused steps gain 0.2 %).
        const int64_t total = (int64_t)gridDim.x * gridDim.y * gridDim.z;
        const int64_t id = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        int64_t s = total % 8 == 0 ? (id & 7) * (total / 8) + (id >> 3) : id;
        tm = (int)(s % gridDim.y); s /= gridDim.y;
        tn = (int)(s % gridDim.x); w = (int)(s / gridDim.x);
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const uint16_t* A = g.A + (int64_t)w * g.sA + (int64_t)m0 * g.lda;
    const uint16_t* B = g.B + (int64_t)w * g.sB;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // two register stages: the loads of k-steps kt+1 and kt+2 are in flight while kt is multiplied
    constexpr int RB = B_CHUNKS;
    u32x4 ra0[A_CHUNKS], ra1[STAGES == 2 ? A_CHUNKS : 1];
    u32x4 rb0[RB], rb1[STAGES == 2 ? RB : 1];

    auto load_global = [&](int kt, u32x4* ra, u32x4* rb) {
        const int k0 = kt * kBK;
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) {
            const int id = tid + c * kGemmThreads, row = id >> 3, ch = id & 7;
            ra[c] = *reinterpret_cast<const u32x4*>(A + (int64_t)row * g.lda + k0 + ch * 8);
        }
        if (TRANS_B) {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) {
                const int id = tid + c * kGemmThreads, row = id / (BN / 8), ch = id % (BN / 8);
                const u32x4* p = reinterpret_cast<const u32x4*>(B + (int64_t)(k0 + row) * g.ldb + n0 + ch * 8);
                rb[c] = EPI == EPI_DX ? __builtin_nontemporal_load(p) : *p;      // weights: once per tile row
            }
        } else {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) {
                const int id = tid + c * kGemmThreads, row = id >> 3, ch = id & 7;
                rb[c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(B + (int64_t)(n0 + row) * g.ldb + k0 + ch * 8));
            }
        }
    };
    auto store_lds = [&](int buf, const u32x4* ra, const u32x4* rb) {
        uint16_t* as = As + buf * BM * kLdk;
        uint16_t* bs = Bs + buf * B_TILE;
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) {
            const int id = tid + c * kGemmThreads, row = id >> 3, ch = id & 7;
            *reinterpret_cast<u32x4*>(as + row * kLdk + ch * 8) = ra[c];
        }
        if (TRANS_B) {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) {
                const int id = tid + c * kGemmThreads, row = id / (BN / 8), ch = id % (BN / 8);
                *reinterpret_cast<u32x4*>(bs + row * LDN + ch * 8) = rb[c];
            }
        } else {
#pragma unroll
            for (int c = 0; c < B_CHUNKS; ++c) {
                const int id = tid + c * kGemmThreads, row = id >> 3, ch = id & 7;
                *reinterpret_cast<u32x4*>(bs + row * kLdk + ch * 8) = rb[c];
            }
        }
    };

    // The first tile column of a d-weight product also sums its rows of delta^T: the bias gradients.
    constexpr bool BIAS = EPI == EPI_DW || EPI == EPI_DWU;
    const bool bias_rows = BIAS && tn == 0;               // uniform
    BiasSum<BM, kGemmThreads, kBK, kLdk> bsum;
    auto compute = [&](int buf) {
        const uint16_t* as = As + buf * BM * kLdk;
        const uint16_t* bs = Bs + buf * B_TILE;
        if (BIAS && bias_rows) bsum.add(as, tid);
#pragma unroll
        for (int kk = 0; kk < kBK / 16; ++kk) {
            bf16x8 af[TM], bfr[TN];
            const int ch = kk * 2 + (lane >> 5);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * WTM + i * 32 + (lane & 31);
                af[i] = *reinterpret_cast<const bf16x8*>(as + row * kLdk + ch * 8);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (TRANS_B) {
                    // lane (n = lane % 32, k-half = lane / 32): k = 16 kk + 8 (lane / 32) + 0..7 of column n
                    const int i = lane & 15;
                    const int col = wn * WTN + j * 32 + (lane & 16) + 4 * (i & 3);
                    const int row = kk * 16 + 8 * (lane >> 5) + (i >> 2);
                    const s16x4 lo = lds_read_tr(bs + row * LDN + col);
                    const s16x4 hi = lds_read_tr(bs + (row + 4) * LDN + col);
                    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    bfr[j] = __builtin_bit_cast(bf16x8, v);
                } else {
                    const int row = wn * WTN + j * 32 + (lane & 31);
                    bfr[j] = *reinterpret_cast<const bf16x8*>(bs + row * kLdk + ch * 8);
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
    };

    // Pipeline.  LDS holds k-steps kt (being multiplied) and kt+1.  Each iteration first hands the
    // register stage that has arrived to LDS (into the buffer nobody reads now) and re-issues it for
    // a later k-step, then multiplies: LDS writes and global loads drain underneath the MFMAs.
    // Two register stages (k-steps kt+1 and kt+2 in flight) where registers allow, else one.
    const int nk = g.K / kBK;
    if (STAGES == 2) {
        load_global(0, ra0, rb0);
        if (nk > 1) load_global(1, ra1, rb1);
        store_lds(0, ra0, rb0);
        if (nk > 2) load_global(2, ra0, rb0);
        __syncthreads();
        int kt = 0;
        // No load in here is conditional: behind a branch that may or may not have issued loads, the compiler has to
        // wait for every load in flight, and the second register stage would be worth nothing.
        for (; kt + 4 < nk; kt += 2) {
            store_lds(1, ra1, rb1);
            load_global(kt + 3, ra1, rb1);
            compute(0);
            __syncthreads();
            store_lds(0, ra0, rb0);
            load_global(kt + 4, ra0, rb0);
            compute(1);
            __syncthreads();
        }
        const int left = nk - kt;                         // 1 .. 4 k-steps, the first already in buffer 0
        if (left > 1) store_lds(1, ra1, rb1);
        if (left > 3) load_global(kt + 3, ra1, rb1);
        compute(0);
        __syncthreads();
        if (left > 1) {
            if (left > 2) store_lds(0, ra0, rb0);
            compute(1);
            __syncthreads();
        }
        if (left > 2) {
            if (left > 3) store_lds(1, ra1, rb1);
            compute(0);
            __syncthreads();
        }
        if (left > 3) {
            compute(1);
            __syncthreads();
        }
    } else {
        load_global(0, ra0, rb0);
        store_lds(0, ra0, rb0);
        if (nk > 1) load_global(1, ra0, rb0);
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            const int buf = kt & 1;
            if (kt + 1 < nk) store_lds(buf ^ 1, ra0, rb0);
            if (kt + 2 < nk) load_global(kt + 2, ra0, rb0);
            compute(buf);
            __syncthreads();
        }
    }

    if (BIAS && bias_rows) {
        const float db = bsum.row_sum();
        if (bsum.first(tid)) store_bias_grad<EPI>(g, w, m0 + bsum.row(tid), db);
    }

    // epilogue: lane holds column n = lane%32 and rows (lane/32)*4 + 8*(v/4) + v%4 of each 32x32 tile
    if (EPI == EPI_DWU) {
        // The update streams x, m and the leader copies, so it wants whole rows per wavefront: the
        // accumulators go through LDS (reusing the operand buffers), 32 rows of every wavefront row at a
        // time, and come back as float4 per thread with a wavefront covering contiguous row segments.
        constexpr int LDC = BN + 4;                       // padded fp32 row
        constexpr int CH_ROWS = WVM * 32;                 // rows staged at a time
        constexpr int C4 = BN / 4;                        // float4 per row
        constexpr int RPP = kGemmThreads / C4;            // rows covered by one pass of all threads
        constexpr int PASSES = CH_ROWS / RPP;
        constexpr int R = PASSES < 4 ? PASSES : 4;        // rows in flight per thread
        static_assert(CH_ROWS % RPP == 0 && PASSES % R == 0, "tile shape");
        float* stage = reinterpret_cast<float*>(smem);
        const FusedRow fr = fused_row(g.fu, w, g.sC);
        const int c4 = tid % C4, r0 = tid / C4;
        constexpr int BPR = PASSES / R;                   // batches per staged block of rows
        constexpr int NB = TM * BPR;
        FusedBatch<R> fb[2];
        auto set_cols = [&](int bi, FusedBatch<R>& b) {   // batch bi = (staged block, pass group)
            const int i = bi / BPR, p0 = (bi % BPR) * R;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int rr = r0 + (p0 + q) * RPP;        // row inside the staged block
                const int m = m0 + (rr >> 5) * WTM + i * 32 + (rr & 31);
                b.off[q] = g.colC + (int64_t)m * g.ldc + n0 + c4 * 4;
            }
        };
        set_cols(0, fb[0]);
        fused_load4<R>(fr, fb[0]);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            __syncthreads();                              // operand buffers / previous block no longer read
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int rl = wm * 32 + (lane >> 5) * 4 + 8 * (v >> 2) + (v & 3);
                    stage[rl * LDC + wn * WTN + j * 32 + (lane & 31)] = acc[i][j][v];
                }
            __syncthreads();
#pragma unroll
            for (int qb = 0; qb < BPR; ++qb) {
                const int bi = i * BPR + qb;
                if (bi + 1 < NB) {                        // next batch's loads fly while this one is finished
                    set_cols(bi + 1, fb[(bi + 1) & 1]);
                    fused_load4<R>(fr, fb[(bi + 1) & 1]);
                }
                f32x4 gv[R];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int rr = r0 + (qb * R + q) * RPP;
                    gv[q] = *reinterpret_cast<const f32x4*>(stage + rr * LDC + c4 * 4);
                }
                fused_store4<R>(fr, fb[bi & 1], gv);
            }
        }
        return;
    }
    if (EPI == EPI_FWD || EPI == EPI_DX) {
        // bf16 results leave through LDS (the operand buffers are free now): lanes hold single columns, a
        // row-major tile in LDS turns them into 16-byte pieces of rows, 256 contiguous bytes per 16 lanes.
        constexpr int LDT = BN + kPadN;                   // rows shift by 64 bytes, as for the transposing read
        constexpr int T_CHUNKS = BM * (BN / 8) / kGemmThreads;
        static_assert((size_t)BM * LDT <= (size_t)2 * (BM * kLdk + B_TILE), "result tile fits the operand buffers");
        uint16_t* T = smem;
        uint16_t* out = g.out + (int64_t)w * g.sOut;
        if (EPI == EPI_DX) {
            // the ReLU mask (h_{k-1} != 0) arrives as 16-byte pieces too and is read back per lane with the
            // transposing read: rows R .. R+3 of the lane's own column, the layout of four accumulators
            const uint16_t* mask = g.mask + (int64_t)w * g.sMask;
            u32x4 mk[T_CHUNKS];
#pragma unroll
            for (int c = 0; c < T_CHUNKS; ++c) {
                const int id = tid + c * kGemmThreads, row = id / (BN / 8), ch = id % (BN / 8);
                mk[c] = *reinterpret_cast<const u32x4*>(mask + (int64_t)(m0 + row) * g.ldmask + n0 + ch * 8);
            }
#pragma unroll
            for (int c = 0; c < T_CHUNKS; ++c) {
                const int id = tid + c * kGemmThreads, row = id / (BN / 8), ch = id % (BN / 8);
                *reinterpret_cast<u32x4*>(T + row * LDT + ch * 8) = mk[c];
            }
            __syncthreads();
        }
        uint16_t* outT = (EPI == EPI_DX) ? g.outT + (int64_t)w * g.sOutT : nullptr;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int nl = wn * WTN + j * 32 + (lane & 31);               // column inside the tile
                const int rb = wm * WTM + i * 32 + (lane >> 5) * 4;            // first row inside the tile
                if (EPI == EPI_FWD) {
                    const float b = g.bias[(int64_t)w * g.sBias + n0 + nl];
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float z = acc[i][j][v] + b;
                        T[(rb + 8 * (v >> 2) + (v & 3)) * LDT + nl] = f32_to_bf16_rne(z > 0.f ? z : 0.f);
                    }
                } else {
                    const int l16 = lane & 15;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // every 4 x 16 block of the tile is read and then overwritten by the same 16 lanes
                        const s16x4 on = lds_read_tr(T + (rb + 8 * q + (l16 >> 2)) * LDT + wn * WTN + j * 32 + (lane & 16) + 4 * (l16 & 3));
                        uint32_t pk[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const uint16_t d = on[r] != 0 ? f32_to_bf16_rne(acc[i][j][q * 4 + r]) : (uint16_t)0;
                            T[(rb + 8 * q + r) * LDT + nl] = d;
                            pk[r] = d;
                        }
                        // the transposed copy: the lane's four rows are 8 contiguous bytes of it
                        const u32x2 o = {pk[0] | (pk[1] << 16), pk[2] | (pk[3] << 16)};
                        *reinterpret_cast<u32x2*>(outT + (int64_t)(n0 + nl) * g.ldoutT + m0 + rb + 8 * q) = o;
                    }
                }
            }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < T_CHUNKS; ++c) {
            const int id = tid + c * kGemmThreads, row = id / (BN / 8), ch = id % (BN / 8);
            *reinterpret_cast<u32x4*>(out + (int64_t)(m0 + row) * g.ldout + n0 + ch * 8) = *reinterpret_cast<const u32x4*>(T + row * LDT + ch * 8);
        }
        return;
    }
    float* C = g.C + (int64_t)w * g.sC;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + wn * WTN + j * 32 + (lane & 31);
            const int mb = m0 + wm * WTM + i * 32 + (lane >> 5) * 4;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = mb + 8 * (v >> 2) + (v & 3);
                __builtin_nontemporal_store(acc[i][j][v], C + (int64_t)m * g.ldc + n);
            }
        }
}

template <int BM, int BN, int WVM, int WVN, bool TRANS_B, int EPI>
static void launch_gemm(const GemmArgs& g, int W, hipStream_t s)
{
    const size_t lds = (size_t)2 * (BM * kLdk + (TRANS_B ? kBK * (BN + kPadN) : BN * kLdk)) * sizeof(uint16_t);
    static bool configured = false;
    if (!configured) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<BM, BN, WVM, WVN, TRANS_B, EPI>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        configured = true;
    }
    dim3 grid((unsigned)(g.N / BN), (unsigned)(g.M / BM), (unsigned)W);
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WVM, WVN, TRANS_B, EPI>), grid, dim3(64 * WVM * WVN), lds, s, g);
}

static bool aligned_for_mfma(const GemmArgs& g)
{
    auto a16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    return a16(g.A) && a16(g.B) && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.sA % 8 == 0 && g.sB % 8 == 0;
}

// Whether the shape is whole tiles of aligned rows.
template <bool TRANS_B, int EPI>
static bool mfma_fits(const GemmArgs& g)
{
    if (g.K % kBK || g.M % 128 || g.N % 64 || !aligned_for_mfma(g)) return false;
    if (EPI == EPI_DX && (g.ldoutT % 4 || (reinterpret_cast<uintptr_t>(g.outT) & 7u) || g.sOutT % 4)) return false;
    if (EPI == EPI_FWD || EPI == EPI_DX) {                 // 16-byte pieces of the result rows (and of the mask rows)
        auto a16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
        if (!a16(g.out) || g.ldout % 8 || g.sOut % 8) return false;
        if (EPI == EPI_DX && (!a16(g.mask) || g.ldmask % 8 || g.sMask % 8)) return false;
    }
    if (EPI == EPI_DWU) {                                  // float4 rows of x, m, Z; 8-byte groups of the bf16 copy
        auto a16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
        if (g.colC % 4 || g.ldc % 4 || g.sC % 4 || !a16(g.fu.x) || !a16(g.fu.m) || !a16(g.fu.Z) ||
            (reinterpret_cast<uintptr_t>(g.fu.xb) & 7u))
            return false;
    }
    return true;
}

// Picks the largest tile whose grid still fills the chip; returns false when no MFMA tile fits the shape.
template <bool TRANS_B, int EPI>
static bool try_mfma(const GemmArgs& g, int W, hipStream_t s)
{
    if (!mfma_fits<TRANS_B, EPI>(g)) return false;
    const int64_t blocks256 = (g.M % 256 == 0 && g.N % 256 == 0) ? (int64_t)(g.M / 256) * (g.N / 256) * W : 0;
    const int64_t blocks128 = (int64_t)(g.M / 128) * (g.N / 128) * W;
    // the fused update keeps two batches of x, m and leader values in registers: no room beside a 256x256 tile
    if constexpr (EPI != EPI_DWU) {
        if (blocks256 >= 256) { launch_gemm<256, 256, 2, 4, TRANS_B, EPI>(g, W, s); return true; }
    }
    // forward and d-input products of more than two K steps go straight to LDS; shorter ones end before its three steps are
    // under way (objective of 64-64-64-64-10, 4 workers, batch 128, 18.5 us that way, 16.4 this way; 128-128-10, batch 1024,
    // 8 workers, 11.2 / 10.7; 192-64-10 11.0 / 11.2)
    if ((EPI == EPI_FWD || EPI == EPI_DX) && g.K > 2 * kBK && better_direct(g, W, EPI)) { launch_gemm_direct(g, W, EPI, s); return true; }
    if (g.N % 128 == 0 && blocks128 >= 256) launch_gemm<128, 128, 2, 2, TRANS_B, EPI>(g, W, s);
    else launch_gemm<128, 64, 2, 2, TRANS_B, EPI>(g, W, s);
    return true;
}

// Softmax cross-entropy of one worker's batch: loss = mean_b(lse - z[y]); delta = bf16((p - onehot)/B),
// stored as [B][C] and [C][B].  One workgroup per worker.
__global__ __launch_bounds__(256) void loss_delta_kernel(const float* __restrict__ logits, int64_t sLogits, const int32_t* __restrict__ y,
                                                         int B, int C, uint16_t* __restrict__ delta, uint16_t* __restrict__ deltaT,
                                                         int64_t sDelta, float* __restrict__ losses, float* __restrict__ g,
                                                         int64_t P, int64_t ld)
{
    const int w = blockIdx.x;
    if (g)                                                 // a gradient pass follows: the padding columns of g are zero
        for (int64_t c = P + threadIdx.x; c < ld; c += 256) g[(int64_t)w * ld + c] = 0.f;
    const float* lg = logits + (int64_t)w * sLogits;
    uint16_t* d = delta + (int64_t)w * sDelta;
    uint16_t* dT = deltaT + (int64_t)w * sDelta;
    const float invB = 1.0f / (float)B;
    double part = 0.0;
    for (int b = threadIdx.x; b < B; b += 256) {
        const float* z = lg + (int64_t)b * C;
        float mx = z[0];
        for (int c = 1; c < C; ++c) mx = fmaxf(mx, z[c]);
        float se = 0.f;
        for (int c = 0; c < C; ++c) se += expf(z[c] - mx);
        const float lse = mx + logf(se);
        const int yb = y[(int64_t)w * B + b];
        part += (double)(lse - z[yb]);
        for (int c = 0; c < C; ++c) {
            const float p = expf(z[c] - lse);
            const uint16_t q = f32_to_bf16_rne((p - (c == yb ? 1.f : 0.f)) * invB);
            d[(int64_t)b * C + c] = q;
            dT[(int64_t)c * B + b] = q;
        }
    }
    __shared__ double red[256];
    red[threadIdx.x] = part;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) losses[w] = (float)(red[0] / (double)B);
}

// losses[w] = sum of the head's row-tile sums / B.  One wavefront per worker.
__global__ __launch_bounds__(256) void loss_finish_kernel(const double* __restrict__ sums, int64_t stride, int n, int W, double B,
                                                          float* __restrict__ losses)
{
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (w >= W) return;
    double acc = 0.0;
    for (int i = lane; i < n; i += 64) acc += sums[(int64_t)w * stride + i];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d, 64);
    if (lane == 0) losses[w] = (float)(acc / B);
}

// h_0 = bf16(X) for fp32 inputs: n values per worker, rounded to nearest even
__global__ __launch_bounds__(256) void cast_input_kernel(const float* __restrict__ X, int64_t n, uint16_t* __restrict__ out, int64_t sOut)
{
    const int w = blockIdx.y;
    const float* src = X + (int64_t)w * n;
    uint16_t* dst = out + (int64_t)w * sOut;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] = f32_to_bf16_rne(src[i]);
}

// ------------------------------------------------------------------------------------------
// Host orchestration
// ------------------------------------------------------------------------------------------
namespace {

struct MlpPlan {
    int L;
    std::size_t bytes;
    // per-worker element offsets inside the scratch (bf16 elements unless noted)
    int64_t h[64];      // h[k], k = 1..L-1  [B][d_k]
    int64_t d[64];      // delta[k], k = 1..L [B][d_k]
    int64_t dT[64];     // delta^T[k]         [d_k][B]
    int64_t logits;     // fp32 [B][C], offset in bytes from the worker's base
    int64_t x0;         // bf16 copy of fp32 inputs [B][d_0] (only when the batch brings fp32 inputs)
    int64_t per_worker; // bytes per worker
};

inline int64_t up16(int64_t v) { return (v + 15) / 16 * 16; }

MlpPlan make_plan(const lsgd_mlp_batch& b, int W)
{
    MlpPlan p{};
    p.L = b.n_layers;
    int64_t o = 0; // bytes
    for (int k = 1; k <= p.L; ++k) {
        const int64_t n = (int64_t)b.B * b.dims[k] * 2;
        if (k < p.L) { p.h[k] = o / 2; o = up16(o + n); }
        p.d[k] = o / 2; o = up16(o + n);
        p.dT[k] = o / 2; o = up16(o + n);
    }
    p.logits = o; o = up16(o + (int64_t)b.B * b.dims[p.L] * 4);
    if (b.x_is_fp32) { p.x0 = o / 2; o = up16(o + (int64_t)b.B * b.dims[0] * 2); }
    p.per_worker = (o + 255) / 256 * 256;
    p.bytes = (std::size_t)p.per_worker * (std::size_t)W;
    return p;
}

} // namespace

bool mlp_shape_supported(const lsgd_mlp_batch& b, const char** why)
{
    if (b.n_layers > 60) { *why = "more than 60 layers"; return false; }
    if (b.dims[b.n_layers] > 4096) { *why = "more than 4096 classes"; return false; }
    return true;
}

size_t mlp_scratch_bytes(int W, const lsgd_mlp_batch& b) { return make_plan(b, W).bytes; }

hipError_t launch_mlp_grad_loss(const uint16_t* xb, const float* x, float* g, float* losses, int W, int64_t P,
                                int64_t ld, const lsgd_mlp_batch& b, const DeviceState& st, LossParts* parts, hipStream_t s)
{
    hipError_t e = launch_mlp_forward(xb, x, g, losses, W, P, ld, b, st, true, parts, s);
    if (e != hipSuccess) return e;
    return launch_mlp_backward(xb, x, g, W, P, ld, b, st, nullptr, s);
}

// Whether the launch of the classifier also forms its d-input product, on its W B / 32 workgroups alone: a launch less,
// but fewer workgroups than the product of its own has, and wavefronts that take more and more columns each.  Whole
// gradient calls and steps, own launch = 1: 10 classes behind 64 units 0.85 to 0.88, 256 0.94, 512 0.95, 768 0.97, 1024
// 1.01 to 1.07, 4096 1.07 to 1.5; behind 1024 to 4096 with 256 workgroups 0.92; 60 classes (four wavefronts) behind 512
// units 1.08.
static bool head_forms_dx(const lsgd_mlp_batch& b, int W)
{
    const int L = b.n_layers;
    if (L < 2 || b.dims[L] > 64) return false;
    const int64_t units = b.dims[L - 1];
    if (b.dims[L] > 32) return units <= 256;
    return units <= 768 || (units <= 4096 && (int64_t)W * ((b.B + 31) / 32) >= 256);
}

hipError_t launch_mlp_forward(const uint16_t* xb, const float* x, float* g, float* losses, int W, int64_t P, int64_t ld,
                              const lsgd_mlp_batch& b, const DeviceState& st, bool backward, LossParts* parts, hipStream_t s)
{
    const MlpPlan p = make_plan(b, W);
    const int L = p.L, B = b.B;
    uint16_t* sc16 = reinterpret_cast<uint16_t*>(st.scratch);
    const int64_t sW16 = p.per_worker / 2;     // per-worker stride in bf16 elements
    const int64_t sW32 = p.per_worker / 4;     // ... in fp32 elements
    float* logits = reinterpret_cast<float*>(st.scratch + p.logits);

    int64_t woff[64];
    { int64_t o = 0; for (int k = 1; k <= L; ++k) { woff[k] = o; o += (int64_t)b.dims[k] * b.dims[k - 1] + b.dims[k]; } }

    // ---- forward ----
    const uint16_t* X0 = static_cast<const uint16_t*>(b.X);
    int64_t sX0 = (int64_t)B * b.dims[0];
    bool first_done = false;
    if (b.x_is_fp32) {                                     // the bf16 copy both passes read
        if (L > 1 && (b.B % 128 || b.dims[1] % 64 || b.dims[0] % kBK)) {      // (whole tiles: the aligned kernels)
            GemmArgs a{};
            a.A32 = static_cast<const float*>(b.X); a.sA = sX0; a.lda = b.dims[0];
            if (backward) { a.copy = sc16 + p.x0; a.sCopy = sW16; }
            a.B = xb + woff[1]; a.sB = ld; a.ldb = b.dims[0];
            a.M = B; a.N = b.dims[1]; a.K = b.dims[0];
            a.bias = x + woff[1] + (int64_t)b.dims[1] * b.dims[0]; a.sBias = ld;
            a.out = sc16 + p.h[1]; a.sOut = sW16; a.ldout = b.dims[1];
            first_done = launch_gemm_ragged_f32(a, W, s);
        }
        const int64_t n = (int64_t)B * b.dims[0];
        int64_t blocks = (n + 255) / 256;
        if (blocks > 4096) blocks = 4096;
        if (!first_done)
            hipLaunchKernelGGL(cast_input_kernel, dim3((unsigned)blocks, (unsigned)W), dim3(256), 0, s, static_cast<const float*>(b.X), n,
                               sc16 + p.x0, sW16);
        X0 = sc16 + p.x0; sX0 = sW16;
    }
    for (int k = first_done ? 2 : 1; k <= L; ++k) {
        const int din = b.dims[k - 1], dout = b.dims[k];
        const uint16_t* Hin = (k == 1) ? X0 : sc16 + p.h[k - 1];
        const int64_t sHin = (k == 1) ? sX0 : sW16;
        const float* bias = x + woff[k] + (int64_t)dout * din;
        GemmArgs a{};
        a.A = Hin; a.sA = sHin; a.lda = din;
        a.B = xb + woff[k]; a.sB = ld; a.ldb = din;
        a.M = B; a.N = dout; a.K = din;
        a.bias = bias; a.sBias = ld;
        if (k < L) {
            a.out = sc16 + p.h[k]; a.sOut = sW16; a.ldout = dout;
            a.updated = backward && !g;
            if (!try_mfma<false, EPI_FWD>(a, W, s) && !launch_gemm_direct_any(a, W, EPI_FWD, s)) launch_gemm_ragged(a, W, EPI_FWD, s);
        } else if (dout <= 64) {                               // logits, loss and output delta in one launch
            const int tiles = (B + 31) / 32;
            a.y = b.y;
            a.losses = losses;
            // the tiles' loss sums lie where the worker's logits would (4 B C bytes hold B / 32 doubles)
            a.loss_parts = reinterpret_cast<double*>(logits); a.sLoss = p.per_worker / 8;
            if (backward) { a.out = sc16 + p.d[L]; a.outT = sc16 + p.dT[L]; a.sOut = sW16; }
            if (backward && head_forms_dx(b, W)) { a.dx = sc16 + p.d[L - 1]; a.dxT = sc16 + p.dT[L - 1]; }
            a.pad = ld > P ? g : nullptr; a.pad_from = P; a.pad_to = ld;
            launch_gemm_ragged(a, W, EPI_HEAD, s);
            if (tiles > 1 && loss_parts_ok(W, tiles)) {        // one order, whoever adds them up
                LossParts q;
                q.sums = nullptr; q.sums64 = a.loss_parts; q.stride = a.sLoss; q.n = tiles; q.c = 1.0; q.div = B;
                if (!parts) return launch_loss_parts(q, W, losses, s);
                *parts = q;
            } else if (tiles > 1) {
                hipLaunchKernelGGL(loss_finish_kernel, dim3((unsigned)((W + 3) / 4)), dim3(256), 0, s, a.loss_parts, a.sLoss, tiles, W, (double)B, losses);
            }
            return hipGetLastError();
        } else {
            a.C = logits; a.sC = sW32; a.ldc = dout;
            launch_gemm_ragged(a, W, EPI_LOGITS, s);
        }
    }
    // ---- loss and output delta ----
    hipLaunchKernelGGL(loss_delta_kernel, dim3((unsigned)W), dim3(256), 0, s, logits, sW32, b.y, B, b.dims[L],
                       sc16 + p.d[L], sc16 + p.dT[L], sW16, losses, g, P, ld);
    return hipGetLastError();
}

// Backward pass.  Per layer, from the top: delta_{k-1} first (it reads W_k, which the fused update
// of dW_k overwrites), then dW_k and db_k; small ones without an aligned tile that follow each other in one launch.
hipError_t launch_mlp_backward(const uint16_t* xb, const float* x, float* g, int W, int64_t P, int64_t ld,
                               const lsgd_mlp_batch& b, const DeviceState& st, const FusedUpdate* fu_in, hipStream_t s)
{
    const MlpPlan p = make_plan(b, W);
    const int L = p.L, B = b.B;
    uint16_t* sc16 = reinterpret_cast<uint16_t*>(st.scratch);
    const int64_t sW16 = p.per_worker / 2;     // per-worker stride in bf16 elements
    FusedUpdate fu{};
    if (fu_in) fu = *fu_in;
    const bool fused = fu.enabled != 0;

    int64_t woff[64];
    { int64_t o = 0; for (int k = 1; k <= L; ++k) { woff[k] = o; o += (int64_t)b.dims[k] * b.dims[k - 1] + b.dims[k]; } }

    // fp32 inputs: the forward pass of this step left their bf16 copy in the scratch
    const uint16_t* X0 = b.x_is_fp32 ? sc16 + p.x0 : static_cast<const uint16_t*>(b.X);
    const int64_t sX0 = b.x_is_fp32 ? sW16 : (int64_t)B * b.dims[0];
    const int epi = fused ? EPI_DWU : EPI_DW;
    GemmGroup rest{};
    for (int k = L; k >= 1; --k) {
        const int din = b.dims[k - 1], dout = b.dims[k];
        const uint16_t* Hin = (k == 1) ? X0 : sc16 + p.h[k - 1];
        const int64_t sHin = (k == 1) ? sX0 : sW16;
        // delta_{k-1}
        if (k > 1 && !(k == L && head_forms_dx(b, W))) {
            GemmArgs a{};
            a.A = sc16 + p.d[k]; a.sA = sW16; a.lda = dout;
            a.B = xb + woff[k]; a.sB = ld; a.ldb = din;
            a.M = B; a.N = din; a.K = dout;
            a.mask = Hin; a.sMask = sHin; a.ldmask = din;
            a.out = sc16 + p.d[k - 1]; a.sOut = sW16; a.ldout = din;
            a.outT = sc16 + p.dT[k - 1]; a.sOutT = sW16; a.ldoutT = B;
            if (!try_mfma<true, EPI_DX>(a, W, s) && !launch_gemm_direct_any(a, W, EPI_DX, s)) launch_gemm_ragged(a, W, EPI_DX, s);
        }
        // dW_k
        {
            GemmArgs a{};
            a.A = sc16 + p.dT[k]; a.sA = sW16; a.lda = B;
            a.B = Hin; a.sB = sHin; a.ldb = din;
            a.M = dout; a.N = din; a.K = B;
            a.C = g + woff[k]; a.sC = ld; a.ldc = din;
            a.fu = fu; a.colC = woff[k];
            // (what waits goes before an aligned product: it is small, and its operands are in the caches)
            const bool whole = fused ? mfma_fits<true, EPI_DWU>(a) : mfma_fits<true, EPI_DW>(a);
            if (rest.n && (whole || rest.n == kGroupMax)) { launch_gemm_group(rest, W, epi, s); rest.n = 0; }
            if (!whole && gemm_joins_group(a, W, epi)) rest.g[rest.n++] = a;
            else if (!whole) launch_gemm_ragged(a, W, epi, s);
            else if (fused) try_mfma<true, EPI_DWU>(a, W, s);
            else try_mfma<true, EPI_DW>(a, W, s);
        }
    }
    if (rest.n) launch_gemm_group(rest, W, epi, s);
    return hipGetLastError();
}

} // namespace lsgd
