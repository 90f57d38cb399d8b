// Forward and d-input products of the MLP path on 16-byte aligned operands with more than 64 samples per worker:
// operands go from global memory straight to LDS, three or four K steps deep.
//
//   forward   out[m][n] = bf16(relu(<A[m,:], B[n,:]> + bias[n]))      A = h_{k-1}, B = W_k       (both [.][k])
//   d-input   out[m][n] = bf16(sum_k A[m][k] B[k][n]) * [mask != 0]   A = delta_k, B = W_k       (B as [k][n]); outT transposed
//
// What bounds these products is what reaches the compute units (a batch of 128 to 256 rows per weight: 17 TB/s of
// tiles out of L2 measured without the products), and for the largest the chip's power limit: 256 x 4096 x 4096, 8
// workers, takes 68 us on zeros and 80 us on normal values, at 1.8 to 2.1 instead of 2.4 GHz, in every tile and
// wavefront shape.  Loads that go straight to LDS need no registers, so three K steps or more are under way per
// workgroup, and no vector instructions to store them.  A wavefront's load writes 64 consecutive 16-byte pieces, so
// rows cannot be padded: the pieces of a row are stored in another order instead (exclusive or with half the row
// number: two rows fill the banks once), which spreads the fragment reads over all banks (with the row number itself
// half of the LDS cycles were conflicts).  Fragments are read a quarter step ahead of their products, across the
// barrier too.
//
// ANY: any M and N, K a multiple of 8.  Row numbers past the end are clamped to the last row, pieces past the end of a
// row to its last piece (fragments past K become zeros in the last step).  Sums are carried as in the any-shape kernel's
// 128-row tiles, in double after every eight matrix instructions, bit for bit.  !ANY: whole tiles, one fp32 chain.
//
// Measured, us, through registers -> straight to LDS: objective of 3072-1024-10, 16 workers, batch 128: 38 -> 32;
// gradients of 1024-2048-2048-10, 8 workers, batch 256: 169 -> 159; 256-512-512-10, 8 workers, batch 128: 46.5 -> 43.
// ANY, kernels alone: forward 500 x 1024 x 3072, 16 workers, 91 -> 76, 128 x 1912 x 1208 34 -> 22; d-input 200 x 1912 x
// 1208 72 -> 44, 256 x 784 x 1000 34 -> 22.  With four buffers the additions to the double sums run beside the next two
// steps' matrix instructions, which go into other accumulators: objective of 3072-1024-10, 16 x 500, 85.8 -> 82.9 us, of
// 3072-1000-10, 8 x 1000, 84.7 -> 81.3 (same bits).
#include <type_traits>

#include "mlp_common.h"

namespace lsgd {

namespace {

constexpr int kBK = 64;              // contraction per K step: one 128-byte line of every row

constexpr int kNonTemporal = 2;      // cache policy of a load

typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* global_ptr;

template <int N>
__device__ __forceinline__ void wait_loads()     // all LDS reads and all but the N youngest global loads of this wavefront are done
{
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}

// The K step handed over: every wavefront's part has arrived, and nobody reads the buffer that is filled next.
__device__ __forceinline__ void step_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int N, int I = 0, class F>
__device__ __forceinline__ void for_each(const F& f)
{
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); for_each<N, I + 1>(f); }
}

// ST: K steps in LDS; NT: B past the caches
template <int BM, int BN, int WVM, int WVN, int ST, bool TRANS_B, int EPI, bool ANY, bool NT>
__global__ __launch_bounds__(64 * WVM * WVN) void gemm_direct_kernel(GemmArgs g, int tiles_m, int tiles_n)
{
    constexpr int THREADS = 64 * WVM * WVN;
    constexpr int WTM = BM / WVM, WTN = BN / WVN, TM = WTM / 32, TN = WTN / 32;
    constexpr int A_OPS = BM * 8 / THREADS, B_OPS = BN * 8 / THREADS, OPS = A_OPS + B_OPS;   // 16-byte pieces per thread and step
    constexpr int NCH = BN / 8;                                       // pieces of a [k][n] row
    constexpr int TILE = (BM + BN) * kBK;
    // separate objects, so that the compiler sees that a read of one does not wait for loads into another
    __shared__ __attribute__((aligned(16))) uint16_t buf0[TILE], buf1[TILE], buf2[TILE], buf3[ST > 3 ? TILE : 8];
    static_assert(ST == 3 || ST == 4, "buffers");
    auto bufs = [&](int q) -> uint16_t* {
        if constexpr (ST > 3) { if (q == 3) return buf3; }
        return q == 0 ? buf0 : q == 1 ? buf1 : buf2;
    };

    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WVN, wn = wid % WVN;
    // a die (workgroup id modulo 8) takes a contiguous run of tiles, row tiles varying fastest
    int64_t s = gridDim.x % 8 == 0 ? (int64_t)(blockIdx.x & 7) * (gridDim.x / 8) + (blockIdx.x >> 3) : blockIdx.x;
    const int tm = (int)(s % tiles_m); s /= tiles_m;
    const int tn = (int)(s % tiles_n), w = (int)(s / tiles_n);
    const int m0 = tm * BM, n0 = tn * BN, M = g.M, N = g.N, K = g.K;
    const uint16_t* A = g.A + (int64_t)w * g.sA;
    const uint16_t* B = g.B + (int64_t)w * g.sB;

    // this thread's pieces: where they come from.  [.][k]: row tid / 8 + c * THREADS / 8, piece (tid % 8) ^ (row / 2 % 8)
    const uint16_t *pa[A_OPS], *pb[B_OPS];
    const int kc = ((tid & 7) ^ ((tid >> 4) & 7)) * 8;
#pragma unroll
    for (int c = 0; c < A_OPS; ++c) {
        int r = m0 + (tid >> 3) + c * (THREADS / 8);
        if (ANY && r >= M) r = M - 1;
        pa[c] = A + (int64_t)r * g.lda + (ANY ? 0 : kc);
    }
    const int krow = tid / NCH;                                       // [k][n]: first k row
    if (TRANS_B) {
        const int swz = BN == 128 ? (krow & 3) << 2 : ((krow >> 1) & 1) << 2;
        int col = n0 + ((tid % NCH) ^ swz) * 8;
        if (ANY && col > N - 8) col = N - 8;
#pragma unroll
        for (int c = 0; c < B_OPS; ++c) pb[c] = B + (ANY ? 0 : (int64_t)(krow + c * (THREADS / NCH)) * g.ldb) + col;
    } else {
#pragma unroll
        for (int c = 0; c < B_OPS; ++c) {
            int r = n0 + (tid >> 3) + c * (THREADS / 8);
            if (ANY && r >= N) r = N - 1;
            pb[c] = B + (int64_t)r * g.ldb + (ANY ? 0 : kc);
        }
    }
    auto issue = [&](int kt, uint16_t* buf) {
        const int k0 = kt * kBK;
        const int k = ANY ? (k0 + kc < K - 8 ? k0 + kc : K - 8) : k0;
#pragma unroll
        for (int c = 0; c < A_OPS; ++c)
            __builtin_amdgcn_global_load_lds((global_ptr)(pa[c] + k), (lds_ptr)(buf + (c * THREADS + wid * 64) * 8), 16, 0, 0);
#pragma unroll
        for (int c = 0; c < B_OPS; ++c) {
            const uint16_t* p;
            if (TRANS_B) {
                int r = k0;
                if (ANY) { r = k0 + krow + c * (THREADS / NCH); r = r < K ? r : K - 1; }
                p = pb[c] + (int64_t)r * g.ldb;
            } else {
                p = pb[c] + k;
            }
            __builtin_amdgcn_global_load_lds((global_ptr)p, (lds_ptr)(buf + (BM * kBK + (c * THREADS + wid * 64) * 8)), 16, 0, NT ? kNonTemporal : 0);
        }
    };

    f32x16 acc[TM][TN];
    double sum[ANY ? TM : 1][ANY ? TN : 1][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][j][v] = 0.f;
                if (ANY) sum[i][j][v] = 0.0;
            }
    // DEFER (an even number of buffers): the accumulators of two K steps are added to the sums while the next two are
    // multiplied into others, a quarter at a time
    constexpr bool DEFER = ANY && ST % 2 == 0;
    f32x16 old[DEFER ? TM : 1][DEFER ? TN : 1];
    auto put_off = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                old[DEFER ? i : 0][DEFER ? j : 0] = acc[i][j];
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
            }
    };
    auto add_old = [&](int part) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 4 * part; v < 4 * part + 4; ++v) sum[ANY ? i : 0][ANY ? j : 0][v] += (double)old[DEFER ? i : 0][DEFER ? j : 0][v];
    };
    auto promote = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) { sum[i][j][v] += (double)acc[i][j][v]; acc[i][j][v] = 0.f; }
    };

    const int half = lane >> 5, l16 = lane & 15;
    const int sw = half ^ ((lane >> 1) & 7);                          // piece of k step 0, swizzled
    const int arow = (wm * WTM + (lane & 31)) * kBK, brow = (BM + wn * WTN + (lane & 31)) * kBK;
    struct Frags { bf16x8 a[TM], b[TN]; };
    // (offsets are summed up first: behind a longer chain of address steps the compiler loses track of which buffer is read)
    auto read = [&](const uint16_t* buf, int kk, Frags& f) {
#pragma unroll
        for (int i = 0; i < TM; ++i) f.a[i] = *reinterpret_cast<const bf16x8*>(buf + (arow + ((kk * 2) ^ sw) * 8 + i * 32 * kBK));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (TRANS_B) {
                // lane (n = lane % 32, k-half = lane / 32): k = 16 kk + 8 (lane / 32) + 0..7 of column n
                const int row = kk * 16 + 8 * half + (l16 >> 2);
                const int col = wn * WTN + j * 32 + (lane & 16) + 4 * (l16 & 3);
                const int swz = BN == 128 ? (l16 >> 2) << 5 : ((l16 >> 3) & 1) << 5;
                const s16x4 lo = lds_read_tr(buf + (BM * kBK + row * BN + (col ^ swz)));
                const s16x4 hi = lds_read_tr(buf + (BM * kBK + (row + 4) * BN + (col ^ swz)));
                const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                f.b[j] = __builtin_bit_cast(bf16x8, v);
            } else {
                f.b[j] = *reinterpret_cast<const bf16x8*>(buf + (brow + ((kk * 2) ^ sw) * 8 + j * 32 * kBK));
            }
        }
    };
    auto multiply = [&](const Frags& f) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
    };

    const int nk = (K + kBK - 1) / kBK;
    Frags f0, f1;
    auto clear_past = [&](Frags& f, int kk, int live) {               // a ragged last step: past the end lies some other piece
        if (kk * 16 + half * 8 < live) return;
#pragma unroll
        for (int i = 0; i < TM; ++i) f.a[i] = (bf16x8)(__bf16)0.f;
#pragma unroll
        for (int j = 0; j < TN; ++j) f.b[j] = (bf16x8)(__bf16)0.f;
    };
    // One K step: the fragments of its first quarter are in f0; its last quarter is multiplied behind the barrier that
    // hands over the next step, whose first fragments are then on their way.
    auto step = [&](auto q, int kt, auto in_flight, auto last_steps) {
        constexpr bool LAST = decltype(last_steps)::value;
        const uint16_t* const buf = bufs(q);
        const int live = K - kt * kBK;
        constexpr bool ADD = DEFER && decltype(q)::value % 2 == 0;    // (before the first step there are only zeros to add)
        read(buf, 1, f1); if (ANY && LAST) clear_past(f0, 0, live); multiply(f0);
        if (ADD) add_old(0);
        read(buf, 2, f0); if (ANY && LAST) clear_past(f1, 1, live); multiply(f1);
        if (ADD) add_old(1);
        read(buf, 3, f1); if (ANY && LAST) clear_past(f0, 2, live); multiply(f0);
        if (ADD) add_old(2);
        __builtin_amdgcn_sched_barrier(0);
        wait_loads<decltype(in_flight)::value * OPS>();
        step_barrier();
        if (!LAST) issue(kt + ST < nk ? kt + ST : nk - 1, bufs(q));
        if (ANY && LAST) clear_past(f1, 3, live);
        read(bufs((q + 1) % ST), 0, f0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f1);
        if (DEFER) {
            if (ADD) add_old(3);
            if (decltype(q)::value % 2 == 1) put_off();
        } else if (ANY && ((kt & 1) || (LAST && kt == nk - 1))) {
            promote();
        }
    };
    if (DEFER) put_off();
    for_each<ST>([&](auto q) { issue(q < nk ? q : nk - 1, bufs(q)); });
    wait_loads<(ST - 1) * OPS>();
    step_barrier();
    read(bufs(0), 0, f0);
    int kt = 0;
    for (; kt + ST < nk; kt += ST)
        for_each<ST>([&](auto q) { step(q, kt + q, std::integral_constant<int, ST - 2>{}, std::false_type{}); });
    // 1 to ST steps left, all under way
    for_each<ST>([&](auto q) {
        constexpr int after = ST - 2 - decltype(q)::value;
        if (q == 0 || kt + q < nk) step(q, kt + q, std::integral_constant<int, (after > 0 ? after : 0)>{}, std::true_type{});
    });
    if (DEFER) {
        if (!(nk & 1)) for_each<4>([&](auto part) { add_old(part); });
        else promote();
    }
    wait_loads<0>();
    __syncthreads();

    // Results leave through LDS (lanes hold single columns) as 16-byte pieces of rows.  Lane: column lane % 32, rows
    // (lane / 32) * 4 + 8 (v / 4) + v % 4 of each 32x32 tile.  The tile's rows are spread over the buffers.
    constexpr int LDT = BN + kPadN;
    constexpr int RPB = TILE / LDT / 64 * 64;                         // rows per buffer
    static_assert(RPB > 0 && (BM + RPB - 1) / RPB <= ST && WTM <= RPB && RPB % WTM == 0, "result tile fits the buffers");
    auto trow = [&](int r) { return bufs(r / RPB) + (r % RPB) * LDT; };
    constexpr int ROWS = THREADS / NCH;                               // rows per pass
    const int cr = tid / NCH, cc = (tid % NCH) * 8;
    uint16_t* out = g.out + (int64_t)w * g.sOut;
    if (EPI == EPI_DX) {
        const uint16_t* mask = g.mask + (int64_t)w * g.sMask;
        u32x4 mk[BM / ROWS];
#pragma unroll
        for (int c = 0; c < BM / ROWS; ++c) {
            int m = m0 + c * ROWS + cr, n = n0 + cc;
            if (ANY) { m = m < M ? m : M - 1; n = n < N - 8 ? n : N - 8; }    // (rows of a multiple of 8 elements)
            mk[c] = *reinterpret_cast<const u32x4*>(mask + (int64_t)m * g.ldmask + n);
        }
#pragma unroll
        for (int c = 0; c < BM / ROWS; ++c) *reinterpret_cast<u32x4*>(trow(c * ROWS) + cr * LDT + cc) = mk[c];
        __syncthreads();
    }
    uint16_t* outT = (EPI == EPI_DX) ? g.outT + (int64_t)w * g.sOutT : nullptr;
    uint16_t* const T = trow(wm * WTM) + half * 4 * LDT;              // this wavefront's rows
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int nl = wn * WTN + j * 32 + (lane & 31);
            uint16_t* const t = T + i * 32 * LDT;
            if (EPI == EPI_FWD) {
                const float b = g.bias[(int64_t)w * g.sBias + (ANY && n0 + nl >= N ? N - 1 : n0 + nl)];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float z = ANY ? (float)(sum[i][j][v] + (double)b) : acc[i][j][v] + b;
                    t[(8 * (v >> 2) + (v & 3)) * LDT + nl] = f32_to_bf16_rne(z > 0.f ? z : 0.f);
                }
            } else {
                const int mb = m0 + wm * WTM + i * 32 + half * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // every 4 x 16 block of the mask is read and then overwritten by the same 16 lanes
                    const s16x4 on = lds_read_tr(t + (8 * q + (l16 >> 2)) * LDT + wn * WTN + j * 32 + (lane & 16) + 4 * (l16 & 3));
                    uint32_t pk[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = ANY ? (float)sum[i][j][q * 4 + r] : acc[i][j][q * 4 + r];
                        const uint16_t d = on[r] != 0 ? f32_to_bf16_rne(v) : (uint16_t)0;
                        t[(8 * q + r) * LDT + nl] = d;
                        pk[r] = d;
                    }
                    const u32x2 o = {pk[0] | (pk[1] << 16), pk[2] | (pk[3] << 16)};     // four samples of one column, adjacent in the transposed copy
                    uint16_t* dst = outT + (int64_t)(n0 + nl) * g.ldoutT + mb + 8 * q;
                    if (!ANY) {
                        *reinterpret_cast<u32x2*>(dst) = o;
                    } else if (n0 + nl < N) {
                        if (mb + 8 * q + 4 <= M) *reinterpret_cast<u32x2_any*>(dst) = o;
                        else
#pragma unroll
                            for (int r = 0; r < 3; ++r)
                                if (mb + 8 * q + r < M) dst[r] = (uint16_t)pk[r];
                    }
                }
            }
        }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < BM / ROWS; ++c) {
        const int m = m0 + c * ROWS + cr, n = n0 + cc;
        const u32x4 v = *reinterpret_cast<const u32x4*>(trow(c * ROWS) + cr * LDT + cc);
        uint16_t* dst = out + (int64_t)m * g.ldout + n;
        if (!ANY) {
            *reinterpret_cast<u32x4*>(dst) = v;
        } else if (m < M) {
            if (n + 8 <= N) *reinterpret_cast<u32x4_any*>(dst) = v;
            else
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (n + e < N) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
    }
}

// Whether a forward product reads its weights past the caches: more than about half of the memory-side cache holds of one
// layer's weights will not be there again at the next pass, and takes the room of what the passes behind it write.
// Plain / past the caches, us: 16 workers, batch 128, 3072-2048-10, objective 56.9 / 52.5, gradients 162 / 150, fused step 314 /
// 309; batch 100, 3072-2000-1000-10, gradients 286 / 260; 3072-1536-10 (151 MB) 51.7 / 48.2, 135 / 127; but 2048-1536-10 (101 MB)
// 31.5 / 36.4, 90 / 94, batch 100, 1000-3000-10 (96 MB) 43.7 / 55.  With a second row tile the L2s are to keep them: batch 200,
// 3072-2000-1000-10, 114 / 119, fused step 685 / 708.  A fused update's own streams have pushed out smaller weights too: batch 128,
// 3072-1024-10 (101 MB), fused step with momentum 262.2 / 260.6.
bool streams(const GemmArgs& g, int W, int rows) { return g.M <= rows && 2.0 * W * (double)g.N * g.K > (g.updated ? 95e6 : 120e6); }

template <int BM, int BN, int WVM, int WVN, int ST, bool ANY>
void launch_forward(const GemmArgs& g, int W, hipStream_t s)
{
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const dim3 grid((unsigned)(tiles_m * tiles_n * W)), block(64 * WVM * WVN);
    if (streams(g, W, BM)) hipLaunchKernelGGL((gemm_direct_kernel<BM, BN, WVM, WVN, ST, false, EPI_FWD, ANY, true>), grid, block, 0, s, g, tiles_m, tiles_n);
    else hipLaunchKernelGGL((gemm_direct_kernel<BM, BN, WVM, WVN, ST, false, EPI_FWD, ANY, false>), grid, block, 0, s, g, tiles_m, tiles_n);
}

template <int BM, int BN, int WVM, int WVN, int ST, bool ANY>
void launch_direct(const GemmArgs& g, int W, int epi, hipStream_t s)
{
    if (epi == EPI_FWD) { launch_forward<BM, BN, WVM, WVN, ST, ANY>(g, W, s); return; }
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    hipLaunchKernelGGL((gemm_direct_kernel<BM, BN, WVM, WVN, ST, true, EPI_DX, ANY, false>), dim3((unsigned)(tiles_m * tiles_n * W)),
                       dim3(64 * WVM * WVN), 0, s, g, tiles_m, tiles_n);
}

// 128 columns as long as that leaves few compute units without a tile (forward 500 x 300 x 784, 16 workers, 192 tiles of
// 128 columns: 14.6 us, of 64: 17.1; 200 x 512 x 512, 128 tiles: 10.3 against 9.2), 64 for the short contractions of
// d-input products, where the results' way out counts (200 x 2048 x 256, 16 workers: 21 against 19).
bool wide_tile(const GemmArgs& g, int W, int epi)
{
    return (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128) * W >= 160 && !(epi == EPI_DX && g.K <= 512);
}

} // namespace

// One row tile per weight tile and more tiles than compute units: nothing is used twice, and a second workgroup on a compute
// unit is worth more than loads that take no registers.  Through registers / straight to LDS, us, 16 workers, batch 128: objective
// of 1024-4096-10 47 / 52, of 3072-4096-10 97 / 103, gradients 283 / 291; 256 tiles (3072-2048-10) 54 / 52.
bool better_direct(const GemmArgs& g, int W, int epi)
{
    return !(epi == EPI_FWD && g.M == 128 && g.N % 128 == 0 && (int64_t)(g.N / 128) * W > 256 && streams(g, W, 128));
}

void launch_gemm_direct(const GemmArgs& g, int W, int epi, hipStream_t s)
{
    // a 256-row tile covers a whole batch of 256: the weights are then read once
    if (g.M % 256 == 0 && g.N % 128 == 0 && (int64_t)(g.M / 256) * (g.N / 128) * W >= 256) launch_direct<256, 128, 4, 2, 3, false>(g, W, epi, s);
    else if (g.N % 128 == 0 && wide_tile(g, W, epi)) launch_direct<128, 128, 2, 4, 3, false>(g, W, epi, s);
    else launch_direct<128, 64, 2, 2, 3, false>(g, W, epi, s);
}

bool launch_gemm_direct_any(const GemmArgs& g, int W, int epi, hipStream_t s)
{
    auto a16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    if (g.K % 8 || g.K < 128 || g.lda % 8 || g.ldb % 8 || g.sA % 8 || g.sB % 8 || !a16(g.A) || !a16(g.B)) return false;
    if (epi == EPI_DX && (g.N % 8 || !a16(g.mask) || g.ldmask % 8 || g.sMask % 8)) return false;
    // Only where the any-shape kernel takes 128-row tiles too: its smaller tiles round less often (and with fewer
    // workgroups than compute units they are the faster ones, 128 x 1000 x 784, 4 workers: 8.5 against 10.9 us).
    if (g.M <= 64 || (int64_t)((g.M + 127) / 128) * ((g.N + 63) / 64) * W < 256) return false;
    // One K step more in LDS where the contraction is long: with double sums a step takes longer than its loads, and the
    // 128 x 128 tile has a compute unit to itself (forward 500 x 3072 x 1024, 16 workers, 79.5 -> 76.8 us; whole tiles and
    // the 64-column tile, two workgroups per compute unit, gain nothing, contractions of 256 lose 2 %).
    if (wide_tile(g, W, epi) && g.K >= 1024 && epi == EPI_FWD) launch_forward<128, 128, 2, 4, 4, true>(g, W, s);
    else if (wide_tile(g, W, epi)) launch_direct<128, 128, 2, 4, 3, true>(g, W, epi, s);
    else launch_direct<128, 64, 2, 2, 3, true>(g, W, epi, s);
    return true;
}

} // namespace lsgd
