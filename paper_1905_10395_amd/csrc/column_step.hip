// The update of a small or medium population in one launch: leader selection, the leader pull (+ momentum) update,
// Algorithm 1's communication pull and the elastic-averaging center, by workgroups that own a tile of columns for
// all rows.
//
// The update is independent per parameter column, and a thread that owns its columns for every row can read the
// leaders' values before it writes anything: nothing has to be ordered between workgroups, so what takes three to
// five launches on the row-streaming path (selection, rows, leader rows, copies of the losses) is one.  Every
// workgroup repeats the selection (at most 64 losses: one wavefront, a segmented minimum scan over lanes); the first
// one also records its result for the calls that follow.
//
// Which path.  A launch costs about 3 to 5 us here whatever it does, while a workgroup that hops between W rows gets
// less out of HBM than the row-streaming kernels (5.2 against 5.9 TB/s at 1.6 GB per update); up to about 300 MB read
// and written per update (the caller's rule) the saved launches weigh more.  Measured, whole lsgd_step on external
// gradients, row streams -> this kernel, us: 4 x 1003 14.6 -> 4.5; 12 x 271 117 with momentum and kept leaders
// 24.6 -> 16.5; 16 x 250 000 with momentum 30.0 -> 17.3;
// 16 x 1 250 000 without 62.5 -> 41.5; elastic averaging, 16 x 1 250 000 with momentum 85.3 -> 73.3.
#include "pull_common.h"
#include "select_common.h"

#include <type_traits>

namespace lsgd {

namespace {

constexpr int kThreads = 256;
template <int VEC> constexpr int kRowsInFlight = VEC == 1 ? 8 : 4;

struct ColumnDev {
    PullDev a;                   // the update (lamL, lamG: its coefficients)
    int update, comm;            // stages present
    float commL, commG;          // coefficients of the communication pull
    int select;                  // 0: leaders as recorded, 1: selection before the update, 2: after it
    uint64_t sel, cap;           // groups re-selected now / captured by the next stage
    int selG, capG;
    const float* losses;
    float* losses_out;           // the population's own loss buffer when the losses come from elsewhere, else NULL
    LossParts parts;             // partial sums to finish instead
    int32_t *lead, *glead, *refreshed;
    RowPlan* plan;
    float* center;               // elastic averaging: the center takes the global leader's place
    double center_rate;
};

struct Leaders {
    int lead[kColumnMaxWorkers]; // of each group
    int fresh[kColumnMaxWorkers];
    int gl, freshG;
};

// A few rows of one group.
template <int VEC>
struct RowBatch {
    typename Vec<VEC>::type x[kRowsInFlight<VEC>], g[kRowsInFlight<VEC>], m[kRowsInFlight<VEC>];
};

template <int VEC, int KIND, bool NT>
__device__ __forceinline__ void load_rows(const PullDev& a, int i, int end, int64_t col, RowBatch<VEC>& b)
{
    using V = typename Vec<VEC>::type;
#pragma unroll
    for (int u = 0; u < kRowsInFlight<VEC>; ++u)
        if (i + u < end) {
            const int64_t o = (int64_t)(i + u) * a.ld + col;
            b.x[u] = NT ? ld_stream<VEC>(a.x + o) : ld_vec<VEC>(a.x + o);
            b.g[u] = ld_stream<VEC>(a.g + o);
            b.m[u] = (KIND == 1) ? (NT ? ld_stream<VEC>(a.m + o) : ld_vec<VEC>(a.m + o)) : zero_of(V());
        }
}

// Rows that one pass treats alike: a group, or all of them where the center is what they are pulled to (no local pull
// then; asked at run time all the same: a loop known to have one pass keeps twice the registers, 84 us instead of 73 for
// 16 x 1 250 000).
template <bool CENTER>
__device__ __forceinline__ int pass_end(const PullDev& a, int j) { return CENTER && a.lamL == 0.0f ? a.W : a.offsets[j + 1]; }

// The rows in order, the loads of the next few under way while a few are updated and stored.  `first` holds the first
// rows of the first pass, loaded before the leaders were known.
template <int VEC, int KIND, bool NT, bool CENTER>
__device__ __forceinline__ void update_columns(const ColumnDev& s, const Leaders& L, int64_t col, const RowBatch<VEC>& first)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    const bool pullL = a.lamL != 0.0f, pullG = a.lamG != 0.0f;
    const bool exempt = (a.flags & LSGD_LEADER_EXEMPT) != 0;
    const Coef c = make_coef<V>(a);
    // a re-selected leader's row belongs to the group that reads it, and the global leader's is read before any row
    // is written: both are as they were
    auto local_leader = [&](int j) { return ld_vec<VEC>((L.fresh[j] ? a.x + (int64_t)L.lead[j] * a.ld : a.Z + (int64_t)j * a.ld) + col); };
    V zg = zero_of(V()), zl = zero_of(V());
    if (pullG) zg = ld_vec<VEC>((L.freshG ? a.x + (int64_t)L.gl * a.ld : a.Z + (int64_t)a.G * a.ld) + col);
    if (pullL) zl = local_leader(0);
    if (pullG && L.freshG && a.Z) st_vec(a.Z + (int64_t)a.G * a.ld + col, zg);
    RowBatch<VEC> cur = first, next;
    const int passes = CENTER && !pullL ? 1 : a.G;
    int j = 0, i = 0, end = pass_end<CENTER>(a, 0);
    while (true) {
        int nj = j, ni = i + kRowsInFlight<VEC>, nend = end;
        if (ni >= end) {
            nj = j + 1; ni = end;
            nend = nj < passes ? pass_end<CENTER>(a, nj) : end;
        }
        V nzl = zl;
        if (nj < passes) {
            load_rows<VEC, KIND, NT>(a, ni, nend, col, next);
            if (pullL && nj != j) nzl = local_leader(nj);
        }
        if (pullL && L.fresh[j] && a.Z && i == a.offsets[j]) st_vec(a.Z + (int64_t)j * a.ld + col, zl);
#pragma unroll
        for (int u = 0; u < kRowsInFlight<VEC>; ++u)
            if (i + u < end) {
                const int64_t o = (int64_t)(i + u) * a.ld + col;
                Coef cr = c;
                if (exempt && pullL && i + u == L.lead[j]) cr.cL = 0.0f;
                if (exempt && pullG && i + u == L.gl) cr.cG = 0.0f;
                update_vec<KIND, V>(cur.x[u], cur.g[u], cur.m[u], zl, zg, cr);
                if (NT) st_stream(a.x + o, cur.x[u]); else st_vec(a.x + o, cur.x[u]);
                if (KIND == 1) { if (NT) st_stream(a.m + o, cur.m[u]); else st_vec(a.m + o, cur.m[u]); }
                if (a.xb) st_bf16(a.xb + o, cur.x[u]);
            }
        if (nj >= passes) break;
        cur = next; zl = nzl; j = nj; i = ni; end = nend;
    }
}

// Algorithm 1's communication pull: every re-selected leader is captured, groups that communicate are pulled to
// their leader, then everyone to the global leader if that was re-selected.
template <int VEC>
__device__ __forceinline__ void comm_columns(const ColumnDev& s, const Leaders& L, int64_t col)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    Coef c = make_coef<V>(a);
    c.cG = L.freshG ? s.commG : 0.0f;
    V zg = zero_of(V());
    if (L.freshG) {
        zg = ld_vec<VEC>(a.x + (int64_t)L.gl * a.ld + col);
        if (a.Z) st_vec(a.Z + (int64_t)a.G * a.ld + col, zg);
    }
    for (int j = 0; j < a.G; ++j) {
        const int ll = L.lead[j];
        const bool fresh = L.fresh[j] != 0;
        V zl = zero_of(V());
        if (fresh) {
            zl = ld_vec<VEC>(a.x + (int64_t)ll * a.ld + col);
            if (a.Z) st_vec(a.Z + (int64_t)j * a.ld + col, zl);
        }
        c.cL = fresh ? s.commL : 0.0f;
        if (c.cL == 0.0f && c.cG == 0.0f) continue;
        for (int i = a.offsets[j]; i < a.offsets[j + 1]; ++i) {
            if (fresh && i == ll && c.cG == 0.0f) continue;          // a leader's pull to itself is zero
            const int64_t o = (int64_t)i * a.ld + col;
            V xv = ld_vec<VEC>(a.x + o), none = zero_of(V());
            update_vec<2, V>(xv, none, none, zl, zg, c);
            st_vec(a.x + o, xv);
            if (a.xb) st_bf16(a.xb + o, xv);
        }
    }
}

// The same with both coefficients zero: nobody moves, the re-selected leaders are copied to Z, eight rows of loads in
// flight.
template <int VEC>
__device__ __forceinline__ void capture_columns(const ColumnDev& s, const Leaders& L, int64_t col)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    if (!a.Z) return;
    int j = L.freshG ? -1 : 0;                           // -1: the global leader
    while (j < a.G) {
        V v[8];
        int to[8], n = 0;
        for (; j < a.G && n < 8; ++j) {
            if (j >= 0 && !L.fresh[j]) continue;
            to[n] = j < 0 ? a.G : j;
            ++n;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (u < n) v[u] = ld_vec<VEC>(a.x + (int64_t)(to[u] == a.G ? L.gl : L.lead[to[u]]) * a.ld + col);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (u < n) st_vec(a.Z + (int64_t)to[u] * a.ld + col, v[u]);
    }
}

// The center's step (mean in double, rows in order, rounded once) and the update that pulls every row to the center
// as it was, which also goes to the global leader's row of Z.
template <int VEC>
__device__ __forceinline__ void easgd_columns(const ColumnDev& s, int64_t col)
{
#pragma clang fp contract(off)      // (1-a)*c + a*mean as two products and a sum, rounded like the plain expression
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    double sum[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) sum[v] = 0.0;
    const V old = ld_vec<VEC>(s.center + col);
    for (int i = 0; i < a.W; i += 8) {
        V r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i + u < a.W) r[u] = ld_vec<VEC>(a.x + (int64_t)(i + u) * a.ld + col);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i + u < a.W) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) sum[v] += (double)reinterpret_cast<const float*>(&r[u])[v];
            }
    }
    V next;
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        reinterpret_cast<float*>(&next)[v] =
            (float)((1.0 - s.center_rate) * (double)reinterpret_cast<const float*>(&old)[v] + s.center_rate * (sum[v] / (double)a.W));
    st_vec(a.Z + (int64_t)a.G * a.ld + col, old);
    st_vec(s.center + col, next);
}

template <int VEC, int KIND, bool NT, bool CENTER>
__device__ __forceinline__ void step_columns(const ColumnDev& s, const Leaders& before, const Leaders& after, int64_t col, const RowBatch<VEC>& first)
{
    if (CENTER) easgd_columns<VEC>(s, col);
    if (CENTER || s.update) update_columns<VEC, KIND, NT, CENTER>(s, before, col, first);
    if (!CENTER && s.comm) comm_columns<VEC>(s, after, col);
}

// The losses from their partial sums: a team of 4 to 256 lanes per worker, in double, in an order that depends on the
// number of workers alone.  All kThreads threads; at most kColumnMaxWorkers workers.
__device__ __forceinline__ void finish_losses(const LossParts& parts, int W, float* losses)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    int team = kThreads;
    while (team * W > kThreads) team >>= 1;
    const int w = tid / team, l = tid % team;
    double acc = 0.0;
    if (w < W)
        for (int i = l; i < parts.n; i += team) {
            const int64_t at = (int64_t)w * parts.stride + i;
            acc += parts.sums64 ? parts.sums64[at] : (double)parts.sums[at];
        }
    if (team > kWave) {                                  // one or two workers
        __shared__ double cross[kThreads / kWave];
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) acc += __shfl_xor(acc, d, kWave);
        if (lane == 0) cross[tid / kWave] = acc;
        __syncthreads();
        acc = 0.0;
        for (int q = 0; q < team / kWave; ++q) acc += cross[(w * team) / kWave + q];
    } else {
        for (int d = 1; d < team; d <<= 1) acc += __shfl_xor(acc, d, kWave);
    }
    if (w < W && l == 0) losses[w] = (float)(parts.c * acc / (double)parts.div);
}

__global__ __launch_bounds__(kThreads) void loss_parts_kernel(LossParts parts, int W, float* losses) { finish_losses(parts, W, losses); }

// Leaders as recorded by earlier calls (now) and, when the call selects, as they stand after the selection (chosen);
// the first workgroup records the latter, and the losses.  All threads; ends behind a barrier.
__device__ __forceinline__ void choose_leaders(const ColumnDev& s, Leaders& now, Leaders& chosen)
{
    __shared__ float loss_s[kColumnMaxWorkers];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int W = s.a.W, G = s.a.G;
    if (s.parts.n > 0) {                                 // every workgroup adds up the partial sums itself
        finish_losses(s.parts, W, loss_s);
        __syncthreads();
    }
    if (tid < kWave) {
        if (lane < G) {                                  // as recorded by earlier calls
            now.lead[lane] = s.a.lead[lane];
            now.fresh[lane] = s.a.use_refreshed ? s.a.refreshed[lane] : 0;
        }
        if (lane == 0) {
            now.gl = s.a.glead[0];
            now.freshG = s.a.use_refreshed ? s.a.refreshed[G] : 0;
        }
        if (s.select) {
            uint64_t key = ~0ull;
            int gid = -1;
            if (lane < W) {
                key = loss_key(s.parts.n > 0 ? loss_s[lane] : s.losses[lane], lane);
                gid = s.a.group_of[lane];
            }
            uint64_t seg = key;                          // segmented inclusive minimum: keys of the lane's own group only
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint64_t ok = shfl_up_u64(seg, d);
                const int og = __shfl_up(gid, d, kWave);
                if (lane >= d && og == gid && ok < seg) seg = ok;
            }
            const uint64_t all = wave_min_u64(key);
            const int next_gid = __shfl_down(gid, 1, kWave);
            if (lane < G) {
                chosen.lead[lane] = now.lead[lane];
                chosen.fresh[lane] = (int)((s.cap >> lane) & 1ull);
            }
            if (lane == 0) {
                chosen.gl = s.selG ? (int32_t)(uint32_t)all : now.gl;
                chosen.freshG = s.capG;
            }
            __builtin_amdgcn_wave_barrier();
            if (lane < W && (lane == W - 1 || next_gid != gid) && ((s.sel >> gid) & 1ull)) chosen.lead[gid] = (int32_t)(uint32_t)seg;
        }
    }
    __syncthreads();
    if (s.losses_out && blockIdx.x == 0 && tid < W) s.losses_out[tid] = s.parts.n > 0 ? loss_s[tid] : s.losses[tid];
    if (s.select && blockIdx.x == 0) {                   // recorded for the calls that follow
        if (tid < G) {
            if ((s.sel >> tid) & 1ull) s.lead[tid] = chosen.lead[tid];
            s.refreshed[tid] = chosen.fresh[tid];
        }
        if (tid == 0) {
            if (s.selG) s.glead[0] = chosen.gl;
            s.refreshed[G] = chosen.freshG;
        }
        if (tid < W) {
            const int j = s.a.group_of[tid];
            RowPlan r;
            r.ll = chosen.lead[j]; r.gl = chosen.gl; r.freshL = chosen.fresh[j]; r.freshG = chosen.freshG; r.j = j;
            r.pad[0] = r.pad[1] = r.pad[2] = 0;
            s.plan[tid] = r;
        }
    }
}

// Capture alone (nobody moves): few registers, so that enough workgroups are resident, and each walks several tiles so
// that the selection is not repeated for every one of them.
template <int VEC>
__global__ __launch_bounds__(kThreads) void capture_kernel(ColumnDev s)
{
    __shared__ Leaders now, chosen;
    choose_leaders(s, now, chosen);
    const Leaders& L = s.select ? chosen : now;
    for (int64_t col = s.a.col0 + ((int64_t)blockIdx.x * kThreads + threadIdx.x) * VEC; col < s.a.col1;
         col += (int64_t)gridDim.x * kThreads * VEC) {
        if (col + VEC <= s.a.col1) capture_columns<VEC>(s, L, col);
        else
            for (int64_t cc = col; cc < s.a.col1; ++cc) capture_columns<1>(s, L, cc);
    }
}

template <int VEC, int KIND, bool NT, bool CENTER>
__global__ __launch_bounds__(kThreads) void column_step_kernel(ColumnDev s)
{
    __shared__ Leaders now, chosen;
    const int64_t col = s.a.col0 + ((int64_t)blockIdx.x * kThreads + threadIdx.x) * VEC;
    const bool whole = col + VEC <= s.a.col1;
    RowBatch<VEC> first;
    if (s.update && whole) load_rows<VEC, KIND, NT>(s.a, 0, pass_end<CENTER>(s.a, 0), col, first);   // under way during the selection
    choose_leaders(s, now, chosen);
    const Leaders& before = s.select == 1 ? chosen : now;
    const Leaders& after = s.select ? chosen : now;
    if (whole) step_columns<VEC, KIND, NT, CENTER>(s, before, after, col, first);
    else
        for (int64_t cc = col; cc < s.a.col1; ++cc) {
            RowBatch<1> one;
            if (s.update) load_rows<1, KIND, NT>(s.a, 0, pass_end<CENTER>(s.a, 0), cc, one);
            step_columns<1, KIND, NT, CENTER>(s, before, after, cc, one);
        }
}

template <int VEC>
void launch_vec(const ColumnDev& s, bool mom, bool nt, hipStream_t st)
{
    const int64_t cols = s.a.col1 - s.a.col0, per = (int64_t)kThreads * VEC;
    const dim3 grid((unsigned)((cols + per - 1) / per));
    auto go = [&](auto kind, auto stream, auto center) {
        hipLaunchKernelGGL((column_step_kernel<VEC, decltype(kind)::value, decltype(stream)::value, decltype(center)::value>),
                           grid, dim3(kThreads), 0, st, s);
    };
    auto with_kind = [&](auto stream, auto center) {
        if constexpr (VEC < 4) {                             // four columns per thread: without momentum only
            if (mom) { go(std::integral_constant<int, 1>{}, stream, center); return; }
        }
        go(std::integral_constant<int, 0>{}, stream, center);
    };
    auto with_stream = [&](auto center) {
        if (nt) with_kind(std::true_type{}, center);
        else with_kind(std::false_type{}, center);
    };
    if (s.center) with_stream(std::true_type{});
    else with_stream(std::false_type{});
}

} // namespace

hipError_t launch_loss_parts(const LossParts& parts, int W, float* losses, hipStream_t stream)
{
    hipLaunchKernelGGL(loss_parts_kernel, dim3(1), dim3(kThreads), 0, stream, parts, W, losses);
    return hipGetLastError();
}

hipError_t launch_column_step(const ColumnStep& q, const DeviceState& st, hipStream_t stream)
{
    const PullParams& p = q.pull;
    ColumnDev s{};
    PullDev& a = s.a;
    a.x = p.x; a.g = p.g; a.m = p.m; a.Z = p.Z; a.xb = p.xb;
    a.col0 = 0; a.col1 = p.P; a.ld = p.ld; a.W = p.W; a.G = p.G;
    a.eta = p.eta; a.lamL = p.lamL; a.lamG = p.lamG; a.mu = p.mu; a.wd = p.wd;
    a.flags = p.flags; a.use_refreshed = p.use_refreshed; a.group_size = p.group_size;
    a.offsets = st.offsets; a.group_of = st.group_of; a.lead = st.lead; a.glead = st.glead; a.refreshed = st.refreshed; a.plan = st.plan;
    s.update = q.update; s.comm = q.comm; s.commL = q.commL; s.commG = q.commG;
    s.select = q.select; s.sel = q.sel; s.cap = q.cap; s.selG = q.selG; s.capG = q.capG;
    s.losses = q.losses; s.losses_out = q.losses_out; s.parts = q.parts;
    s.lead = st.lead; s.glead = st.glead; s.refreshed = st.refreshed; s.plan = st.plan;
    s.center = q.center; s.center_rate = q.center_rate;
    const bool mom = q.update && p.mu != 0.0f;
    auto aligned = [](const void* v, unsigned n) { return (reinterpret_cast<uintptr_t>(v) & (n - 1u)) == 0; };
    auto layout_ok = [&](unsigned v) {      // every row start and every thread's group of v columns is v*4-byte aligned
        return p.ld % v == 0 && aligned(p.x, 4 * v) && (!q.update || aligned(p.g, 4 * v)) && (!mom || aligned(p.m, 4 * v)) &&
               (!p.Z || aligned(p.Z, 4 * v)) && (!p.xb || aligned(p.xb, 2 * v)) && (!q.center || aligned(q.center, 4 * v));
    };
    // Columns per thread: one, so that small rows still make enough wavefronts; more once there are plenty (16 workers
    // without momentum: 600 000 columns 27.0 / 25.6 / 24.5 us with 1 / 2 / 4, 250 000 columns 13.8 / 13.7 / 14.1;
    // with momentum two columns are never more than 2 % ahead, four mostly behind)
    int vec = 1;
    if (q.update && !mom && p.P >= 500000) vec = p.P >= 1000000 ? 4 : 2;
    // (a bf16 copy is written two bytes per lane with one column: 8 workers x 266 610 columns, whole step 62.9 -> 61.0 us)
    if (q.update && p.xb && p.P >= 100000 && vec < 2) vec = 2;
    if (!q.update) vec = 4;
    while (vec > 1 && !layout_ok((unsigned)vec)) vec >>= 1;
    // Streaming accesses (x, m past the caches) where the population neither lives in the L2s from step to step nor in
    // the memory-side cache as it is: plain / streaming, us: 16 workers with momentum, 250 000 columns (80 MB) 18.9 / 17.3,
    // 600 000 (192 MB) 37.3 / 39.1, 1 250 000 (400 MB) 80.3 / 73.7, elastic averaging there 86.4 / 73.3; pairs of workers,
    // 16 x 250 000, 26.8 / 25.3.
    // Not before a communication pull, which reads x again.
    const double bytes = (mom ? 20.0 : 12.0) * (double)p.W * (double)p.P;
    const bool nt = !q.comm && bytes >= 16e6 && (bytes < 90e6 || bytes > 280e6);
    if (!q.update && q.comm && q.commL == 0.0f && q.commG == 0.0f) {
        const int64_t tiles = (p.P + (int64_t)kThreads * vec - 1) / ((int64_t)kThreads * vec);
        const dim3 grid((unsigned)(tiles < 2048 ? tiles : 2048));
        if (vec == 4) hipLaunchKernelGGL((capture_kernel<4>), grid, dim3(kThreads), 0, stream, s);
        else if (vec == 2) hipLaunchKernelGGL((capture_kernel<2>), grid, dim3(kThreads), 0, stream, s);
        else hipLaunchKernelGGL((capture_kernel<1>), grid, dim3(kThreads), 0, stream, s);
        return hipGetLastError();
    }
    if (vec == 4) launch_vec<4>(s, mom, nt, stream);
    else if (vec == 2) launch_vec<2>(s, mom, nt, stream);
    else launch_vec<1>(s, mom, nt, stream);
    return hipGetLastError();
}

} // namespace lsgd
