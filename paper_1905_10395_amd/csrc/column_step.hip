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
// less out of HBM than the row-streaming kernels (5.2 against 5.9 TB/s at 1.6 GB per update); up to 300 MB read and
// written per update, 450 for groups of one and Algorithm 1, 650 for elastic averaging (the caller's rules), the saved
// launches weigh more.  Measured, whole lsgd_step on external
// gradients, row streams -> this kernel, us: 4 x 1003 14.6 -> 4.5; 12 x 271 117 with momentum and kept leaders
// 24.6 -> 13.3; 16 x 250 000 with momentum 30.0 -> 17.3 (by groups);
// 16 x 1 250 000 without 62.5 -> 41.5; elastic averaging, 16 x 1 250 000 with momentum 85.3 -> 73.3.
//
// What bounds a small call is not memory but one wavefront's instructions, 2.7 ns each, and the loads that it waits for
// one after the other.  So what the selection reads is asked for first, all at once and by the wavefront that selects
// alone; the selection scans by data-parallel-primitive moves; and where rows are held in registers a row is one addition
// to a 32-bit offset.  Against a chain of dependent loads, scans by LDS shuffles and 64-bit row addresses: 4 x 1003 4.5 ->
// 3.6 us, 16 in 4 groups x 40 001 with momentum 10.1 -> 6.5.
//
// Medium calls whose workgroups are all resident at once hold their stores back until the chip has read its rows
// (holds_stores_*): reads among stores come slower.
//
// The ways through the rows (launch_column_step), by what a thread has to wait for:
//   the update of groups of several workers     every row in registers, leaders found in an LDS copy (held_update); nothing but
//                                               the selection is waited for twice: 12 in 3 groups x 271 117 with momentum 18.2 ->
//                                               15.5 (13.3 with stores held back), pairs, 16 x 140 001, 18.5 -> 8.7
//   ... of more than 16 workers beyond 100 MB   group by group, the next rows' loads under way (update_columns)
//   ... of groups of one, and Algorithm 1's     one pass over all rows, two batches ahead, whatever group they are in
//   iterations of more than 8 workers           (stream_columns): groups one after the other would leave a single row in
//                                               flight, and a communication pull behind the update would read x again.
//                                               16 groups of one x 140 001 36 -> 16 us, x 1 250 001 102 -> 67; iteration of
//                                               16 workers in 4 groups x 1 250 001 74 -> 60, of 24 144 -> 79
//   Algorithm 1's iterations of up to 8         every row in registers (regs_update, regs_comm): 8 workers in 2 groups x
//                                               2 500 000 81 -> 57
//   iterations and pulls in which few           group by group (pull_columns): the other ways read or work on every row,
//   groups communicate                          whoever communicates
//   elastic averaging                           every row in registers, x read once: 4 x 1003 6.5 -> 4.0, 16 x 1 250 001
//                                               without momentum 54 -> 46, 32 x 140 001 34 -> 17 (two passes for 13 to
//                                               16 rows with momentum between 300 and 430 MB)
#include "pull_common.h"
#include "select_common.h"

#include <type_traits>

namespace lsgd {

namespace {

constexpr int kThreads = 256;
template <int VEC> constexpr int kRowsInFlight = VEC == 1 ? 8 : 4;
constexpr int kHoldLoads = 3;

struct ColumnDev {
    PullDev a;                   // the update (lamL, lamG: its coefficients)
    int update, comm;            // stages present
    float commL, commG;          // coefficients of the communication pull
    int select;                  // 0: leaders as recorded, 1: selection before the update, 2: after it
    uint64_t sel, cap;           // groups re-selected now / captured by the next stage
    int selG, capG;
    uint32_t pitch;              // bytes from row to row, for the ways that hold every row
    int group_inv;               // 65536 / rows of a group, rounded up, where all groups are alike, else 0
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
    alignas(16) int row[kColumnMaxWorkers];  // kUpdateRegs: a word per row (row_word)
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
    const bool exempt = !CENTER && (a.flags & LSGD_LEADER_EXEMPT) != 0;
    const Coef c = make_coef<V>(a);
    // a re-selected leader's row belongs to the group that reads it, and the global leader's is read before any row
    // is written: both are as they were
    auto local_leader = [&](int j) { return ld_vec<VEC>((L.fresh[j] ? a.x + (int64_t)L.lead[j] * a.ld : a.Z + (int64_t)j * a.ld) + col); };
    V zg = zero_of(V()), zl = zero_of(V());
    const bool freshG = !CENTER && L.freshG;             // (elastic averaging pulls to the center and has no leaders)
    if (pullG) zg = ld_vec<VEC>((freshG ? a.x + (int64_t)L.gl * a.ld : a.Z + (int64_t)a.G * a.ld) + col);
    if (pullL) zl = local_leader(0);
    if (pullG && freshG && a.Z) st_vec(a.Z + (int64_t)a.G * a.ld + col, zg);
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

// A thread's columns of row i of p: the row's address is the same in every lane, the column's is an offset of 32 bits
// (launch_column_step refuses more), which keeps addresses out of the vector registers.  (Bytes are added to a pointer:
// through an integer the compiler loses that it is global memory, and its flat loads are waited for with every LDS
// access and scalar load.)
template <class T>
__device__ __forceinline__ T* at(T* p, int64_t ld, int i, uint32_t col)
{
    using B = std::conditional_t<std::is_const_v<T>, const char, char>;
    return reinterpret_cast<T*>(reinterpret_cast<B*>(p + (int64_t)i * ld) + col * (uint32_t)sizeof(T));
}

// The same where whole matrices span less than 4 GB (launch_column_step sees to it): the matrix's address is the same for
// all of a call's accesses, a row is one addition to a lane's offset in bytes.  (With 64-bit row addresses a row of an
// update took 30 scalar instructions, and a small call is the instructions of one wavefront.)
template <class T>
__device__ __forceinline__ T* at(T* p, uint32_t off)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 2, "");
    using B = std::conditional_t<std::is_const_v<T>, const char, char>;
    return reinterpret_cast<T*>(reinterpret_cast<B*>(p) + (sizeof(T) == 4 ? off : off / 2));
}

// Every row's values at a thread's columns.
template <int VEC, int NR>
struct Rows {
    typename Vec<VEC>::type x[NR], g[NR], m[NR];
};

template <int VEC, int KIND, bool NT>
__device__ __forceinline__ void load_row(const ColumnDev& s, int i, uint32_t col, typename Vec<VEC>::type& x, typename Vec<VEC>::type& g,
                                         typename Vec<VEC>::type& m)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    x = NT ? ld_stream<VEC>(at(a.x, a.ld, i, col)) : ld_vec<VEC>(at(a.x, a.ld, i, col));
    g = s.update ? ld_stream<VEC>(at(a.g, a.ld, i, col)) : zero_of(V());
    m = (KIND == 1) ? (NT ? ld_stream<VEC>(at(a.m, a.ld, i, col)) : ld_vec<VEC>(at(a.m, a.ld, i, col))) : zero_of(V());
}

// UPDATE: gradients and momentum too.
template <int VEC, int KIND, bool NT, bool UPDATE, int NR>
__device__ __forceinline__ void load_rows(const ColumnDev& s, uint32_t off, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            r.x[u] = NT ? ld_stream<VEC>(at(a.x, off + (uint32_t)u * s.pitch)) : ld_vec<VEC>(at(a.x, off + (uint32_t)u * s.pitch));
            r.g[u] = r.m[u] = zero_of(V());
            if (UPDATE) r.g[u] = ld_stream<VEC>(at(a.g, off + (uint32_t)u * s.pitch));
            if (UPDATE && KIND == 1) r.m[u] = NT ? ld_stream<VEC>(at(a.m, off + (uint32_t)u * s.pitch)) : ld_vec<VEC>(at(a.m, off + (uint32_t)u * s.pitch));
        }
}

// Row `i` (the same in every lane).
template <int VEC, int NR>
__device__ __forceinline__ typename Vec<VEC>::type row_of(const Rows<VEC, NR>& r, int i)
{
    typename Vec<VEC>::type v = r.x[0];
#pragma unroll
    for (int u = 1; u < NR; ++u) {
        const typename Vec<VEC>::type at = r.x[u];
        v = u == i ? at : v;
    }
    return v;
}

template <int VEC, int KIND, bool NT>
__device__ __forceinline__ void load_batch(const ColumnDev& s, int i, uint32_t col, RowBatch<VEC>& b)
{
#pragma unroll
    for (int u = 0; u < kRowsInFlight<VEC>; ++u)
        if (i + u < s.a.W) load_row<VEC, KIND, NT>(s, i + u, col, b.x[u], b.g[u], b.m[u]);
}

// !COMM: the update of groups of one worker.  COMM: the update, if there is one, and Algorithm 1's communication pull
// behind it: every leader re-selected by then is captured, groups that communicate are pulled to their leader, then
// everyone to the global leader if that was re-selected.  One pass over the rows, two batches of loads ahead; what the
// pull needs of a leader's row is its value after the update, which is worked out from that row when its group begins.
// `before`: the leaders that the update pulls to, `after`: those of the communication pull.
template <int VEC, int KIND, bool NT, bool COMM>
__device__ __forceinline__ void stream_columns(const ColumnDev& s, const Leaders& before, const Leaders& after, uint32_t col, RowBatch<VEC>& cur,
                                               RowBatch<VEC>& next)
{
    using V = typename Vec<VEC>::type;
    constexpr int R = kRowsInFlight<VEC>;
    const PullDev& a = s.a;
    const bool pullL = a.lamL != 0.0f && s.update, pullG = a.lamG != 0.0f && s.update;
    const bool exempt = !COMM && (a.flags & LSGD_LEADER_EXEMPT) != 0;
    const Coef c = make_coef<V>(a);
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    // a re-selected leader's row belongs to the group that reads it, and the global leader's is read before any row
    // is written: both are as they were
    auto local_leader = [&](int j, int lead, int fresh) { return ld_vec<VEC>(fresh ? at(a.x, a.ld, lead, col) : at(a.Z, a.ld, j, col)); };
    const int gl = uni(before.gl), freshG = uni(before.freshG);
    V zg = zero_of(V());
    if (pullG) zg = ld_vec<VEC>(freshG ? at(a.x, a.ld, gl, col) : at(a.Z, a.ld, a.G, col));
    int lead = uni(before.lead[0]), fresh = uni(before.fresh[0]);
    const bool own = !COMM;                              // groups of one: a re-selected leader is the row itself
    V nzl = zero_of(V());
    if (pullL && !(own && fresh)) nzl = local_leader(0, lead, fresh);
    // communication pull: the leaders' values after the update
    V zgc = zero_of(V()), nlx = zero_of(V()), nlg = zero_of(V()), nlm = zero_of(V());
    int clead = 0, cfresh = 0, cfreshG = 0;
    if (COMM) {
        cfreshG = uni(after.freshG);
        if (cfreshG) {
            const int cgl = uni(after.gl), j = uni(a.group_of[cgl]);
            V g, m, zl = zero_of(V());
            load_row<VEC, KIND, false>(s, cgl, col, zgc, g, m);
            if (pullL) zl = local_leader(j, uni(before.lead[j]), uni(before.fresh[j]));
            if (s.update) update_vec<KIND, V>(zgc, g, m, zl, zg, c);
        }
        clead = uni(after.lead[0]); cfresh = uni(after.fresh[0]);
        if (cfresh) load_row<VEC, KIND, false>(s, clead, col, nlx, nlg, nlm);
    }
    if (pullG && freshG && a.Z) st_vec(at(a.Z, a.ld, a.G, col), zg);
    if (COMM && cfreshG && a.Z) st_vec(at(a.Z, a.ld, a.G, col), zgc);
    V zl = zero_of(V()), zlc = zero_of(V());
    Coef cc = c;
    cc.cG = cfreshG ? s.commG : 0.0f;
    int j = -1, end = 0, crow = -1;                      // group, its end, and (COMM) the leader its rows are pulled to
    for (int at_row = 0; at_row < a.W; at_row += R) {
        int i = at_row;
        asm("" : "+s"(i));                               // (or every row's address becomes a loop variable of its own: scalar registers spill)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int row = i + u;
            if (row >= a.W) break;
            if (row == end) {                            // a group begins
                ++j; end = a.offsets[j + 1];
                zl = own && fresh ? cur.x[u] : nzl;
                if (pullL && fresh && a.Z) st_vec(at(a.Z, a.ld, j, col), zl);
                if (COMM) {
                    crow = cfresh ? clead : -1;
                    cc.cL = cfresh ? s.commL : 0.0f;
                    zlc = zero_of(V());                  // (the last group's may be infinite: not even times zero)
                    if (cfresh) {
                        zlc = nlx;
                        if (s.update) update_vec<KIND, V>(zlc, nlg, nlm, zl, zg, c);
                        if (a.Z) st_vec(at(a.Z, a.ld, j, col), zlc);
                    }
                }
                if (j + 1 < a.G) {
                    lead = uni(before.lead[j + 1]); fresh = uni(before.fresh[j + 1]);
                    if (pullL && !(own && fresh)) nzl = local_leader(j + 1, lead, fresh);
                    if (COMM) {
                        clead = uni(after.lead[j + 1]); cfresh = uni(after.fresh[j + 1]);
                        if (cfresh) load_row<VEC, KIND, false>(s, clead, col, nlx, nlg, nlm);
                    }
                }
            }
            if (s.update) {
                Coef cr = c;
                if (exempt) {
                    if (pullL && row == uni(before.lead[j])) cr.cL = 0.0f;
                    if (pullG && row == gl) cr.cG = 0.0f;
                }
                update_vec<KIND, V>(cur.x[u], cur.g[u], cur.m[u], zl, zg, cr);
                if (KIND == 1) { if (NT) st_stream(at(a.m, a.ld, row, col), cur.m[u]); else st_vec(at(a.m, a.ld, row, col), cur.m[u]); }
            }
            bool store = s.update;
            if (COMM && ((cc.cL != 0.0f && row != crow) || cc.cG != 0.0f)) {   // (a leader's pull to itself is zero)
                V none = zero_of(V());
                update_vec<2, V>(cur.x[u], none, none, zlc, zgc, cc);
                store = true;
            }
            if (store) {
                if (NT) st_stream(at(a.x, a.ld, row, col), cur.x[u]); else st_vec(at(a.x, a.ld, row, col), cur.x[u]);
                if (a.xb) st_bf16(at(a.xb, a.ld, row, col), cur.x[u]);
            }
        }
        if (i + R < a.W) {
            cur = next;
            load_batch<VEC, KIND, NT>(s, i + 2 * R, col, next);
        }
    }
}

// The update with every row in registers.  Nothing that is loaded waits for the selection: rows and kept copies are on
// their way before it, and a leader is then found among them by its number, in an LDS copy of the thread's own columns
// (rows 0 .. W-1, behind them the groups' kept copies).  No barrier for that: a thread reads only what it wrote.
// What a row has to know is one word: its local leader's place in that copy, its group, and
constexpr int kRowCaptureL = 1 << 8, kRowCaptureG = 1 << 9;     // it is a leader to be captured
constexpr int kRowExemptL = 1 << 10, kRowExemptG = 1 << 11;     // it is a leader that takes no pull
constexpr int kRowGroupShift = 16;

template <int NR> constexpr int kHeldGroups = NR / 2;           // at most

template <int VEC, int NR>
struct HeldRows {
    typename Vec<VEC>::type x[NR], g[NR], m[NR], kept[kHeldGroups<NR>], keptG;
};

template <int VEC, int KIND, bool NT, int NR>
__device__ __forceinline__ void held_load(const ColumnDev& s, uint32_t off, HeldRows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    uint32_t o = off;                                    // (no branch around a load: past the end the last row again)
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        r.x[u] = NT ? ld_stream<VEC>(at(a.x, o)) : ld_vec<VEC>(at(a.x, o));
        r.g[u] = ld_stream<VEC>(at(a.g, o));
        r.m[u] = (KIND == 1) ? (NT ? ld_stream<VEC>(at(a.m, o)) : ld_vec<VEC>(at(a.m, o))) : zero_of(V());
        o += u + 1 < a.W ? s.pitch : 0u;
    }
    if (a.lamL != 0.0f) {
#pragma unroll
        for (int j = 0; j < kHeldGroups<NR>; ++j)
            if (j < a.G && !((s.cap >> j) & 1ull)) r.kept[j] = ld_vec<VEC>(at(a.Z, off + (uint32_t)j * s.pitch));
    }
    if (a.lamG != 0.0f && !s.capG) r.keptG = ld_vec<VEC>(at(a.Z, off + (uint32_t)a.G * s.pitch));
}

template <int VEC, int KIND, bool NT, int NR>
__device__ __forceinline__ void held_update(const ColumnDev& s, const Leaders& L, uint32_t off, HeldRows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    extern __shared__ __align__(16) char held_lds[];
    V* const own = reinterpret_cast<V*>(held_lds) + threadIdx.x;
    const bool pullL = a.lamL != 0.0f, pullG = a.lamG != 0.0f;
    const Coef c = make_coef<V>(a);
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) own[u * kThreads] = r.x[u];
    if (pullL) {
#pragma unroll
        for (int j = 0; j < kHeldGroups<NR>; ++j)
            if (j < a.G && !((s.cap >> j) & 1ull)) own[(a.W + j) * kThreads] = r.kept[j];
    }
    V zg = zero_of(V());
    if (pullG) zg = s.capG ? own[__builtin_amdgcn_readfirstlane(L.gl) * kThreads] : r.keptG;
    uint32_t o = off;
#pragma unroll
    for (int i = 0; i < NR; i += 4) {
        if (i >= a.W) break;
        const int4 words = *reinterpret_cast<const int4*>(L.row + i);
        const int word[4] = {words.x, words.y, words.z, words.w};
        int row[4];
        V zl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            row[u] = __builtin_amdgcn_readfirstlane(word[u]);
            zl[u] = pullL ? own[(row[u] & 0xff) * kThreads] : zero_of(V());
        }
#pragma unroll
        for (int v = 0; v < 4; ++v, o += s.pitch) {
            const int u = i + v;
            if (u >= a.W) break;
            Coef cr = c;
            if (row[v] & (kRowCaptureL | kRowCaptureG | kRowExemptL | kRowExemptG)) {
                if (row[v] & kRowCaptureL) st_vec(at(a.Z, off + (uint32_t)(row[v] >> kRowGroupShift) * s.pitch), r.x[u]);
                if (row[v] & kRowCaptureG) st_vec(at(a.Z, off + (uint32_t)a.G * s.pitch), r.x[u]);
                if (row[v] & kRowExemptL) cr.cL = 0.0f;
                if (row[v] & kRowExemptG) cr.cG = 0.0f;
            }
            update_vec<KIND, V>(r.x[u], r.g[u], r.m[u], zl[v], zg, cr);
            if (NT) st_stream(at(a.x, o), r.x[u]); else st_vec(at(a.x, o), r.x[u]);
            if (KIND == 1) { if (NT) st_stream(at(a.m, o), r.m[u]); else st_vec(at(a.m, o), r.m[u]); }
            if (a.xb) st_bf16(at(a.xb, o), r.x[u]);
        }
    }
}

// The word of row `lane`, pulled to `own`, the global leader being `gl`.
__device__ __forceinline__ int row_word(const ColumnDev& s, int lane, int gid, int own, int gl)
{
    const PullDev& a = s.a;
    const bool fresh = (s.cap >> gid) & 1ull, pullL = a.lamL != 0.0f, pullG = a.lamG != 0.0f, exempt = (a.flags & LSGD_LEADER_EXEMPT) != 0;
    int word = (fresh ? own : a.W + gid) | gid << kRowGroupShift;
    if (pullL && own == lane) word |= (fresh && a.Z ? kRowCaptureL : 0) | (exempt ? kRowExemptL : 0);
    if (pullG && gl == lane) word |= (s.capG && a.Z ? kRowCaptureG : 0) | (exempt ? kRowExemptG : 0);
    return word;
}

// Algorithm 1's iteration, or a communication pull alone, with every row in registers.  The update's leaders are kept copies.
template <int VEC, int KIND, bool NT, int NR>
__device__ __forceinline__ void regs_update(const ColumnDev& s, uint32_t off, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    const bool pullL = a.lamL != 0.0f, pullG = a.lamG != 0.0f;
    const Coef c = make_coef<V>(a);
    V zg = zero_of(V()), zl = zero_of(V()), nzl = zero_of(V());
    if (pullG) zg = ld_vec<VEC>(at(a.Z, off + (uint32_t)a.G * s.pitch));
    if (pullL) zl = ld_vec<VEC>(at(a.Z, off));
    if (pullL && a.G > 1) nzl = ld_vec<VEC>(at(a.Z, off + s.pitch));
    int j = 0, end = a.offsets[1];
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            if (u == end) {                              // the next group
                ++j; end = a.offsets[j + 1];
                zl = nzl;
                if (pullL && j + 1 < a.G) nzl = ld_vec<VEC>(at(a.Z, off + (uint32_t)(j + 1) * s.pitch));
            }
            update_vec<KIND, V>(r.x[u], r.g[u], r.m[u], zl, zg, c);
            if (KIND == 1) { if (NT) st_stream(at(a.m, off + (uint32_t)u * s.pitch), r.m[u]); else st_vec(at(a.m, off + (uint32_t)u * s.pitch), r.m[u]); }
        }
}

template <int VEC, bool NT, bool UPDATE, int NR>
__device__ __forceinline__ void regs_comm(const ColumnDev& s, const Leaders& L, uint32_t off, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    Coef c = make_coef<V>(a);
    c.cG = L.freshG ? s.commG : 0.0f;
    // (eight rows of one column: asked at run time, or their branches are joined: 8 workers x 95 180 7.3 us instead of 6.5)
    const bool stores = UPDATE && (VEC > 1 || NR < 8 || s.update);
    V zg = zero_of(V());
    if (L.freshG) {
        zg = row_of<VEC, NR>(r, __builtin_amdgcn_readfirstlane(L.gl));
        if (a.Z) st_vec(at(a.Z, off + (uint32_t)a.G * s.pitch), zg);
    }
    int j = -1, end = 0, lead = 0;
    bool fresh = false;
    V zl = zero_of(V());
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            if (u == end) {
                ++j; end = a.offsets[j + 1];
                lead = __builtin_amdgcn_readfirstlane(L.lead[j]);
                fresh = L.fresh[j] != 0;
                c.cL = fresh ? s.commL : 0.0f;
                zl = zero_of(V());                       // (the last group's may be infinite: not even times zero)
                if (fresh) {                             // (no row of the group has moved yet)
                    zl = row_of<VEC, NR>(r, lead);
                    if (a.Z) st_vec(at(a.Z, off + (uint32_t)j * s.pitch), zl);
                }
            }
            const bool moves = (c.cL != 0.0f && !(fresh && u == lead)) || c.cG != 0.0f;   // (a leader's pull to itself is zero)
            V none = zero_of(V());
            if (moves) update_vec<2, V>(r.x[u], none, none, zl, zg, c);
            if (moves || stores) {
                if (NT) st_stream(at(a.x, off + (uint32_t)u * s.pitch), r.x[u]); else st_vec(at(a.x, off + (uint32_t)u * s.pitch), r.x[u]);
                if (a.xb) st_bf16(at(a.xb, off + (uint32_t)u * s.pitch), r.x[u]);
            }
        }
}

// A communication pull group by group, alone or behind update_columns: rows of groups that do not communicate are not touched at all.
template <int VEC>
__device__ __forceinline__ void pull_columns(const ColumnDev& s, const Leaders& L, int64_t col)
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
        const int lead = L.lead[j];
        const bool fresh = L.fresh[j] != 0;
        V zl = zero_of(V());
        if (fresh) {                                     // (no row of the group has moved yet)
            zl = ld_vec<VEC>(a.x + (int64_t)lead * a.ld + col);
            if (a.Z) st_vec(a.Z + (int64_t)j * a.ld + col, zl);
        }
        c.cL = fresh ? s.commL : 0.0f;
        if (c.cL == 0.0f && c.cG == 0.0f) continue;
        for (int i = a.offsets[j]; i < a.offsets[j + 1]; ++i) {
            if (fresh && i == lead && c.cG == 0.0f) continue;        // a leader's pull to itself is zero
            const int64_t o = (int64_t)i * a.ld + col;
            V xv = ld_vec<VEC>(a.x + o), none = zero_of(V());
            update_vec<2, V>(xv, none, none, zl, zg, c);
            st_vec(a.x + o, xv);
            if (a.xb) st_bf16(a.xb + o, xv);
        }
    }
}

// A communication pull with both coefficients zero: nobody moves, the re-selected leaders are copied to Z, eight rows of loads in
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

// Elastic averaging in two passes: the center's step (mean in double, rows in order, rounded once), the center as it was,
// which the update pulls every row to, to the global leader's row of Z; then update_columns.
template <int VEC>
__device__ __forceinline__ void center_columns(const ColumnDev& s, int64_t col)
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

// The same with every row's values in registers.
template <int VEC, int KIND, bool NT, int NR>
__device__ __forceinline__ void regs_easgd(const ColumnDev& s, uint32_t off, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    const V old = ld_vec<VEC>(at(s.center, off));
    V next;
    {
#pragma clang fp contract(off)      // (1-a)*c + a*mean as two products and a sum, rounded like the plain expression
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            double sum = 0.0;
#pragma unroll
            for (int u = 0; u < NR; ++u)
                if (u < a.W) sum += (double)reinterpret_cast<const float*>(&r.x[u])[v];
            reinterpret_cast<float*>(&next)[v] =
                (float)((1.0 - s.center_rate) * (double)reinterpret_cast<const float*>(&old)[v] + s.center_rate * (sum / (double)a.W));
        }
    }
    st_vec(at(a.Z, off + (uint32_t)a.G * s.pitch), old);
    st_vec(at(s.center, off), next);
    const Coef c = make_coef<V>(a);
    const V none = zero_of(V());
    const V zg = a.lamG != 0.0f ? old : none;
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            update_vec<KIND, V>(r.x[u], r.g[u], r.m[u], none, zg, c);
            if (NT) st_stream(at(a.x, off + (uint32_t)u * s.pitch), r.x[u]); else st_vec(at(a.x, off + (uint32_t)u * s.pitch), r.x[u]);
            if (KIND == 1) { if (NT) st_stream(at(a.m, off + (uint32_t)u * s.pitch), r.m[u]); else st_vec(at(a.m, off + (uint32_t)u * s.pitch), r.m[u]); }
            if (a.xb) st_bf16(at(a.xb, off + (uint32_t)u * s.pitch), r.x[u]);
        }
}

// What the selection reads, requested before anything else: loads return in order, so that it waits for none of the rows'.
struct Pick {
    float loss;                  // of row `lane`
    int gid;                     // its group
    int lead, fresh;             // of group `lane`, as recorded
    int gl, freshG;
    uint64_t part[4];            // partial sums of the losses, as they lie in memory
};

// The losses from their partial sums: a team of 4 to 256 lanes per worker, in double, in an order that depends on the
// number of workers alone.  All kThreads threads; at most kColumnMaxWorkers workers.
__device__ __forceinline__ int parts_team(int W)
{
    int team = kThreads;
    while (team * W > kThreads) team >>= 1;
    return team;
}
__device__ __forceinline__ void load_parts(const LossParts& parts, int W, uint64_t (&part)[4], int first)
{
    const int team = parts_team(W), w = (int)threadIdx.x / team, l = first + (int)threadIdx.x % team;
    const int64_t row = (w < W ? w : 0) * parts.stride;
    if (parts.sums64) {
#pragma unroll
        for (int u = 0; u < 4; ++u) part[u] = reinterpret_cast<const uint64_t*>(parts.sums64)[row + (l + u * team < parts.n ? l + u * team : 0)];
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) part[u] = reinterpret_cast<const uint32_t*>(parts.sums)[row + (l + u * team < parts.n ? l + u * team : 0)];
    }
}
__device__ __forceinline__ void finish_losses(const LossParts& parts, int W, uint64_t (&part)[4], float* losses)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), team = parts_team(W), w = tid / team, l = tid % team;
    double acc = 0.0;
    for (int first = 0; first < parts.n; first += 4 * team) {
        if (first) load_parts(parts, W, part, first);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double v = parts.sums64 ? __longlong_as_double((long long)part[u]) : (double)__uint_as_float((uint32_t)part[u]);
            if (w < W && first + l + u * team < parts.n) acc += v;
        }
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

__global__ __launch_bounds__(kThreads) void loss_parts_kernel(LossParts parts, int W, float* losses)
{
    uint64_t part[4];
    load_parts(parts, W, part, 0);
    finish_losses(parts, W, part, losses);
}

// By the wavefront that selects, and no more than it needs: every workgroup asks for the same few lines, which holds up
// the rows' loads behind them.  Leaders as recorded count where a call does not select, or captures one that an earlier call
// selected, or exempts kept leaders, and for what the first workgroup records.
__device__ __forceinline__ void load_pick(const ColumnDev& s, Pick& p)
{
    if (s.parts.n > 0) load_parts(s.parts, s.a.W, p.part, 0);
    if (threadIdx.x >= kWave) return;
    const int lane = threadIdx.x, W = s.a.W, G = s.a.G;
    const int i = lane < W ? lane : W - 1, j = lane < G ? lane : G - 1;
    p.loss = 0.f;
    if (s.select && s.parts.n == 0) p.loss = s.losses[i];
    if (s.group_inv) p.gid = (i * s.group_inv) >> 16;
    else p.gid = s.a.group_of[i];
    p.lead = p.gl = p.fresh = p.freshG = 0;
    if (blockIdx.x == 0 || !s.select || (s.cap & ~s.sel) || (s.capG && !s.selG) || (s.a.flags & LSGD_LEADER_EXEMPT)) {
        p.lead = s.a.lead[j];
        p.gl = s.a.glead[0];
    }
    if (s.a.use_refreshed && s.select != 1) {
        p.fresh = s.a.refreshed[j];
        p.freshG = s.a.refreshed[G];
    }
}

// Loads one after the other, by the wavefront that selects, behind the rows' (holds_stores_*).
__device__ __forceinline__ void hold_stores(const ColumnDev& s)
{
    if (threadIdx.x >= kWave) return;
    for (int h = 0; h < kHoldLoads; ++h) {
        const int v = s.a.lead[(int)threadIdx.x < s.a.G ? threadIdx.x : 0];
        asm volatile("" :: "v"(v) : "memory");           // (here it has arrived)
    }
}

// The selection's loads behind the rows', where registers are full while those are on their way, or stores are to be held back.
template <bool HOLD>
__device__ __forceinline__ void load_pick_behind(const ColumnDev& s, Pick& p)
{
    __builtin_amdgcn_sched_barrier(0);
    if (HOLD) hold_stores(s);
    load_pick(s, p);
}

// One step of a segmented minimum scan: the key of the lane that CTRL names counts if it is of the same group.  Lanes
// that have none keep theirs (ROWS: the rows of 16 lanes that take part).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t scan_min(uint32_t key, int gid)
{
    const uint32_t ok = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, CTRL, ROWS, 0xF, false);
    const int og = __builtin_amdgcn_update_dpp(-1, gid, CTRL, ROWS, 0xF, false);
    return og == gid && ok < key ? ok : key;
}

// Every row's local leader, in its lane, and the global leader: selected from the losses, or as recorded.  The smallest
// key of a group stands in its last lane after a scan (keys are the losses alone: of equal ones the lowest lane is taken),
// by data-parallel-primitive moves: a scan by LDS shuffles waits for twelve of them one after the other.
__device__ __forceinline__ void pick_leaders(const ColumnDev& s, const Pick& p, float loss, int& own, int& gl, bool& starts)
{
    const int lane = threadIdx.x & (kWave - 1), W = s.a.W;
    const bool row = lane < W;
    const uint32_t key = row ? (uint32_t)(loss_key(loss, 0) >> 32) : ~0u;
    auto scan = [&](uint32_t v, int gid) {
        v = scan_min<0x111, 0xF>(v, gid);                // row_shr:1, 2, 4, 8
        v = scan_min<0x112, 0xF>(v, gid);
        v = scan_min<0x114, 0xF>(v, gid);
        v = scan_min<0x118, 0xF>(v, gid);
        v = scan_min<0x142, 0xA>(v, gid);                // lane 15 of a row to the row behind it
        return scan_min<0x143, 0xC>(v, gid);             // lane 31 to the upper half
    };
    const int before = __builtin_amdgcn_update_dpp(-1, p.gid, 0x138, 0xF, 0xF, false);      // wave_shr:1
    starts = row && before != p.gid;
    const uint64_t lanes = ~0ull >> (kWave - W), starting = __ballot(starts);
    const int start = kWave - 1 - __builtin_clzll((starting & (~0ull >> (kWave - 1 - lane))) | 1ull);
    const uint64_t later = ((starting | ~lanes) >> lane) >> 1;
    const int last = later ? lane + __builtin_ctzll(later) : kWave - 1;
    const uint32_t seg = scan(key, row ? p.gid : -2), all = scan(key, 0);
    // (no branch from here on: behind one that only rows take, lane 63 would not have the scan's last step)
    const uint32_t least = (uint32_t)__builtin_amdgcn_ds_bpermute(last * 4, (int)seg);
    const uint32_t leastG = (uint32_t)__builtin_amdgcn_readlane((int)all, kWave - 1);
    const uint64_t best = __ballot(key == least) & lanes, bestG = __ballot(key == leastG) & lanes;
    const int picked = start + __builtin_ctzll((best >> start) | (1ull << (kWave - 1)));
    const int recorded = __builtin_amdgcn_ds_bpermute(p.gid * 4, p.lead);
    own = s.select && ((s.sel >> p.gid) & 1ull) ? picked : recorded;
    gl = s.select && s.selG ? __builtin_ctzll(bestG) : p.gl;
}

// Leaders as recorded by earlier calls (now) and, when the call selects, as they stand after the selection (chosen);
// the first workgroup records the latter, and the losses.  All threads; ends behind a barrier.
template <bool WORDS = false>
__device__ __forceinline__ void choose_leaders(const ColumnDev& s, Pick& p, Leaders& now, Leaders& chosen)
{
    __shared__ float loss_s[kColumnMaxWorkers];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int W = s.a.W, G = s.a.G;
    if (s.parts.n > 0) {                                 // every workgroup adds up the partial sums itself
        finish_losses(s.parts, W, p.part, loss_s);
        __syncthreads();
    }
    if (tid < kWave) {
        if (lane < G) {                                  // as recorded by earlier calls
            now.lead[lane] = p.lead;
            now.fresh[lane] = p.fresh;
        }
        if (lane == 0) {
            now.gl = p.gl;
            now.freshG = p.freshG;
        }
        if (s.select) {
            int own, gl;
            bool starts;
            pick_leaders(s, p, s.parts.n > 0 ? loss_s[lane < W ? lane : 0] : p.loss, own, gl, starts);
            if (starts) chosen.lead[p.gid] = own;
            if (WORDS) chosen.row[lane] = lane < W ? row_word(s, lane, p.gid, own, gl) : 0;
            if (lane < G) chosen.fresh[lane] = (int)((s.cap >> lane) & 1ull);
            if (lane == 0) {
                chosen.gl = gl;
                chosen.freshG = s.capG;
            }
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
            const int j = p.gid;
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
    Pick pick;
    load_pick(s, pick);
    choose_leaders(s, pick, now, chosen);
    const Leaders& L = s.select ? chosen : now;
    for (int64_t col = s.a.col0 + ((int64_t)blockIdx.x * kThreads + threadIdx.x) * VEC; col < s.a.col1;
         col += (int64_t)gridDim.x * kThreads * VEC) {
        if (col + VEC <= s.a.col1) capture_columns<VEC>(s, L, col);
        else
            for (int64_t cc = col; cc < s.a.col1; ++cc) capture_columns<1>(s, L, cc);
    }
}

enum { kUpdate, kUpdateOnes, kComm, kCommRegs, kCenter, kCenterRegs, kPull, kUpdatePull, kUpdateRegs, kPullRegs };

// What one thread does at its columns.  Loads are under way during the selection.  NR: rows in registers (*Regs).
template <int VEC, int KIND, bool NT, int MODE, int NR, bool HOLD>
__device__ __forceinline__ void step_thread(const ColumnDev& s, Leaders& now, Leaders& chosen, int64_t col, bool live)
{
    const Leaders& before = s.select == 1 ? chosen : now;
    const Leaders& after = s.select ? chosen : now;
    Pick pick;
    // (eight rows of four columns: with what the selection reads, and every row's offset kept from its load to its store, 100
    // registers, one wavefront less per SIMD than with 96: 8 workers in 2 groups x 1 250 001 30.9 us instead of 28.0)
    constexpr bool FULL = MODE == kCommRegs && VEC == 4 && NR == 8, BEHIND = HOLD || FULL;
    if (MODE == kCenter || MODE == kCenterRegs) {
        if (blockIdx.x == 0) load_pick(s, pick);
    } else if (!BEHIND) {
        load_pick(s, pick);
    }
    if constexpr (MODE == kUpdate || MODE == kCenter || MODE == kUpdatePull) {
        constexpr bool CENTER = MODE == kCenter;
        RowBatch<VEC> first;
        if (live) load_rows<VEC, KIND, NT>(s.a, 0, pass_end<CENTER>(s.a, 0), col, first);
        if constexpr (BEHIND) load_pick_behind<HOLD>(s, pick);
        if (!CENTER || blockIdx.x == 0) choose_leaders(s, pick, now, chosen);              // (CENTER: the losses alone)
        if (!live) return;
        if (CENTER) center_columns<VEC>(s, col);
        update_columns<VEC, KIND, NT, CENTER>(s, before, col, first);
        if (MODE == kUpdatePull) pull_columns<VEC>(s, after, col);
    } else if constexpr (MODE == kUpdateRegs) {
        HeldRows<VEC, NR> r;
        const uint32_t off = (uint32_t)col * 4u;
        if (live) held_load<VEC, KIND, NT, NR>(s, off, r);
        if constexpr (BEHIND) load_pick_behind<HOLD>(s, pick);
        choose_leaders<true>(s, pick, now, chosen);
        if (live) held_update<VEC, KIND, NT, NR>(s, chosen, off, r);
    } else if constexpr (MODE == kPull) {
        choose_leaders(s, pick, now, chosen);
        if (live) pull_columns<VEC>(s, after, col);
    } else if constexpr (MODE == kUpdateOnes || MODE == kComm) {
        RowBatch<VEC> cur, next;
        if (live) {
            load_batch<VEC, KIND, NT>(s, 0, (uint32_t)col, cur);
            load_batch<VEC, KIND, NT>(s, kRowsInFlight<VEC>, (uint32_t)col, next);
        }
        if constexpr (BEHIND) load_pick_behind<HOLD>(s, pick);
        choose_leaders(s, pick, now, chosen);
        if (live) stream_columns<VEC, KIND, NT, MODE == kComm>(s, before, after, (uint32_t)col, cur, next);
    } else {
        Rows<VEC, NR> r;
        if constexpr (MODE == kCenterRegs) {
            if (live) load_rows<VEC, KIND, NT, true, NR>(s, (uint32_t)col * 4u, r);
            if constexpr (HOLD) {
                __builtin_amdgcn_sched_barrier(0);
                hold_stores(s);
                __syncthreads();
            }
            if (blockIdx.x == 0) choose_leaders(s, pick, now, chosen);                   // the losses alone
            if (live) regs_easgd<VEC, KIND, NT, NR>(s, (uint32_t)col * 4u, r);
            return;
        }
        constexpr bool UPDATE = MODE == kCommRegs;
        uint32_t off = (uint32_t)col * 4u;
        if (live) load_rows<VEC, KIND, NT, UPDATE, NR>(s, off, r);
        if constexpr (BEHIND) load_pick_behind<HOLD>(s, pick);
        // (stores count in the same counter: with one column per thread rows that are waited for between them take 5 % longer)
        if constexpr (VEC == 1) __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt 0
        choose_leaders(s, pick, now, chosen);
        if (!live) return;
        if constexpr (FULL) asm("" : "+v"(off));         // (the compiler works it out anew)
        if constexpr (UPDATE) regs_update<VEC, KIND, NT, NR>(s, off, r);
        regs_comm<VEC, NT, UPDATE, NR>(s, after, off, r);
    }
}

// The last workgroup takes the columns that are left over, one per thread, if there are any.
// HOLD: stores are held back.
template <int VEC, int KIND, bool NT, int MODE, int NR, bool HOLD>
__global__ __launch_bounds__(kThreads) void column_step_kernel(ColumnDev s)
{
    __shared__ Leaders now, chosen;
    const int64_t whole = s.a.col1 - (s.a.col1 - s.a.col0) % VEC, first = s.a.col0 + (int64_t)blockIdx.x * kThreads * VEC;
    if (VEC == 1 || first < whole) {
        const int64_t col = first + threadIdx.x * VEC;
        step_thread<VEC, KIND, NT, MODE, NR, HOLD>(s, now, chosen, col, col < whole);
    } else {
        const int64_t col = whole + threadIdx.x;
        step_thread<1, KIND, NT, MODE, NR, HOLD>(s, now, chosen, col, col < s.a.col1);
    }
}

size_t held_bytes(int W, int G) { return (size_t)(W + G) * kThreads * sizeof(float); }     // (one column per thread)

int64_t workgroups(int64_t cols, int vec)
{
    const int64_t per = (int64_t)kThreads * vec, whole = cols / vec * vec;
    return (whole + per - 1) / per + (whole < cols);
}

// Kernels that hold their stores back: those that ask for all rows, or all they have room for, before they store any, where the
// rules below (holds_stores_*) can send a call to them.
template <int VEC, int KIND, int MODE, int NR>
constexpr bool kCanHold = MODE == kCommRegs ? (KIND ? 20.0 : 12.0) * NR * 1536 * kThreads * VEC >= 40e6
                        : MODE == kUpdateOnes ? VEC == 4 || (VEC == 2 && KIND == 1)
                        : MODE == kUpdateRegs ? NR > 4 : MODE == kCenterRegs || (MODE == kUpdate && VEC == 4 && KIND == 0);

// How many workgroups of a kernel that holds its stores back are resident at once, on 256 compute units: by its registers,
// which are asked for once, and the LDS it is launched with.
template <int VEC, int KIND, int MODE, int NR>
int64_t resident(size_t lds)
{
    static const int by_registers = [] {
        int n = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, column_step_kernel<VEC, KIND, true, MODE, NR, true>, kThreads, 0) == hipSuccess ? n : 0;
    }();
    const int by_lds = (int)(160 * 1024 / (lds + 2048));
    return 256 * (int64_t)(by_registers < by_lds ? by_registers : by_lds);
}

template <int VEC, int KIND, int MODE, int NR>
void launch_vec(const ColumnDev& s, bool nt, bool hold, hipStream_t st)
{
    const dim3 grid((unsigned)workgroups(s.a.col1 - s.a.col0, VEC));
    // one kernel where a way has but one kind of accesses: what is walked group by group is read again, rows in registers and
    // the two passes of elastic averaging stream, and so does most of what holds its stores back
    constexpr bool PLAIN = MODE == kPull || MODE == kUpdatePull, STREAMS = MODE == kCommRegs || MODE == kPullRegs || MODE == kCenter;
    const size_t lds = MODE == kUpdateRegs ? held_bytes(s.a.W, s.a.G) : 0;
    if constexpr (kCanHold<VEC, KIND, MODE, NR>) {
        if (hold) {
            if constexpr (MODE == kUpdateOnes)
                if (!nt) { hipLaunchKernelGGL((column_step_kernel<VEC, KIND, false, MODE, NR, true>), grid, dim3(kThreads), lds, st, s); return; }
            hipLaunchKernelGGL((column_step_kernel<VEC, KIND, true, MODE, NR, true>), grid, dim3(kThreads), lds, st, s);
            return;
        }
    }
    if constexpr (!PLAIN)
        if (nt || STREAMS) { hipLaunchKernelGGL((column_step_kernel<VEC, KIND, true, MODE, NR, false>), grid, dim3(kThreads), lds, st, s); return; }
    if constexpr (!STREAMS) hipLaunchKernelGGL((column_step_kernel<VEC, KIND, false, MODE, NR, false>), grid, dim3(kThreads), lds, st, s);
}

// vec: columns per thread; with momentum no more than two.
template <int MODE, int NR = 0>
void launch_mode(const ColumnDev& s, int vec, bool mom, bool nt, bool hold, hipStream_t st)
{
    if (mom) {
        if (vec >= 2) launch_vec<2, 1, MODE, NR>(s, nt, hold, st);
        else launch_vec<1, 1, MODE, NR>(s, nt, hold, st);
    } else {
        if (vec == 4) launch_vec<4, 0, MODE, NR>(s, nt, hold, st);
        else if (vec >= 2) launch_vec<2, 0, MODE, NR>(s, nt, hold, st);
        else launch_vec<1, 0, MODE, NR>(s, nt, hold, st);
    }
}

// The update of groups of several workers: whether every row in registers beats a walk by groups.  By groups / registers,
// us: 24 workers in 4 groups with momentum x 140 001 (67 MB) 19.4 / 17.1, x 271 117 (130 MB) nothing re-selected 27.3 / 27.8,
// x 600 001 (288 MB) 56 / 59; 32 in 4 groups x 271 117 (104 MB) 23.2 / 24.1; 16 in 4 groups x 1 250 001 (240 MB) 48 / 46.  4 workers
// without momentum, nothing re-selected, x 271 117 (13 MB) 6.5 / 5.1, x 1 250 001 (60 MB) 12.5 / 14.4 (15.6 / 15.4 where it is).
// 313 populations of 4 to 32 workers, 1003 to 1 250 001 columns: 0.82 of the time.
bool update_in_registers(const ColumnStep& q, double bytes)
{
    const PullParams& p = q.pull;
    if (p.W > 16) return bytes <= 100e6;
    return p.W > 4 || p.mu != 0.0f || q.cap || q.capG || bytes <= 35e6;
}

// Holding stores back.  Where all workgroups of a launch are resident at once and ask for all their rows at once, those whose
// rows come first would store while the others still wait for theirs, and reads among stores come slower: of 1221 workgroups
// (4 workers x 1 250 001 without momentum, nothing re-selected) the last had its rows after 11.8 us, held back after 9.2.  So
// the wavefront that selects first sends kHoldLoads loads one after the other.  They queue behind the rows of all: long while
// the chip reads, short when it no longer does.  (A fixed number of clocks instead: 14.1 us and more where these take 12.5 and
// nothing 13.8.  That the selection itself was once such a chain is why it was the faster one at these sizes.)  It costs up to
// 0.5 us where there is nothing to hold apart: smaller calls, or more workgroups than are resident, which store in turns anyway.
//
// Rows in registers, us, without / with: 12 in 3 groups x 271 117 with momentum (65 MB) 15.9 / 13.5, 8 in one x 271 117 with
// (43 MB) 10.5 / 9.4, 16 in 4 x 170 001 with (54 MB, 665 workgroups) 12.6 / 11.4, 28 in 7 x 140 001 with (78 MB, 547) 20.3 / 17.3;
// not 24 in 4 x 140 001 without (40 MB, 547) 10.6 / 11.2, 16 in 4 x 100 001 with (32 MB) 8.5 / 9.0, 16 in 4 x 450 001 without
// (1758 workgroups on 1536 places) 20.0 / 21.0, 32 in 8 x 230 001 without (899 on 768) 22.4 / 23.6.
template <int KIND, int NR>
bool holds_stores_regs(const ColumnDev& s, double bytes)
{
    const int64_t n = workgroups(s.a.col1 - s.a.col0, 1);
    return (bytes >= 55e6 || (bytes >= 40e6 && n >= 640)) && n <= resident<1, KIND, kUpdateRegs, NR>(held_bytes(s.a.W, s.a.G));
}
// By groups: only where one batch holds all rows (4 in 2 groups x 1 250 001 14.2 / 15.2).  4 in one x 1 250 001 13.8 / 12.5, x
// 1 000 001 11.2 / 10.6, 3 x 1 250 001 11.3 / 10.3; not x 1 400 001 (1367 workgroups on 1280 places) 15.5 / 17.0.
bool holds_stores_batch(const ColumnDev& s, int vec, double bytes)
{
    return s.select == 1 && vec == 4 && s.a.G == 1 && s.a.W <= kRowsInFlight<4> && bytes >= 36e6 &&
           workgroups(s.a.col1 - s.a.col0, 4) <= resident<4, 0, kUpdate, 0>(0);
}
// Algorithm 1's iteration: 4 x 1 250 001 15.6 / 13.7, 4 x 700 001 with momentum 13.4 / 11.7, 8 in 2 groups x 600 001 with 23.0 /
// 21.2, without 15.6 / 14.1, x 271 117 with (43 MB) 12.1 / 11.3; not 4 x 1 600 001 (1563 workgroups) 19.5 / 20.1, 8 in 2 x 140 001
// with (547 workgroups) 8.3 / 8.6.
bool holds_stores_comm(const ColumnDev& s, int vec, double bytes)
{
    const int64_t n = workgroups(s.a.col1 - s.a.col0, vec);
    return bytes >= (vec == 4 ? 36e6 : 40e6) && n >= 768 && n <= 1536;
}

// Groups of one, while the batches ahead hold all rows: 8 x 800 001 without momentum (77 MB, 782 workgroups), one re-selected, 23.1 /
// 20.8, x 400 001 with (64 MB) 19.3 / 17.6; x 400 001 without (38 MB) no sure difference; not 4 x 1 250 001 without (1221 workgroups
// on 1024 places) 17.1 / 19.1.
template <int VEC, int KIND>
bool holds_stores_ones(const ColumnDev& s, double bytes)
{
    return bytes >= 55e6 && bytes <= 100e6 && s.a.W <= 2 * kRowsInFlight<VEC> && workgroups(s.a.col1 - s.a.col0, VEC) <= resident<VEC, KIND, kUpdateOnes, 0>(0);
}

// Elastic averaging with every row in registers, plain accesses without / streaming with: 4 x 400 001 with momentum 7.8 / 6.8, 5 x
// 500 001 with 11.1 / 9.4, 8 x 400 001 without 9.1 / 8.3, with 13.8 / 11.9, 16 x 200 001 with 14.1 / 13.2, 32 x 140 001 with (90 MB, 547
// workgroups) 19.3 / 18.3; not 16 x 100 001 with (391 workgroups) 7.6 / 7.8, 4 x 600 001 with (2344 on 2048 places) 11.4 / 12.0, 4 x
// 1 250 001 without 13.8 / 15.9, and nothing gained below 24 MB.
template <int KIND, int NR>
bool holds_stores_center(const ColumnDev& s, double bytes)
{
    const int64_t n = workgroups(s.a.col1 - s.a.col0, 1);
    return bytes >= 24e6 && bytes < 90e6 && n >= (bytes >= 55e6 ? 512 : 640) && n <= resident<1, KIND, kCenterRegs, NR>(0);
}

// One column per thread.
template <int MODE, int NR = 0>
void launch_narrow(const ColumnDev& s, bool mom, bool nt, bool hold, hipStream_t st)
{
    if (mom) launch_vec<1, 1, MODE, NR>(s, nt, hold, st);
    else launch_vec<1, 0, MODE, NR>(s, nt, hold, st);
}

template <int MODE, int NR>
void launch_pull(const ColumnDev& s, int vec, hipStream_t st)
{
    if (vec == 4) launch_vec<4, 0, MODE, NR>(s, false, false, st);
    else if (vec == 2) launch_vec<2, 0, MODE, NR>(s, false, false, st);
    else launch_vec<1, 0, MODE, NR>(s, false, false, st);
}

// The update of groups of several workers, every row in registers.
template <int NR>
void launch_held(const ColumnDev& s, bool mom, bool nt, double bytes, hipStream_t st)
{
    bool hold = false;
    if constexpr (kCanHold<1, 0, kUpdateRegs, NR>) hold = nt && (mom ? holds_stores_regs<1, NR>(s, bytes) : holds_stores_regs<0, NR>(s, bytes));
    launch_narrow<kUpdateRegs, NR>(s, mom, nt, hold, st);
}

// Elastic averaging with every row in registers.
template <int NR>
void launch_center_regs(const ColumnDev& s, bool mom, bool nt, double bytes, hipStream_t st)
{
    const bool hold = mom ? holds_stores_center<1, NR>(s, bytes) : holds_stores_center<0, NR>(s, bytes);
    launch_narrow<kCenterRegs, NR>(s, mom, nt || hold, hold, st);
}

// A pull alone: whether one pass over all rows beats a walk group by group, which touches only rows that move.  One pass / by
// groups, us, selection included: 8 workers in 2 groups x 400 001 one group communicates 9.0 / 9.2, both 10.3 / 12.9, the global
// leader too 11.6 / 14.7; 16 in 4 x 140 001 one 11.3 / 7.6, all 13.2 / 15.5, x 1 000 001 all 31 / 25; 32 in 8 x 400 001 one 20 / 9,
// all 27 / 30; 16 in 8 x 40 001 all 13.1 / 12.1, x 400 001 23 / 20.  Over 1190 pulls, 2 to 32 workers in 1 to 32 groups, 1003 to
// 3 million columns, none more than 5 % slower than with the walk (row streams for groups of one), 13 % faster together.
bool pull_in_one_pass(const ColumnStep& q)
{
    const PullParams& p = q.pull;
    const double bytes = 12.0 * (double)p.W * (double)p.P;
    const bool large_groups = p.W >= 4 * p.G;
    if (p.W <= 8) return q.capG && (p.W > 4 || p.W < 2 * p.G || bytes <= 100e6);        // 4 in 2 x 2 500 000 25.6 / 23.8
    if (!q.capG && !(large_groups && __builtin_popcountll(q.cap) == p.G)) return false;
    return large_groups ? p.W > 16 || bytes <= 70e6 : bytes <= 40e6;
}

// An iteration of Algorithm 1: whether its pull is better walked group by group behind the update, which reads rows a second
// time, but only those that move.  One pass / behind the update, us: 24 workers in 4 groups x 1003 one group communicates
// 10.6 / 9.5, three 11.1 / 11.6, x 400 001 (115 MB) one 29.4 / 28.7, two 29.7 / 31.9; 16 in 8 x 1 000 001 (192 MB) one 55 / 41,
// all 65 / 59; with momentum 32 in 8 x 140 001 (90 MB) one 31 / 27, all 36 / 34, 16 in 8 (45 MB) all 25.8 / 23.2.  To a global
// leader everybody moves: 24 in 4 x 140 001 18.0 / 19.6, but 16 in 8 with momentum 26.6 / 24.8.  Registers of eight rows with momentum are slower than a walk while
// rows are short: 8 in 1 x 40 001 7.5 / 6.7, x 140 001 9.3 / 9.5.
bool pull_behind_update(const ColumnStep& q, double bytes)
{
    const PullParams& p = q.pull;
    const int fresh = __builtin_popcountll(q.cap);
    const bool mom = p.mu != 0.0f, large_groups = p.W >= 4 * p.G;
    if (p.W <= 8) return mom && p.W > 4 && p.P < 100000 && large_groups && (p.G == 1 || (!q.capG && 2 * fresh <= p.G));
    if (p.W < 2 * p.G || bytes > 300e6) return false;
    if (mom && bytes >= 30e6 && bytes < (q.capG ? 60e6 : 95e6) && (!q.capG || (fresh == p.G && p.W <= 16))) return true;
    if (q.capG) return false;
    return large_groups ? fresh * (bytes < 100e6 ? 2 : 4) <= p.G : p.W <= 16 && bytes >= (2 * fresh <= p.G ? 70e6 : 150e6);
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
    s.group_inv = p.group_size > 0 ? (65535 + p.group_size) / p.group_size : 0;          // (exact for up to 64 rows)
    const bool mom = q.update && p.mu != 0.0f;
    auto aligned = [](const void* v, unsigned n) { return (reinterpret_cast<uintptr_t>(v) & (n - 1u)) == 0; };
    auto layout_ok = [&](unsigned v) {      // every row start and every thread's group of v columns is v*4-byte aligned
        return p.ld % v == 0 && aligned(p.x, 4 * v) && (!q.update || aligned(p.g, 4 * v)) && (!mom || aligned(p.m, 4 * v)) &&
               (!p.Z || aligned(p.Z, 4 * v)) && (!p.xb || aligned(p.xb, 2 * v)) && (!q.center || aligned(q.center, 4 * v));
    };
    const double bytes = (mom ? 20.0 : 12.0) * (double)p.W * (double)p.P;
    // whole matrices within reach of 32-bit offsets (rows may lie far apart)
    const bool near = (double)(p.W + 1) * (double)p.ld < (double)(1u << 30);
    const bool by_groups = q.comm && ((p.W <= 8 && !near) || (q.update ? pull_behind_update(q, bytes) : !pull_in_one_pass(q)));
    const bool held = near && q.select == 1 && p.W >= 2 * p.G && update_in_registers(q, bytes);
    s.pitch = (uint32_t)p.ld * 4u;
    // 13 to 16 rows with momentum, while much of x is still in the memory-side cache at its second reading: twice costs less than
    // registers for sixteen rows of three values.  Twice / once, us: 16 x 1 250 001 (400 MB) 73 / 79, 15 x 1 250 001 69 / 74, 14 x
    // 1 250 001 65 / 68, 13 x 1 250 001 (325 MB) 62 / 65, 15 x 1 400 001 (420 MB) 82 / 83; 16 x 1 400 001 (448 MB) 89 / 90, 14 x
    // 1 666 667 (467 MB) 94 / 87, 16 x 1 866 667 (597 MB) 135 / 123, 13 x 2 000 001 109 / 94; 12 x 1 250 001 (300 MB) 60 / 59.
    const int mode = q.center ? ((mom && p.W > 12 && p.W <= 16 && bytes > 300e6 && bytes <= 430e6) || !near ? kCenter : kCenterRegs)
                   : !q.comm ? (p.W == p.G ? kUpdateOnes : held ? kUpdateRegs : kUpdate)
                   : by_groups ? (q.update ? kUpdatePull : kPull) : p.W <= 8 ? (q.update ? kCommRegs : kPullRegs) : kComm;
    // Columns per thread: one, so that small rows still make enough wavefronts; more once there are plenty, but not where
    // every row's loads are under way at once, which wait less with one.  Update by groups: 16
    // workers without momentum, 600 000 columns 27.0 / 25.6 / 24.5 us with 1 / 2 / 4, 250 000 columns 13.8 / 13.7 / 14.1;
    // with momentum two columns are never more than 2 % ahead, four mostly behind.  From registers, 16 workers in 4 groups,
    // 140 001 columns 8.1 / 9.3 / 9.2, with momentum 10.5 / 13.7 / 13.8, 1 250 001 46 / 52 / 59.  Algorithm 1's iteration,
    // 8 workers in 2 groups with momentum, 271 117 columns 11.9 / 13.4 / 13.4, 600 001 25.1 / 23.0 / 23.0; 4 workers without x
    // 800 001 12.9 / 11.4 with 2 / 4, x 1 250 001 19.8 / 17.6 / 14.1.  Groups of one, 8 x 271 117, 13.6 / 12.8 / 12.5.
    // Elastic averaging, 16 without momentum x 600 001 22 / 29 / 29, with momentum x 140 001 10.0 / 12.8 / 12.8.
    int vec = 1;
    if (mode == kUpdate || mode == kUpdatePull) {
        if (!mom && p.P >= 500000) vec = p.P >= 1000000 ? 4 : 2;
        // (a bf16 copy is written two bytes per lane with one column: 8 workers x 266 610 columns, whole step 62.9 -> 61.0 us)
        if (p.xb && p.P >= 100000 && vec < 2) vec = 2;
    } else if (mode == kCommRegs) {
        vec = p.P < 400000 ? 1 : mom || p.P < 750000 ? 2 : 4;
    } else if (mode != kUpdateRegs && mode != kCenterRegs && mode != kCenter) {
        vec = p.P < (mode == kComm ? 100000 : 200000) ? 1 : p.P < 500000 ? 2 : 4;
    }
    if (!q.update) vec = 4;
    while (vec > 1 && !layout_ok((unsigned)vec)) vec >>= 1;
    // Streaming accesses (x, m past the caches) where the population neither lives in the L2s from step to step nor in
    // the memory-side cache as it is: plain / streaming, us: 16 workers with momentum, 250 000 columns (80 MB) 18.9 / 17.3,
    // 600 000 (192 MB) 37.3 / 39.1, 1 250 000 (400 MB) 80.3 / 73.7, elastic averaging there 86.4 / 73.3; pairs of workers,
    // 16 x 250 000, 26.8 / 25.3.  Groups of one with their leaders re-selected write a copy of every row as well: 8 x 271 117
    // (26 MB) 13.6 / 17.3, 16 x 1 250 001 with momentum (400 MB) 106 / 90; with most of them kept 8 x 1 250 001 (120 MB) 43 / 39.
    // Elastic averaging from registers reads x once; beside the calls that hold their stores back those of few workers stream: 2 x
    // 600 001 with momentum (24 MB) 7.1 / 6.3, 3 x 800 001 without 8.2 / 7.8, 4 x 600 001 without 8.0 / 7.2; not 12 x 600 001 without
    // (86 MB) 17.3 / 18.0, 4 x 1 250 001 without 14.0 / 14.4.
    const bool center_streams = p.W <= 4 && bytes >= 24e6 && p.P <= 1000000;
    const bool all_fresh = q.select == 1 && (q.cap & (~0ull >> (64 - p.G))) == (~0ull >> (64 - p.G));
    const bool nt = mode == kUpdateOnes ? (all_fresh ? bytes > 200e6 : true)
                  : bytes > 280e6 || (bytes >= 16e6 && bytes < 90e6 && (mode != kCenterRegs || center_streams));
    if (!q.update && q.comm && q.commL == 0.0f && q.commG == 0.0f) {
        const int64_t tiles = (p.P + (int64_t)kThreads * vec - 1) / ((int64_t)kThreads * vec);
        const dim3 grid((unsigned)(tiles < 2048 ? tiles : 2048));
        if (vec == 4) hipLaunchKernelGGL((capture_kernel<4>), grid, dim3(kThreads), 0, stream, s);
        else if (vec == 2) hipLaunchKernelGGL((capture_kernel<2>), grid, dim3(kThreads), 0, stream, s);
        else hipLaunchKernelGGL((capture_kernel<1>), grid, dim3(kThreads), 0, stream, s);
        return hipGetLastError();
    }
    // (captures alone, above, take any number of columns)
    if (p.P > ((int64_t)1 << 30) && mode != kUpdate && mode != kPull && mode != kUpdatePull && mode != kCenter) return hipErrorInvalidValue;
    const bool hold_comm = holds_stores_comm(s, mom && vec > 2 ? 2 : vec, bytes);
    switch (mode) {
    case kUpdate: launch_mode<kUpdate>(s, vec, mom, nt, nt && !mom && holds_stores_batch(s, vec, bytes), stream); break;
    case kUpdateOnes:
        launch_mode<kUpdateOnes>(s, vec, mom, nt, mom ? vec >= 2 && holds_stores_ones<2, 1>(s, bytes) : vec == 4 && holds_stores_ones<4, 0>(s, bytes), stream);
        break;
    case kUpdateRegs:
        if (p.W <= 4) launch_held<4>(s, mom, nt, bytes, stream);
        else if (p.W <= 8) launch_held<8>(s, mom, nt, bytes, stream);
        else if (p.W <= 12) launch_held<12>(s, mom, nt, bytes, stream);
        else if (p.W <= 16) launch_held<16>(s, mom, nt, bytes, stream);
        else if (p.W <= 24) launch_held<24>(s, mom, nt, bytes, stream);
        else launch_held<32>(s, mom, nt, bytes, stream);
        break;
    case kComm: launch_mode<kComm>(s, vec, mom, nt, false, stream); break;
    case kUpdatePull: launch_mode<kUpdatePull>(s, vec, mom, nt, false, stream); break;
    case kPull: launch_pull<kPull, 0>(s, vec, stream); break;
    case kCommRegs:
        if (p.W <= 4) launch_mode<kCommRegs, 4>(s, vec, mom, nt, hold_comm, stream);
        else launch_mode<kCommRegs, 8>(s, vec, mom, nt, hold_comm, stream);
        break;
    case kPullRegs:
        if (p.W <= 4) launch_pull<kPullRegs, 4>(s, vec, stream);
        else launch_pull<kPullRegs, 8>(s, vec, stream);
        break;
    case kCenter: launch_narrow<kCenter>(s, mom, nt, false, stream); break;
    case kCenterRegs:
        if (p.W <= 8) launch_center_regs<8>(s, mom, nt, bytes, stream);
        else if (p.W <= 16) launch_center_regs<16>(s, mom, nt, bytes, stream);
        else launch_center_regs<32>(s, mom, nt, bytes, stream);
        break;
    }
    return hipGetLastError();
}

} // namespace lsgd
