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
// 24.6 -> 16.5; 16 x 250 000 with momentum 30.0 -> 17.3;
// 16 x 1 250 000 without 62.5 -> 41.5; elastic averaging, 16 x 1 250 000 with momentum 85.3 -> 73.3.
//
// The ways through the rows (launch_column_step), by what a thread has to wait for:
//   the update of groups of several workers     group by group, the next rows' loads under way (update_columns)
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

// A thread's columns of row i of p: the row's address is the same in every lane, the column's is an offset of 32 bits
// (launch_column_step refuses more), which keeps addresses out of the vector registers.
template <class T>
__device__ __forceinline__ T* at(T* p, int64_t ld, int i, uint32_t col)
{
    T* const row = p + (int64_t)i * ld;
    return reinterpret_cast<T*>(reinterpret_cast<uintptr_t>(row) + (uintptr_t)(col * (uint32_t)sizeof(T)));
}

// Every row's values at a thread's columns.
template <int VEC, int NR>
struct Rows {
    typename Vec<VEC>::type x[NR], g[NR], m[NR];
};

template <int VEC, int KIND, bool NT, int NR>
__device__ __forceinline__ void load_rows(const ColumnDev& s, uint32_t col, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            r.x[u] = NT ? ld_stream<VEC>(at(a.x, a.ld, u, col)) : ld_vec<VEC>(at(a.x, a.ld, u, col));
            r.g[u] = s.update ? ld_stream<VEC>(at(a.g, a.ld, u, col)) : zero_of(V());
            r.m[u] = (KIND == 1) ? (NT ? ld_stream<VEC>(at(a.m, a.ld, u, col)) : ld_vec<VEC>(at(a.m, a.ld, u, col))) : zero_of(V());
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
__device__ __forceinline__ void load_row(const ColumnDev& s, int i, uint32_t col, typename Vec<VEC>::type& x, typename Vec<VEC>::type& g,
                                         typename Vec<VEC>::type& m)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    x = NT ? ld_stream<VEC>(at(a.x, a.ld, i, col)) : ld_vec<VEC>(at(a.x, a.ld, i, col));
    g = s.update ? ld_stream<VEC>(at(a.g, a.ld, i, col)) : zero_of(V());
    m = (KIND == 1) ? (NT ? ld_stream<VEC>(at(a.m, a.ld, i, col)) : ld_vec<VEC>(at(a.m, a.ld, i, col))) : zero_of(V());
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

// Algorithm 1's iteration, or a communication pull alone, with every row in registers.  The update's leaders are kept copies.
template <int VEC, int KIND, bool NT, int NR>
__device__ __forceinline__ void regs_update(const ColumnDev& s, uint32_t col, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    const bool pullL = a.lamL != 0.0f, pullG = a.lamG != 0.0f;
    const Coef c = make_coef<V>(a);
    V zg = zero_of(V()), zl = zero_of(V()), nzl = zero_of(V());
    if (pullG) zg = ld_vec<VEC>(at(a.Z, a.ld, a.G, col));
    if (pullL) zl = ld_vec<VEC>(at(a.Z, a.ld, 0, col));
    if (pullL && a.G > 1) nzl = ld_vec<VEC>(at(a.Z, a.ld, 1, col));
    int j = 0, end = a.offsets[1];
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            if (u == end) {                              // the next group
                ++j; end = a.offsets[j + 1];
                zl = nzl;
                if (pullL && j + 1 < a.G) nzl = ld_vec<VEC>(at(a.Z, a.ld, j + 1, col));
            }
            update_vec<KIND, V>(r.x[u], r.g[u], r.m[u], zl, zg, c);
            if (KIND == 1) { if (NT) st_stream(at(a.m, a.ld, u, col), r.m[u]); else st_vec(at(a.m, a.ld, u, col), r.m[u]); }
        }
}

template <int VEC, bool NT, int NR>
__device__ __forceinline__ void regs_comm(const ColumnDev& s, const Leaders& L, uint32_t col, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    Coef c = make_coef<V>(a);
    c.cG = L.freshG ? s.commG : 0.0f;
    V zg = zero_of(V());
    if (L.freshG) {
        zg = row_of<VEC, NR>(r, __builtin_amdgcn_readfirstlane(L.gl));
        if (a.Z) st_vec(at(a.Z, a.ld, a.G, col), zg);
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
                    if (a.Z) st_vec(at(a.Z, a.ld, j, col), zl);
                }
            }
            const bool moves = (c.cL != 0.0f && !(fresh && u == lead)) || c.cG != 0.0f;   // (a leader's pull to itself is zero)
            V none = zero_of(V());
            if (moves) update_vec<2, V>(r.x[u], none, none, zl, zg, c);
            if (moves || s.update) {
                if (NT) st_stream(at(a.x, a.ld, u, col), r.x[u]); else st_vec(at(a.x, a.ld, u, col), r.x[u]);
                if (a.xb) st_bf16(at(a.xb, a.ld, u, col), r.x[u]);
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
__device__ __forceinline__ void regs_easgd(const ColumnDev& s, uint32_t col, Rows<VEC, NR>& r)
{
    using V = typename Vec<VEC>::type;
    const PullDev& a = s.a;
    const V old = ld_vec<VEC>(at(s.center, 0, 0, col));
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
    st_vec(at(a.Z, a.ld, a.G, col), old);
    st_vec(at(s.center, 0, 0, col), next);
    const Coef c = make_coef<V>(a);
    const V none = zero_of(V());
    const V zg = a.lamG != 0.0f ? old : none;
#pragma unroll
    for (int u = 0; u < NR; ++u)
        if (u < a.W) {
            update_vec<KIND, V>(r.x[u], r.g[u], r.m[u], none, zg, c);
            if (NT) st_stream(at(a.x, a.ld, u, col), r.x[u]); else st_vec(at(a.x, a.ld, u, col), r.x[u]);
            if (KIND == 1) { if (NT) st_stream(at(a.m, a.ld, u, col), r.m[u]); else st_vec(at(a.m, a.ld, u, col), r.m[u]); }
            if (a.xb) st_bf16(at(a.xb, a.ld, u, col), r.x[u]);
        }
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

enum { kUpdate, kUpdateOnes, kComm, kCommRegs, kCenter, kCenterRegs, kPull, kUpdatePull };

// What one thread does at its columns.  Loads are under way during the selection.  NR: rows in registers (*Regs).
template <int VEC, int KIND, bool NT, int MODE, int NR>
__device__ __forceinline__ void step_thread(const ColumnDev& s, Leaders& now, Leaders& chosen, int64_t col, bool live)
{
    const Leaders& before = s.select == 1 ? chosen : now;
    const Leaders& after = s.select ? chosen : now;
    if constexpr (MODE == kUpdate || MODE == kCenter || MODE == kUpdatePull) {
        constexpr bool CENTER = MODE == kCenter;
        RowBatch<VEC> first;
        if (live) load_rows<VEC, KIND, NT>(s.a, 0, pass_end<CENTER>(s.a, 0), col, first);
        choose_leaders(s, now, chosen);
        if (!live) return;
        if (CENTER) center_columns<VEC>(s, col);
        update_columns<VEC, KIND, NT, CENTER>(s, before, col, first);
        if (MODE == kUpdatePull) pull_columns<VEC>(s, after, col);
    } else if constexpr (MODE == kPull) {
        choose_leaders(s, now, chosen);
        if (live) pull_columns<VEC>(s, after, col);
    } else if constexpr (MODE == kUpdateOnes || MODE == kComm) {
        RowBatch<VEC> cur, next;
        if (live) {
            load_batch<VEC, KIND, NT>(s, 0, (uint32_t)col, cur);
            load_batch<VEC, KIND, NT>(s, kRowsInFlight<VEC>, (uint32_t)col, next);
        }
        choose_leaders(s, now, chosen);
        if (live) stream_columns<VEC, KIND, NT, MODE == kComm>(s, before, after, (uint32_t)col, cur, next);
    } else {
        Rows<VEC, NR> r;
        if (live) load_rows<VEC, KIND, NT, NR>(s, (uint32_t)col, r);
        choose_leaders(s, now, chosen);
        if (!live) return;
        if (MODE == kCenterRegs) {
            regs_easgd<VEC, KIND, NT, NR>(s, (uint32_t)col, r);
        } else {
            if (s.update) regs_update<VEC, KIND, NT, NR>(s, (uint32_t)col, r);
            regs_comm<VEC, NT, NR>(s, after, (uint32_t)col, r);
        }
    }
}

// The last workgroup takes the columns that are left over, one per thread, if there are any.
template <int VEC, int KIND, bool NT, int MODE, int NR>
__global__ __launch_bounds__(kThreads) void column_step_kernel(ColumnDev s)
{
    __shared__ Leaders now, chosen;
    const int64_t whole = s.a.col1 - (s.a.col1 - s.a.col0) % VEC, first = s.a.col0 + (int64_t)blockIdx.x * kThreads * VEC;
    if (VEC == 1 || first < whole) {
        const int64_t col = first + threadIdx.x * VEC;
        step_thread<VEC, KIND, NT, MODE, NR>(s, now, chosen, col, col < whole);
    } else {
        const int64_t col = whole + threadIdx.x;
        step_thread<1, KIND, NT, MODE, NR>(s, now, chosen, col, col < s.a.col1);
    }
}

template <int VEC, int KIND, int MODE, int NR>
void launch_vec(const ColumnDev& s, bool nt, hipStream_t st)
{
    const int64_t cols = s.a.col1 - s.a.col0, per = (int64_t)kThreads * VEC, whole = cols / VEC * VEC;
    const dim3 grid((unsigned)((whole + per - 1) / per + (whole < cols)));
    // one kernel where a way has but one kind of accesses: what is walked group by group is read again, rows in registers and
    // the two passes of elastic averaging stream
    constexpr bool PLAIN = MODE == kPull || MODE == kUpdatePull, STREAMS = MODE == kCommRegs || MODE == kCenter;
    if constexpr (!PLAIN)
        if (nt || STREAMS) { hipLaunchKernelGGL((column_step_kernel<VEC, KIND, true, MODE, NR>), grid, dim3(kThreads), 0, st, s); return; }
    if constexpr (!STREAMS) hipLaunchKernelGGL((column_step_kernel<VEC, KIND, false, MODE, NR>), grid, dim3(kThreads), 0, st, s);
}

// vec: columns per thread wished for; no more than the registers hold.
template <int MODE, int NR = 0>
void launch_mode(const ColumnDev& s, int vec, bool mom, bool nt, hipStream_t st)
{
    if (mom) {
        if constexpr (NR <= 16) {
            if (vec >= 2) { launch_vec<2, 1, MODE, NR>(s, nt, st); return; }
        }
        launch_vec<1, 1, MODE, NR>(s, nt, st);
    } else {
        if constexpr (NR <= 16) {
            if (vec == 4) { launch_vec<4, 0, MODE, NR>(s, nt, st); return; }
        }
        if (vec >= 2) launch_vec<2, 0, MODE, NR>(s, nt, st);
        else launch_vec<1, 0, MODE, NR>(s, nt, st);
    }
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
    const bool mom = q.update && p.mu != 0.0f;
    auto aligned = [](const void* v, unsigned n) { return (reinterpret_cast<uintptr_t>(v) & (n - 1u)) == 0; };
    auto layout_ok = [&](unsigned v) {      // every row start and every thread's group of v columns is v*4-byte aligned
        return p.ld % v == 0 && aligned(p.x, 4 * v) && (!q.update || aligned(p.g, 4 * v)) && (!mom || aligned(p.m, 4 * v)) &&
               (!p.Z || aligned(p.Z, 4 * v)) && (!p.xb || aligned(p.xb, 2 * v)) && (!q.center || aligned(q.center, 4 * v));
    };
    const double bytes = (mom ? 20.0 : 12.0) * (double)p.W * (double)p.P;
    // 13 to 16 rows with momentum, while much of x is still in the memory-side cache at its second reading: twice costs less than
    // registers for sixteen rows of three values.  Twice / once, us: 16 x 1 250 001 (400 MB) 73 / 79, 15 x 1 250 001 69 / 74, 14 x
    // 1 250 001 65 / 68, 13 x 1 250 001 (325 MB) 62 / 65, 15 x 1 400 001 (420 MB) 82 / 83; 16 x 1 400 001 (448 MB) 89 / 90, 14 x
    // 1 666 667 (467 MB) 94 / 87, 16 x 1 866 667 (597 MB) 135 / 123, 13 x 2 000 001 109 / 94; 12 x 1 250 001 (300 MB) 60 / 59.
    const bool by_groups = q.comm && (q.update ? pull_behind_update(q, bytes) : !pull_in_one_pass(q));
    const int mode = q.center ? (mom && p.W > 12 && p.W <= 16 && bytes > 300e6 && bytes <= 430e6 ? kCenter : kCenterRegs)
                   : !q.comm ? (p.W == p.G ? kUpdateOnes : kUpdate)
                   : by_groups ? (q.update ? kUpdatePull : kPull) : p.W <= 8 ? kCommRegs : kComm;
    // Columns per thread: one, so that small rows still make enough wavefronts; more once there are plenty.  Update: 16
    // workers without momentum, 600 000 columns 27.0 / 25.6 / 24.5 us with 1 / 2 / 4, 250 000 columns 13.8 / 13.7 / 14.1;
    // with momentum two columns are never more than 2 % ahead, four mostly behind.  Algorithm 1's iteration, 8 workers in 2
    // groups: 140 001 columns 8.8 / 9.4 / 10.0, 1 250 001 37 / 35 / 32.  Groups of one, 8 x 271 117, 13.6 / 12.8 / 12.5.
    // Elastic averaging, 16 x 271 117 with momentum, 18.3 / 21.1, 4 x 1 250 001 without 18.8 / 17.8 / 16.3.
    int vec = 1;
    if (mode == kUpdate || mode == kUpdatePull || mode == kCenter) {
        if (!mom && p.P >= 500000) vec = p.P >= 1000000 ? 4 : 2;
        // (a bf16 copy is written two bytes per lane with one column: 8 workers x 266 610 columns, whole step 62.9 -> 61.0 us)
        if (p.xb && p.P >= 100000 && vec < 2) vec = 2;
    } else if (mode == kCenterRegs) {
        vec = p.P < 500000 ? 1 : p.P < 1000000 ? 2 : 4;
    } else {
        vec = p.P < (mode == kComm ? 100000 : 200000) ? 1 : p.P < 500000 ? 2 : 4;
    }
    if (!q.update) vec = 4;
    while (vec > 1 && !layout_ok((unsigned)vec)) vec >>= 1;
    // Streaming accesses (x, m past the caches) where the population neither lives in the L2s from step to step nor in
    // the memory-side cache as it is: plain / streaming, us: 16 workers with momentum, 250 000 columns (80 MB) 18.9 / 17.3,
    // 600 000 (192 MB) 37.3 / 39.1, 1 250 000 (400 MB) 80.3 / 73.7, elastic averaging there 86.4 / 73.3; pairs of workers,
    // 16 x 250 000, 26.8 / 25.3.  Groups of one with their leaders re-selected write a copy of every row as well: 8 x 271 117
    // (26 MB) 13.6 / 17.3, 16 x 1 250 001 with momentum (400 MB) 106 / 90; with most of them kept 8 x 1 250 001 (120 MB) 43 / 39.
    const bool all_fresh = q.select == 1 && (q.cap & (~0ull >> (64 - p.G))) == (~0ull >> (64 - p.G));
    const bool nt = mode == kUpdateOnes ? (all_fresh ? bytes > 200e6 : true)
                  : bytes >= 16e6 && (bytes < 90e6 || bytes > 280e6);
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
    switch (mode) {
    case kUpdate: launch_mode<kUpdate>(s, vec, mom, nt, stream); break;
    case kUpdateOnes: launch_mode<kUpdateOnes>(s, vec, mom, nt, stream); break;
    case kComm: launch_mode<kComm>(s, vec, mom, nt, stream); break;
    case kUpdatePull: launch_mode<kUpdatePull>(s, vec, mom, nt, stream); break;
    case kPull:
        if (vec == 4) launch_vec<4, 0, kPull, 0>(s, false, stream);
        else if (vec == 2) launch_vec<2, 0, kPull, 0>(s, false, stream);
        else launch_vec<1, 0, kPull, 0>(s, false, stream);
        break;
    case kCommRegs:
        if (p.W <= 4) launch_mode<kCommRegs, 4>(s, vec, mom, nt, stream);
        else launch_mode<kCommRegs, 8>(s, vec, mom, nt, stream);
        break;
    case kCenter: launch_vec<1, 1, kCenter, 0>(s, nt, stream); break;
    case kCenterRegs:
        if (p.W <= 8) launch_mode<kCenterRegs, 8>(s, vec, mom, nt, stream);
        else if (p.W <= 16) launch_mode<kCenterRegs, 16>(s, vec, mom, nt, stream);
        else launch_mode<kCenterRegs, 32>(s, vec, mom, nt, stream);
        break;
    }
    return hipGetLastError();
}

} // namespace lsgd
