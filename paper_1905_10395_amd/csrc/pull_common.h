// Vector accesses and the per-row update shared by the kernels that apply the leader pull.
#pragma once

#include "common.h"
#include "update_math.h"

namespace lsgd {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

template <int VEC> struct Vec;
template <> struct Vec<4> { using type = v4f; };
template <> struct Vec<2> { using type = v2f; };
template <> struct Vec<1> { using type = float; };

template <int VEC> __device__ __forceinline__ typename Vec<VEC>::type ld_vec(const float* p)
{
    return *reinterpret_cast<const typename Vec<VEC>::type*>(p);
}
template <int VEC> __device__ __forceinline__ typename Vec<VEC>::type ld_stream(const float* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const typename Vec<VEC>::type*>(p));
}

__device__ __forceinline__ void st_vec(float* p, v4f v) { *reinterpret_cast<v4f*>(p) = v; }
__device__ __forceinline__ void st_vec(float* p, v2f v) { *reinterpret_cast<v2f*>(p) = v; }
__device__ __forceinline__ void st_vec(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_stream(float* p, v4f v) { __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(p)); }
__device__ __forceinline__ void st_stream(float* p, v2f v) { __builtin_nontemporal_store(v, reinterpret_cast<v2f*>(p)); }
__device__ __forceinline__ void st_stream(float* p, float v) { __builtin_nontemporal_store(v, p); }

__device__ __forceinline__ void st_bf16(uint16_t* p, v4f v)
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    const v2u o = {f32x2_to_bf16x2(v.x, v.y), f32x2_to_bf16x2(v.z, v.w)};
    *reinterpret_cast<v2u*>(p) = o;
}
__device__ __forceinline__ void st_bf16(uint16_t* p, v2f v) { *reinterpret_cast<unsigned int*>(p) = f32x2_to_bf16x2(v.x, v.y); }
__device__ __forceinline__ void st_bf16(uint16_t* p, float v) { *p = f32_to_bf16_rne(v); }

__device__ __forceinline__ v4f zero_of(v4f) { return (v4f)(0.f); }
__device__ __forceinline__ v2f zero_of(v2f) { return (v2f)(0.f); }
__device__ __forceinline__ float zero_of(float) { return 0.f; }

constexpr int kPullThreads = 256;

struct PullDev {
    float* x;
    const float* g;
    float* m;
    float* Z;
    uint16_t* xb;
    int64_t col0, col1, ld; // columns [col0, col1)
    int row0;               // first row of this launch of the streaming kernel
    int W, G;
    float eta, lamL, lamG, mu, wd;
    int flags, use_refreshed;
    int group_size;     // l when all groups have l rows (group = row / l), else 0: look the group up
    const int32_t* offsets;
    const int32_t* group_of;
    const int32_t* lead;
    const int32_t* glead;
    const int32_t* refreshed;
    const RowPlan* plan;
};

template <class V>
__device__ __forceinline__ Coef make_coef(const PullDev& a)
{
    Coef c;
    c.eta = a.eta; c.mu = a.mu; c.wd = a.wd; c.cL = a.lamL; c.cG = a.lamG;
    c.nesterov = (a.flags & LSGD_NESTEROV) != 0;
    c.grad_only = (a.flags & LSGD_MOMENTUM_GRAD_ONLY) != 0;
    return c;
}

template <int VEC, int KIND>
__device__ __forceinline__ void apply_row(const PullDev& a, int64_t o, typename Vec<VEC>::type xv, typename Vec<VEC>::type gv,
                                          typename Vec<VEC>::type mv, const typename Vec<VEC>::type zl,
                                          const typename Vec<VEC>::type zg, const Coef& c)
{
    using V = typename Vec<VEC>::type;
    update_vec<KIND, V>(xv, gv, mv, zl, zg, c);
    st_stream(a.x + o, xv);
    if (KIND == 1) st_stream(a.m + o, mv);
    if (a.xb) st_bf16(a.xb + o, xv);
}

template <int VEC, int KIND>
__device__ __forceinline__ void update_row(const PullDev& a, int64_t o, typename Vec<VEC>::type xv,
                                           const typename Vec<VEC>::type zl, const typename Vec<VEC>::type zg, const Coef& c)
{
    using V = typename Vec<VEC>::type;
    V gv = (KIND != 2) ? ld_stream<VEC>(a.g + o) : zero_of(V());
    V mv = (KIND == 1) ? ld_stream<VEC>(a.m + o) : zero_of(V());
    apply_row<VEC, KIND>(a, o, xv, gv, mv, zl, zg, c);
}

} // namespace lsgd
