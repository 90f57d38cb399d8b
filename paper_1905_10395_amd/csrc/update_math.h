// The per-parameter arithmetic of the LSGD update (supplement B.1 / Eq. 3 of arXiv 1905.10395,
// with the optional momentum, Nesterov and weight-decay forms of Section 4.1), shared by the
// streaming update kernels and by the gradient kernels that apply the update in their epilogue.
#pragma once

namespace lsgd {

struct Coef {
    float eta, cL, cG, mu, wd;
    int nesterov, grad_only;
};

// One parameter (V = float) or several (V = a vector), element-wise.  The fused multiply-adds are written out, so that
// every kernel rounds alike wherever this is inlined: the one-launch update works out a leader's new value a second time
// and the paths are compared bit for bit.  Of the two pulls one product is rounded by itself: the global one's, whose
// coefficient is the smaller in use (the other way round the error of the momentum grows by 1 %).
// KIND 0: gradient step, 1: gradient step with momentum, 2: Algorithm 1's communication pull
// (x <- x - cL (x - zl), then x <- x - cG (x - zg); no gradient, momentum untouched).
template <class V>
__device__ __forceinline__ V mul_add(float a, V b, V c) { return __builtin_elementwise_fma((V)(a), b, c); }

template <int KIND, class V>
__device__ __forceinline__ void update_vec(V& x, const V g, V& m, const V zl, const V zg, const Coef& c)
{
#pragma clang fp contract(off)
    constexpr bool MOM = KIND == 1;
    if (KIND == 2) {
        const V y = mul_add(-c.cL, x - zl, x);
        x = mul_add(-c.cG, y - zg, y);
        return;
    }
    V d = mul_add(c.wd, x, g);
    const V pull = mul_add(c.cL, x - zl, c.cG * (x - zg));
    V step;
    if (MOM) {
        if (c.grad_only) {
            m = mul_add(c.mu, m, d);
            step = (c.nesterov ? mul_add(c.mu, m, d) : m) + pull;
        } else {
            d += pull;
            m = mul_add(c.mu, m, d);
            step = c.nesterov ? mul_add(c.mu, m, d) : m;
        }
    } else {
        step = d + pull;
    }
    x = mul_add(-c.eta, step, x);
}

} // namespace lsgd
