// 3x3 complex matrix products (row-major, any arithmetic type).
#pragma once

#include "cs_internal.hpp"

namespace cs {

// c = op(a) op(b) (ACC = 0), c += op(a) op(b) (1) or c -= op(a) op(b) (-1), op
// the adjoint where DA / DB is set.  c must not overlap a or b.  Sums start
// from the first product (or from c) rather than from zero, so no register is
// cleared and no sum is added afterwards.
template <bool DA, bool DB, int ACC, typename R>
__device__ __forceinline__ void m3_prod(const cpx<R>* a, const cpx<R>* b, cpx<R>* c) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<R> s;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const cpx<R> u = DA ? a[k * 3 + i] : a[i * 3 + k], v = DB ? b[j * 3 + k] : b[k * 3 + j];
                // (u or conj u) times (v or conj v), ACC < 0 with the sign of u turned
                const R sg = ACC < 0 ? (R)-1 : (R)1;
                const R ur = sg * u.re, ui = DA ? -sg * u.im : sg * u.im, vi = DB ? -v.im : v.im;
                if (k == 0 && ACC == 0) {
                    s.re = ur * v.re;
                    s.im = ur * vi;
                } else {
                    const cpx<R> o = k == 0 ? c[i * 3 + j] : s;
                    s.re = fma(ur, v.re, o.re);
                    s.im = fma(ur, vi, o.im);
                }
                s.re = fma(-ui, vi, s.re);
                s.im = fma(ui, v.re, s.im);
            }
            c[i * 3 + j] = s;
        }
}

// c = a b (c may alias a or b)
template <typename R>
__device__ __forceinline__ void m3_mul(const cpx<R>* a, const cpx<R>* b, cpx<R>* c) {
    cpx<R> t[9];
    m3_prod<false, false, 0>(a, b, t);
#pragma unroll
    for (int i = 0; i < 9; ++i) c[i] = t[i];
}

// c = (or, ACC: +=) h a for a Hermitian h packed as nine reals: the diagonal,
// then re and im of (0,1), (0,2), (1,2); RIGHT: c = (+=) a h.  c must not
// overlap a.
template <bool RIGHT, bool ACC, typename R>
__device__ __forceinline__ void m3_herm(const R* h, const cpx<R>* a, cpx<R>* c) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int d = RIGHT ? j : i;  // the index of h's row (left) or column (right)
            cpx<R> s = a[i * 3 + j];
            if (ACC) s = {fma(h[d], s.re, c[i * 3 + j].re), fma(h[d], s.im, c[i * 3 + j].im)};
            else s = {h[d] * s.re, h[d] * s.im};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (k == d) continue;
                const int lo = k < d ? k : d, hi = k < d ? d : k, e = 3 + 2 * (lo + hi - 1);
                const R hr = h[e], him = h[e + 1];
                // h[d][k] (left) is the stored entry for d < k, its conjugate else;
                // h[k][d] (right) is the stored entry for k < d
                const bool stored = RIGHT ? k < d : d < k;
                const cpx<R> x = RIGHT ? a[i * 3 + k] : a[k * 3 + j];
                s.re = fma(hr, x.re, s.re);
                s.im = fma(hr, x.im, s.im);
                s.re = fma(stored ? -him : him, x.im, s.re);
                s.im = fma(stored ? him : -him, x.re, s.im);
            }
            c[i * 3 + j] = s;
        }
}

template <typename R>
__device__ __forceinline__ void m3_dag(const cpx<R>* a, cpx<R>* c) {
    cpx<R> t[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) t[i * 3 + j] = conj(a[j * 3 + i]);
#pragma unroll
    for (int i = 0; i < 9; ++i) c[i] = t[i];
}

}  // namespace cs
