// Field setup, run once per gauge field: link compression into the internal
// layout, the clover term C = 1 + T of the paper's Eq. (1) (Section 2; the
// paper leaves building C from the gauge field to the user), and conversion
// of spinors between the canonical and the internal layouts.
#include "fields.hpp"
#include "su3.hpp"

namespace cs {

namespace {

constexpr int TPB = BLOCK_SITES;

__global__ __launch_bounds__(TPB) void k_import_links(Geom g, const double2* __restrict__ U,
                                                      void* l64, void* l32, void* l16, void* lbf) {
    const int blk = blockIdx.x, l = threadIdx.x;
    const long long s = canonical_site(g, blk, l);
    for (int mu = 0; mu < 4; ++mu) {
        cpx<double> u[6];
        const double2* src = U + (s * 4 + mu) * 9;  // rows 0 and 1 are entries 0..5
#pragma unroll
        for (int k = 0; k < 6; ++k) u[k] = {src[k].x, src[k].y};
        LinkIO<P_F64>::store6(l64, blk, l, mu, u);
        LinkIO<P_F32>::store6(l32, blk, l, mu, u);
        LinkIO<P_F16>::store6(l16, blk, l, mu, u);
        LinkIO<P_BF16>::store6(lbf, blk, l, mu, u);
    }
}

using C64 = cpx<double>;

// Offsets, in double2 elements of the FP64 link array, from a site's links to
// those of its neighbours: one value per direction and sign, added up for a
// neighbour reached in two directions (block and in-block coordinates change
// independently in every direction).
struct LinkOffsets {
    long long up[4], dn[4];
};

constexpr int LINK_BLOCK = 4 * 6 * BLOCK_SITES;  // double2 elements of one block's links

__device__ __forceinline__ LinkOffsets link_offsets(const Geom& g, const BlockPos& p, int l) {
    LinkOffsets o;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        int nl;
        bool in;
        int nb = neighbour(g, p, l, d, +1, &nl, &in);
        o.up[d] = (long long)(nb - p.blk) * LINK_BLOCK + (nl - l);
        nb = neighbour(g, p, l, d, -1, &nl, &in);
        o.dn[d] = (long long)(nb - p.blk) * LINK_BLOCK + (nl - l);
    }
    return o;
}

// The link of direction d at the site whose link words start at p
__device__ __forceinline__ void link_at(const double2* p, int d, C64* u) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double2 v = p[(d * 6 + k) * BLOCK_SITES];
        u[k] = {v.x, v.y};
    }
    su3_row2<false>(u);
}

// A = Q - Q^dag of the plane (MU, NU) with Q_{mu nu}(x) the four
// counter-clockwise plaquettes starting at x:
//   U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//   U_nu(x) U_mu(x-mu+nu)^dag U_nu(x-mu)^dag U_mu(x-mu)
//   U_mu(x-mu)^dag U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_nu(x-nu)
//   U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu) U_mu(x)^dag
// Only the anti-Hermitian part of Q counts, so the last two may be replaced
// by minus their adjoints; the first and last then share the factor U_mu(x)
// on the left and the other two U_mu(x-mu) on the right: ten products, and
// the plane's twelve distinct links are loaded once each.  A is anti-Hermitian
// and is returned as the Hermitian i A: three diagonal reals h[0..2], then the
// entries (0,1), (0,2), (1,2).
template <int MU, int NU>
__device__ __forceinline__ void plane_field(const double2* x, const LinkOffsets& o, double* h) {
    // links shared with other planes are loaded again (from cache) rather than
    // kept in registers, and no plane's loads are issued ahead of its turn:
    // with all six planes' links in flight the registers spill
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    C64 s[9], t[9], a[9], b[9], Q[9];
    // U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag - U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
    link_at(x + o.up[MU], NU, a);
    link_at(x + o.up[NU], MU, b);
    m3_prod<false, true, 0>(a, b, t);
    link_at(x, NU, a);
    m3_prod<false, true, 0>(t, a, s);
    link_at(x + o.dn[NU], MU, a);
    link_at(x + o.dn[NU], NU, b);
    m3_prod<true, false, 0>(a, b, t);
    link_at(x + o.up[MU] + o.dn[NU], NU, a);
    m3_prod<true, false, -1>(a, t, s);
    link_at(x, MU, a);
    m3_prod<false, false, 0>(a, s, Q);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // U_nu(x) U_mu(x-mu+nu)^dag U_nu(x-mu)^dag - U_nu(x-nu)^dag U_mu(x-mu-nu)^dag U_nu(x-mu-nu)
    link_at(x, NU, a);
    link_at(x + o.dn[MU] + o.up[NU], MU, b);
    m3_prod<false, true, 0>(a, b, t);
    link_at(x + o.dn[MU], NU, a);
    m3_prod<false, true, 0>(t, a, s);
    link_at(x + o.dn[MU] + o.dn[NU], MU, a);
    link_at(x + o.dn[MU] + o.dn[NU], NU, b);
    m3_prod<true, false, 0>(a, b, t);
    link_at(x + o.dn[NU], NU, a);
    m3_prod<true, false, -1>(a, t, s);
    link_at(x + o.dn[MU], MU, a);
    m3_prod<false, false, 1>(s, a, Q);
    // i (Q - Q^dag)
    h[0] = -2.0 * Q[0].im;
    h[1] = -2.0 * Q[4].im;
    h[2] = -2.0 * Q[8].im;
    const int e[3][2] = {{1, 3}, {2, 6}, {5, 7}};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const C64 q = Q[e[k][0]], c = Q[e[k][1]];
        h[3 + 2 * k] = -(q.im + c.im);
        h[4 + 2 * k] = q.re - c.re;
    }
    // computed here, not where the packed matrix is stored
#pragma unroll
    for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(h[k]));
}

// Upper-triangle slot of entry (i, j), i < j, of a 6x6 matrix, row-major.
__device__ __forceinline__ int up_slot(int i, int j) { return i * 6 - i * (i + 1) / 2 + (j - i - 1); }

// Entry (a, b) of a Hermitian 3x3 matrix packed as plane_field packs it
__device__ __forceinline__ C64 herm_entry(const double* h, int a, int b) {
    if (a == b) return {h[a], 0.0};
    const int lo = a < b ? a : b, hi = a < b ? b : a, k = lo + hi - 1;  // (0,1), (0,2), (1,2)
    return {h[3 + 2 * k], a < b ? h[4 + 2 * k] : -h[4 + 2 * k]};
}

// In the chiral basis T = diag(T+, T-), and with G1, G2, G3 the colour
// matrices multiplying sigma_1, sigma_2, sigma_3 (on the local spin pair),
//   T(h) = i kappa c_sw [[G3, G1 - i G2], [G1 + i G2, -G3]]
// where, from sigma_{kl} = -eps_{klm} diag(s_m, s_m) and
// sigma_{kt} = diag(s_k, -s_k):
//   G1 = -F_yz + sgn F_xt,  G2 = F_xz + sgn F_yt,  G3 = -F_xy + sgn F_zt,
// sgn = +1 for h = 0 and -1 for h = 1.
// One lane per site; planes and directions are compile-time and every entry
// of the packed matrix is stored as soon as its planes are done: with the six
// planes in a loop over tables and the matrix held to the end, 1.5 KB per lane
// lived in scratch memory, and 32^3 x 64 took 8.7 ms where it now takes 1.3
// (FP64 issue: 9,000 instructions a wave of 64 sites, 60 products of 108 FMA and
// the third rows of 72 links, are 0.5 to 0.6 ms at the 4.2 to 5 cycles that one
// takes; the rest waits for those links, 6.9 KB a site from cache, with two
// waves per SIMD).  The FP32 copy is left to k_clover_invert, which reads the
// result anyway.
__global__ __launch_bounds__(TPB, 2) void k_clover_build(Geom g, const double2* links, double kappa, double csw,
                                                         double2* c64) {
    const int blk = block_of_item(g, xcd_remap(blockIdx.x, g.nblk)), l = threadIdx.x;
    const BlockPos p = block_pos(g, blk);
    const LinkOffsets o = link_offsets(g, p, l);
    const double2* x = links + (size_t)blk * LINK_BLOCK + l;
    double2* out = c64 + (size_t)blk * 36 * BLOCK_SITES + l;
    const double w = kappa * csw * 0.125;
    auto put = [&](int h, int i, int j, double re, double im) {
        out[(18 * h + 3 + up_slot(i, j)) * BLOCK_SITES] = make_double2(re, im);
    };
    double a[9], b[9];
    // w i G3 on the diagonal blocks
    plane_field<0, 1>(x, o, a);
    plane_field<2, 3>(x, o, b);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        double m[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) m[i] = w * (h == 0 ? b[i] - a[i] : -a[i] - b[i]);
        double2* q = out + 18 * h * BLOCK_SITES;
        q[0] = make_double2(1.0 + m[0], 1.0 + m[1]);
        q[BLOCK_SITES] = make_double2(1.0 + m[2], 1.0 - m[0]);
        q[2 * BLOCK_SITES] = make_double2(1.0 - m[1], 1.0 - m[2]);
        put(h, 0, 1, m[3], m[4]);
        put(h, 0, 2, m[5], m[6]);
        put(h, 1, 2, m[7], m[8]);
        put(h, 3, 4, -m[3], -m[4]);
        put(h, 3, 5, -m[5], -m[6]);
        put(h, 4, 5, -m[7], -m[8]);
    }
    // w i (G1 - i G2) on the upper right block
    double c[9], d[9];
    plane_field<1, 2>(x, o, a);
    plane_field<0, 3>(x, o, b);
    plane_field<0, 2>(x, o, c);
    plane_field<1, 3>(x, o, d);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const C64 u = herm_entry(a, i, j), v = herm_entry(b, i, j);
            const C64 s = herm_entry(c, i, j), t = herm_entry(d, i, j);
            put(0, i, 3 + j, w * (v.re - u.re + (s.im + t.im)), w * (v.im - u.im - (s.re + t.re)));
            put(1, i, 3 + j, w * (-u.re - v.re + (s.im - t.im)), w * (-u.im - v.im - (s.re - t.re)));
        }
}

// Canonical [V][12][12] matrix of a packed field: T = (1 + T) - 1 for the
// clover term (minus_one), or the packed matrix itself (its inverse).
__global__ __launch_bounds__(TPB) void k_clover_export(Geom g, const double2* __restrict__ c64,
                                                       double2* __restrict__ out, double minus_one) {
    const int blk = blockIdx.x, l = threadIdx.x;
    const long long s = canonical_site(g, blk, l);
    double m[72];
    CloverIO<double>::load(c64, blk, l, m);
    double2* T = out + s * 144;
    for (int i = 0; i < 144; ++i) T[i] = make_double2(0.0, 0.0);
    for (int h = 0; h < 2; ++h) {
        const double* d = m + 36 * h;
        const double* up = d + 6;
        const int o = 6 * h;
        for (int i = 0; i < 6; ++i) T[(o + i) * 12 + o + i] = make_double2(d[i] - minus_one, 0.0);
        for (int i = 0; i < 6; ++i)
            for (int j = i + 1; j < 6; ++j) {
                const int k = up_slot(i, j);
                T[(o + i) * 12 + o + j] = make_double2(up[2 * k], up[2 * k + 1]);
                T[(o + j) * 12 + o + i] = make_double2(up[2 * k], -up[2 * k + 1]);
            }
    }
}

// (1 + T)^-1 per site and chirality (grid.y): each 6x6 block of 1 + T is
// Hermitian positive definite (the clover term is small against the unit
// matrix: its norm is below 6 kappa c_SW times the norm of F), so in-place
// Gauss-Jordan elimination without pivoting inverts it; the result is
// symmetrised and packed like the clover term, in FP64 and FP32; the FP32
// copy of 1 + T itself is written on the way.
__device__ __forceinline__ void store_packed32(float4* q, const double* m) {
#pragma unroll
    for (int k = 0; k < 9; ++k)
        q[k * BLOCK_SITES] = make_float4((float)m[4 * k], (float)m[4 * k + 1], (float)m[4 * k + 2],
                                         (float)m[4 * k + 3]);
}

__global__ __launch_bounds__(TPB) void k_clover_invert(Geom g, const double2* __restrict__ c64,
                                                       float4* __restrict__ c32, double2* __restrict__ ci64,
                                                       float4* __restrict__ ci32) {
    const int blk = blockIdx.x, h = blockIdx.y, l = threadIdx.x;
    const double2* p = c64 + ((size_t)blk * 36 + 18 * h) * BLOCK_SITES + l;
    double m[36];
    for (int k = 0; k < 18; ++k) {
        const double2 v = p[k * BLOCK_SITES];
        m[2 * k] = v.x;
        m[2 * k + 1] = v.y;
    }
    const size_t q32 = ((size_t)blk * 18 + 9 * h) * BLOCK_SITES + l;
    store_packed32(c32 + q32, m);
    cpx<double> a[6][6];
    for (int i = 0; i < 6; ++i) {
        a[i][i] = {m[i], 0.0};
        for (int j = i + 1; j < 6; ++j) {
            const int k = up_slot(i, j);
            a[i][j] = {m[6 + 2 * k], m[7 + 2 * k]};
            a[j][i] = {m[6 + 2 * k], -m[7 + 2 * k]};
        }
    }
    for (int k = 0; k < 6; ++k) {
        const cpx<double> piv = a[k][k];
        const double n2 = piv.re * piv.re + piv.im * piv.im;
        const cpx<double> ip = {piv.re / n2, -piv.im / n2};
        a[k][k] = {1.0, 0.0};
        for (int j = 0; j < 6; ++j) a[k][j] = a[k][j] * ip;
        for (int i = 0; i < 6; ++i) {
            if (i == k) continue;
            const cpx<double> f = a[i][k];
            a[i][k] = {0.0, 0.0};
            for (int j = 0; j < 6; ++j) a[i][j] = a[i][j] - f * a[k][j];
        }
    }
    for (int i = 0; i < 6; ++i) {
        m[i] = a[i][i].re;
        for (int j = i + 1; j < 6; ++j) {
            const int k = up_slot(i, j);
            m[6 + 2 * k] = 0.5 * (a[i][j].re + a[j][i].re);
            m[7 + 2 * k] = 0.5 * (a[i][j].im - a[j][i].im);
        }
    }
    double2* q64 = ci64 + ((size_t)blk * 36 + 18 * h) * BLOCK_SITES + l;
    for (int k = 0; k < 18; ++k) q64[k * BLOCK_SITES] = make_double2(m[2 * k], m[2 * k + 1]);
    store_packed32(ci32 + q32, m);
}

template <int P>
__global__ __launch_bounds__(TPB) void k_field_import(Geom g, void* dst, const double2* src,
                                                      size_t dst_stride, long long V) {
    const int blk = blockIdx.x, l = threadIdx.x, r = blockIdx.y;
    using R = typename SpinorIO<P>::R;
    const long long s = canonical_site(g, blk, l);
    const double2* p = src + ((long long)r * V + s) * 12;
    cpx<R> c[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) c[k] = {(R)p[k].x, (R)p[k].y};
    SpinorIO<P>::store((char*)dst + r * dst_stride, g.nblk, blk, l, c);
}

template <int P>
__global__ __launch_bounds__(TPB) void k_field_export(Geom g, double2* dst, const void* src,
                                                      size_t src_stride, long long V) {
    const int blk = blockIdx.x, l = threadIdx.x, r = blockIdx.y;
    using R = typename SpinorIO<P>::R;
    const long long s = canonical_site(g, blk, l);
    cpx<R> c[12];
    SpinorIO<P>::load((const char*)src + r * src_stride, g.nblk, blk, l, c);
    double2* p = dst + ((long long)r * V + s) * 12;
#pragma unroll
    for (int k = 0; k < 12; ++k) p[k] = make_double2((double)c[k].re, (double)c[k].im);
}

}  // namespace

hipError_t launch_import_links(const Geom& g, const void* U, void* l64, void* l32, void* l16,
                               void* lbf, hipStream_t s) {
    ProfScope ps("setup", s);
    hipLaunchKernelGGL(k_import_links, dim3(g.nblk), dim3(TPB), 0, s, g, (const double2*)U, l64, l32,
                       l16, lbf);
    return hipGetLastError();
}

hipError_t launch_clover_build(const Geom& g, const void* links64, double kappa, double csw, void* c64,
                               hipStream_t s) {
    ProfScope ps("clover_build", s);
    hipLaunchKernelGGL(k_clover_build, dim3(g.nblk), dim3(TPB), 0, s, g, (const double2*)links64, kappa, csw,
                       (double2*)c64);
    return hipGetLastError();
}

hipError_t launch_clover_export(const Geom& g, const void* c64, void* dst, bool inverse, hipStream_t s) {
    hipLaunchKernelGGL(k_clover_export, dim3(g.nblk), dim3(TPB), 0, s, g, (const double2*)c64,
                       (double2*)dst, inverse ? 0.0 : 1.0);
    return hipGetLastError();
}

hipError_t launch_clover_invert(const Geom& g, const void* c64, void* c32, void* ci64, void* ci32,
                                hipStream_t s) {
    ProfScope ps("clover_build", s);
    hipLaunchKernelGGL(k_clover_invert, dim3(g.nblk, 2), dim3(TPB), 0, s, g, (const double2*)c64,
                       (float4*)c32, (double2*)ci64, (float4*)ci32);
    return hipGetLastError();
}

hipError_t launch_field_import(const Geom& g, int prec, void* dst, const void* src, int nrhs,
                               hipStream_t s) {
    const size_t stride = spinor_bytes_per_site(prec) * g.V;
    const dim3 grid(g.nblk, nrhs);
    switch (prec) {
    case P_F64: hipLaunchKernelGGL(k_field_import<P_F64>, grid, dim3(TPB), 0, s, g, dst, (const double2*)src, stride, g.V); break;
    case P_F32: hipLaunchKernelGGL(k_field_import<P_F32>, grid, dim3(TPB), 0, s, g, dst, (const double2*)src, stride, g.V); break;
    case P_F16: hipLaunchKernelGGL(k_field_import<P_F16>, grid, dim3(TPB), 0, s, g, dst, (const double2*)src, stride, g.V); break;
    case P_BF16: hipLaunchKernelGGL(k_field_import<P_BF16>, grid, dim3(TPB), 0, s, g, dst, (const double2*)src, stride, g.V); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_field_export(const Geom& g, int prec, void* dst, const void* src, int nrhs,
                               hipStream_t s) {
    const size_t stride = spinor_bytes_per_site(prec) * g.V;
    const dim3 grid(g.nblk, nrhs);
    switch (prec) {
    case P_F64: hipLaunchKernelGGL(k_field_export<P_F64>, grid, dim3(TPB), 0, s, g, (double2*)dst, src, stride, g.V); break;
    case P_F32: hipLaunchKernelGGL(k_field_export<P_F32>, grid, dim3(TPB), 0, s, g, (double2*)dst, src, stride, g.V); break;
    case P_F16: hipLaunchKernelGGL(k_field_export<P_F16>, grid, dim3(TPB), 0, s, g, (double2*)dst, src, stride, g.V); break;
    case P_BF16: hipLaunchKernelGGL(k_field_export<P_BF16>, grid, dim3(TPB), 0, s, g, (double2*)dst, src, stride, g.V); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cs
