// Gradient of a real function of the solution x = D^{-1} b with respect to
// the gauge links (the force), for the operator of the paper's Eq. (1)
// (Section 2).  With y = D^{-dag} eta (eta = dL/dx from the caller), every
// variation dD of the operator changes L by -Re(y^dag dD x).  Links are varied
// in left Lie-algebra coordinates, U -> exp(i w T^a) U with T^a = lambda^a / 2,
// and the kernel returns g_{mu,a}(x) = dL/dw for all eight generators, plus
// optionally the 3x3 tangent-space gradient G = 2 i (sum_a g_a T^a) U.
//
// Hopping part (U_mu(x) appears once forward at row x, once backward at row
// x+mu):  g_a = -kappa Im tr[T^a (U X1 - X2 U^dag)], with
//   X1 = sum over the two projected spins of h (x) k^dag,
//        h = P_-(x(x+mu)), k = P_-(y(x))      (P_-: spin projection of 1 - gamma_mu)
//   X2 = same with h = P_+(x(x)), k = P_+(y(x+mu)).
// Clover part: y^dag (sigma (x) F) x = tr(F Lambda) with the insertion matrix
// Lambda_{rho sigma}(z) = sum_{s s'} sigma_{s s'} x_{s'}(z) y_s(z)^dag, so that
//   dL = (kappa c_sw / 8) sum_z sum_{rho<sigma} Im tr(dQ_{rho sigma}(z) H(z)),
//   H = Lambda + Lambda^dag.
// Each link sits in 24 plaquette leaves (3 planes x 2 plaquettes x 4
// corners).  For a leaf L U R the derivative contributes U R H L, for a leaf
// L U^dag R it contributes -R H L U^dag, which Re tr(T^a .) does not tell
// from its adjoint -U L^dag H R^dag (H and T^a are Hermitian).  So every term
// is U times a path from x + mu to x with H inserted at one corner, and
// g_a = (kappa c_sw / 8) Re tr(T^a U V) for the signed sum V of the paths.
#include <mutex>

#include "dslash_core.hpp"
#include "su3.hpp"

namespace cs {

namespace {

using C64 = cpx<double>;
constexpr int TPB = BLOCK_SITES;

// Insertion matrices, Hermitian: double [nblk][6 planes][9][256], planes
// ordered (x,y), (x,z), (x,t), (y,z), (y,t), (z,t); the nine reals are the
// diagonal, then re and im of the entries (0,1), (0,2), (1,2).
constexpr int HERM_PLANE = 9 * BLOCK_SITES;        // doubles of one plane
constexpr int HERM_BLOCK = 6 * HERM_PLANE;         // doubles of one block

__device__ __forceinline__ int plane_of(int r, int s) {
    // r < s
    return r == 0 ? s - 1 : (r == 1 ? s + 1 : 5);
}

// outer product accumulation o += w * u (x) v^dag, w = (wr + i wi)
__device__ __forceinline__ void outer_acc(C64* o, const C64* u, const C64* v, double wr, double wi) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const C64 p = u[a] * conj(v[b]);
            o[a * 3 + b].re += wr * p.re - wi * p.im;
            o[a * 3 + b].im += wr * p.im + wi * p.re;
        }
}

// In the chiral basis sigma_{rho sigma} = diag(c0 s_m, c1 s_m) (Pauli s_m on
// the two spins of each chirality): (x,y): -s3, -s3; (x,z): s2, s2;
// (x,t): s1, -s1; (y,z): -s1, -s1; (y,t): s2, -s2; (z,t): s3, -s3.
__global__ __launch_bounds__(TPB) void k_force_insertion(Geom g, const void* __restrict__ xs,
                                                         const void* __restrict__ ys,
                                                         double* __restrict__ H) {
    const int blk = blockIdx.x, l = threadIdx.x;
    C64 x[12], y[12];
    SpinorIO<P_F64>::load(xs, g.nblk, blk, l, x);
    SpinorIO<P_F64>::load(ys, g.nblk, blk, l, y);
    const int pm[6] = {3, 2, 1, 1, 2, 3};
    const double c0[6] = {-1, 1, 1, -1, 1, 1};
    const double c1[6] = {-1, 1, -1, -1, -1, -1};
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        C64 L[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) L[i] = {0.0, 0.0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double c = h == 0 ? c0[p] : c1[p];
            const C64* x0 = x + 6 * h;      // spin 2h
            const C64* x1 = x + 6 * h + 3;  // spin 2h+1
            const C64* y0 = y + 6 * h;
            const C64* y1 = y + 6 * h + 3;
            // sum_{s s'} (s_m)_{s s'} x_{s'} y_s^dag
            if (pm[p] == 1) {          // s1: (0,1) = (1,0) = 1
                outer_acc(L, x1, y0, c, 0);
                outer_acc(L, x0, y1, c, 0);
            } else if (pm[p] == 2) {   // s2: (0,1) = -i, (1,0) = i
                outer_acc(L, x1, y0, 0, -c);
                outer_acc(L, x0, y1, 0, c);
            } else {                   // s3: (0,0) = 1, (1,1) = -1
                outer_acc(L, x0, y0, c, 0);
                outer_acc(L, x1, y1, -c, 0);
            }
        }
        double* dst = H + (size_t)blk * HERM_BLOCK + p * HERM_PLANE + l;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            dst[a * TPB] = 2.0 * L[4 * a].re;
#pragma unroll
            for (int b = a + 1; b < 3; ++b) {
                const C64 v = L[a * 3 + b] + conj(L[b * 3 + a]);
                dst[(1 + 2 * (a + b)) * TPB] = v.re;  // a + b - 1 = 0, 1, 2 for (0,1), (0,2), (1,2)
                dst[(2 + 2 * (a + b)) * TPB] = v.im;
            }
        }
    }
}

__device__ __forceinline__ void load_H(const double* h, double* m) {
#pragma unroll
    for (int i = 0; i < 9; ++i) m[i] = h[i * TPB];
}

// A site as (block, local index) relative to another: differences add up over
// directions, since the block and in-block coordinates of different
// directions are independent.
struct Step {
    int blk, l;
    __device__ __forceinline__ Step operator+(Step o) const { return {blk + o.blk, l + o.l}; }
};

__device__ __forceinline__ Step step(const Geom& g, const BlockPos& p, int l, int mu, int dir) {
    // selected by masks: a select between members of p would be turned into an
    // indexed load, and p into memory
    const int e0 = -(mu == 0), e1 = -(mu == 1), e2 = -(mu == 2), e3 = -(mu == 3);
    const int bc = (e0 & p.bc[0]) | (e1 & p.bc[1]) | (e2 & p.bc[2]) | (e3 & p.bc[3]);
    const int nb = (e0 & g.NB[0]) | (e1 & g.NB[1]) | (e2 & g.NB[2]) | (e3 & g.NB[3]);
    const int st = (e0 & p.stride[0]) | (e1 & p.stride[1]) | (e2 & p.stride[2]) | (e3 & p.stride[3]);
    const int sh = 2 * mu, lc = (l >> sh) & 3;
    if (dir > 0) {
        if (lc < 3) return {0, 1 << sh};
        return {bc == nb - 1 ? -(nb - 1) * st : st, -(3 << sh)};
    }
    if (lc > 0) return {0, -(1 << sh)};
    return {bc == 0 ? (nb - 1) * st : -st, 3 << sh};
}

// V += the eight paths of the plane (mu, nu) through H (mu < nu; the caller
// takes the sign of the other order).  Above the link, with A = U_nu(x+mu),
// B = U_mu(x+nu)^dag, C = U_nu(x)^dag and H_i at the corners x, x+mu,
// x+mu+nu, x+nu:
//   H_1 A B C + A H_2 B C + A B H_3 C + A B C H_0
//     = (H_1 A + A H_2)(B C) + (A B)(H_3 C + C H_0),
// and below it, with the opposite sign, A = U_nu(x+mu-nu)^dag, B = U_mu(x-nu)^dag,
// C = U_nu(x-nu) and the corners x, x+mu, x+mu-nu, x-nu: eight products each
// where the four leaves one by one take twenty.
__device__ __forceinline__ void clover_paths(const Geom& g, const BlockPos& p, int l, const void* links,
                                             const double* H, int mu, int nu, C64* V) {
    const Step m = step(g, p, l, mu, +1);
    const double* Hp = H + (mu < nu ? plane_of(mu, nu) : plane_of(nu, mu)) * HERM_PLANE;
    auto link = [&](Step d, int dir, C64* u) {
        load_link<P_F64, double, false>(links, p.blk + d.blk, l + d.l, dir, u);
    };
    auto ins = [&](Step d, double* h) { load_H(Hp + (size_t)(p.blk + d.blk) * HERM_BLOCK + l + d.l, h); };
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {
        // side 0: C = c^dag with c = U_nu(x), A = a; side 1: C = c = U_nu(x-nu), A = a^dag
        const Step s = step(g, p, l, nu, side == 0 ? +1 : -1), z = {0, 0};
        const bool up = side == 0;
        const double sg = up == (mu < nu) ? 1.0 : -1.0;
        C64 A[9], C[9], b[9], t[9], q[9];
        double h[9];
        asm volatile("" ::: "memory");  // the H both sides read are loaded on each (cached), not kept
        link(up ? z : s, nu, C);
        if (up) m3_dag(C, C);
#pragma unroll
        for (int i = 0; i < 9; ++i) C[i] = sg * C[i];  // every path holds C once (C itself or b^dag C)
        link(s, mu, b);
        m3_prod<true, false, 0>(b, C, t);
        link(up ? m : m + s, nu, A);
        if (!up) m3_dag(A, A);
        ins(m, h);
        m3_herm<false, false>(h, A, q);
        ins(m + s, h);
        m3_herm<true, true>(h, A, q);
        m3_prod<false, false, 1>(q, t, V);  // (H_1 A + A H_2)(b^dag C)
        __builtin_amdgcn_sched_barrier(0);
        m3_prod<false, true, 0>(A, b, q);
        ins(s, h);
        m3_herm<false, false>(h, C, t);
        ins(z, h);
        m3_herm<true, true>(h, C, t);
        m3_prod<false, false, 1>(q, t, V);  // (A b^dag)(H_3 C + C H_0)
    }
}

// Re / Im tr(T^a M), T^a = lambda^a / 2
__device__ __forceinline__ void trace_generators(const C64* M, double* re, double* im) {
    const double is3 = 0.57735026918962576451;  // 1/sqrt(3)
    C64 t[8];
    t[0] = M[3] + M[1];
    t[1] = mul_i(M[1] - M[3]);
    t[2] = M[0] - M[4];
    t[3] = M[6] + M[2];
    t[4] = mul_i(M[2] - M[6]);
    t[5] = M[7] + M[5];
    t[6] = mul_i(M[5] - M[7]);
    t[7] = is3 * (M[0] + M[4] - 2.0 * M[8]);
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        re[a] = 0.5 * t[a].re;
        im[a] = 0.5 * t[a].im;
    }
}

// h = the projected half spinor P_-(psi) (S = -1) or P_+(psi) (S = +1) of the
// field f at a site
template <int S>
__device__ __forceinline__ void project_at(const Geom& g, const void* f, int blk, int l, int mu, C64* h) {
    C64 c[12];
    SpinorIO<P_F64>::load(f, g.nblk, blk, l, c);
    switch (mu) {
    case 0: spin_project<0, S>(c, h); break;
    case 1: spin_project<1, S>(c, h); break;
    case 2: spin_project<2, S>(c, h); break;
    default: spin_project<3, S>(c, h); break;
    }
}

// X = the sum over the two projected spins of h (x) k^dag
__device__ __forceinline__ void hop_outer(const C64* h, const C64* k, C64* X) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            C64 t = h[a] * conj(k[b]);
            cmac_conj(t, k[3 + b], h[3 + a]);
            X[a * 3 + b] = t;
        }
}

// One lane per link; the four directions of a block are consecutive
// workgroups of one XCD, which share the block's links and insertion matrices
// in its L2.  About 55 products of 3x3 matrices a link; at 24^3 x 48 it takes
// 1.4 ms (5.2 ms with the leaves taken one by one, 120 products a link), 0.5
// of it FP64 issue and the rest waiting for the 4.5 KB a link reads from
// cache with two waves per SIMD to hide it.
__global__ __launch_bounds__(TPB, 2) void k_force_link(Geom g, const void* links, double kappa,
                                                    double csw, const void* __restrict__ xs,
                                                    const void* __restrict__ ys,
                                                    const double* H, double* glie,
                                                    double2* gradU) {
    const int w = xcd_remap(blockIdx.x, 4 * g.nblk);
    const int blk = block_of_item(g, w >> 2), mu = w & 3, l = threadIdx.x;
    const BlockPos p = block_pos(g, blk);
    const long long site = canonical_site(g, blk, l);

    // hopping part
    double gh[8];
    {
        C64 U[9];
        load_link<P_F64, double, false>(links, blk, l, mu, U);
        const Step fw = step(g, p, l, mu, +1);
        const int nb = blk + fw.blk, nl = l + fw.l;
        C64 h[6], k[6], X[9], M[9];
        project_at<-1>(g, xs, nb, nl, mu, h);
        project_at<-1>(g, ys, blk, l, mu, k);
        hop_outer(h, k, X);
        m3_prod<false, false, 0>(U, X, M);
        asm volatile("" ::: "memory");
        project_at<+1>(g, xs, blk, l, mu, h);
        project_at<+1>(g, ys, nb, nl, mu, k);
        hop_outer(h, k, X);
        m3_prod<false, true, -1>(X, U, M);
        double re[8], im[8];
        trace_generators(M, re, im);
        // both hop terms of the link U_t(x) on the last time slice cross the
        // time boundary: with antiperiodic fields they carry a factor -1
        const double hs = (mu == 3 && g.antiperiodic_t && p.bc[3] == g.NB[3] - 1 && (l >> 6) == 3) ? -1.0 : 1.0;
#pragma unroll
        for (int a = 0; a < 8; ++a) gh[a] = -hs * kappa * im[a];
        // computed here, not after the clover part: only these eight values
        // stay in registers through it
#pragma unroll
        for (int a = 0; a < 8; ++a) asm volatile("" : "+v"(gh[a]));
    }

    // clover part
    double gc[8];
    {
        C64 W[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) W[i] = {0.0, 0.0};
        if (csw != 0.0) {
#pragma unroll 1
            for (int nu = 0; nu < 4; ++nu)
                if (nu != mu) clover_paths(g, p, l, links, H, mu, nu, W);
        }
        // the link is loaded again (from cache): kept through the loop above it
        // would cost it 36 registers
        asm volatile("" ::: "memory");
        C64 U[9];
        load_link<P_F64, double, false>(links, blk, l, mu, U);
        m3_mul(U, W, W);
        double re[8], im[8];
        trace_generators(W, re, im);
        const double pref = kappa * csw / 8.0;
#pragma unroll
        for (int a = 0; a < 8; ++a) gc[a] = pref * re[a];
    }

    double gt[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) gt[a] = gh[a] + gc[a];
    if (glie) {
        double* o = glie + (site * 4 + mu) * 8;
#pragma unroll
        for (int a = 0; a < 8; ++a) o[a] = gt[a];
    }
    if (gradU) {
        // P = sum_a g_a T^a, G = 2 i P U
        const double is3 = 0.57735026918962576451;
        C64 P[9];
        P[0] = {0.5 * (gt[2] + gt[7] * is3), 0.0};
        P[4] = {0.5 * (-gt[2] + gt[7] * is3), 0.0};
        P[8] = {-gt[7] * is3, 0.0};
        P[1] = {0.5 * gt[0], -0.5 * gt[1]};
        P[3] = {0.5 * gt[0], 0.5 * gt[1]};
        P[2] = {0.5 * gt[3], -0.5 * gt[4]};
        P[6] = {0.5 * gt[3], 0.5 * gt[4]};
        P[5] = {0.5 * gt[5], -0.5 * gt[6]};
        P[7] = {0.5 * gt[5], 0.5 * gt[6]};
        C64 U[9], G[9];
        load_link<P_F64, double, false>(links, blk, l, mu, U);
        m3_mul(P, U, G);
        double2* o = gradU + (site * 4 + mu) * 9;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const C64 v = mul_i(G[i]);
            o[i] = make_double2(2.0 * v.re, 2.0 * v.im);
        }
    }
}

// Workspace of the allocation-free entry point: the insertion matrices of
// up to FORCE_SCRATCH_BYTES / FORCE_SITE_BYTES sites, in a fixed device array that every
// GPU the library runs on holds until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is a stand-in, not a
// device address): the address comes from hipGetSymbolAddress, once per
// device, on that device.
__device__ __align__(256) double2 scratch[FORCE_SCRATCH_BYTES / sizeof(double2)];

std::mutex g_scratch_mu;
void* g_scratch_ptr[FORCE_SCRATCH_MAX_DEVICES] = {};

}  // namespace

hipError_t force_scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= FORCE_SCRATCH_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_force(const Geom& g, const void* links64, double kappa, double csw, const void* x,
                        const void* y, void* Hbuf, double* glie, void* gradU, hipStream_t s) {
    ProfScope ps("force", s);
    hipLaunchKernelGGL(k_force_insertion, dim3(g.nblk), dim3(TPB), 0, s, g, x, y, (double*)Hbuf);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_force_link, dim3(4 * g.nblk), dim3(TPB), 0, s, g, links64, kappa, csw, x, y,
                       (const double*)Hbuf, glie, (double2*)gradU);
    return hipGetLastError();
}

}  // namespace cs
