// Two-level multigrid pieces of the paper's Section 3 (FP32 storage and
// arithmetic; reductions in FP64 where a result feeds a solver scalar).
//
// Aggregates are the 4^4 SAP blocks (one workgroup, one lane per site).  A
// coarse site carries nc = 2 nv values, index c = chi * nv + i, chi the
// chirality (spins 0, 1 / spins 2, 3).  The prolongator P is stored as nv FP32
// spinor fields: field i holds p_{a,chi,i} on every aggregate a and chirality
// chi.  Coarse vectors are float2[nblk][nc]; the coarse operator
// D_c = P^dag D P is a 9-point stencil float2[nblk][9][nc (column)][nc (row)],
// direction d = 0 the aggregate itself, 1 + 2 mu its +mu neighbour, 2 + 2 mu
// its -mu neighbour (entries that reach the same aggregate through different
// faces stay separate, so the stencil is exact on any lattice).
#include <type_traits>
#include <utility>

#include "blas.hpp"
#include "dslash_core.hpp"
#include "wave.hpp"
#include "mg.hpp"

namespace cs {

namespace {

constexpr int TPB = BLOCK_SITES;

// Sum N values over the workgroup; afterwards out[k] (LDS) holds total k.  The
// folded wave sums carry the restriction of many fields: with one sum per value
// 32^3 x 64, 16 vectors took 2.30 ms, with these 1.61 ms.
template <int N>
__device__ __forceinline__ void block_sum(const float* v, float (*red)[N], float* out) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float t[N];
#pragma unroll
    for (int k = 0; k < N; ++k) t[k] = v[k];
    wave_sums<N>(t);
    if (lane % 16 == 0) {
#pragma unroll
        for (int k = 0; k < N / 4; ++k) red[wave][k + lane / 16 * (N / 4)] = t[k];
    }
    __syncthreads();
    if ((int)threadIdx.x < N) {
        const int k = threadIdx.x;
        out[k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
    }
    __syncthreads();
}

// Block index one step in direction mu (dir = +1 / -1) with periodic wrap.
__device__ __forceinline__ int block_step(const Geom& g, const BlockPos& p, int mu, int dir) {
    // selected by masks: a select between members of p would be turned into an
    // indexed load, and p into memory
    const int e0 = -(mu == 0), e1 = -(mu == 1), e2 = -(mu == 2), e3 = -(mu == 3);
    const int bc = (e0 & p.bc[0]) | (e1 & p.bc[1]) | (e2 & p.bc[2]) | (e3 & p.bc[3]);
    const int nb = (e0 & g.NB[0]) | (e1 & g.NB[1]) | (e2 & g.NB[2]) | (e3 & g.NB[3]);
    const int st = (e0 & p.stride[0]) | (e1 & p.stride[1]) | (e2 & p.stride[2]) | (e3 & p.stride[3]);
    if (dir > 0) return bc == nb - 1 ? p.blk - (nb - 1) * st : p.blk + st;
    return bc == 0 ? p.blk + (nb - 1) * st : p.blk - st;
}

// ---------------------------------------------------------------- setup

// Modified Gram-Schmidt of the nv fields per aggregate and chirality, in place.
// One workgroup per (aggregate, chirality), lane = site, ORTHO_V vectors in
// registers at a time: as soon as vector i is done, its dot products with all
// later vectors of the group are summed together (one barrier per vector) and
// it is projected out of them, so every v_j loses its components along q_0,
// q_1, ... in that order and each field is read and written once, and read once
// more by every later group.  The dots are taken with v_i before its norm is
// known; the norm is inverted in 64 bits.  Groups of 8 leave room for three
// workgroups per CU, which cover one another's chain of sums: 32^3 x 64 with 16
// vectors takes 1.42 ms for 8 GB (16 vectors at a time, two workgroups per CU:
// 1.47 ms for 6.4 GB).  Reading every earlier vector again for each one, with a
// reduction per pair, took 4.4 ms.
constexpr int ORTHO_V = 8;

__device__ __forceinline__ void ortho_dot(const cpx<float>* q, const cpx<float>* v, float& re, float& im) {
    re = im = 0.f;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        re += q[k].re * v[k].re + q[k].im * v[k].im;
        im += q[k].re * v[k].im - q[k].im * v[k].re;
    }
}

// Sums over the workgroup: the waves' parts of N values into red (one float4
// per value), in order of the value; the total of value k is the sum of red[k].
template <int N>
__device__ __forceinline__ void ortho_put(float* t, float4* red) {
    wave_sums<N>(t);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane % 16 == 0) {
#pragma unroll
        for (int k = 0; k < N / 4; ++k) ((float*)&red[k + lane / 16 * (N / 4)])[wave] = t[k];
    }
}

// The dots of q with v_J, v_{J + 1}, ... into red[2 J], ...
template <int J>
__device__ __forceinline__ void ortho_dots(const cpx<float>* q, const cpx<float> (*v)[6], float4* red) {
    constexpr int W = (ORTHO_V - J + 1) / 2 * 2;  // a multiple of 4 sums
    float t[2 * W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        t[2 * j] = t[2 * j + 1] = 0.f;
        if (J + j < ORTHO_V) ortho_dot(q, v[J + j < ORTHO_V ? J + j : 0], t[2 * j], t[2 * j + 1]);
        __builtin_amdgcn_sched_barrier(0);  // one dot at a time: interleaved, they need more registers
    }
    ortho_put<2 * W>(t, red + 2 * J);
}
__device__ __forceinline__ float ortho_total(const float4* red, int k) {
    const float4 t = red[k];
    return (t.x + t.y) + (t.z + t.w);
}

// One step within a group: vector I is finished and projected out of the later ones.
template <int I>
__device__ __forceinline__ void ortho_step(cpx<float> (*v)[6], float4 (*red)[2 * ORTHO_V + 2], int& buf) {
    float4* r = red[buf];
    float nn32 = 0.f;
#pragma unroll
    for (int k = 0; k < 6; ++k) nn32 += v[I][k].re * v[I][k].re + v[I][k].im * v[I][k].im;
    nn32 = wave_sum(nn32);
    if ((threadIdx.x & 63) == 0) ((float*)&r[2 * I])[threadIdx.x >> 6] = nn32;
    if constexpr (I + 1 < ORTHO_V) ortho_dots<I + 1>(v[I], v, r);
    __syncthreads();
    const float4 n4 = r[2 * I];
    const double nn = ((double)n4.x + n4.y) + ((double)n4.z + n4.w);
    const float s = nn > 0. ? (float)(1. / sqrt(nn)) : 0.f;
#pragma unroll
    for (int k = 0; k < 6; ++k) v[I][k] = s * v[I][k];
#pragma unroll
    for (int j = I + 1; j < ORTHO_V; ++j) {
        const cpx<float> c = {s * ortho_total(r, 2 * j), s * ortho_total(r, 2 * j + 1)};
#pragma unroll
        for (int k = 0; k < 6; ++k) v[j][k] = v[j][k] - c * v[I][k];
        __builtin_amdgcn_sched_barrier(0);
    }
    buf ^= 1;
}
template <int... I>
__device__ __forceinline__ void ortho_steps(cpx<float> (*v)[6], float4 (*red)[2 * ORTHO_V + 2], int n, int& buf,
                                            std::integer_sequence<int, I...>) {
    ((I < n ? ortho_step<I>(v, red, buf) : (void)0), ...);
}

__global__ __launch_bounds__(TPB) void k_mg_orthonormalize(Geom g, char* P, size_t fs, int nv) {
    const int blk = blockIdx.x, chi = blockIdx.y, l = threadIdx.x;
    __shared__ float4 red[2][2 * ORTHO_V + 2];
    int buf = 0;  // two buffers, so that one barrier per sum is enough
    // uniform row address + lane offset, so that no per-lane pointers are held
    auto row = [&](int i, int k) {
        return P + (size_t)i * fs + ((size_t)blk * 6 + 3 * chi + k) * (BLOCK_SITES * sizeof(float4));
    };
    const unsigned lane_off = l * sizeof(float4);
    auto load = [&](int i, cpx<float>* v) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float4 t = *(const float4*)(row(i, k) + lane_off);
            v[2 * k] = {t.x, t.y};
            v[2 * k + 1] = {t.z, t.w};
        }
    };
#pragma unroll 1
    for (int j0 = 0; j0 < nv; j0 += ORTHO_V) {
        const int n = nv - j0 < ORTHO_V ? nv - j0 : ORTHO_V;
        cpx<float> v[ORTHO_V][6];
#pragma unroll
        for (int j = 0; j < ORTHO_V; ++j) {
#pragma unroll
            for (int k = 0; k < 6; ++k) v[j][k] = {0.f, 0.f};  // past the last vector
            if (j < n) load(j0 + j, v[j]);
        }
        // against the finished vectors of earlier groups, read back by the lane that stored them
#pragma unroll 1
        for (int i = 0; i < j0; ++i) {
            cpx<float> q[6];
            load(i, q);
            ortho_dots<0>(q, v, red[buf]);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < ORTHO_V; ++j) {
                const cpx<float> c = {ortho_total(red[buf], 2 * j), ortho_total(red[buf], 2 * j + 1)};
#pragma unroll
                for (int k = 0; k < 6; ++k) v[j][k] = v[j][k] - c * q[k];
                __builtin_amdgcn_sched_barrier(0);
            }
            buf ^= 1;
        }
        ortho_steps(v, red, n, buf, std::make_integer_sequence<int, ORTHO_V>{});
#pragma unroll
        for (int j = 0; j < ORTHO_V; ++j)
            if (j < n) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    *(float4*)(row(j0 + j, k) + lane_off) =
                        make_float4(v[j][2 * k].re, v[j][2 * k].im, v[j][2 * k + 1].re, v[j][2 * k + 1].im);
            }
    }
}

// Assembly of D_c[a][d][col][row] = <p_{a,row}, D p_{n(a,d),col}> restricted
// to the terms of D that couple aggregate a to its neighbour in direction d
// (d = 0 and the -mu faces; the +mu blocks follow from gamma5-hermiticity,
// k_mg_assemble_fwd).
//
// Every block of D_c is a contraction over the sites and components of an
// aggregate (self) or a face, so it runs on the matrix cores in FP32
// (v_mfma_f32_16x16x4_f32).  While D is applied a lane of a wave is (site
// lane % 4 of the step, column lane / 4), so that four lanes read 64 consecutive
// bytes of their column's null vector: it loads the vector at its site and the
// neighbours and applies D to the two chirality halves.  The vector and the two
// results then change lanes to (column lane % 16, site lane / 16) and are exactly
// the operands of the products, the vector itself as row j of P^dag and D p as
// column j, for four sites and one component at a time; nothing is reduced
// across lanes.  (Loading in the products' lane order needs no such change, but
// sixteen neighbouring lanes then read sixteen vectors, 16 bytes each: 404 us at
// 16^3 x 32 with 16 vectors, 362 now.)  Workgroup = (aggregate, 16 columns j of
// either chirality): first the self term, a quarter of the sites per wave, summed
// over the waves in LDS; then the faces, wave mu the -mu face.  RT row tiles of 16
// cover nv (rows and columns past nv repeat field nv - 1 and are not stored).
// Per site and column about 1400 VALU instructions apply D and 96 products of
// 32 cycles contract: 5.9 ms at 32^3 x 64 with 16 vectors; with one column per
// workgroup and dot products reduced through LDS the same work took 17.6 ms.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// y0 += (1 + S gamma_mu) U' psi_0, y1 += (1 + S gamma_mu) U' psi_1 for the
// chirality halves psi_0 (spins 0, 1) and psi_1 (spins 2, 3) of psi
template <int MU, int S>
__device__ __forceinline__ void hop_halves(const cpx<float>* u, const cpx<float>* psi, cpx<float>* y0,
                                           cpx<float>* y1) {
    cpx<float> h[6], v[6];
    su3_mul_half<(S > 0)>(u, psi, v);
    spin_reconstruct_add<MU, S>(v, y0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {  // S A_mu psi_lo
        const cpx<float> s2 = psi[6 + a], s3 = psi[9 + a], n2 = {-s2.re, -s2.im}, n3 = {-s3.re, -s3.im};
        if (MU == 0) {
            h[a] = S > 0 ? mul_mi(s3) : mul_i(s3);
            h[3 + a] = S > 0 ? mul_mi(s2) : mul_i(s2);
        } else if (MU == 1) {
            h[a] = S > 0 ? n3 : s3;
            h[3 + a] = S > 0 ? s2 : n2;
        } else if (MU == 2) {
            h[a] = S > 0 ? mul_mi(s2) : mul_i(s2);
            h[3 + a] = S > 0 ? mul_i(s3) : mul_mi(s3);
        } else {
            h[a] = S > 0 ? s2 : n2;
            h[3 + a] = S > 0 ? s3 : n3;
        }
    }
    su3_mul_half<(S > 0)>(u, h, v);
    spin_reconstruct_add<MU, S>(v, y1);
}

// The two hops of direction MU inside the aggregate into site l
template <int MU>
__device__ __forceinline__ void hops_inside(int blk, int l, const void* links, const char* Pj, int nblk,
                                            cpx<float>* y0, cpx<float>* y1) {
    constexpr int sh = 2 * MU;
    const int lc = (l >> sh) & 3;
    if (lc < 3) {
        cpx<float> psi[12], u[9];
        SpinorIO<P_F32>::load(Pj, nblk, blk, l + (1 << sh), psi);
        load_link<P_F32, float, false>(links, blk, l, MU, u);
        hop_halves<MU, -1>(u, psi, y0, y1);
    }
    if (lc > 0) {
        cpx<float> psi[12], u[9];
        SpinorIO<P_F32>::load(Pj, nblk, blk, l - (1 << sh), psi);
        load_link<P_F32, float, false>(links, blk, l - (1 << sh), MU, u);
        hop_halves<MU, +1>(u, psi, y0, y1);
    }
}

// The hop across the -MU face of block p into site l (lc_mu = 0)
template <int MU>
__device__ __forceinline__ void hop_back_face(const Geom& g, const BlockPos& p, int l, const void* links,
                                              const char* Pj, cpx<float>* y0, cpx<float>* y1) {
    int nl;
    bool in;
    const int nb = neighbour(g, p, l, MU, -1, &nl, &in);
    cpx<float> psi[12], u[9];
    SpinorIO<P_F32>::load(Pj, g.nblk, nb, nl, psi);
    if (MU == 3) time_boundary_phase(g, wraps_time(g, p, MU, -1, in), &psi[0].re, 24);
    load_link<P_F32, float, false>(links, nb, nl, MU, u);  // U_mu(x - mu)
    hop_halves<MU, +1>(u, psi, y0, y1);
}

// Sums of the products of rows and columns: [row chirality][column chirality]
struct AsmTile {
    f32x4 re[2][2], im[2][2];
};

__device__ __forceinline__ void asm_clear(AsmTile& t) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) t.re[i][j] = t.im[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// acc += conj(q_row) y_col over four sites and the twelve components.  The
// products of a step are summed on their own and then added: one chain of
// products through all 16 steps of a wave would round each of its 768 terms
// against the whole sum (2.2e-7 relative to 64 bits, 0.8e-7 before; now 0.6e-7).
__device__ __forceinline__ void asm_products(const cpx<float>* q, const cpx<float>* y0, const cpx<float>* y1,
                                             AsmTile& acc) {
    AsmTile t;
    asm_clear(t);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        const int r = c / 6;
        const float ar = q[c].re, ai = q[c].im;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const cpx<float> y = j ? y1[c] : y0[c];
            t.re[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, y.re, t.re[r][j], 0, 0, 0);
            t.im[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, y.im, t.im[r][j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const cpx<float> y = j ? y1[c] : y0[c];
            t.re[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai, y.im, t.re[r][j], 0, 0, 0);
            t.im[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(-ai, y.re, t.im[r][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            acc.re[i][j] += t.re[i][j];
            acc.im[i][j] += t.im[i][j];
        }
}

// Lane site + 4 column -> lane column + 16 site, for twelve values
__device__ __forceinline__ void asm_turn(cpx<float>* v) {
    const int lane = threadIdx.x & 63, src = 4 * ((lane >> 4) + 4 * (lane & 15));
#pragma unroll
    for (int k = 0; k < 12; ++k)
        v[k] = {__int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(v[k].re))),
                __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(v[k].im)))};
}

template <int RT>
__global__ __launch_bounds__(TPB, RT == 1 ? 2 : 1) void k_mg_assemble(Geom g, const void* links, const void* clover,
                                                                      float kappa, const char* P, size_t fs, int nv,
                                                                      float2* Dc) {
    const int nc = 2 * nv, w = xcd_remap(blockIdx.x, g.nblk * RT), blk = w / RT, ct = w % RT;
    const BlockPos p = block_pos(g, blk);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15, kk = lane >> 4;
    const int col = 16 * ct + j;
    // while D is applied: column lj, site lk of the step
    const int lj = lane >> 2, lk = lane & 3;
    const char* Pj = P + (size_t)(16 * ct + lj < nv ? 16 * ct + lj : nv - 1) * fs;
    const char* Pi[RT];  // the rows this lane loads
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) Pi[rt] = P + (size_t)(16 * rt + lj < nv ? 16 * rt + lj : nv - 1) * fs;
    AsmTile acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) asm_clear(acc[rt]);
    // rows of this lane's sums: 4 kk + r of every row tile
    auto store = [&](int d, int rt, int ri, int ci, int r, float re, float im) {
        const int row = 16 * rt + 4 * kk + r;
        if (col < nv && row < nv)
            Dc[(((size_t)blk * 9 + d) * nc + ci * nv + col) * nc + ri * nv + row] = make_float2(re, im);
    };

    // ---- self term: a step is an xy plane of the aggregate, a wave one of its
    // x rows, so that the waves' neighbours meet in the L1
#pragma unroll 1
    for (int s = 0; s < 16; ++s) {
        const int l = lk + 4 * wave + 16 * s;
        cpx<float> q[12], y0[12], y1[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) y0[k] = y1[k] = {0.f, 0.f};
        hops_inside<0>(blk, l, links, Pj, g.nblk, y0, y1);
        hops_inside<1>(blk, l, links, Pj, g.nblk, y0, y1);
        hops_inside<2>(blk, l, links, Pj, g.nblk, y0, y1);
        hops_inside<3>(blk, l, links, Pj, g.nblk, y0, y1);
        SpinorIO<P_F32>::load(Pj, g.nblk, blk, l, q);
        cpx<float> cq[12];
        {
            float cl[72];
            CloverIO<float>::template load<false>(clover, blk, l, cl);
            clover_apply(cl, q, cq);
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const cpx<float> c0 = k < 6 ? cq[k] : cpx<float>{0.f, 0.f}, c1 = k < 6 ? cpx<float>{0.f, 0.f} : cq[k];
            y0[k] = {fmaf(-kappa, y0[k].re, c0.re), fmaf(-kappa, y0[k].im, c0.im)};
            y1[k] = {fmaf(-kappa, y1[k].re, c1.re), fmaf(-kappa, y1[k].im, c1.im)};
        }
        asm_turn(y0);
        asm_turn(y1);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if (RT > 1) SpinorIO<P_F32>::load(Pi[rt], g.nblk, blk, l, q);
            asm_turn(q);
            asm_products(q, y0, y1, acc[rt]);
        }
    }
    // the four waves' sums in LDS, added in order by the wave of each
    // (row, column) chirality pair
    __shared__ float2 red[4][4][4][64];  // [wave][chirality pair][r][lane]
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        __syncthreads();  // the previous tile's readers are done
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[wave][q][r][lane] = make_float2(acc[rt].re[q >> 1][q & 1][r], acc[rt].im[q >> 1][q & 1][r]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 a = red[0][wave][r][lane], b = red[1][wave][r][lane], c = red[2][wave][r][lane],
                         d = red[3][wave][r][lane];
            store(0, rt, wave >> 1, wave & 1, r, (a.x + b.x) + (c.x + d.x), (a.y + b.y) + (c.y + d.y));
        }
        asm_clear(acc[rt]);
    }

    // ---- faces: wave mu takes the 64 sites of the -mu face, four to a step
    // (an x row, or a y row of the x face)
    const int mu = wave;
#pragma unroll 1
    for (int s = 0; s < 16; ++s) {
        const int lo = s & 3, hi = s >> 2;
        const int l = mu == 0 ? 4 * lk + 16 * lo + 64 * hi : mu == 1 ? lk + 16 * lo + 64 * hi
                      : mu == 2 ? lk + 4 * lo + 64 * hi : lk + 4 * lo + 16 * hi;
        cpx<float> y0[12], y1[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) y0[k] = y1[k] = {0.f, 0.f};
        switch (mu) {
        case 0: hop_back_face<0>(g, p, l, links, Pj, y0, y1); break;
        case 1: hop_back_face<1>(g, p, l, links, Pj, y0, y1); break;
        case 2: hop_back_face<2>(g, p, l, links, Pj, y0, y1); break;
        default: hop_back_face<3>(g, p, l, links, Pj, y0, y1); break;
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            y0[k] = {-kappa * y0[k].re, -kappa * y0[k].im};
            y1[k] = {-kappa * y1[k].re, -kappa * y1[k].im};
        }
        asm_turn(y0);
        asm_turn(y1);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            cpx<float> q[12];
            SpinorIO<P_F32>::load(Pi[rt], g.nblk, blk, l, q);
            asm_turn(q);
            asm_products(q, y0, y1, acc[rt]);
        }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                store(2 + 2 * mu, rt, q >> 1, q & 1, r, acc[rt].re[q >> 1][q & 1][r], acc[rt].im[q >> 1][q & 1][r]);
}

// D_c[a][1 + 2 mu] from gamma5-hermiticity of D (P keeps chirality):
// D_c[a][+mu][col][row] = g5(col) g5(row) conj(D_c[b][-mu][row][col]) with
// b the +mu neighbour of a and g5 = +1 on chirality 0, -1 on chirality 1.
__global__ __launch_bounds__(TPB) void k_mg_assemble_fwd(Geom g, int nv, float2* Dc) {
    const int a = blockIdx.x, mu = blockIdx.y, nc = 2 * nv;
    const BlockPos p = block_pos(g, a);
    const int b = block_step(g, p, mu, +1);
    const float2* src = Dc + ((size_t)b * 9 + 2 + 2 * mu) * nc * nc;
    float2* dst = Dc + ((size_t)a * 9 + 1 + 2 * mu) * nc * nc;
    for (int idx = threadIdx.x; idx < nc * nc; idx += TPB) {
        const int col = idx / nc, row = idx % nc;
        const float sg = ((col < nv) == (row < nv)) ? 1.f : -1.f;
        const float2 v = src[(size_t)row * nc + col];
        dst[idx] = make_float2(sg * v.x, -sg * v.y);
    }
}

// --------------------------------------------------------------- transfer

// rc[a][chi * nv + i] = <p_{a,chi,i}, r> (r an FP32 field)
template <int PP>
__global__ __launch_bounds__(TPB) void k_mg_restrict(Geom g, const char* P, size_t fs, int nv, const void* r,
                                                     float2* rc) {
    const int blk = blockIdx.x, l = threadIdx.x;
    __shared__ float red[4][8];
    __shared__ float tot[8];
    cpx<float> rv[12];
    SpinorIO<P_F32>::load(r, g.nblk, blk, l, rv);
    for (int i0 = 0; i0 < nv; i0 += 2) {
        float dd[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (i0 + u < nv) {
                cpx<float> q[12];
                SpinorIO<PP>::load(P + (size_t)(i0 + u) * fs, g.nblk, blk, l, q);
#pragma unroll
                for (int k = 0; k < 12; ++k) {
                    const int o = 4 * u + (k < 6 ? 0 : 2);
                    dd[o] += q[k].re * rv[k].re + q[k].im * rv[k].im;
                    dd[o + 1] += q[k].re * rv[k].im - q[k].im * rv[k].re;
                }
            }
        }
        block_sum<8>(dd, red, tot);
        if (l < 4) {
            const int u = l >> 1, chi = l & 1, i = i0 + u;
            if (i < nv) rc[(size_t)blk * 2 * nv + chi * nv + i] = make_float2(tot[4 * u + 2 * chi], tot[4 * u + 2 * chi + 1]);
        }
    }
}

// Workgroup -> (aggregate, part of the fields) for the transfers of many fields.
// All parts of an aggregate read the same rows of P: they are consecutive
// workgroups of one XCD (workgroup b runs on XCD b % 8), so that its L2 serves
// all parts but the first.  32^3 x 64, 16 vectors, 4 parts: with the parts in
// grid y every part read P from HBM (prolong 3.03 ms, now 1.49 ms).
struct MgManyPlace {
    int blk, part;
};
__device__ __forceinline__ MgManyPlace mg_many_place(int nblk, int parts, int b) {
    const int whole = nblk / 8 * 8 * parts;
    if (b >= whole) return {(nblk / 8 * 8) + (b - whole) / parts, (b - whole) % parts};
    const int k = b / 8;
    return {k / parts * 8 + b % 8, k % parts};
}

// The restriction of nr FP32 fields r_j (stride rs) into nr coarse vectors
// (stride rcs), R fields per workgroup: each P row read serves all R, and
// every r_j gets the sums of k_mg_restrict (same terms, same order).
template <int PP, int R>
__global__ __launch_bounds__(TPB) void k_mg_restrict_many(Geom g, const char* P, size_t fs, int nv,
                                                          const char* rbase, size_t rs, int nr, float2* rcbase,
                                                          size_t rcs) {
    const auto [blk, part] = mg_many_place(g.nblk, (nr + R - 1) / R, blockIdx.x);
    const int l = threadIdx.x, j0 = part * R;
    __shared__ float red[4][8 * R];
    __shared__ float tot[8 * R];
    cpx<float> rv[R][12];
#pragma unroll
    for (int u = 0; u < R; ++u)
        SpinorIO<P_F32>::load(rbase + (size_t)(j0 + u < nr ? j0 + u : nr - 1) * rs, g.nblk, blk, l, rv[u]);
    for (int i0 = 0; i0 < nv; i0 += 2) {
        float dd[8 * R];
#pragma unroll
        for (int k = 0; k < 8 * R; ++k) dd[k] = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (i0 + u < nv) {
                cpx<float> q[12];
                SpinorIO<PP>::load(P + (size_t)(i0 + u) * fs, g.nblk, blk, l, q);
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int k = 0; k < 12; ++k) {
                        const int o = 8 * j + 4 * u + (k < 6 ? 0 : 2);
                        dd[o] += q[k].re * rv[j][k].re + q[k].im * rv[j][k].im;
                        dd[o + 1] += q[k].re * rv[j][k].im - q[k].im * rv[j][k].re;
                    }
            }
        }
        block_sum<8 * R>(dd, red, tot);
        if (l < 4 * R) {
            const int j = l >> 2, u = (l >> 1) & 1, chi = l & 1, i = i0 + u;
            if (i < nv && j0 + j < nr)
                rcbase[(size_t)(j0 + j) * rcs + (size_t)blk * 2 * nv + chi * nv + i] =
                    make_float2(tot[8 * j + 4 * u + 2 * chi], tot[8 * j + 4 * u + 2 * chi + 1]);
        }
    }
}

// z = P ec (an FP32 field)
template <int PP>
__global__ __launch_bounds__(TPB) void k_mg_prolong(Geom g, const char* P, size_t fs, int nv, const float2* ec,
                                                    void* z) {
    const int blk = blockIdx.x, l = threadIdx.x;
    cpx<float> o[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) o[k] = {0.f, 0.f};
    const float2* e = ec + (size_t)blk * 2 * nv;
    for (int i = 0; i < nv; ++i) {
        cpx<float> q[12];
        SpinorIO<PP>::load(P + (size_t)i * fs, g.nblk, blk, l, q);
        const float2 e0 = e[i], e1 = e[nv + i];
        const cpx<float> c0 = {e0.x, e0.y}, c1 = {e1.x, e1.y};
#pragma unroll
        for (int k = 0; k < 12; ++k) cmac(o[k], k < 6 ? c0 : c1, q[k]);
    }
    SpinorIO<P_F32>::store(z, g.nblk, blk, l, o);
}

// The prolongation of nr coarse vectors (stride ecs) into nr FP32 fields
// (stride zs), R per workgroup: each P row read serves all R, every z_j
// gets the sums of k_mg_prolong (same terms, same order).
template <int PP, int R>
__global__ __launch_bounds__(TPB) void k_mg_prolong_many(Geom g, const char* P, size_t fs, int nv,
                                                         const float2* ecbase, size_t ecs, int nr, char* zbase,
                                                         size_t zs) {
    const auto [blk, part] = mg_many_place(g.nblk, (nr + R - 1) / R, blockIdx.x);
    const int l = threadIdx.x, j0 = part * R;
    cpx<float> o[R][12];
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
        for (int k = 0; k < 12; ++k) o[j][k] = {0.f, 0.f};
    for (int i = 0; i < nv; ++i) {
        cpx<float> q[12];
        SpinorIO<PP>::load(P + (size_t)i * fs, g.nblk, blk, l, q);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float2* e = ecbase + (size_t)(j0 + j < nr ? j0 + j : nr - 1) * ecs + (size_t)blk * 2 * nv;
            const float2 e0 = e[i], e1 = e[nv + i];
            const cpx<float> c0 = {e0.x, e0.y}, c1 = {e1.x, e1.y};
#pragma unroll
            for (int k = 0; k < 12; ++k) cmac(o[j][k], k < 6 ? c0 : c1, q[k]);
        }
    }
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (j0 + j < nr) SpinorIO<P_F32>::store(zbase + (size_t)(j0 + j) * zs, g.nblk, blk, l, o[j]);
}

// ---------------------------------------------------------- coarse solver
//
// Matrix-vector products with D_c read 5 of the 9 stencil blocks of every
// aggregate.  The +mu blocks are fixed by the -mu blocks of the neighbours
// through gamma5-hermiticity, D_c[b - mu][+mu] = G5 D_c[b][-mu]^dag G5 (G5 =
// +1 on chirality 0, -1 on chirality 1), so the product runs in two passes:
//   pass 1, one workgroup of 256 lanes per aggregate a: y_a = D_c[a][0] x_a
//     + sum_mu D_c[a][-mu] x_{a - mu}, and tau[a][mu] = G5 D_c[a][-mu]^dag G5
//     x_a, the +mu contribution of a to the aggregate a - mu;
//   pass 2, elementwise: y_a += sum_mu tau[a + mu][mu], mu in increasing order.
// Each -mu block is read from HBM once (its adjoint re-reads it from cache).
// In pass 1 the five blocks are one K5 x nc matrix M[k][row] (k = slot nc +
// col, slot 0 the aggregate itself, slot 1 + mu its -mu block, row fastest)
// applied to the gathered vector xg[k] = x_{n(a, slot), col} staged in LDS.
// Lane t owns row t % nc and the column chunk t / nc (every (256 / nc)-th
// k), so a wave reads whole consecutive rows of M (coalesced) and each lane
// keeps several independent loads in flight; the chunks are then added in a
// fixed order.  The adjoints give lane t the outputs o = t, t + 256, ... of
// the 4 nc values tau[a][mu][i] (o = mu nc + i), each a sum over the nc
// entries of one stored column.

constexpr int CMV_TPB = 256;
constexpr int CMV_KMAX = 5 * 2 * MG_MAX_NV;

__device__ __forceinline__ int coarse_nb(const Geom& g, const BlockPos& p, int d) {
    return d == 0 ? p.blk : block_step(g, p, (d - 1) >> 1, (d & 1) ? +1 : -1);
}

// stencil direction of gather slot sl: the aggregate itself, then -mu
__device__ __forceinline__ int slot_dir(int sl) { return sl == 0 ? 0 : 2 * sl; }

// Entry i of the coarse matrices, FP32 or FP16 storage
template <bool HALF>
__device__ __forceinline__ float2 cm_load(const void* M, size_t i) {
    if (HALF) {
        float a, b;
        unpack2<P_F16>(((const unsigned int*)M)[i], a, b);
        return make_float2(a, b);
    }
    return ((const float2*)M)[i];
}

// R right-hand sides share one pass over the matrices: xs[j], y[j] and
// tau + j * rs are those of right-hand side j, each with the sums it has alone.

// y[j]_row = sum over the self and -mu blocks of aggregate a of M[k][row]
// xs[j][k]; valid in lanes t < nc
template <bool HALF, int R>
__device__ __forceinline__ void cmv_rows5(const void* __restrict__ Dc, int a, int nc, const float2 (*xs)[CMV_KMAX],
                                          float2* red, float2* y) {
    const int t = threadIdx.x, kch = CMV_TPB / nc, row = t % nc, kc = t / nc, K5 = 5 * nc;
    const size_t base = (size_t)a * 9 * nc * nc + row;
    float re[R], im[R], re2[R], im2[R];
#pragma unroll
    for (int j = 0; j < R; ++j) re[j] = im[j] = re2[j] = im2[j] = 0.f;
    auto mac = [](float2 m, float2 x, float& re_, float& im_) {
        re_ = fmaf(m.x, x.x, re_);
        re_ = fmaf(-m.y, x.y, re_);
        im_ = fmaf(m.x, x.y, im_);
        im_ = fmaf(m.y, x.x, im_);
    };
    if (kc < kch) {
        int k = kc;
        for (; k + kch < K5; k += 2 * kch) {
            const int k1 = k + kch;
            const float2 m0 = cm_load<HALF>(Dc, base + (size_t)(slot_dir(k / nc) * nc + k % nc) * nc);
            const float2 m1 = cm_load<HALF>(Dc, base + (size_t)(slot_dir(k1 / nc) * nc + k1 % nc) * nc);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                mac(m0, xs[j][k], re[j], im[j]);
                mac(m1, xs[j][k1], re2[j], im2[j]);
            }
        }
        if (k < K5) {
            const float2 m0 = cm_load<HALF>(Dc, base + (size_t)(slot_dir(k / nc) * nc + k % nc) * nc);
#pragma unroll
            for (int j = 0; j < R; ++j) mac(m0, xs[j][k], re[j], im[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (j > 0) __syncthreads();  // the previous right-hand side's readers of red are done
        red[t] = make_float2(re[j] + re2[j], im[j] + im2[j]);
        __syncthreads();
        y[j] = make_float2(0.f, 0.f);
        if (t < nc)
            for (int c = 0; c < kch; ++c) {
                const float2 v = red[c * nc + t];
                y[j].x += v.x;
                y[j].y += v.y;
            }
    }
}

// tau[a][mu][i] = sum_c g5(i) g5(c) conj(D_c[a][-mu][col i][row c]) xa[c],
// xa the aggregate's own entries (LDS); written where bit j of live is set
template <bool HALF, int R>
__device__ __forceinline__ void cmv_adjoint4(const void* __restrict__ Dc, int a, int nc, const float2 (*xs)[CMV_KMAX],
                                             float2* __restrict__ tau, size_t rs, int live) {
    const int nv = nc / 2;
    for (int o = threadIdx.x; o < 4 * nc; o += CMV_TPB) {
        const int mu = o / nc, i = o % nc;
        const size_t base = (((size_t)a * 9 + 2 + 2 * mu) * nc + i) * nc;
        float re[R], im[R];
#pragma unroll
        for (int j = 0; j < R; ++j) re[j] = im[j] = 0.f;
        for (int c = 0; c < nc; ++c) {
            const float2 m = cm_load<HALF>(Dc, base + c);
            const float sg = (i < nv) == (c < nv) ? 1.f : -1.f;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const float2 x = xs[j][c];
                // conj(m) x
                re[j] = fmaf(sg * m.x, x.x, re[j]); re[j] = fmaf(sg * m.y, x.y, re[j]);
                im[j] = fmaf(sg * m.x, x.y, im[j]); im[j] = fmaf(-sg * m.y, x.x, im[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (live >> j & 1) tau[j * rs + ((size_t)a * 4 + mu) * nc + i] = make_float2(re[j], im[j]);
    }
}

// Sum over aligned groups of G = 16, 32 or 64 lanes (a row of the wave, a
// half or the whole wave); every lane of the group receives the total.
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    using namespace wave_detail;
    v += dpp_move<DPP_XOR1>(v);
    v += dpp_move<DPP_XOR2>(v);
    v += dpp_move<DPP_HALF_MIRROR>(v);
    v += dpp_move<DPP_MIRROR>(v);
    if constexpr (G >= 32) v = cross_add<16>(v);
    if constexpr (G >= 64) v = cross_add<32>(v);
    return v;
}

// Pass 1 of the product for nc = NC in {16, 32, 64}: the adjoint terms come
// from the same loads as the forward ones.  The NC lanes of the group kc
// all hold entry k of one stored column (rows 0..NC-1), so each lane forms
// g5(col) g5(row) conj(M[k][row]) xa[row] and a group sum gives
// tau[a][mu][col] for the -mu slots (it is formed, and dropped, for the
// self slot too, so that every lane takes part in every exchange).  The
// loads of a lane are issued in batches before their arithmetic, the first
// batch (for one right-hand side and nc = 16 or 32 all of them) before the
// entries of x are gathered, so that the two waits overlap; the sums are stored after the
// loop, so no store sits between loads.
// The forward chunks are reduced as in cmv_rows5.
template <bool HALF, int NC, int R>
struct FusedBatch {
    static constexpr int KCH = CMV_TPB / NC, NJ = 5 * NC / KCH;  // NJ is 5, 20 or 80
    static constexpr int MOST = R == 1 ? 20 : 10, CH = NJ < MOST ? NJ : MOST;  // entries of a batch
    static_assert(NJ % CH == 0 && NJ <= 2 * NC, "batches cover the loop; a lane keeps at most two sums");
    float2 m[CH];
    __device__ __forceinline__ void load(const void* __restrict__ Dc, int a, int j0) {
        const int row = threadIdx.x % NC, kc = threadIdx.x / NC;
        const size_t base = (size_t)a * 9 * NC * NC + row;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int k = kc + (j0 + c) * KCH;
            m[c] = cm_load<HALF>(Dc, base + (size_t)(slot_dir(k / NC) * NC + k % NC) * NC);
        }
    }
};

template <bool HALF, int NC, int R>
__device__ __forceinline__ void cmv5_fused(const void* __restrict__ Dc, int a, FusedBatch<HALF, NC, R>& fb,
                                           const float2 (*xs)[CMV_KMAX], float2* red, float2* __restrict__ tau,
                                           size_t rs, int live, float2* y) {
    using FB = FusedBatch<HALF, NC, R>;
    constexpr int KCH = FB::KCH, NJ = FB::NJ, CH = FB::CH, NV = NC / 2;
    const int t = threadIdx.x, row = t % NC, kc = t / NC;
    float2 xa[R];
    float re[R], im[R];
    // the adjoint sums this lane stores: j = row and j = row + NC
    float2 keep0[R], keep1[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        xa[q] = xs[q][row];
        re[q] = im[q] = 0.f;
        keep0[q] = keep1[q] = make_float2(0.f, 0.f);
    }
#pragma unroll 1
    for (int j0 = 0; j0 < NJ; j0 += CH) {
        if (j0 > 0) fb.load(Dc, a, j0);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int j = j0 + c, k = kc + j * KCH, col = k % NC;
            const float2 m = fb.m[c];
            const float sg = (col < NV) == (row < NV) ? 1.f : -1.f;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const float2 x = xs[q][k];
                re[q] = fmaf(m.x, x.x, re[q]);
                re[q] = fmaf(-m.y, x.y, re[q]);
                im[q] = fmaf(m.x, x.y, im[q]);
                im[q] = fmaf(m.y, x.x, im[q]);
                float ar = sg * fmaf(m.x, xa[q].x, m.y * xa[q].y), ai = sg * fmaf(m.x, xa[q].y, -m.y * xa[q].x);
                ar = group_sum<NC>(ar);
                ai = group_sum<NC>(ai);
                if (j == row) keep0[q] = make_float2(ar, ai);
                if (j == row + NC) keep1[q] = make_float2(ar, ai);
            }
            // the selections are made here: left to the end of the batch they
            // would keep all of its sums in registers
#pragma unroll
            for (int q = 0; q < R; ++q)
                asm volatile("" : "+v"(keep0[q].x), "+v"(keep0[q].y), "+v"(keep1[q].x), "+v"(keep1[q].y));
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int j = i * NC + row;
        if (j < NJ) {
            const int k = kc + j * KCH, sl = k / NC;
            if (sl > 0) {
#pragma unroll
                for (int q = 0; q < R; ++q)
                    if (live >> q & 1) tau[q * rs + ((size_t)a * 4 + sl - 1) * NC + k % NC] = i ? keep1[q] : keep0[q];
            }
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (q > 0) __syncthreads();  // the previous right-hand side's readers of red are done
        red[t] = make_float2(re[q], im[q]);
        __syncthreads();
        y[q] = make_float2(0.f, 0.f);
        if (t < NC)
            for (int c = 0; c < KCH; ++c) {
                const float2 v = red[c * NC + t];
                y[q].x += v.x;
                y[q].y += v.y;
            }
    }
}

// Pass 1 for any nc: NC = 0 takes the two-step form.  gather() fills xs and
// returns after every lane can read it.
template <bool HALF, int NC, int R, typename G>
__device__ __forceinline__ void cmv5(const void* __restrict__ Dc, int a, int nc, const float2 (*xs)[CMV_KMAX],
                                     float2* red, float2* __restrict__ tau, size_t rs, int live, float2* y,
                                     G&& gather) {
    if constexpr (NC > 0) {
        FusedBatch<HALF, NC, R> fb;
        fb.load(Dc, a, 0);
        gather();
        cmv5_fused<HALF, NC, R>(Dc, a, fb, xs, red, tau, rs, live, y);
    } else {
        gather();
        cmv_rows5<HALF, R>(Dc, a, nc, xs, red, y);
        cmv_adjoint4<HALF, R>(Dc, a, nc, xs, tau, rs, live);
    }
}

// Gather of slot sl's entries of x for aggregate p (n(a, slot))
__device__ __forceinline__ size_t gather_index(const Geom& g, const BlockPos& p, int nc, int k) {
    return (size_t)coarse_nb(g, p, slot_dir(k / nc)) * nc + k % nc;
}

// Pass 2 for entry i = a nc + row: the +mu contributions of the four +mu
// neighbours, in increasing mu
__device__ __forceinline__ float2 tau_sum(const Geom& g, int nc, const float2* __restrict__ tau, size_t i) {
    const int a = (int)(i / nc), row = (int)(i % nc);
    const BlockPos p = block_pos(g, a);
    float2 s = make_float2(0.f, 0.f);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        const int b = block_step(g, p, mu, +1);
        const float2 v = tau[((size_t)b * 4 + mu) * nc + row];
        s.x += v.x;
        s.y += v.y;
    }
    return s;
}

__device__ __forceinline__ double2 cdot_d(float2 a, float2 b) {  // conj(a) b
    return make_double2((double)a.x * b.x + (double)a.y * b.y, (double)a.x * b.y - (double)a.y * b.x);
}

// y = D_c x, pass 1 (y holds the self and -mu terms afterwards, tau the
// adjoint terms)
template <bool HALF, int NC>
__global__ __launch_bounds__(CMV_TPB) void k_mg_coarse_apply(Geom g, const void* __restrict__ Dc, int nc,
                                                             const float2* __restrict__ x, float2* __restrict__ y,
                                                             float2* __restrict__ tau) {
    __shared__ float2 xs[1][CMV_KMAX];
    __shared__ float2 red[CMV_TPB];
    const int a = blockIdx.x, K5 = 5 * nc;
    const BlockPos p = block_pos(g, a);
    float2 v[1];
    cmv5<HALF, NC, 1>(Dc, a, nc, xs, red, tau, 0, 1, v, [&]() {
        for (int k = threadIdx.x; k < K5; k += CMV_TPB) xs[0][k] = x[gather_index(g, p, nc, k)];
        __syncthreads();
    });
    if ((int)threadIdx.x < nc) y[(size_t)a * nc + threadIdx.x] = v[0];
}

// y = D_c x, pass 2
__global__ __launch_bounds__(256) void k_mg_coarse_complete(Geom g, int nc, float2* __restrict__ y,
                                                            const float2* __restrict__ tau) {
    const size_t n = (size_t)g.nblk * nc;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float2 t = tau_sum(g, nc, tau, i);
        const float2 v = y[i];
        y[i] = make_float2(v.x + t.x, v.y + t.y);
    }
}

__device__ __forceinline__ double2 cdiv2(double2 a, double2 b) {
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}
__device__ __forceinline__ double2 cmul_d(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Coarse BiCGStab, for one right-hand side or for several at once (each with
// its own vectors cv.rs apart, scalars, partial sums and stops; the second
// grid dimension, or the first of the one-workgroup kernels, runs over them).
// The start (x = 0, r = rh = r_c) is followed by the stop
// test F1 of iteration 0; iteration it (parity q = it & 1) is then eight
// launches, the last of which is the stop test of iteration it + 1:
//   M1  p = r + beta (p_prev - omega v_prev) formed while gathering, pass 1
//       of v = D_c p
//   C1  pass 2 of v = D_c p, partials B = <rh, v>
//   F2  alpha = rho_new / <rh, v> (a zero denominator ends the solve)
//   M2  s = r - alpha v formed while gathering, pass 1 of t = D_c s
//   C2  pass 2 of t = D_c s, partials C = <t, s>, |t|^2
//   F3  omega = <t, s> / |t|^2 (0 when t = 0)
//   U   x += alpha p + omega s, r = s - omega t, partials A
//   F1  rho_new = <rh, r>, |r|^2 from the partials A; stop before the next
//       iteration when rho_new = 0, omega = 0, |r| <= tol |r_0| or an earlier
//       stop; beta = (rho_new / rho_old) (alpha / omega)
// p and v alternate between two buffers by parity, so the gathers of M1 read
// the previous iteration's values while its own entries are written.  A
// kernel reads only scalars written by earlier kernels (slots by parity
// where a kernel would otherwise read what it writes), and every later
// kernel returns at once after a stop, so a fixed number of iterations can be
// launched or captured; stopped[it & 1] tells whether iteration it runs.

// Fixed-order sum of the first three reals (re, im of slot 0; re of slot 1)
// of nwg two-slot partials by one workgroup of 1024 lanes; valid in lane 0.
__device__ __forceinline__ void sum3_partials(const double2* partials, int nwg, double* out) {
    __shared__ double red[3][1024];
    const int t = threadIdx.x;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int i = t; i < nwg; i += 1024) {
        const double2 a = partials[(size_t)i * 2], b = partials[(size_t)i * 2 + 1];
        s0 += a.x;
        s1 += a.y;
        s2 += b.x;
    }
    red[0][t] = s0;
    red[1][t] = s1;
    red[2][t] = s2;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (t < w) {
            red[0][t] += red[0][t + w];
            red[1][t] += red[1][t + w];
            red[2][t] += red[2][t + w];
        }
        __syncthreads();
    }
    out[0] = red[0][0];
    out[1] = red[1][0];
    out[2] = red[2][0];
}

__global__ __launch_bounds__(1024) void k_cb_f1(const double2* partials, int nwg, CbScalars* sc, int it,
                                                double tol2) {
    const int q = it & 1;
    partials += (size_t)blockIdx.x * CB_PARTIALS;
    sc += blockIdx.x;
    double tot[3];
    sum3_partials(partials, nwg, tot);
    if (threadIdx.x != 0) return;
    const double2 rho = make_double2(tot[0], tot[1]);
    const double rr = tot[2];
    int stop;
    if (it == 0) {
        sc->stop2 = tol2 * rr;
        sc->alpha = sc->omega = make_double2(1.0, 0.0);
        sc->beta[q] = make_double2(0.0, 0.0);
        stop = 0;
    } else {
        const bool w0 = sc->omega.x == 0.0 && sc->omega.y == 0.0;
        stop = sc->stopped[q ^ 1] || sc->brk[q ^ 1] || w0 || rr <= sc->stop2;
        sc->beta[q] = stop ? make_double2(0.0, 0.0) : cmul_d(cdiv2(rho, sc->rho[q ^ 1]), cdiv2(sc->alpha, sc->omega));
    }
    if (rho.x == 0.0 && rho.y == 0.0) stop = 1;
    sc->rho[q] = rho;
    sc->rr = rr;
    sc->stopped[q] = stop;
}

// Workgroup partials (a, b) over 256-entry chunks: partials A of <rh, r>,
// |r|^2, B of <rh, v> and C of <t, s>, |t|^2
__device__ __forceinline__ void chunk_partials(double2 a, double b, double2* partials) {
    __shared__ double red[3][4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    a = make_double2(wave_sum(a.x), wave_sum(a.y));
    b = wave_sum(b);
    if (lane == 0) {
        red[0][wave] = a.x;
        red[1][wave] = a.y;
        red[2][wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        partials += (size_t)blockIdx.y * CB_PARTIALS;
        partials[(size_t)blockIdx.x * 2] = make_double2((red[0][0] + red[0][1]) + (red[0][2] + red[0][3]),
                                                        (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
        partials[(size_t)blockIdx.x * 2 + 1] =
            make_double2((red[2][0] + red[2][1]) + (red[2][2] + red[2][3]), 0.0);
    }
}

template <bool HALF, int NC, int R>
__global__ __launch_bounds__(CMV_TPB) void k_cb_m1(Geom g, const void* __restrict__ Dc, int nc, CbVecs cv,
                                                   const CbScalars* sc, int q, int nr) {
    const int r0 = blockIdx.y * R;
    int live = 0;  // bit j: right-hand side r0 + j is still being solved
    for (int j = 0; j < R; ++j) live |= (r0 + j < nr && !sc[r0 + j].stopped[q]) << j;
    if (!live) return;
    __shared__ float2 xs[R][CMV_KMAX];
    __shared__ float2 red[CMV_TPB];
    const int a = blockIdx.x, K5 = 5 * nc;
    const BlockPos p = block_pos(g, a);
    float2 v[R];
    cmv5<HALF, NC, R>(Dc, a, nc, xs, red, cv.tau + r0 * cv.rs, cv.rs, live, v, [&]() {
        for (int j = 0; j < R; ++j) {
            if (!(live >> j & 1)) continue;  // xs[j] goes into no stored value then
            const CbScalars& S = sc[r0 + j];
            const float br = (float)S.beta[q].x, bi = (float)S.beta[q].y;
            const float wr = (float)S.omega.x, wi = (float)S.omega.y;
            const size_t o = (r0 + j) * cv.rs;
            const float2 *rp = cv.r + o, *pp = cv.pp(q ^ 1) + o, *vp = cv.vv(q ^ 1) + o;
            float2* pn = cv.pp(q) + o;
            for (int k = threadIdx.x; k < K5; k += CMV_TPB) {
                const size_t i = gather_index(g, p, nc, k);
                const float2 r = rp[i], po = pp[i], vo = vp[i];
                const float tr = po.x - (wr * vo.x - wi * vo.y), ti = po.y - (wr * vo.y + wi * vo.x);
                const float2 pv = make_float2(r.x + (br * tr - bi * ti), r.y + (br * ti + bi * tr));
                xs[j][k] = pv;
                if (k < nc) pn[i] = pv;
            }
        }
        __syncthreads();
    });
#pragma unroll
    for (int j = 0; j < R; ++j)
        if ((live >> j & 1) && (int)threadIdx.x < nc) cv.vv(q)[(r0 + j) * cv.rs + (size_t)a * nc + threadIdx.x] = v[j];
}

// v += the +mu terms, partials B of <rh, v>
__global__ __launch_bounds__(256) void k_cb_c1(Geom g, int nc, CbVecs cv, const CbScalars* sc, int q,
                                               double2* partials) {
    sc += blockIdx.y;
    if (sc->stopped[q]) return;
    cv = cv.of(blockIdx.y);
    const size_t n = (size_t)g.nblk * nc;
    float2* vq = cv.vv(q);
    double2 d = make_double2(0.0, 0.0);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float2 t = tau_sum(g, nc, cv.tau, i), v0 = vq[i];
        const float2 v = make_float2(v0.x + t.x, v0.y + t.y);
        vq[i] = v;
        const double2 hv = cdot_d(cv.rh[i], v);
        d.x += hv.x;
        d.y += hv.y;
    }
    chunk_partials(d, 0.0, partials);
}

__global__ __launch_bounds__(1024) void k_cb_f2(const double2* partials, int nwg, CbScalars* sc, int q) {
    partials += (size_t)blockIdx.x * CB_PARTIALS;
    sc += blockIdx.x;
    if (sc->stopped[q]) return;
    double tot[3];
    sum3_partials(partials, nwg, tot);
    if (threadIdx.x != 0) return;
    const double2 rv = make_double2(tot[0], tot[1]);
    const bool brk = rv.x == 0.0 && rv.y == 0.0;
    sc->brk[q] = brk;
    if (!brk) sc->alpha = cdiv2(sc->rho[q], rv);
}

template <bool HALF, int NC, int R>
__global__ __launch_bounds__(CMV_TPB) void k_cb_m2(Geom g, const void* __restrict__ Dc, int nc, CbVecs cv,
                                                   const CbScalars* sc, int q, int nr) {
    const int r0 = blockIdx.y * R;
    int live = 0;
    for (int j = 0; j < R; ++j) live |= (r0 + j < nr && !sc[r0 + j].stopped[q] && !sc[r0 + j].brk[q]) << j;
    if (!live) return;
    __shared__ float2 xs[R][CMV_KMAX];
    __shared__ float2 red[CMV_TPB];
    const int a = blockIdx.x, K5 = 5 * nc;
    const BlockPos p = block_pos(g, a);
    float2 t[R];
    cmv5<HALF, NC, R>(Dc, a, nc, xs, red, cv.tau + r0 * cv.rs, cv.rs, live, t, [&]() {
        for (int j = 0; j < R; ++j) {
            if (!(live >> j & 1)) continue;
            const float ar = (float)sc[r0 + j].alpha.x, ai = (float)sc[r0 + j].alpha.y;
            const size_t o = (r0 + j) * cv.rs;
            const float2 *rp = cv.r + o, *vq = cv.vv(q) + o;
            float2* sp = cv.s + o;
            for (int k = threadIdx.x; k < K5; k += CMV_TPB) {
                const size_t i = gather_index(g, p, nc, k);
                const float2 r = rp[i], v = vq[i];
                const float2 sv = make_float2(r.x - (ar * v.x - ai * v.y), r.y - (ar * v.y + ai * v.x));
                xs[j][k] = sv;
                if (k < nc) sp[i] = sv;
            }
        }
        __syncthreads();
    });
#pragma unroll
    for (int j = 0; j < R; ++j)
        if ((live >> j & 1) && (int)threadIdx.x < nc) cv.t[(r0 + j) * cv.rs + (size_t)a * nc + threadIdx.x] = t[j];
}

// t += the +mu terms, partials C of <t, s>, |t|^2
__global__ __launch_bounds__(256) void k_cb_c2(Geom g, int nc, CbVecs cv, const CbScalars* sc, int q,
                                               double2* partials) {
    sc += blockIdx.y;
    if (sc->stopped[q] || sc->brk[q]) return;
    cv = cv.of(blockIdx.y);
    const size_t n = (size_t)g.nblk * nc;
    double2 ts = make_double2(0.0, 0.0);
    double tt = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float2 u = tau_sum(g, nc, cv.tau, i), t0 = cv.t[i];
        const float2 t = make_float2(t0.x + u.x, t0.y + u.y);
        cv.t[i] = t;
        const double2 d = cdot_d(t, cv.s[i]);
        ts.x += d.x;
        ts.y += d.y;
        tt += (double)t.x * t.x + (double)t.y * t.y;
    }
    chunk_partials(ts, tt, partials);
}

__global__ __launch_bounds__(1024) void k_cb_f3(const double2* partials, int nwg, CbScalars* sc, int q) {
    partials += (size_t)blockIdx.x * CB_PARTIALS;
    sc += blockIdx.x;
    if (sc->stopped[q] || sc->brk[q]) return;
    double tot[3];
    sum3_partials(partials, nwg, tot);
    if (threadIdx.x != 0) return;
    const double tt = tot[2];
    sc->omega = tt > 0.0 ? make_double2(tot[0] / tt, tot[1] / tt) : make_double2(0.0, 0.0);
}

// x = 0, r = rh = rc, p_prev = v_prev = 0 (slot 1), partials A
__global__ __launch_bounds__(256) void k_cb_init(int n, const float2* rc, CbVecs cv, double2* partials) {
    cv = cv.of(blockIdx.y);
    rc += (size_t)blockIdx.y * n;
    double2 a = make_double2(0.0, 0.0);
    double b = 0.0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float2 r = rc[i];
        cv.x[i] = cv.p[1][i] = cv.v[1][i] = make_float2(0.f, 0.f);
        cv.r[i] = cv.rh[i] = r;
        const double rr = (double)r.x * r.x + (double)r.y * r.y;
        a.x += rr;
        b += rr;
    }
    chunk_partials(a, b, partials);
}

__global__ __launch_bounds__(256) void k_cb_update(int n, const CbScalars* sc, int q, CbVecs cv,
                                                   double2* partials) {
    sc += blockIdx.y;
    if (sc->stopped[q] || sc->brk[q]) return;
    cv = cv.of(blockIdx.y);
    const float ar = (float)sc->alpha.x, ai = (float)sc->alpha.y, wr = (float)sc->omega.x, wi = (float)sc->omega.y;
    const float2* pq = cv.pp(q);
    double2 a = make_double2(0.0, 0.0);
    double b = 0.0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float2 x = cv.x[i], p = pq[i], s = cv.s[i], t = cv.t[i], h = cv.rh[i];
        cv.x[i] = make_float2(x.x + (ar * p.x - ai * p.y) + (wr * s.x - wi * s.y),
                              x.y + (ar * p.y + ai * p.x) + (wr * s.y + wi * s.x));
        const float2 r = make_float2(s.x - (wr * t.x - wi * t.y), s.y - (wr * t.y + wi * t.x));
        cv.r[i] = r;
        const double2 hr = cdot_d(h, r);
        a.x += hr.x;
        a.y += hr.y;
        b += (double)r.x * r.x + (double)r.y * r.y;
    }
    chunk_partials(a, b, partials);
}

// FP16 copy of the FP32 coarse matrices
__global__ __launch_bounds__(256) void k_mg_dc_half(const float2* __restrict__ src, unsigned int* __restrict__ dst,
                                                    size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float2 v = src[i];
        dst[i] = pack2<P_F16>(v.x, v.y);
    }
}

int cb_grid(int n) {
    const int b = (n + 255) / 256;
    return b < MG_ELEM_WG ? b : MG_ELEM_WG;
}

// f(half, nc) with the storage flag and the product's nc as compile-time
// constants: 16, 32 and 64 take the fused pass 1, other sizes NC = 0
template <typename F>
void with_nc(int nc, bool half, F&& f) {
    auto go = [&](auto h) {
        switch (nc) {
        case 16: f(h, std::integral_constant<int, 16>{}); break;
        case 32: f(h, std::integral_constant<int, 32>{}); break;
        case 64: f(h, std::integral_constant<int, 64>{}); break;
        default: f(h, std::integral_constant<int, 0>{}); break;
        }
    };
    if (half) go(std::true_type{});
    else go(std::false_type{});
}

}  // namespace

hipError_t mg_orthonormalize(const Geom& g, void* P, int nv, hipStream_t s) {
    ProfScope ps("mg", s);
    hipLaunchKernelGGL(k_mg_orthonormalize, dim3(g.nblk, 2), dim3(TPB), 0, s, g, (char*)P,
                       spinor_bytes_per_site(P_F32) * g.V, nv);
    return hipGetLastError();
}

hipError_t mg_assemble(const OpData& op, const void* P, int nv, float2* Dc, hipStream_t s) {
    ProfScope ps("mg", s);
    static_assert(MG_MAX_NV <= 32, "two row tiles of 16");
    const size_t fs = spinor_bytes_per_site(P_F32) * op.g.V;
    if (nv <= 16)
        hipLaunchKernelGGL(k_mg_assemble<1>, dim3(op.g.nblk), dim3(TPB), 0, s, op.g, op.links[P_F32], op.clover32,
                           (float)op.kappa, (const char*)P, fs, nv, Dc);
    else
        hipLaunchKernelGGL(k_mg_assemble<2>, dim3(2 * op.g.nblk), dim3(TPB), 0, s, op.g, op.links[P_F32],
                           op.clover32, (float)op.kappa, (const char*)P, fs, nv, Dc);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mg_assemble_fwd, dim3(op.g.nblk, 4), dim3(TPB), 0, s, op.g, nv, Dc);
    return hipGetLastError();
}

hipError_t mg_restrict(const Geom& g, Transfer T, int nv, const void* r, float2* rc, hipStream_t s) {
    ProfScope ps("mg", s);
    const size_t fs = spinor_bytes_per_site(T.prec) * g.V;
    if (T.prec == P_F16)
        hipLaunchKernelGGL(k_mg_restrict<P_F16>, dim3(g.nblk), dim3(TPB), 0, s, g, (const char*)T.P, fs, nv, r, rc);
    else
        hipLaunchKernelGGL(k_mg_restrict<P_F32>, dim3(g.nblk), dim3(TPB), 0, s, g, (const char*)T.P, fs, nv, r, rc);
    return hipGetLastError();
}

hipError_t mg_prolong(const Geom& g, Transfer T, int nv, const float2* ec, void* z, hipStream_t s) {
    ProfScope ps("mg", s);
    const size_t fs = spinor_bytes_per_site(T.prec) * g.V;
    if (T.prec == P_F16)
        hipLaunchKernelGGL(k_mg_prolong<P_F16>, dim3(g.nblk), dim3(TPB), 0, s, g, (const char*)T.P, fs, nv, ec, z);
    else
        hipLaunchKernelGGL(k_mg_prolong<P_F32>, dim3(g.nblk), dim3(TPB), 0, s, g, (const char*)T.P, fs, nv, ec, z);
    return hipGetLastError();
}

hipError_t mg_restrict_many(const Geom& g, Transfer T, int nv, const void* r, int nr, float2* rc,
                            hipStream_t s) {
    ProfScope ps("mg", s);
    constexpr int R = 4;
    const size_t fs = spinor_bytes_per_site(T.prec) * g.V, rs = spinor_bytes_per_site(P_F32) * g.V;
    const size_t rcs = (size_t)g.nblk * 2 * nv;
    const dim3 grid(g.nblk * ((nr + R - 1) / R));
    if (T.prec == P_F16)
        hipLaunchKernelGGL((k_mg_restrict_many<P_F16, R>), grid, dim3(TPB), 0, s, g, (const char*)T.P, fs, nv,
                           (const char*)r, rs, nr, rc, rcs);
    else
        hipLaunchKernelGGL((k_mg_restrict_many<P_F32, R>), grid, dim3(TPB), 0, s, g, (const char*)T.P, fs, nv,
                           (const char*)r, rs, nr, rc, rcs);
    return hipGetLastError();
}

hipError_t mg_prolong_many(const Geom& g, Transfer T, int nv, const float2* ec, size_t ecs, int nr, void* z,
                           hipStream_t s) {
    ProfScope ps("mg", s);
    constexpr int R = 4;
    const size_t fs = spinor_bytes_per_site(T.prec) * g.V, zs = spinor_bytes_per_site(P_F32) * g.V;
    const dim3 grid(g.nblk * ((nr + R - 1) / R));
    if (T.prec == P_F16)
        hipLaunchKernelGGL((k_mg_prolong_many<P_F16, R>), grid, dim3(TPB), 0, s, g, (const char*)T.P, fs, nv, ec,
                           ecs, nr, (char*)z, zs);
    else
        hipLaunchKernelGGL((k_mg_prolong_many<P_F32, R>), grid, dim3(TPB), 0, s, g, (const char*)T.P, fs, nv, ec,
                           ecs, nr, (char*)z, zs);
    return hipGetLastError();
}

hipError_t mg_coarse_half(const float2* Dc, void* Dc16, size_t n, hipStream_t s) {
    ProfScope ps("mg", s);
    const size_t b = (n + 255) / 256;
    hipLaunchKernelGGL(k_mg_dc_half, dim3((unsigned)(b < 4096 ? b : 4096)), dim3(256), 0, s, Dc, (unsigned int*)Dc16,
                       n);
    return hipGetLastError();
}

hipError_t mg_coarse_apply(const Geom& g, CoarseMat M, int nc, const float2* x, float2* y, float2* tau,
                           hipStream_t s) {
    ProfScope ps("mg", s);
    with_nc(nc, M.half, [&](auto half, auto ncc) {
        hipLaunchKernelGGL((k_mg_coarse_apply<decltype(half)::value, decltype(ncc)::value>), dim3(g.nblk),
                           dim3(CMV_TPB), 0, s, g, M.m, nc, x, y, tau);
    });
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mg_coarse_complete, dim3(cb_grid(g.nblk * nc)), dim3(256), 0, s, g, nc, y, tau);
    return hipGetLastError();
}

#define CB_CHECK()                               \
    do {                                         \
        hipError_t e_ = hipGetLastError();       \
        if (e_ != hipSuccess) return e_;         \
    } while (0)
#define CB_LAUNCH(...)                           \
    do {                                         \
        hipLaunchKernelGGL(__VA_ARGS__);         \
        CB_CHECK();                              \
    } while (0)

// Right-hand sides that share one pass over D_c in a batch: four, so that the
// sums and kept adjoints of a lane (7 floats each) stay in registers beside
// the loads in flight.  At 16^3 x 32 with 16 null vectors a product of all 16
// takes 57 us, one alone 20; the coarse solves of four adaptive passes 2 ms
// side by side, 14 one after another.
constexpr int CB_BATCH = 4;

hipError_t mg_coarse_begin(const Geom& g, int nc, int nr, const float2* rc, const CbVecs& cv, CbScalars* sc,
                           const CbPartials& pa, double tol, hipStream_t s) {
    ProfScope ps("mg", s);
    const int n = g.nblk * nc, grid = cb_grid(n);
    CB_LAUNCH(k_cb_init, dim3(grid, nr), dim3(256), 0, s, n, rc, cv, pa.A);
    CB_LAUNCH(k_cb_f1, dim3(nr), dim3(1024), 0, s, pa.A, grid, sc, 0, tol * tol);
    return hipSuccess;
}

hipError_t mg_coarse_iters(const Geom& g, CoarseMat M, int nc, int nr, const CbVecs& cv, CbScalars* sc,
                           const CbPartials& pa, int it0, int it1, hipStream_t s) {
    ProfScope ps("mg", s);
    const int n = g.nblk * nc, grid = cb_grid(n);
    // pass 1 of a product: one right-hand side per workgroup, or CB_BATCH
    auto product = [&](auto m1, int q) {
        with_nc(nc, M.half, [&](auto half, auto ncc) {
            constexpr bool H = decltype(half)::value;
            constexpr int NC = decltype(ncc)::value;
            if (nr == 1) {
                const dim3 wgs(g.nblk);
                if constexpr (decltype(m1)::value) hipLaunchKernelGGL((k_cb_m1<H, NC, 1>), wgs, dim3(CMV_TPB), 0, s, g, M.m, nc, cv, sc, q, nr);
                else hipLaunchKernelGGL((k_cb_m2<H, NC, 1>), wgs, dim3(CMV_TPB), 0, s, g, M.m, nc, cv, sc, q, nr);
            } else {
                const dim3 wgs(g.nblk, (nr + CB_BATCH - 1) / CB_BATCH);
                if constexpr (decltype(m1)::value) hipLaunchKernelGGL((k_cb_m1<H, NC, CB_BATCH>), wgs, dim3(CMV_TPB), 0, s, g, M.m, nc, cv, sc, q, nr);
                else hipLaunchKernelGGL((k_cb_m2<H, NC, CB_BATCH>), wgs, dim3(CMV_TPB), 0, s, g, M.m, nc, cv, sc, q, nr);
            }
        });
    };
    for (int it = it0; it < it1; ++it) {
        const int q = it & 1;
        product(std::true_type{}, q);
        CB_CHECK();
        CB_LAUNCH(k_cb_c1, dim3(grid, nr), dim3(256), 0, s, g, nc, cv, sc, q, pa.B);
        CB_LAUNCH(k_cb_f2, dim3(nr), dim3(1024), 0, s, pa.B, grid, sc, q);
        product(std::false_type{}, q);
        CB_CHECK();
        CB_LAUNCH(k_cb_c2, dim3(grid, nr), dim3(256), 0, s, g, nc, cv, sc, q, pa.C);
        CB_LAUNCH(k_cb_f3, dim3(nr), dim3(1024), 0, s, pa.C, grid, sc, q);
        CB_LAUNCH(k_cb_update, dim3(grid, nr), dim3(256), 0, s, n, sc, q, cv, pa.A);
        CB_LAUNCH(k_cb_f1, dim3(nr), dim3(1024), 0, s, pa.A, grid, sc, it + 1, 0.0);
    }
    return hipSuccess;
}

#undef CB_LAUNCH
#undef CB_CHECK

hipError_t mg_coarse_bicgstab(const Geom& g, CoarseMat M, int nc, const float2* rc, const CbVecs& cv,
                              CbScalars* sc, const CbPartials& pa, int max_iter, double tol, hipStream_t s) {
    hipError_t e = mg_coarse_begin(g, nc, 1, rc, cv, sc, pa, tol, s);
    if (e != hipSuccess) return e;
    return mg_coarse_iters(g, M, nc, 1, cv, sc, pa, 0, max_iter, s);
}

}  // namespace cs
