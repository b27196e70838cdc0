// Clover-Wilson operator (paper Section 2, Eq. (1), with C = 1 + T):
//   (D psi)(x) = (1 + T(x)) psi(x)
//     - kappa sum_mu [(1 - gamma_mu) U_mu(x) psi(x+mu) + (1 + gamma_mu) U_mu(x-mu)^dag psi(x-mu)]
// One workgroup per 4^4 block, one lane per site; every load is unit-stride
// across the lanes because fields are component-major within a block.  The
// kernel is bound by HBM bandwidth: per site it reads the spinor (the eight
// neighbours come from cache), four compressed links (the backward links are
// the neighbours' forward links) and the clover term, and writes one spinor.
#include <type_traits>

#include "dslash_core.hpp"

namespace cs {

namespace {

// The hopping sum with the loads of AHEAD hops in flight while a hop is
// computed, as straight code: for launches of few workgroups, whose time is
// the chain of one workgroup's loads.  The same terms in the same order as
// hopping_sum_rolled.  A fetched hop is kept as loaded (16-bit words packed,
// third link row not yet rebuilt), so that nothing waits for it before its
// turn.
template <int P>
struct RawSpinor {  // FP64, FP32
    using R = typename SpinorIO<P>::R;
    cpx<R> c[12];
    __device__ __forceinline__ void load(const void* base, int nblk, int blk, int l) {
        SpinorIO<P>::load(base, nblk, blk, l, c);
    }
    __device__ __forceinline__ void get(cpx<R>* o) const {
#pragma unroll
        for (int k = 0; k < 12; ++k) o[k] = c[k];
    }
};
template <int P>
struct RawSpinor16 {
    typename SpinorIO16<P>::Raw r;
    __device__ __forceinline__ void load(const void* base, int nblk, int blk, int l) {
        SpinorIO16<P>::load_raw(base, nblk, blk, l, r);
    }
    __device__ __forceinline__ void get(cpx<float>* o) const {
        SpinorIO16<P>::unpack(r, o);
        keep_rounding(o);
    }
};
template <>
struct RawSpinor<P_F16> : RawSpinor16<P_F16> {};
template <>
struct RawSpinor<P_BF16> : RawSpinor16<P_BF16> {};

template <int P>
struct RawLink {  // FP64, FP32
    using R = typename LinkIO<P>::R;
    cpx<R> u[6];
    __device__ __forceinline__ void load(const void* base, int blk, int l, int mu) {
        LinkIO<P>::template load6<false>(base, blk, l, mu, u);
    }
    __device__ __forceinline__ void get(cpx<R>* o) const {
#pragma unroll
        for (int k = 0; k < 6; ++k) o[k] = u[k];
    }
};
template <int P>
struct RawLink16 {
    uint2 w[3];
    __device__ __forceinline__ void load(const void* base, int blk, int l, int mu) {
        const uint2* p = (const uint2*)base + ((size_t)blk * 4 + mu) * 3 * BLOCK_SITES + l;
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = p[k * BLOCK_SITES];
    }
    __device__ __forceinline__ void get(cpx<float>* o) const {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            unpack2<P>(w[k].x, o[2 * k].re, o[2 * k].im);
            unpack2<P>(w[k].y, o[2 * k + 1].re, o[2 * k + 1].im);
        }
    }
};
template <>
struct RawLink<P_F16> : RawLink16<P_F16> {};
template <>
struct RawLink<P_BF16> : RawLink16<P_BF16> {};

// One hop's operands for G right-hand sides, fields in_stride apart.
template <int PIN, int PLINK, int G>
struct RawHop {
    RawSpinor<PIN> psi[G];
    RawLink<PLINK> link;
    template <int H>
    __device__ __forceinline__ void load(const Geom& g, const BlockPos& p, int l, const void* in, size_t in_stride,
                                         const void* links) {
        constexpr int MU = H >> 1, DIR = (H & 1) ? -1 : +1;
        int nl;
        bool inside;
        const int nb = neighbour(g, p, l, MU, DIR, &nl, &inside);
#pragma unroll
        for (int j = 0; j < G; ++j) psi[j].load((const char*)in + j * in_stride, g.nblk, nb, nl);
        link.load(links, DIR > 0 ? p.blk : nb, DIR > 0 ? l : nl, MU);
    }
    template <int H, bool DAG, typename R>
    __device__ __forceinline__ void apply(const Geom& g, const BlockPos& p, int l, cpx<R> (*acc)[12]) const {
        constexpr int MU = H >> 1, DIR = (H & 1) ? -1 : +1, lc = DIR > 0 ? 3 : 0;
        cpx<R> u[9];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            cpx<R> c[12];
            psi[j].get(c);
            if (DAG) negate_lower(c);
            if (MU == 3) time_boundary_phase(g, wraps_time(g, p, MU, DIR, ((l >> 6) & 3) != lc), &c[0].re, 24);
            if (j == 0) {
                link.get(u);
                su3_row2<std::is_same<R, float>::value>(u);
            }
            hop_term<MU, -DIR>(u, c, acc[j]);
#pragma unroll
            for (int k = 0; k < 12; ++k) asm volatile("" : "+v"(acc[j][k].re), "+v"(acc[j][k].im));
        }
    }
};

template <int H, int AHEAD, bool DAG, int G, typename HOP, typename R>
__device__ __forceinline__ void hops_ahead(const Geom& g, const BlockPos& p, int l, const void* in, size_t in_stride,
                                           const void* links, HOP* f, cpx<R> (*acc)[12]) {
    if constexpr (H < 8) {
        constexpr int N = AHEAD + 1;
        if constexpr (H + AHEAD < 8) f[(H + AHEAD) % N].template load<H + AHEAD>(g, p, l, in, in_stride, links);
        // the fetch stays before this hop's arithmetic and the arithmetic here,
        // or the compiler would issue all loads first and spill
        __builtin_amdgcn_sched_barrier(0);
        f[H % N].template apply<H, DAG>(g, p, l, acc);
        __builtin_amdgcn_sched_barrier(0);
        hops_ahead<H + 1, AHEAD, DAG, G>(g, p, l, in, in_stride, links, f, acc);
    }
}

template <int PIN, int PLINK, int AHEAD, bool DAG, int G, typename R>
__device__ __forceinline__ void hopping_sum_ahead(const Geom& g, const BlockPos& p, int l, const void* in,
                                                  size_t in_stride, const void* links, cpx<R> (*acc)[12]) {
    static_assert(AHEAD >= 1 && AHEAD <= 3, "the first hops fetched here");
    RawHop<PIN, PLINK, G> f[AHEAD + 1];
    f[0].template load<0>(g, p, l, in, in_stride, links);
    if constexpr (AHEAD > 1) f[1].template load<1>(g, p, l, in, in_stride, links);
    if constexpr (AHEAD > 2) f[2].template load<2>(g, p, l, in, in_stride, links);
    hops_ahead<0, AHEAD, DAG, G>(g, p, l, in, in_stride, links, f, acc);
}

// One right-hand side per workgroup.  Bound by HBM on large lattices (per
// site the FP32 operator cannot do without 672 bytes: 32^3 x 64 takes 300 us,
// 4.7 TB/s of them, with 1.18 times as many crossing the L2) and by the chain
// of loads on small ones, where a launch is a round or two of workgroups.
// With the loop over hops not unrolled every hop waited for its own loads:
// 13.3 us at 8^4 in FP64 and 13.1 in FP32 against 9.9 and 7.8 now, 47 and 21.6
// against 33 and 18.4 at 16^3 x 32, 719 against 614 for FP64 at 32^3 x 64.
// Hops in flight: two in FP64, three below, measured best of 1-3 and 2-5 on
// lattices of 512 blocks and more (registers: two waves per SIMD in FP32, four
// in the 16-bit formats, which are asked for: the BF16 kernel would take one or
// two registers too many).
template <int P>
constexpr int hops_in_flight() { return P == P_F64 ? 2 : 3; }

template <int PIN, int POUT, int PLINK, bool DAG, bool SUB>
__global__ __launch_bounds__(BLOCK_SITES, PLINK == P_F16 || PLINK == P_BF16 ? 4 : 1) void k_dslash(
    Geom g, const void* __restrict__ links, const void* __restrict__ clover, double kappa, void* __restrict__ out,
    const void* __restrict__ in, const void* __restrict__ sub, size_t in_stride, size_t out_stride) {
    using R = typename Arith<PIN>::R;
    const int blk = block_of_item(g, xcd_remap(blockIdx.x, g.nblk)), l = threadIdx.x, r = blockIdx.y;
    const char* src = (const char*)in + r * in_stride;
    const BlockPos p = block_pos(g, blk);

    cpx<R> acc[1][12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[0][k] = {(R)0, (R)0};
    hopping_sum_ahead<PIN, PLINK, hops_in_flight<PIN>(), DAG, 1>(g, p, l, src, 0, links, acc);

    GlobalSpinor<PIN, DAG> ld{src, g.nblk};
    cpx<R> self[12], res[12];
    ld.load(blk, l, self);
    R cl[72];
    CloverIO<R>::load(clover, blk, l, cl);
    clover_apply(cl, self, res);
    const R k = (R)kappa;
#pragma unroll
    for (int i = 0; i < 12; ++i) res[i] = {res[i].re - k * acc[0][i].re, res[i].im - k * acc[0][i].im};
    if (DAG) negate_lower(res);
    using RO = typename SpinorIO<POUT>::R;
    cpx<RO> o[12];
    if (SUB) {
        SpinorIO<POUT>::load((const char*)sub + r * out_stride, g.nblk, blk, l, o);
#pragma unroll
        for (int i = 0; i < 12; ++i) o[i] = {o[i].re - (RO)res[i].re, o[i].im - (RO)res[i].im};
    } else {
#pragma unroll
        for (int i = 0; i < 12; ++i) o[i] = {(RO)res[i].re, (RO)res[i].im};
    }
    SpinorIO<POUT>::store((char*)out + r * out_stride, g.nblk, blk, l, o);
}

// Variant for several right-hand sides in FP64, and in FP32 for tiles of three
// and more: work item = (block, tile of right-hand sides).  The block's links go
// to LDS once and its clover term to registers once per item; every right-hand
// side of the tile reuses them.  Backward links of neighbours outside the block
// come from HBM (cache).  With gridDim.x < nitems the workgroups stride over the
// items (persistent).
template <typename RS, int PLINK>
struct MixedLinks {
    const lds_cpx<RS> (*sm)[6][BLOCK_SITES];
    const void* base;
    template <typename R>
    __device__ __forceinline__ void load(int blk, int l, int mu, bool inside, cpx<R>* u) const {
        if (inside) {
#pragma unroll
            for (int k = 0; k < 6; ++k) u[k] = {(R)sm[mu][k][l].re, (R)sm[mu][k][l].im};
            su3_row2<std::is_same<R, float>::value>(u);
        } else {
            load_link<PLINK, R, false, std::is_same<R, float>::value>(base, blk, l, mu, u);
        }
    }
};

// The rolled hopping sum for two right-hand sides at once: each hop loads
// its link once and the two neighbour spinors together, so two loads are in
// flight where the one-right-hand-side loop waits on one.  Each sum gets the
// same terms in the same order as hopping_sum_rolled.
template <typename R, typename LS, typename LL>
__device__ __forceinline__ void hopping_sum_rolled2(const Geom& g, const BlockPos& p, int l, const LS& ls0,
                                                    const LS& ls1, const LL& lk, cpx<R>* acc0, cpx<R>* acc1) {
#pragma unroll 1
    for (int h = 0; h < 8; ++h) {
        const int mu = h >> 1, dir = (h & 1) ? -1 : +1;
        const int bc = mu == 0 ? p.bc[0] : mu == 1 ? p.bc[1] : mu == 2 ? p.bc[2] : p.bc[3];
        const int nbm = mu == 0 ? g.NB[0] : mu == 1 ? g.NB[1] : mu == 2 ? g.NB[2] : g.NB[3];
        const int st = mu == 0 ? p.stride[0] : mu == 1 ? p.stride[1] : mu == 2 ? p.stride[2] : p.stride[3];
        const int sh = 2 * mu, lc = (l >> sh) & 3;
        int nl, nb;
        bool in;
        if (dir > 0) {
            in = lc < 3;
            nl = in ? l + (1 << sh) : l - (3 << sh);
            nb = in ? p.blk : (bc == nbm - 1 ? p.blk - (nbm - 1) * st : p.blk + st);
        } else {
            in = lc > 0;
            nl = in ? l - (1 << sh) : l + (3 << sh);
            nb = in ? p.blk : (bc == 0 ? p.blk + (nbm - 1) * st : p.blk - st);
        }
        cpx<R> psi0[12], psi1[12], u[9];
        ls0.template load_nb<R>(nb, nl, in, psi0);
        ls1.template load_nb<R>(nb, nl, in, psi1);
        if (mu == 3) {
            const bool wraps = !in && (dir > 0 ? bc == nbm - 1 : bc == 0);
            time_boundary_phase(g, wraps, &psi0[0].re, 24);
            time_boundary_phase(g, wraps, &psi1[0].re, 24);
        }
        if (dir > 0) lk.template load<R>(p.blk, l, mu, true, u);
        else lk.template load<R>(nb, nl, mu, in, u);
        switch (h) {
        case 0: hop_term<0, -1>(u, psi0, acc0); hop_term<0, -1>(u, psi1, acc1); break;
        case 1: hop_term<0, +1>(u, psi0, acc0); hop_term<0, +1>(u, psi1, acc1); break;
        case 2: hop_term<1, -1>(u, psi0, acc0); hop_term<1, -1>(u, psi1, acc1); break;
        case 3: hop_term<1, +1>(u, psi0, acc0); hop_term<1, +1>(u, psi1, acc1); break;
        case 4: hop_term<2, -1>(u, psi0, acc0); hop_term<2, -1>(u, psi1, acc1); break;
        case 5: hop_term<2, +1>(u, psi0, acc0); hop_term<2, +1>(u, psi1, acc1); break;
        case 6: hop_term<3, -1>(u, psi0, acc0); hop_term<3, -1>(u, psi1, acc1); break;
        default: hop_term<3, +1>(u, psi0, acc0); hop_term<3, +1>(u, psi1, acc1); break;
        }
    }
}

template <int PIN, int POUT, int PLINK, bool DAG, bool SUB>
__global__ CS_DSLASH_BOUNDS void k_dslash_tiled(Geom g, const void* __restrict__ links,
                                                const void* __restrict__ clover, double kappa,
                                                void* __restrict__ out, const void* __restrict__ in,
                                                const void* __restrict__ sub, size_t in_stride,
                                                size_t out_stride, int nrhs, int tile, int nitems) {
    using R = typename Arith<PIN>::R;
    using RS = typename LinkIO<PLINK>::R;
    __shared__ lds_cpx<RS> s_lk[4][6][BLOCK_SITES];
    const int l = threadIdx.x;
    for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int w = xcd_remap(item, nitems);
        const int blk = block_of_item(g, w % g.nblk);
        const int r0 = (w / g.nblk) * tile;
        const int r1 = r0 + tile < nrhs ? r0 + tile : nrhs;
        const BlockPos p = block_pos(g, blk);
        __syncthreads();
        for (int mu = 0; mu < 4; ++mu) {
            cpx<RS> u[6];
            LinkIO<PLINK>::load6(links, blk, l, mu, u);
#pragma unroll
            for (int k = 0; k < 6; ++k) s_lk[mu][k][l].set(u[k]);
        }
        R cl[72];
        CloverIO<R>::load(clover, blk, l, cl);
        __syncthreads();
        MixedLinks<RS, PLINK> lk{s_lk, links};
        const R k = (R)kappa;
        // the clover term and the output of one right-hand side
        auto finish = [&](int r, const GlobalSpinor<PIN, DAG>& ld, const cpx<R>* acc) {
            cpx<R> self[12], res[12];
            ld.load(blk, l, self);
            clover_apply(cl, self, res);
#pragma unroll
            for (int i = 0; i < 12; ++i) res[i] = {res[i].re - k * acc[i].re, res[i].im - k * acc[i].im};
            if (DAG) negate_lower(res);
            using RO = typename SpinorIO<POUT>::R;
            cpx<RO> o[12];
            if constexpr (SUB) {
                SpinorIO<POUT>::load((const char*)sub + (size_t)r * out_stride, g.nblk, blk, l, o);
#pragma unroll
                for (int i = 0; i < 12; ++i) o[i] = {o[i].re - (RO)res[i].re, o[i].im - (RO)res[i].im};
            } else {
#pragma unroll
                for (int i = 0; i < 12; ++i) o[i] = {(RO)res[i].re, (RO)res[i].im};
            }
            SpinorIO<POUT>::store((char*)out + (size_t)r * out_stride, g.nblk, blk, l, o);
        };
        int r = r0;
        if constexpr (PIN != P_F64) {
            // right-hand sides two at a time (the FP64 form keeps one: its
            // registers are full)
            for (; r + 1 < r1; r += 2) {
                GlobalSpinor<PIN, DAG> ld0{(const char*)in + (size_t)r * in_stride, g.nblk};
                GlobalSpinor<PIN, DAG> ld1{(const char*)in + (size_t)(r + 1) * in_stride, g.nblk};
                cpx<R> acc0[12], acc1[12];
#pragma unroll
                for (int i = 0; i < 12; ++i) acc0[i] = acc1[i] = {(R)0, (R)0};
                hopping_sum_rolled2<R>(g, p, l, ld0, ld1, lk, acc0, acc1);
                finish(r, ld0, acc0);
                finish(r + 1, ld1, acc1);
            }
        }
        for (; r < r1; ++r) {
            GlobalSpinor<PIN, DAG> ld{(const char*)in + (size_t)r * in_stride, g.nblk};
            cpx<R> acc[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) acc[i] = {(R)0, (R)0};
            hopping_sum_rolled<R>(g, p, l, ld, lk, acc);
            finish(r, ld, acc);
        }
    }
}

// Pairs in FP32 and any tile in the 16-bit formats: right-hand sides in groups
// of G, a hop loading its link once for the group, the next hops' loads in
// flight, and the clover term serving the group; nothing is staged in LDS and
// no lane waits for another.  The same terms in the same order as k_dslash.
// Bound by the chain of loads below a few rounds of workgroups and by HBM
// above.  FP16, three right-hand sides: 12 x 20 x 28 x 36 66 us (one workgroup
// each 81, staged tile 81), 32^3 x 64 431 (644, 604); FP32 pairs, 16^3 x 32 with
// twelve 110 (172, staged tiles of four 134), 32^3 x 64 with two 463 (590).
// FP32 tiles of three and more stay with the staged kernel: three spinors a hop
// leave no registers for a hop ahead (32^3 x 64 with three: 727 us, as 2 + 1
// 689, staged 650).
template <int PIN, int G>
constexpr int group_hops_in_flight() { return PIN == P_F32 ? (G == 1 ? 3 : 1) : (G == 3 ? 1 : G == 2 ? 2 : 3); }

template <int G, int PIN, int POUT, int PLINK, bool DAG>
__device__ __forceinline__ void dslash_group(const Geom& g, const BlockPos& p, int lane, const void* links,
                                             const void* clover, float kappa, void* out, const void* in,
                                             size_t in_stride, size_t out_stride) {
    int l = lane;
    asm volatile("" : "+v"(l));  // addresses are made here, not kept from group to group
    cpx<float> acc[G][12];
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[j][k] = {0.f, 0.f};
    hopping_sum_ahead<PIN, PLINK, group_hops_in_flight<PIN, G>(), DAG, G>(g, p, l, in, in_stride, links, acc);
    float cl[72];
    CloverIO<float>::template load<false>(clover, p.blk, l, cl);
#pragma unroll
    for (int j = 0; j < G; ++j) {
        GlobalSpinor<PIN, DAG> ld{(const char*)in + j * in_stride, g.nblk};
        cpx<float> self[12], res[12];
        ld.load(p.blk, l, self);
        clover_apply(cl, self, res);
#pragma unroll
        for (int i = 0; i < 12; ++i)
            res[i] = {res[i].re - kappa * acc[j][i].re, res[i].im - kappa * acc[j][i].im};
        if (DAG) negate_lower(res);
        SpinorIO<POUT>::store((char*)out + j * out_stride, g.nblk, p.blk, l, res);
    }
}

// Work item = (block, tile of right-hand sides); the tiles of a block are
// neighbours on one XCD, whose L2 serves their links and clover term.
template <int PIN, int POUT, int PLINK, bool DAG>
__global__ CS_DSLASH_BOUNDS void k_dslash_groups(Geom g, const void* links, const void* clover, double kappa,
                                                 void* out, const void* in, size_t in_stride, size_t out_stride,
                                                 int nrhs, int tile, int nitems) {
    constexpr int GM = PIN == P_F32 ? 2 : 3;  // as many as leave two waves per SIMD
    const int ntiles = (nrhs + tile - 1) / tile;
    for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int w = xcd_remap(item, nitems);
        const int r0 = w % ntiles * tile, r1 = r0 + tile < nrhs ? r0 + tile : nrhs;
        const BlockPos p = block_pos(g, block_of_item(g, w / ntiles));
        auto go = [&](auto n, int r) {
            dslash_group<decltype(n)::value, PIN, POUT, PLINK, DAG>(
                g, p, threadIdx.x, links, clover, (float)kappa, (char*)out + (size_t)r * out_stride,
                (const char*)in + (size_t)r * in_stride, in_stride, out_stride);
        };
        int r = r0;
#pragma unroll 1
        for (; r + GM <= r1; r += GM) go(std::integral_constant<int, GM>{}, r);
        if constexpr (GM > 2) {
            if (r + 2 <= r1) {
                go(std::integral_constant<int, 2>{}, r);
                r += 2;
            }
        }
        if (r < r1) go(std::integral_constant<int, 1>{}, r);
    }
}

template <int PIN, int POUT, int PLINK>
hipError_t launch_tiled(const OpData& op, bool dagger, void* out, const void* in, int nrhs,
                        const LaunchCfg& cfg, hipStream_t s, const void* sub = nullptr) {
    const int tile = cfg.rhs_tile > nrhs ? nrhs : cfg.rhs_tile;
    const int nitems = op.g.nblk * ((nrhs + tile - 1) / tile);
    const int grid = cfg.persistent_wgs > 0 && cfg.persistent_wgs < nitems ? cfg.persistent_wgs : nitems;
    const size_t is = spinor_bytes_per_site(PIN) * op.g.V, os = spinor_bytes_per_site(POUT) * op.g.V;
    const void* cl = PIN == P_F64 ? op.clover64 : op.clover32;
    const void* lk = op.links[PLINK];
    if constexpr (PIN != P_F64) {
        if (sub) return hipErrorInvalidValue;
        if (PIN != P_F32 || tile == 2) {
            auto go = [&](auto dag) {
                hipLaunchKernelGGL((k_dslash_groups<PIN, POUT, PLINK, decltype(dag)::value>), dim3(grid),
                                   dim3(BLOCK_SITES), 0, s, op.g, lk, cl, op.kappa, out, in, is, os, nrhs, tile,
                                   nitems);
            };
            dagger ? go(std::true_type{}) : go(std::false_type{});
            return hipGetLastError();
        }
    }
    if constexpr (PIN == P_F64 || PIN == P_F32) {
        auto go = [&](auto dag, auto with_sub) {
            hipLaunchKernelGGL((k_dslash_tiled<PIN, POUT, PLINK, decltype(dag)::value, decltype(with_sub)::value>),
                               dim3(grid), dim3(BLOCK_SITES), 0, s, op.g, lk, cl, op.kappa, out, in, sub, is, os,
                               nrhs, tile, nitems);
        };
        if constexpr (PIN == P_F64) {
            if (sub) {  // b - D x only
                if (dagger) return hipErrorInvalidValue;
                go(std::false_type{}, std::true_type{});
                return hipGetLastError();
            }
        }
        dagger ? go(std::true_type{}, std::false_type{}) : go(std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

template <int PIN, int POUT, int PLINK>
hipError_t launch3(const OpData& op, bool dagger, void* out, const void* in, const void* sub,
                   int nrhs, hipStream_t s) {
    const size_t is = spinor_bytes_per_site(PIN) * op.g.V, os = spinor_bytes_per_site(POUT) * op.g.V;
    const void* cl = PIN == P_F64 ? op.clover64 : op.clover32;
    auto go = [&](auto dag, auto with_sub) {
        hipLaunchKernelGGL((k_dslash<PIN, POUT, PLINK, decltype(dag)::value, decltype(with_sub)::value>),
                           dim3(op.g.nblk, nrhs), dim3(BLOCK_SITES), 0, s, op.g, op.links[PLINK], cl, op.kappa, out,
                           in, sub, is, os);
    };
    if (dagger) {
        if (sub) go(std::true_type{}, std::true_type{});
        else go(std::true_type{}, std::false_type{});
    } else {
        if (sub) go(std::false_type{}, std::true_type{});
        else go(std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

}  // namespace

// The kernels for tiles against the one with a workgroup per block and
// right-hand side, as rounds of resident workgroups times what a round takes:
// a staged tile its links and clover term (head), a unit per right-hand side and
// what an odd one costs on top; the grouped kernel for two and for three
// right-hand sides; the untiled kernel.  Fitted at 8^4 to 32^3 x 64 with 2 to 16
// right-hand sides; a unit is about 9 us below FP64 and 14 us in FP64.  In FP64
// sharing pays where links, clover term and a field leave the 256 MB cache
// (24^3 x 48 with 12: 2.41 ms untiled, 2.03 in tiles of six; 16^3 x 32 with 5:
// 151 us untiled, 157 in one tile).  Two workgroups per compute unit or less
// have nothing to gain by sharing (8^4 with 12: 9 us untiled, 11 in pairs).
struct DslashModel {
    int slots;
    double head, odd;
    double group2, group3;  // 0: tiles of that size are staged
    int untiled_slots;
    double untiled_units;
};
static DslashModel dslash_model(const Geom& g, int prec) {
    if (prec == P_F64) return {256, 0.5, 0.0, 0.0, 0.0, 256, g.V * 1344 > (256ll << 20) ? 1.5 : 1.0};
    if (prec == P_F32) return {512, 1.0, 0.6, 2.6, 0.0, 512, 1.65};
    return {512, 1.0, 0.8, 2.0, 2.6, 1024, 2.45};
}

double dslash_tile_units(const Geom& g, int prec, int nrhs, int t) {
    const DslashModel m = dslash_model(g, prec);
    if (t <= 1) return (double)(((long long)g.nblk * nrhs + m.untiled_slots - 1) / m.untiled_slots) * m.untiled_units;
    const long long wgs = (long long)g.nblk * ((nrhs + t - 1) / t);
    double tile = m.head + t + (t & 1 ? m.odd : 0.0);
    if (t == 2 && m.group2 > 0.0) tile = m.group2;
    else if (m.group3 > 0.0) tile = t / 3 * m.group3 + (t % 3 == 2 ? m.group2 : t % 3 ? m.untiled_units : 0.0);
    return (double)((wgs + m.slots - 1) / m.slots) * tile;
}

LaunchCfg dslash_default_cfg(const Geom& g, int prec, int nrhs) {
    LaunchCfg c;
    if (nrhs < 2 || (long long)g.nblk * nrhs <= 512) return c;
    int best = 2;
    for (int t = 3; t <= nrhs && t <= 64; ++t)
        if (dslash_tile_units(g, prec, nrhs, t) < dslash_tile_units(g, prec, nrhs, best)) best = t;
    if (dslash_tile_units(g, prec, nrhs, best) < 0.95 * dslash_tile_units(g, prec, nrhs, 1)) c.rhs_tile = best;
    return c;
}

hipError_t launch_dslash_tiled(const OpData& op, int prec, bool dagger, void* out, const void* in, int nrhs,
                               const LaunchCfg& cfg, hipStream_t s, const void* sub) {
    ProfScope ps("dslash", s);
    if (sub && prec != P_F64) return hipErrorInvalidValue;
    switch (prec) {
    case P_F64: return launch_tiled<P_F64, P_F64, P_F64>(op, dagger, out, in, nrhs, cfg, s, sub);
    case P_F32: return launch_tiled<P_F32, P_F32, P_F32>(op, dagger, out, in, nrhs, cfg, s);
    case P_F16: return launch_tiled<P_F16, P_F16, P_F16>(op, dagger, out, in, nrhs, cfg, s);
    case P_BF16: return launch_tiled<P_BF16, P_BF16, P_BF16>(op, dagger, out, in, nrhs, cfg, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_dslash_tiled_to16(const OpData& op, int out_prec, void* out, const void* in, int nrhs,
                                    const LaunchCfg& cfg, hipStream_t s) {
    ProfScope ps("dslash", s);
    switch (out_prec) {
    case P_F16: return launch_tiled<P_F32, P_F16, P_F32>(op, false, out, in, nrhs, cfg, s);
    case P_BF16: return launch_tiled<P_F32, P_BF16, P_F32>(op, false, out, in, nrhs, cfg, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_dslash(const OpData& op, int in_prec, int out_prec, int link_prec, bool dagger,
                         void* out, const void* in, const void* sub, int nrhs, hipStream_t s) {
    ProfScope ps("dslash", s);
    // Supported combinations: F64 -> F64 (F64 links); float arithmetic with
    // spinors in F32/F16/BF16, links F32 or the spinor's 16-bit type, output
    // F32 or the input type.
    if (in_prec == P_F64) {
        if (out_prec != P_F64) return hipErrorInvalidValue;
        return launch3<P_F64, P_F64, P_F64>(op, dagger, out, in, sub, nrhs, s);
    }
    if (in_prec == P_F32 && out_prec == P_F32 && link_prec == P_F32)
        return launch3<P_F32, P_F32, P_F32>(op, dagger, out, in, sub, nrhs, s);
    if (in_prec == P_F16 && out_prec == P_F16 && link_prec == P_F16)
        return launch3<P_F16, P_F16, P_F16>(op, dagger, out, in, sub, nrhs, s);
    if (in_prec == P_BF16 && out_prec == P_BF16 && link_prec == P_BF16)
        return launch3<P_BF16, P_BF16, P_BF16>(op, dagger, out, in, sub, nrhs, s);
    if (in_prec == P_F16 && out_prec == P_F32 && link_prec == P_F32)
        return launch3<P_F16, P_F32, P_F32>(op, dagger, out, in, sub, nrhs, s);
    if (in_prec == P_BF16 && out_prec == P_F32 && link_prec == P_F32)
        return launch3<P_BF16, P_F32, P_F32>(op, dagger, out, in, sub, nrhs, s);
    // FP32 or 16-bit input with FP32 links, written straight into a 16-bit
    // field (the 16-bit Krylov basis of the outer solver)
    if (link_prec == P_F32 && out_prec == P_F16 && in_prec == P_F32)
        return launch3<P_F32, P_F16, P_F32>(op, dagger, out, in, sub, nrhs, s);
    if (link_prec == P_F32 && out_prec == P_BF16 && in_prec == P_F32)
        return launch3<P_F32, P_BF16, P_F32>(op, dagger, out, in, sub, nrhs, s);
    if (link_prec == P_F32 && out_prec == P_F16 && in_prec == P_F16)
        return launch3<P_F16, P_F16, P_F32>(op, dagger, out, in, sub, nrhs, s);
    if (link_prec == P_F32 && out_prec == P_BF16 && in_prec == P_BF16)
        return launch3<P_BF16, P_BF16, P_F32>(op, dagger, out, in, sub, nrhs, s);
    return hipErrorInvalidValue;
}

}  // namespace cs
