// Wilson Dirac operator D_W and its adjoint (Sec. 5, Eq. app_wils; r = 1), with the optional clover
// term C of Eq. def_clov added at the site (C is hermitian, so (D_W + C)^+ = D_W^+ + C):
//
//   (D_W u)(n)   = (4+m) u(n) - 1/2 sum_mu [(1 - g_mu) U_mu(n) u(n+mu) + (1 + g_mu) U_mu(n-mu)^+ u(n-mu)]
//   (D_W^+ u)(n) = (4+m) u(n) - 1/2 sum_mu [(1 + g_mu) U_mu(n) u(n+mu) + (1 - g_mu) U_mu(n-mu)^+ u(n-mu)]
//
// Each hop uses the spin-projection trick of App. A: (1 +- g_mu) has rank two, so the
// neighbour spinor is first reduced to two spin components h0, h1 (chiral basis), only
// those are multiplied by the Nc x Nc link, and the other two rows are rebuilt from them.
// One thread owns one site and RB consecutive right-hand sides; every output element is
// written once (no atomics).  Fermion fields pick up -1 on t-wrapping hops when
// antiperiodic in t.
#pragma once

#include <algorithm>
#include <type_traits>

#include "clover.h"
#include "common.h"
#include "kernels.h"
#include "tile.h"

namespace dirac {

namespace {

// Half spinor of (1 + SIG g_MU) psi in the chiral basis: rows 0 and 1.
template <int MU, int SIG, typename R>
__device__ __forceinline__ void project(const cx<R> p[4], cx<R>& h0, cx<R>& h1) {
    if constexpr (MU == 0) {  // h0 = p0 - SIG i p3, h1 = p1 - SIG i p2
        if constexpr (SIG > 0) {
            h0 = {p[0].re + p[3].im, p[0].im - p[3].re};
            h1 = {p[1].re + p[2].im, p[1].im - p[2].re};
        } else {
            h0 = {p[0].re - p[3].im, p[0].im + p[3].re};
            h1 = {p[1].re - p[2].im, p[1].im + p[2].re};
        }
    } else if constexpr (MU == 1) {  // h0 = p0 - SIG p3, h1 = p1 + SIG p2
        if constexpr (SIG > 0) {
            h0 = csub(p[0], p[3]);
            h1 = cadd(p[1], p[2]);
        } else {
            h0 = cadd(p[0], p[3]);
            h1 = csub(p[1], p[2]);
        }
    } else if constexpr (MU == 2) {  // h0 = p0 - SIG i p2, h1 = p1 + SIG i p3
        if constexpr (SIG > 0) {
            h0 = {p[0].re + p[2].im, p[0].im - p[2].re};
            h1 = {p[1].re - p[3].im, p[1].im + p[3].re};
        } else {
            h0 = {p[0].re - p[2].im, p[0].im + p[2].re};
            h1 = {p[1].re + p[3].im, p[1].im - p[3].re};
        }
    } else {  // h0 = p0 + SIG p2, h1 = p1 + SIG p3
        if constexpr (SIG > 0) {
            h0 = cadd(p[0], p[2]);
            h1 = cadd(p[1], p[3]);
        } else {
            h0 = csub(p[0], p[2]);
            h1 = csub(p[1], p[3]);
        }
    }
}

// acc[0..3] += s * (full spinor rebuilt from c0, c1): the scale rides on the multiply-adds.
template <int MU, int SIG, typename R>
__device__ __forceinline__ void reconstruct_scaled(cx<R> acc[4], cx<R> c0, cx<R> c1, R s) {
    // a += f v and a += f i v (i v = (-v.im, v.re)), f = +-s
    auto ax = [](cx<R>& a, R f, cx<R> v) __attribute__((always_inline)) {
        a.re += f * v.re;
        a.im += f * v.im;
    };
    auto axi = [](cx<R>& a, R f, cx<R> v) __attribute__((always_inline)) {
        a.re -= f * v.im;
        a.im += f * v.re;
    };
    const R n = -s;
    ax(acc[0], s, c0);
    ax(acc[1], s, c1);
    if constexpr (MU == 0) {  // r2 = SIG i c1, r3 = SIG i c0
        axi(acc[2], SIG > 0 ? s : n, c1);
        axi(acc[3], SIG > 0 ? s : n, c0);
    } else if constexpr (MU == 1) {  // r2 = SIG c1, r3 = -SIG c0
        ax(acc[2], SIG > 0 ? s : n, c1);
        ax(acc[3], SIG > 0 ? n : s, c0);
    } else if constexpr (MU == 2) {  // r2 = SIG i c0, r3 = -SIG i c1
        axi(acc[2], SIG > 0 ? s : n, c0);
        axi(acc[3], SIG > 0 ? n : s, c1);
    } else {  // r2 = SIG c0, r3 = SIG c1
        ax(acc[2], SIG > 0 ? s : n, c0);
        ax(acc[3], SIG > 0 ? s : n, c1);
    }
}

// L = link (ADJ = false) or link^+ (ADJ = true) into registers.
template <int NC, bool ADJ, class P>
__device__ __forceinline__ void load_link(cx<typename P::R> (&l)[NC][NC], const typename P::G* __restrict__ link) {
    using R = typename P::R;
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            cx<R> v = io<R, typename P::G>::ld(link + a * NC + b);
            if constexpr (ADJ) {
                l[b][a] = cconj(v);
            } else {
                l[a][b] = v;
            }
        }
}

// acc += scale * (1 + SIG g_MU) L u_nb for a link matrix L already in registers.  NVC > 0 fixes
// the RHS stride at compile time (else nv).
template <int NC, int RB, int MU, int SIG, class P, int NVC = 0>
__device__ __forceinline__ void hop_with(cx<typename P::R> (&acc)[RB][NC][4], const cx<typename P::R> (&l)[NC][NC],
                                         const typename P::S* __restrict__ nb, int nv, typename P::R scale) {
    using R = typename P::R;
    const int stride = NVC > 0 ? NVC : nv;
#pragma unroll
    for (int k = 0; k < RB; ++k) {
        cx<R> h0[NC], h1[NC];
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            cx<R> p[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) p[s] = io<R, typename P::S>::ld(nb + (b * 4 + s) * stride + k);
            project<MU, SIG>(p, h0[b], h1[b]);
        }
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            cx<R> c0{R(0), R(0)}, c1{R(0), R(0)};
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                cfma(c0, l[a][b], h0[b]);
                cfma(c1, l[a][b], h1[b]);
            }
            reconstruct_scaled<MU, SIG>(acc[k][a], c0, c1, scale);
        }
    }
}

// Direct form: one thread per (site, RB right-hand sides), neighbours read from global memory, the two hops of an axis
// in flight together.  It serves the shapes the row tiles cannot take: a few right-hand sides, or too few or too many
// threads in a row.  NVC > 0 fixes N_v (= RB) at compile time: a site block is then contiguous in a thread and its loads
// are 16 bytes wide.  Bound by the address rate of the loads: with one 8-byte load per element and one hop at a
// time, 100 us at 22 x 18 x 14 x 30 (FP32, N_c = 3, N_v = 1), 1.22 ms at 32^3 x 64 and 19 us (one work-group) at 4^4 in
// FP64; now 46 us, 0.58 ms and less than the 11 us that the call costs the host.
template <int NC, int RB, bool DAG, class P, int NVC>
__global__ __launch_bounds__(256) void wilson_kernel(const typename P::G* __restrict__ U,
                                                      const typename P::S* __restrict__ in,
                                                      typename P::S* __restrict__ out, typename P::R diag, Geom g,
                                                      int nv, SiteOrder order, const typename P::R* __restrict__ clov) {
    using R = typename P::R;
    constexpr int L = NC * NC;
    if constexpr (NVC > 0) nv = NVC;
    const int nrg = NVC > 0 ? NVC / RB : nv / RB;
    const int64_t gid = logical_block() * blockDim.x + threadIdx.x;
    if (gid >= g.vol * nrg) return;
    const int64_t idx = nrg == 1 ? gid : gid / nrg;
    const int r0 = static_cast<int>(gid - idx * nrg) * RB;
    const int64_t site = ordered_site(idx, order, g);
    const Coord c = site_coord(site, g);
    const int64_t vs = static_cast<int64_t>(NC) * 4 * nv;

    cx<R> acc[RB][NC][4];
    const typename P::S* centre = in + site * vs + r0;
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                acc[k][a][s] = cscale(diag, io<R, typename P::S>::ld(centre + (a * 4 + s) * nv + k));
    if (clov) clover_add<NC, RB>(acc, centre, nv, clov + site * clover_reals<NC>());

    // The loads of the next hop (of the next axis, where two hops fit the registers) wait for the sums of this one: an
    // opaque zero that depends on them goes into the addresses.  All hops in flight at once spill.
    constexpr bool PAIR = RB * sizeof(R) <= 8;
    int later = 0;
    auto wait_for_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < RB; ++k)
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(later), "+v"(acc[k][a][s].re), "+v"(acc[k][a][s].im));
    };
    auto axis = [&](auto mu_c, int x, int n, int64_t stride) __attribute__((always_inline)) {
        constexpr int MU = decltype(mu_c)::value;
        constexpr int SF = DAG ? 1 : -1;  // forward projector 1 + SF g_mu
        const bool flip = MU == 3 && g.apbc;  // fermion sign of a hop across the boundary
        const int64_t here = site + later;
        const int64_t fwd = here + (x == n - 1 ? (1 - n) * stride : stride);
        cx<R> l[NC][NC];
        load_link<NC, false, P>(l, U + (here * 4 + MU) * L);
        hop_with<NC, RB, MU, SF, P, NVC>(acc, l, in + fwd * vs + r0, nv, flip && x == n - 1 ? R(0.5) : R(-0.5));
        if constexpr (!PAIR) wait_for_sums();
        const int64_t bwd = site + later - (x == 0 ? (1 - n) * stride : stride);
        load_link<NC, true, P>(l, U + (bwd * 4 + MU) * L);
        hop_with<NC, RB, MU, -SF, P, NVC>(acc, l, in + bwd * vs + r0, nv, flip && x == 0 ? R(0.5) : R(-0.5));
        wait_for_sums();
    };
    axis(std::integral_constant<int, 0>{}, c.x, g.nx, 1);
    axis(std::integral_constant<int, 1>{}, c.y, g.ny, g.nx);
    axis(std::integral_constant<int, 2>{}, c.z, g.nz, static_cast<int64_t>(g.nx) * g.ny);
    axis(std::integral_constant<int, 3>{}, c.t, g.nt, static_cast<int64_t>(g.nx) * g.ny * g.nz);

    typename P::S* o = out + site * vs + r0;
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s) io<R, typename P::S>::st(o + (a * 4 + s) * nv + k, acc[k][a][s]);
}

// Row-tiled variant (see RowTile).  Seven row copies per tile: the own rows (mass term and the
// +-x hops) and the rows one step away in +y, -y, +z, -z, +t, -t.  The copy of the next
// direction is issued into registers before the current direction is consumed from LDS, so the
// loads of one direction overlap the arithmetic of the previous one.  The output tile leaves
// through LDS as one contiguous store.
//
// LL: the links are staged in LDS beside the row copy.  LL 2 (FP32, BF16): the row's own four links per site, one
// contiguous block, once at the start (they serve the four forward hops and the -x hop), and per backward hop the one link
// per site of the neighbour row, an N_c x N_c block of its four.  LL 1 (FP64): one direction at a time, the own links as
// well; a 72-byte block per 288-byte site, the own links are then 128-byte lines touched four times far apart, which costs
// FP32 2 to 3 % (100.6 against 98.0 us at 16^3 x 32, N_c = 3, N_v = 12, bound by the fabric, since a row leaves L2 between
// its seven uses), while FP64, at two wavefronts per SIMD, does not hide the larger first load (216.5 against 224.1 us; N_c = 2
// at 32 x 12 x 12 x 16 83.5 against 96.6).  LL 0: every thread loads its own link one direction ahead.
// CLOV 2: the site's clover record is staged as well (contiguous, 16 bytes a lane) instead of being read by every
// right-hand side's thread (with the links 1.70 against 1.63 ms for BF16 vectors at 32^3 x 64, which the vector
// instructions bound: 1.46 ms with the BF16 stores converted in hardware).  CLOV 1: every thread reads the record; CLOV 0:
// no clover field.  launch_rows chooses.

// Entries of a neighbour row's links (one direction) that a thread moves: N_c^2 over the threads of a site, at most
// three of them where N_v is only known at run time.
template <int NC, int RB, int NVC>
struct RowLinks {
    static constexpr int PER = NVC > 0 ? (NC * NC + NVC / RB - 1) / (NVC / RB) : 3;
};

template <int NC, int RB, bool DAG, class P, int NVC, int LL, int CLOV>
__global__ __launch_bounds__(512) void wilson_rows_kernel(const typename P::G* __restrict__ U,
                                                          const typename P::S* __restrict__ in,
                                                          typename P::S* __restrict__ out, typename P::R diag,
                                                          Geom g, int nv, RowTile rt,
                                                          const typename P::R* __restrict__ clov, Epilogue epi) {
    using R = typename P::R;
    using S = typename P::S;
    constexpr int PER = RowUnits<NC, RB, P>::PER;
    constexpr int L = NC * NC;
    extern __shared__ __align__(16) u32x4 rtile[];

    const int64_t tix = logical_block();
    if (tix >= rt.ntiles) return;
    const RowPos pos = tile_row_pos(static_cast<uint32_t>(tix), rt, g);  // one row per work-group
    const uint32_t rho = row_index(pos, g);
    const uint32_t tid = threadIdx.x;
    const bool active = tid < static_cast<uint32_t>(rt.threads);
    // padding threads (block rounded up to whole wavefronts) shadow a real thread: same loads and
    // LDS writes of the same values, no global store
    const uint32_t tt = active ? tid : tid - rt.threads;
    const uint32_t j = fast_div(tt, rt.magic_nrg);  // x of this thread's site
    const int rg = static_cast<int>(tt - j * rt.nrg);
    const int x = static_cast<int>(j);
    const int64_t rowsite = static_cast<int64_t>(rho) * g.nx;
    const int64_t site = rowsite + x;
    const int ct = pos.t;
    const u32x4* src = reinterpret_cast<const u32x4*>(in);
    if constexpr (NVC > 0) nv = NVC;

    // unit k of this thread: k * threads + tt of the row copy; its padded LDS slot (sites padded to a
    // bank-conflict-free stride)
    const uint32_t PADU = row_pad(rt.units, static_cast<uint32_t>(nv) * static_cast<uint32_t>(sizeof(S)) / 4u);
    const uint32_t SU = rt.units + PADU;  // units per site of the row copy
    uint32_t slot[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint32_t u = k * static_cast<uint32_t>(rt.threads) + tt;
        slot[k] = u + fast_div(u, rt.magic_units) * PADU;
    }
    u32x4 pre[PER];
    const uint32_t row_bytes = static_cast<uint32_t>(rt.row_units) * 16u;
    auto fetch = [&](int64_t row_start) __attribute__((always_inline)) {
        const auto r = raw_buffer(src + row_start * rt.units, row_bytes);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            pre[k] = buffer_load_unit<u32x4>(r, tt * 16u, static_cast<uint32_t>(k * rt.threads) * 16u);
    };
    auto stash = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PER; ++k) rtile[slot[k]] = pre[k];
    };
    auto at = [&](uint32_t jj) __attribute__((always_inline)) {
        return reinterpret_cast<const S*>(rtile + jj * SU) + rg * RB;
    };

    // LDS after the row tile: the own links (LL), the backward links of one neighbour row (LL), the clover records
    using G = typename P::G;
    constexpr int LPER = RowLinks<NC, RB, NVC>::PER;
    const uint32_t nlink = static_cast<uint32_t>(rt.S) * L;  // links of one direction
    u32x4* const lown_u = rtile + rt.S * SU;
    const uint32_t own_units = nlink * 4u * static_cast<uint32_t>(sizeof(G)) / 16u;
    const G* lown = reinterpret_cast<const G*>(lown_u);
    u32x4* const lwin_u = lown_u + (LL == 2 ? own_units : 0u);
    G* const lwin = reinterpret_cast<G*>(lwin_u);
    u32x4* const lclov_u = lwin_u + (LL ? (nlink * static_cast<uint32_t>(sizeof(G)) + 15u) / 16u : 0u);
    auto stage = [&](u32x4* dst, const u32x4* from, uint32_t n) __attribute__((always_inline)) {
        for (uint32_t u0 = tt; u0 < n; u0 += 4u * static_cast<uint32_t>(rt.threads)) {
            u32x4 t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t u = u0 + q * static_cast<uint32_t>(rt.threads);
                if (u < n) t[q] = from[u];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t u = u0 + q * static_cast<uint32_t>(rt.threads);
                if (u < n) dst[u] = t[q];
            }
        }
    };
    G lpre[LPER];
    auto lfetch = [&](int64_t lrow, int mu) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < LPER; ++k) {
            const uint32_t u = k * static_cast<uint32_t>(rt.threads) + tt;
            if (u < nlink) {
                const uint32_t sx = u / L;
                lpre[k] = U[((lrow + sx) * 4 + mu) * L + (u - sx * L)];
            }
        }
    };
    auto lstash = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < LPER; ++k) {
            const uint32_t u = k * static_cast<uint32_t>(rt.threads) + tt;
            if (u < nlink) lwin[u] = lpre[k];
        }
    };

    cx<R> acc[RB][NC][4];
    constexpr int SF = DAG ? 1 : -1;  // forward projector 1 + SF g_mu
    // Per-thread links are loaded one direction ahead and before the next row copy: loads complete in issue
    // order, so waiting for a link never waits for the row copy still in flight.
    const int xp = x + 1 == g.nx ? 0 : x + 1;
    const int xm = x == 0 ? g.nx - 1 : x - 1;
    cx<R> lxp[NC][NC], lxm[NC][NC], lnext[NC][NC];
    fetch(rowsite);
    if constexpr (LL == 2) {
        stage(lown_u, reinterpret_cast<const u32x4*>(U + rowsite * 4 * L), own_units);
    } else if constexpr (LL == 1) {
        lfetch(rowsite, 0);
    } else {
        load_link<NC, false, P>(lxp, U + (site * 4 + 0) * L);
        load_link<NC, true, P>(lxm, U + ((rowsite + xm) * 4 + 0) * L);
    }
    if constexpr (CLOV == 2) {
        constexpr uint32_t CU = clover_reals<NC>() * sizeof(R) / 16;  // units per site
        stage(lclov_u, reinterpret_cast<const u32x4*>(clov) + rowsite * CU, static_cast<uint32_t>(rt.S) * CU);
    }
    stash();
    if constexpr (LL == 1) lstash();
    __syncthreads();
    fetch(row_neighbour_start(pos, 0, g));
    if constexpr (LL == 1) lfetch(rowsite, 1);
    auto mass_term = [&]() __attribute__((always_inline)) {
        const S* mine = at(j);
#pragma unroll
        for (int k = 0; k < RB; ++k)
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int s = 0; s < 4; ++s) acc[k][a][s] = cscale(diag, io<R, S>::ld(mine + (a * 4 + s) * nv + k));
        if constexpr (CLOV == 1) clover_add<NC, RB>(acc, mine, nv, clov + site * clover_reals<NC>());
        if constexpr (CLOV == 2)
            clover_add<NC, RB>(acc, mine, nv, reinterpret_cast<const R*>(lclov_u) + x * clover_reals<NC>());
    };
    // with a clover field the site's clover block is applied from the own row before the x links are
    // taken into registers
    if constexpr (CLOV)
        if (active) mass_term();
    if constexpr (LL == 2) {
        load_link<NC, false, P>(lxp, lown + x * 4 * L);
        load_link<NC, true, P>(lxm, lown + xm * 4 * L);
    } else if constexpr (LL == 1) {
        load_link<NC, false, P>(lxp, lwin + x * L);
        load_link<NC, true, P>(lxm, lwin + xm * L);
    } else {
        load_link<NC, false, P>(lnext, U + (site * 4 + 1) * L);
    }
    // each transported half spinor enters the sum with -1/2 (+1/2 across the antiperiodic t
    // boundary) as the multiplier of the rebuild's multiply-adds
    if (active) {
        if constexpr (!CLOV) mass_term();
        hop_with<NC, RB, 0, SF, P, NVC>(acc, lxp, at(xp), nv, R(-0.5));
        hop_with<NC, RB, 0, -SF, P, NVC>(acc, lxm, at(xm), nv, R(-0.5));
    }
    auto step = [&](auto mu_c, auto back_c) __attribute__((always_inline)) {
        constexpr int MU = decltype(mu_c)::value;
        constexpr bool BACK = decltype(back_c)::value;
        constexpr int DIR = 2 * (MU - 1) + (BACK ? 1 : 0);
        cx<R> lcur[NC][NC];
        if constexpr (LL == 0) {
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) lcur[a][b] = lnext[a][b];
        }
        __syncthreads();
        stash();
        if constexpr (LL == 1 || (LL == 2 && BACK)) lstash();
        __syncthreads();
        if constexpr (DIR < 5) {
            constexpr int ND = DIR + 1;
            constexpr int NMU = ND / 2 + 1;
            const int64_t nrow = row_neighbour_start(pos, ND, g);
            fetch(nrow);
            if constexpr (LL != 0) {
                if constexpr (ND % 2 == 1)
                    lfetch(nrow, NMU);
                else if constexpr (LL == 1)
                    lfetch(rowsite, NMU);
            } else if constexpr (ND % 2 == 0) {
                load_link<NC, false, P>(lnext, U + (site * 4 + NMU) * L);
            } else {
                load_link<NC, true, P>(lnext, U + ((nrow + x) * 4 + NMU) * L);
            }
        }
        if constexpr (LL != 0)
            load_link<NC, BACK, P>(lcur, BACK || LL == 1 ? lwin + x * L : lown + (x * 4 + MU) * L);
        if (active) {
            const bool wrap = MU == 3 && g.apbc && ct == (BACK ? 0 : g.nt - 1);  // fermion sign
            hop_with<NC, RB, MU, (BACK ? -SF : SF), P, NVC>(acc, lcur, at(j), nv,
                                                                        wrap ? R(0.5) : R(-0.5));
        }
    };
    step(std::integral_constant<int, 1>{}, std::false_type{});
    step(std::integral_constant<int, 1>{}, std::true_type{});
    step(std::integral_constant<int, 2>{}, std::false_type{});
    step(std::integral_constant<int, 2>{}, std::true_type{});
    step(std::integral_constant<int, 3>{}, std::false_type{});
    step(std::integral_constant<int, 3>{}, std::true_type{});
    // the thread's outputs as [RB][NC * 4] (element a * 4 + s at offset (a * 4 + s) * nv)
    const auto& flat = reinterpret_cast<const cx<R>(&)[RB][NC * 4]>(acc);
    if (epi.mode == 2) {  // r -= alpha (D^+ t): the output itself is not written
        row_epilogue<RB, NC * 4, R, S>(epi, flat, active, site * (NC * 4 * nv) + rg * RB, nv, rg * RB, j, rt.S, tix,
                                       reinterpret_cast<double*>(rtile));
        return;
    }
    __syncthreads();
    if (active) {
        S* o = const_cast<S*>(at(j));
#pragma unroll
        for (int k = 0; k < RB; ++k)
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    io<R, S>::st(o + (a * 4 + s) * nv + k, acc[k][a][s]);
    }
    __syncthreads();
    u32x4* dst = reinterpret_cast<u32x4*>(out) + rowsite * rt.units;
    const uint32_t total = static_cast<uint32_t>(rt.S) * rt.units;
    // streaming stores: the output is not read again by this launch, so its lines should not
    // displace input rows that neighbouring work-groups still read from L2
    for (uint32_t u = tid; u < total; u += blockDim.x)
        __builtin_nontemporal_store(rtile[u + fast_div(u, rt.magic_units) * PADU], dst + u);
    if (epi.mode == 1)
        row_epilogue<RB, NC * 4, R, S>(epi, flat, active, 0, nv, rg * RB, j, rt.S, tix,
                                       reinterpret_cast<double*>(rtile));
}

template <int NC, int RB, class P>
bool launch_rows(const StencilArgs& a, hipStream_t st) {
    using S = typename P::S;
    const size_t block_bytes = static_cast<size_t>(NC) * 4 * a.nv * sizeof(S);
    if (block_bytes % 16 != 0 || !tile_aligned(a)) return false;
    const int units = static_cast<int>(block_bytes / 16);
    const int nrg = a.nv / RB;
    const int64_t rows = a.g.vol / a.g.nx;
    const uint32_t pad = row_pad(units, static_cast<uint32_t>(a.nv * sizeof(S) / 4));
    const int Rr = choose_tile_rows(a.variant, rows, a.g.nx, units, nrg, pad);
    if (Rr == 0) return false;
    RowTile rt;
    rt.R = Rr;
    rt.S = Rr * a.g.nx;
    rt.nrg = nrg;
    rt.units = units;
    rt.row_units = a.g.nx * units;
    rt.threads = rt.S * nrg;
    rt.ntiles = rows / Rr;
    rt.nseg = 1;
    rt.magic_nrg = div_magic(nrg);
    rt.magic_nx = div_magic(a.g.nx);
    rt.magic_units = div_magic(units);
    rt.magic_row_units = div_magic(rt.row_units);
    if (!row_order(4, a.g, rt)) return false;
    const int block = (rt.threads + 63) / 64 * 64;
    size_t lds = row_tile_lds(rt.S, units, pad);
    // What is staged in LDS after the row tile, with N_c^2 links of a site moved by its threads, at most LPER each, and up to
    // all of the LDS, beyond the row tile's own cap (one work-group per CU instead of two costs nothing: FP32, N_v = 24 at
    // 32 x 16^3 274 against 284 us).
    // FP32, BF16: the links from 8 right-hand sides on, or where links and vectors leave the 256 MB of the Infinity Cache;
    // below that a thread moves two or three entries and waits for them (BF16, N_v = 4: 31.7 against 28.4 us at 32 x 16^3,
    // but 215 against 250 at 32^4).  With them the clover records from 10 on, when they are read by that many threads
    // (FP32 at 16^3 x 32: N_v = 4 55.2 against 48.6 us, 10 97.5 and 98.4, 24 253 and 353); without the links they cost
    // (BF16, N_v = 12: 137 against 108).
    // FP64: the links at N_v = 12 (with N_v known at run time the entries in flight spill: N_v = 4 at 24^3 x 48 0.69 against
    // 0.55 ms), the clover records from 5 right-hand sides on where as many work-groups still share a CU (N_v = 8 at
    // 16^3 x 32 200 against 218 us, N_v = 4 at 64 x 8 x 16^2 135 against 122).
    constexpr bool kFP64 = sizeof(typename P::R) == 8;
    const size_t room = max_lds_per_block();
    const size_t nlink = static_cast<size_t>(rt.S) * NC * NC * sizeof(typename P::G);
    const size_t lds_ll = (kFP64 ? 0 : 4 * nlink) + (nlink + 15) / 16 * 16;
    const size_t lds_cl = static_cast<size_t>(rt.S) * clover_reals<NC>() * sizeof(typename P::R);
    const double data = static_cast<double>(a.g.vol) * (4.0 * NC * NC * sizeof(typename P::G) + 2.0 * block_bytes);
    const bool ll = NC > 1 && NC * NC <= RowLinks<NC, RB, 0>::PER * nrg && lds + lds_ll <= room &&
                    (kFP64 ? a.nv == 12 && RB == 1 : a.nv >= (a.clover ? 10 : 8) || data > 256e6);
    if (ll) lds += lds_ll;
    bool stage_cl = a.clover && reinterpret_cast<uintptr_t>(a.clover) % 16 == 0 && lds + lds_cl <= room;
    if constexpr (kFP64) {
        constexpr size_t kPerSimd = NC == 1 ? (RB == 1 ? 6 : 4) : (NC == 2 && RB == 1 ? 3 : 2);  // wavefronts, by registers
        const size_t by_registers = std::max<size_t>(1, 4 * kPerSimd / (block / 64));
        stage_cl = stage_cl && a.nv >= 5 &&
                   std::min(room / (lds + lds_cl), by_registers) >= std::min(room / lds, by_registers);
        // N_c = 4 spills 456 registers with the record read by every thread: 159 us at 128 x 8^3, N_v = 2, direct 67
        if (NC == 4 && a.clover && !stage_cl) return false;
    } else {
        stage_cl = stage_cl && ll && a.nv >= 10;
    }
    if (stage_cl) lds += lds_cl;
    const dim3 grid(static_cast<unsigned>(grid_blocks_x8(rt.ntiles, 1)));
    using R = typename P::R;
    const R diag = static_cast<R>(4.0 + a.mass);
    auto U = static_cast<const typename P::G*>(a.gauge);
    auto in = static_cast<const S*>(a.in);
    auto out = static_cast<S*>(a.out);
    auto clov = static_cast<const R*>(a.clover);
    bool ok = true;
    auto go = [&](auto kern) {
        if (!allow_lds(reinterpret_cast<const void*>(kern), lds)) {
            ok = false;
            return;
        }
        hipLaunchKernelGGL(kern, grid, dim3(block), lds, st, U, in, out, diag, a.g, a.nv, rt, clov, a.epi);
    };
    // the clover term is a separate instantiation: its registers would otherwise lower the occupancy
    // of the plain kernel
    auto pick = [&](auto clov_c, auto links_c) {
        constexpr int CL = decltype(clov_c)::value, LL = decltype(links_c)::value;
        auto with = [&](auto nvc) {
            constexpr int NVC = decltype(nvc)::value;
            if (a.dagger)
                go(wilson_rows_kernel<NC, RB, true, P, NVC, LL, CL>);
            else
                go(wilson_rows_kernel<NC, RB, false, P, NVC, LL, CL>);
        };
        if constexpr (RB == 1 && LL != 0) {
            if (a.nv == 12) {  // the RHS stride as a compile-time constant
                with(std::integral_constant<int, 12>{});
                return;
            }
        }
        if constexpr (!kFP64 || LL == 0) with(std::integral_constant<int, 0>{});
    };
    const std::integral_constant<int, 0> none;
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    const std::integral_constant<int, kFP64 ? 1 : 2> links;
    if (!clov)
        ll ? pick(none, links) : pick(none, none);
    else if (!stage_cl)
        ll ? pick(one, links) : pick(one, none);
    else if (ll)
        pick(two, links);
    else if constexpr (kFP64)
        pick(two, none);
    return ok;
}

// false: an epilogue was asked for and only the direct kernel could take this shape (nothing launched)
template <int NC, int RB, class P>
bool launch_rb(const StencilArgs& a, hipStream_t st) {
    using R = typename P::R;
    if (a.variant == 4 && launch_rows<NC, RB, P>(a, st)) return true;
    if (a.epi.mode != 0) return false;
    // direct loads (selected, or the row tile does not fit this shape)
    const int64_t threads = a.g.vol * (a.nv / RB);
    const int block = direct_block(threads);
    const dim3 grid(static_cast<unsigned>(grid_blocks_x8(threads, block)));
    const R diag = static_cast<R>(4.0 + a.mass);
    auto U = static_cast<const typename P::G*>(a.gauge);
    auto in = static_cast<const typename P::S*>(a.in);
    auto out = static_cast<typename P::S*>(a.out);
    auto clov = static_cast<const R*>(a.clover);
    const SiteOrder ord = make_site_order(a.g);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(block), 0, st, U, in, out, diag, a.g, a.nv, ord, clov);
    };
    if (a.nv == RB) {
        if (a.dagger)
            go(wilson_kernel<NC, RB, true, P, RB>);
        else
            go(wilson_kernel<NC, RB, false, P, RB>);
    } else {
        if (a.dagger)
            go(wilson_kernel<NC, RB, true, P, 0>);
        else
            go(wilson_kernel<NC, RB, false, P, 0>);
    }
    return true;
}

template <int NC, class P>
bool launch_nc(const StencilArgs& a, hipStream_t st) {
    return a.rb == 2 ? launch_rb<NC, 2, P>(a, st) : launch_rb<NC, 1, P>(a, st);
}

template <class P>
int launch_prec(const StencilArgs& a, hipStream_t st) {
    bool ok;
    switch (a.nc) {
        case 1: ok = launch_nc<1, P>(a, st); break;
        case 2: ok = launch_nc<2, P>(a, st); break;
        case 3: ok = launch_nc<3, P>(a, st); break;
        case 4: ok = launch_nc<4, P>(a, st); break;
        default: return DIRAC_EUNSUPPORTED;
    }
    return ok ? DIRAC_OK : kNoEpilogue;
}

}  // namespace

}  // namespace dirac
