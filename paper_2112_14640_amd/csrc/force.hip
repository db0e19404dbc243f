// Link gradients of Dirac bilinears and their su(Nc) projection (FP64).
//
// Gradient convention: for real L, g = dL/dRe U + i dL/dIm U.  For L = Re sum_rhs psi^+ D chi:
//   Wilson (from Eq. app_wils; U_mu(n) appears in the hops n -> n+mu and n+mu -> n):
//     g_mu(n) = -1/2 b sum_{s,rhs} [((1 - g_mu) psi(n))_s chi_s(n+mu)^+ + chi_s(n) ((1 + g_mu) psi(n+mu))_s^+]
//   Staggered (Eq. def_stag):
//     g_mu(n) = 1/2 eta_mu(n) b sum_rhs [psi(n) chi(n+mu)^+ - chi(n) psi(n+mu)^+]
//   Brillouin (Eq. app_bril), for each stored link W_d(n) (d one of the 40 stored directions), which
//   enters the hop n -> n+d as W_d(n) and the hop n+d -> n as W_{-d}(n+d) = W_d(n)^+:
//     g_d(n) = b sum_{s,rhs} [psi(n) (S_d chi(n+d))^+ + (psi(n+d) (S_{-d} chi(n))^+)^+]  (colour outer
//     products), with S_d = rho_|d| sum_mu d_mu g_mu - lambda_|d|/2 the spin factor of displacement d.
// b is the fermion boundary sign of the hop n -> n+mu (n -> n+d).  A kernel accumulates coeff * g into the output
// (each entry written by exactly one thread).
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace dirac {

namespace {

// Lanes of a gradient kernel: a site has one lane per spin component that the kernel keeps apart (Wilson: two half
// spinor rows, Brillouin: four spins, staggered: none, but directions) and RL right-hand sides r = lane, lane + RL, ...  A vector is
// [site][colour][spin][rhs], so the lanes of a site read one contiguous run, whole lines for N_v = 4, and a line is
// not asked for again once it has left the cache.  RL is 4 (more would leave lanes idle for a few right-hand sides),
// less for fewer than 3 right-hand sides.  The lanes' sums are added inside a row of 16 lanes by DPP moves and lane k
// of a site stores the entries k, k + lanes, ... of the link.  Bound by load latency at two waves per SIMD.  One thread per link,
// whose lanes were whole sites apart, took 1.84 ms for the Wilson gradient at 24^3 x 48 (N_c = 3, N_v = 4) and 0.23 ms
// for the Brillouin one at 8^3 x 16; four lanes (right-hand sides) per site 1.22 and 0.17 ms; these 0.73 and 0.10 ms.
constexpr int kForceThreads = 256;
inline int force_lanes(int nv) { return nv >= 3 ? 4 : nv; }

// v + the value of the lane a DPP pattern names (both halves of a double)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}
// Sum over LANES (1, 2, 4, 8, 16) neighbouring lanes, in every lane: quad permutations for 1 and 2; with the quads'
// sums equal, mirroring 8 and 16 lanes swaps quads and halves.
template <int LANES>
__device__ __forceinline__ double lane_sum(double v) {
    if constexpr (LANES >= 2) v = dpp_add<0xB1>(v);
    if constexpr (LANES >= 4) v = dpp_add<0x4E>(v);
    if constexpr (LANES >= 8) v = dpp_add<0x141>(v);
    if constexpr (LANES >= 16) v = dpp_add<0x140>(v);
    return v;
}

template <int NC>
struct Grad {
    cx<double> e[NC][NC];
};

template <int NC>
__device__ __forceinline__ Grad<NC> grad_zero() {
    Grad<NC> g;
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) g.e[a][b] = {0.0, 0.0};
    return g;
}

// The entries of a link that lane `lane` of a site adds to: lane, lane + LANES, ...  They are read before the sum is
// formed (read one by one behind it, the nine reads of a link were a chain of nine memory latencies: 1.36 ms).
template <int NC, int LANES>
struct GradOut {
    static constexpr int K = (NC * NC + LANES - 1) / LANES;
    double2 w[K];
    __device__ __forceinline__ void load(const double2* __restrict__ o, int lane) {
#pragma unroll
        for (int k = 0; k < K; ++k) w[k] = o[min(k * LANES + lane, NC * NC - 1)];
    }
    // o += f * (sum of acc over the lanes of a site).  Every lane of the site takes part; `store`: a real site.
    __device__ __forceinline__ void add(const Grad<NC>& acc, double f, int lane, bool store, double2* __restrict__ o) {
        cx<double> mine[K];
#pragma unroll
        for (int e = 0; e < NC * NC; ++e) {
            const cx<double> v{lane_sum<LANES>(acc.e[e / NC][e % NC].re), lane_sum<LANES>(acc.e[e / NC][e % NC].im)};
            if (e % LANES == 0 || lane == e % LANES) mine[e / LANES] = v;
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (store && k * LANES + lane < NC * NC)
                o[k * LANES + lane] = make_double2(w[k].x + f * mine[k].re, w[k].y + f * mine[k].im);
    }
};

// Site and lane of a thread; sites past the volume shadow the last one without storing.  Sites are taken brick by
// brick with t next: the sites in flight on an XCD touch more bytes than its L2 holds, and in memory order the z and t
// neighbours had left it (5.4 GB fetched for 1.4 GB of operands at 24^3 x 48, 0.98 ms; in bricks, and with the rows at n kept in registers, 2.1 GB, 0.73 ms).
struct ForceLane {
    int lane;
    int64_t site;
    bool store;
};
template <int LANES>
__device__ __forceinline__ ForceLane force_lane(int64_t block, const SiteOrder& order, const Geom& g) {
    ForceLane f;
    f.lane = static_cast<int>(threadIdx.x) % LANES;
    f.site = block * (kForceThreads / LANES) + static_cast<int>(threadIdx.x) / LANES;
    f.store = f.site < g.vol;
    f.site = ordered_site(f.store ? f.site : g.vol - 1, order, g);
    return f;
}

// Site offset of one step forwards along mu, and whether it wraps
__device__ __forceinline__ int64_t step_forward(const Coord& c, int mu, const Geom& g, bool& wraps) {
    const int x = mu == 0 ? c.x : (mu == 1 ? c.y : (mu == 2 ? c.z : c.t));
    const int n = mu == 0 ? g.nx : (mu == 1 ? g.ny : (mu == 2 ? g.nz : g.nt));
    const int64_t stride = mu == 0 ? 1
                                   : (mu == 1 ? g.nx
                                              : (mu == 2 ? static_cast<int64_t>(g.nx) * g.ny
                                                         : static_cast<int64_t>(g.nx) * g.ny * g.nz));
    wraps = x == n - 1;
    return wraps ? (1 - n) * stride : stride;
}

// g_d(n) for the kForceDirs stored directions of a group (blocks of the groups of one tile are neighbours), see the
// file header.  The spin factor is hermitian, so it is applied to the spinors at n alone:
//   g_d(n) = b sum_{s,rhs} [(S_d psi(n))_a conj(chi(n+d))_b + (S_{-d} chi(n))_a conj(psi(n+d))_b],
// and in the chiral basis row s of it is (S_d u)_s = -l u_s + (e_2 q_2 + i e_1 q_1) u_{3-s} + (q_4 + i e_3 q_3) u_{s^2}
// with q_mu = rho_k d_mu, l = lambda_k / 2 and signs e(s): a lane (s, r) needs three spin components at n and its
// own at n + d.  Those at n stay in registers for the group when one lane has one right-hand side.
constexpr int kForceDirs = 5;  // directions per group: the 8 groups fill the chip at 8^3 x 16 already
template <int NC, int RL>
__global__ __launch_bounds__(kForceThreads) void brillouin_force_kernel(const double2* __restrict__ psi,
                                                                        const double2* __restrict__ chi,
                                                                        double2* __restrict__ gout, double coeff,
                                                                        Geom g, int nv, SiteOrder order, int64_t first) {
    constexpr int LANES = 4 * RL;
    const int64_t block = first + logical_block();
    const int group = static_cast<int>(block % (40 / kForceDirs));
    const int64_t tile = block / (40 / kForceDirs);
    if (tile * (kForceThreads / LANES) >= g.vol) return;
    const ForceLane f = force_lane<LANES>(tile, order, g);
    const int s = f.lane / RL, r0 = f.lane % RL;
    const Coord c = site_coord(f.site, g);
    const int64_t vs = static_cast<int64_t>(NC) * 4 * nv;
    const double rho_k[5] = {0.0, 64.0 / 432.0, 16.0 / 432.0, 4.0 / 432.0, 1.0 / 432.0};
    const double lh_k[5] = {-120.0 / 64.0, 4.0 / 64.0, 2.0 / 64.0, 1.0 / 64.0, 0.5 / 64.0};
    const double e1 = s < 2 ? -1.0 : 1.0, e2 = (s == 0 || s == 3) ? -1.0 : 1.0, e3 = e2;
    cx<double> pn[NC][3], cn[NC][3];  // psi(n), chi(n): spins s, 3 - s, s ^ 2
#pragma unroll 1
    for (int q = 0; q < kForceDirs; ++q) {
        const int dir = group * kForceDirs + q;
        const int dx = dir % 3 - 1, dy = (dir / 3) % 3 - 1, dz = (dir / 9) % 3 - 1, dt = dir / 27 - 1;
        const int k = (dx != 0) + (dy != 0) + (dz != 0) + (dt != 0);
        const double rho = rho_k[k], lh = lh_k[k];
        const int tt = c.t + dt;
        const int64_t nb = site_index(wrap(c.x + dx, g.nx), wrap(c.y + dy, g.ny), wrap(c.z + dz, g.nz), wrap(tt, g.nt), g);
        const cx<double> al{e2 * rho * dy, e1 * rho * dx}, be{rho * dt, e3 * rho * dz};
        const cx<double> mal{-al.re, -al.im}, mbe{-be.re, -be.im};
        GradOut<NC, LANES> out;
        out.load(gout + (f.site * 40 + dir) * NC * NC, f.lane);
        Grad<NC> acc = grad_zero<NC>();
        for (int r = r0; r < nv; r += RL) {
            if (q == 0 || nv > RL) {
#pragma unroll
                for (int a = 0; a < NC; ++a)
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        const int64_t at = f.site * vs + (a * 4 + (t == 0 ? s : (t == 1 ? 3 - s : s ^ 2))) * nv + r;
                        pn[a][t] = io<double, double2>::ld(psi + at);
                        cn[a][t] = io<double, double2>::ld(chi + at);
                    }
            }
            cx<double> pb[NC], cb[NC];
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                cb[b] = io<double, double2>::ld(chi + nb * vs + (b * 4 + s) * nv + r);
                pb[b] = io<double, double2>::ld(psi + nb * vs + (b * 4 + s) * nv + r);
            }
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                cx<double> sp = cscale(-lh, pn[a][0]), sc = cscale(-lh, cn[a][0]);
                cfma(sp, al, pn[a][1]);
                cfma(sp, be, pn[a][2]);
                cfma(sc, mal, cn[a][1]);
                cfma(sc, mbe, cn[a][2]);
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    cfma_conj(acc.e[a][b], cb[b], sp);
                    cfma_conj(acc.e[a][b], pb[b], sc);
                }
            }
        }
        const double bsign = (g.apbc && (tt < 0 || tt >= g.nt)) ? -1.0 : 1.0;  // the same for the hop back
        out.add(acc, bsign * coeff, f.lane, f.store, gout + (f.site * 40 + dir) * NC * NC);
    }
}

// One direction of the Wilson gradient.  P = 1 -+ g_mu is hermitian with P^2 = 2 P and its lower rows are the upper
// ones times a phase, so sum_s (P psi)_s conj(chi)_s is the sum over the two upper rows of (P psi)_s conj((P chi)_s):
// half the products of the four rows.  A lane (i, r) takes row i: (P u)_i = u_i + SIG w u_j with
//   mu = 0: w = -i, j = 3 - i;  mu = 1: w = -1, +1, j = 3 - i;  mu = 2: w = -i, +i, j = 2 + i;  mu = 3: w = 1, j = 2 + i.
// The rows i, 3 - i and 2 + i at n serve the four directions and stay in registers when one lane has one right-hand
// side: read again per direction, they had left the caches in between (5.2 GB fetched instead of 2.1, 0.96 ms).
template <int NC>
struct OwnRows {
    cx<double> p[NC][3], c[NC][3];
    __device__ __forceinline__ void load(const double2* __restrict__ psi, const double2* __restrict__ chi, int64_t at,
                                         int nv, int i) {
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int64_t e = at + (a * 4 + (t == 0 ? i : (t == 1 ? 3 - i : 2 + i))) * nv;
                p[a][t] = io<double, double2>::ld(psi + e);
                c[a][t] = io<double, double2>::ld(chi + e);
            }
    }
};

template <int NC, int RL, int MU>
__device__ __forceinline__ void wilson_force_mu(const double2* __restrict__ psi, const double2* __restrict__ chi,
                                                double2* __restrict__ gout, double coeff, const Geom& g, int nv,
                                                const ForceLane& f, const Coord& c, OwnRows<NC>& own) {
    bool wraps;
    const int64_t fwd = f.site + step_forward(c, MU, g, wraps);
    const int64_t vs = static_cast<int64_t>(NC) * 4 * nv;
    const int i = f.lane / RL;
    const int j = MU < 2 ? 3 - i : 2 + i;
    const double w = MU == 0 ? -1.0 : (MU == 1 ? (i ? 1.0 : -1.0) : (MU == 2 ? (i ? 1.0 : -1.0) : 1.0));
    auto half = [&](double t, cx<double> u, cx<double> x) __attribute__((always_inline)) {  // u + t w x
        if constexpr (MU == 0 || MU == 2)  // w is imaginary
            return cx<double>{fma(-t * w, x.im, u.re), fma(t * w, x.re, u.im)};
        else
            return cx<double>{fma(t * w, x.re, u.re), fma(t * w, x.im, u.im)};
    };
    GradOut<NC, 2 * RL> out;
    out.load(gout + (f.site * 4 + MU) * NC * NC, f.lane);
    Grad<NC> acc = grad_zero<NC>();
    for (int r = f.lane % RL; r < nv; r += RL) {
        if (MU == 0 || nv > RL) own.load(psi, chi, f.site * vs + r, nv, i);
        // (1 - g) chi(n+mu) and (1 + g) psi(n+mu), with (1 - g) psi(n) and (1 + g) chi(n)
        cx<double> cf[NC], pf[NC];
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            const int64_t at = fwd * vs + b * 4 * nv + r;
            cf[b] = half(-1.0, io<double, double2>::ld(chi + at + i * nv), io<double, double2>::ld(chi + at + j * nv));
            pf[b] = half(1.0, io<double, double2>::ld(psi + at + i * nv), io<double, double2>::ld(psi + at + j * nv));
        }
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            const cx<double> pn = half(-1.0, own.p[a][0], own.p[a][MU < 2 ? 1 : 2]);
            const cx<double> cn = half(1.0, own.c[a][0], own.c[a][MU < 2 ? 1 : 2]);
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                cfma_conj(acc.e[a][b], cf[b], pn);
                cfma_conj(acc.e[a][b], pf[b], cn);
            }
        }
    }
    const double b = (MU == 3 && g.apbc && wraps) ? -1.0 : 1.0;
    out.add(acc, -0.5 * b * coeff, f.lane, f.store, gout + (f.site * 4 + MU) * NC * NC);
}

template <int NC, int RL>
__global__ __launch_bounds__(kForceThreads) void wilson_force_kernel(const double2* __restrict__ psi,
                                                                     const double2* __restrict__ chi,
                                                                     double2* __restrict__ gout, double coeff, Geom g,
                                                                     int nv, SiteOrder order, int64_t first) {
    const int64_t block = first + logical_block();
    if (block * (kForceThreads / (2 * RL)) >= g.vol) return;
    const ForceLane f = force_lane<2 * RL>(block, order, g);
    const Coord c = site_coord(f.site, g);
    OwnRows<NC> own;
    wilson_force_mu<NC, RL, 0>(psi, chi, gout, coeff, g, nv, f, c, own);
    wilson_force_mu<NC, RL, 1>(psi, chi, gout, coeff, g, nv, f, c, own);
    wilson_force_mu<NC, RL, 2>(psi, chi, gout, coeff, g, nv, f, c, own);
    wilson_force_mu<NC, RL, 3>(psi, chi, gout, coeff, g, nv, f, c, own);
}

// A lane takes one or two of a site's four directions, and a site has 4 / DIRS RL lanes.  All four in one lane are too long a
// chain of loads: at 24^4 with N_c = 3 126 us for N_v = 1, 168 for 3, 510 for 12; with one each 79, 125 and 296.  Two where 16
// lanes per site do not read whole lines (24^4, N_v = 8: N_c = 1 41 against 47 us, N_c = 4 309 and 314; 16^3 x 32 88 and 112).
template <int NC, int RL>
constexpr int kStaggeredDirs = RL < 4 || NC == 3 ? 1 : 2;
template <int NC, int RL>
__global__ __launch_bounds__(kForceThreads) void staggered_force_kernel(const double2* __restrict__ psi,
                                                                        const double2* __restrict__ chi,
                                                                        double2* __restrict__ gout, double coeff,
                                                                        Geom g, int nv, SiteOrder order, int64_t first) {
    constexpr int DIRS = kStaggeredDirs<NC, RL>, LANES = 4 / DIRS * RL;  // lanes of a site: direction, right-hand side
    const int64_t block = first + logical_block();
    if (block * (kForceThreads / LANES) >= g.vol) return;
    ForceLane f = force_lane<LANES>(block, order, g);
    const int mu0 = f.lane / RL * DIRS;
    f.lane %= RL;
    const Coord c = site_coord(f.site, g);
    const int64_t vs = static_cast<int64_t>(NC) * nv;
#pragma unroll 1
    for (int mu = mu0; mu < mu0 + DIRS; ++mu) {
        bool wraps;
        const int64_t fwd = f.site + step_forward(c, mu, g, wraps);
        GradOut<NC, RL> out;
        out.load(gout + (f.site * 4 + mu) * NC * NC, f.lane);
        Grad<NC> acc = grad_zero<NC>();
        for (int r = f.lane; r < nv; r += RL) {
            cx<double> p0[NC], p1[NC], c0[NC], c1[NC];
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                p0[a] = io<double, double2>::ld(psi + f.site * vs + a * nv + r);
                p1[a] = cscale(-1.0, io<double, double2>::ld(psi + fwd * vs + a * nv + r));
                c0[a] = io<double, double2>::ld(chi + f.site * vs + a * nv + r);
                c1[a] = io<double, double2>::ld(chi + fwd * vs + a * nv + r);
            }
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    cfma_conj(acc.e[a][b], c1[b], p0[a]);  // psi(n)_a conj(chi(n+mu))_b
                    cfma_conj(acc.e[a][b], p1[b], c0[a]);  // -chi(n)_a conj(psi(n+mu))_b
                }
        }
        const double b = (mu == 3 && g.apbc && wraps) ? -1.0 : 1.0;
        const int par = mu == 0 ? 0 : (mu == 1 ? (c.x & 1) : (mu == 2 ? ((c.x + c.y) & 1) : ((c.x + c.y + c.z) & 1)));
        out.add(acc, 0.5 * (par ? -b : b) * coeff, f.lane, f.store, gout + (f.site * 4 + mu) * NC * NC);
    }
}

// F = (i/2)(U g^+ - g U^+) - tr/Nc
template <int NC>
__global__ __launch_bounds__(256) void project_kernel(const double2* __restrict__ U, const double2* g,
                                                       double2* F, int64_t nlinks) {
    const int64_t l = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (l >= nlinks) return;
    cx<double> u[NC][NC], gg[NC][NC], m[NC][NC];
    for (int a = 0; a < NC; ++a)
        for (int b = 0; b < NC; ++b) {
            u[a][b] = io<double, double2>::ld(U + l * NC * NC + a * NC + b);
            gg[a][b] = io<double, double2>::ld(g + l * NC * NC + a * NC + b);
        }
    // M = U g^+ ; F = (i/2)(M - M^+)
    for (int a = 0; a < NC; ++a)
        for (int b = 0; b < NC; ++b) {
            cx<double> s{0.0, 0.0};
            for (int e = 0; e < NC; ++e) cfma_conj(s, gg[b][e], u[a][e]);  // u[a][e] conj(g[b][e])
            m[a][b] = s;
        }
    cx<double> tr{0.0, 0.0};
    cx<double> f[NC][NC];
    for (int a = 0; a < NC; ++a)
        for (int b = 0; b < NC; ++b) {
            cx<double> d = csub(m[a][b], cconj(m[b][a]));
            f[a][b] = cscale(0.5, cmuli(d));
        }
    for (int a = 0; a < NC; ++a) tr = cadd(tr, f[a][a]);
    tr = cscale(1.0 / NC, tr);
    for (int a = 0; a < NC; ++a) f[a][a] = csub(f[a][a], tr);
    for (int a = 0; a < NC; ++a)
        for (int b = 0; b < NC; ++b) io<double, double2>::st(F + l * NC * NC + a * NC + b, f[a][b]);
}

template <int NC, int RL>
void launch_force_rl(dirac_op op, int nv, const Geom& g, const void* psi, const void* chi, void* gout, double coeff,
                     hipStream_t st) {
    const int lanes = RL * (op == DIRAC_BRILLOUIN ? 4 : (op == DIRAC_WILSON ? 2 : 4 / kStaggeredDirs<NC, RL>));  // of a site
    const int64_t tiles = (g.vol + kForceThreads / lanes - 1) / (kForceThreads / lanes);
    const int64_t blocks = op == DIRAC_BRILLOUIN ? tiles * (40 / kForceDirs) : tiles;
    auto p = static_cast<const double2*>(psi);
    auto c = static_cast<const double2*>(chi);
    auto o = static_cast<double2*>(gout);
    const SiteOrder order = make_site_order(g);
    launch_slices(blocks, kForceThreads, [&](int64_t first, unsigned grid) {
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(grid), dim3(kForceThreads), 0, st, p, c, o, coeff, g, nv, order, first);
        };
        if (op == DIRAC_BRILLOUIN)
            go(brillouin_force_kernel<NC, RL>);
        else if (op == DIRAC_WILSON)
            go(wilson_force_kernel<NC, RL>);
        else
            go(staggered_force_kernel<NC, RL>);
    });
}

template <int NC>
int launch_force_nc(dirac_op op, int nv, const Geom& g, const void* psi, const void* chi, void* gout, double coeff,
                    hipStream_t st) {
    // N_c = 1, staggered: a vector is a run of N_v elements, and one lane loads it whole (24^4, N_v = 2: 16 against 25 us)
    switch (NC == 1 && op == DIRAC_STAGGERED && nv <= 3 ? 1 : force_lanes(nv)) {
        case 1: launch_force_rl<NC, 1>(op, nv, g, psi, chi, gout, coeff, st); break;
        case 2: launch_force_rl<NC, 2>(op, nv, g, psi, chi, gout, coeff, st); break;
        default: launch_force_rl<NC, 4>(op, nv, g, psi, chi, gout, coeff, st); break;
    }
    return DIRAC_OK;
}

}  // namespace

int launch_force(dirac_op op, int nc, int nv, const Geom& g, const void* /*U*/, const void* psi, const void* chi,
                 void* gout, double coeff, hipStream_t st) {
    switch (nc) {
        case 1: return launch_force_nc<1>(op, nv, g, psi, chi, gout, coeff, st);
        case 2: return launch_force_nc<2>(op, nv, g, psi, chi, gout, coeff, st);
        case 3: return launch_force_nc<3>(op, nv, g, psi, chi, gout, coeff, st);
        case 4: return launch_force_nc<4>(op, nv, g, psi, chi, gout, coeff, st);
    }
    return DIRAC_EUNSUPPORTED;
}

int launch_project_su(int nc, int64_t nlinks, const void* U, const void* g, void* F, hipStream_t st) {
    const int block = 256;
    const dim3 grid(static_cast<unsigned>((nlinks + block - 1) / block));
    auto u = static_cast<const double2*>(U);
    auto gg = static_cast<const double2*>(g);
    auto f = static_cast<double2*>(F);
    switch (nc) {
        case 1: hipLaunchKernelGGL((project_kernel<1>), grid, dim3(block), 0, st, u, gg, f, nlinks); break;
        case 2: hipLaunchKernelGGL((project_kernel<2>), grid, dim3(block), 0, st, u, gg, f, nlinks); break;
        case 3: hipLaunchKernelGGL((project_kernel<3>), grid, dim3(block), 0, st, u, gg, f, nlinks); break;
        case 4: hipLaunchKernelGGL((project_kernel<4>), grid, dim3(block), 0, st, u, gg, f, nlinks); break;
        default: return DIRAC_EUNSUPPORTED;
    }
    return DIRAC_OK;
}

}  // namespace dirac
