// Brillouin operator (Sec. 6): hypercube links W and the 81-point apply.
//
// Directions d in {-1,0,1}^4 are numbered dir = 27(d_t+1) + 9(d_z+1) + 3(d_y+1) + (d_x+1);
// dir = 40 is the centre.  The 40 directions dir < 40 are stored; W_d(n) for dir > 40 is
// W_{-d}(n+d)^+ (Tab. off-axis), read from the neighbour's direction 80 - dir.
//
// Links: W_d(n) is the plain average over the |d|! orderings of the unit steps of d of the
// ordered products of V along each path (a step -mu from x uses V_mu(x-mu)^+).
//
// Apply, with k = |d| (non-zero components), rho = (64,16,4,1)/432, lambda = (-240,8,4,2,1)/64:
//   (D_B u)(n) = (m - lambda_0/2) u(n) + sum_{d != 0} [(rho_k sum_mu d_mu g_mu - lambda_k/2) x W_d(n)] u(n+d)
// which is Eq. app_bril with the derivative factor of Eq. def_ider written out; the adjoint
// negates the rho part (g_5-hermiticity).  In the chiral basis sum_mu c_mu g_mu is
// [[0, B], [B^+, 0]] with B = [[c4 - i c3, -c2 - i c1], [c2 - i c1, c4 + i c3]] (App. C).
// The optional clover term C of Eq. def_clov is added at the centre (hermitian: the adjoint adds it
// unchanged).  With the flag lap the same kernels apply the Brillouin Laplacian of Eq. app_blap,
//   (-1/2 Delta^bri + m^2/2) u(n) = (m^2/2 - lambda_0/2) u(n) - sum_{d != 0} (lambda_|d|/2) W_d(n) u(n+d),
// the spin-trivial part of the stencil (the rho terms are skipped; the caller passes the diagonal).
#pragma once

#include <algorithm>
#include <type_traits>

#include "brillouin_plan.h"
#include "clover.h"
#include "common.h"
#include "kernels.h"
#include "launch.h"
#include "tile.h"

namespace dirac {

namespace {

__constant__ double c_rho[5] = {0.0, 64.0 / 432.0, 16.0 / 432.0, 4.0 / 432.0, 1.0 / 432.0};
__constant__ double c_halflam[5] = {-120.0 / 64.0, 4.0 / 64.0, 2.0 / 64.0, 1.0 / 64.0, 0.5 / 64.0};

// Spin-factor scalars per direction: {lambda_k / 2, q_1..q_4} with q_mu = rho_k d_mu (negated for the adjoint).
// Wave-uniform, so the row kernel reads them with scalar loads instead of recomputing them in every lane.  A constant of
// the code object, so that a first launch uploads nothing (it may be one that a stream captures).
template <typename R>
struct SpinTable {
    R at[2][81][5];  // [dagger][dir]
};
template <typename R>
constexpr SpinTable<R> make_spin_table() {
    SpinTable<R> t{};
    const double rho[5] = {0.0, 64.0 / 432.0, 16.0 / 432.0, 4.0 / 432.0, 1.0 / 432.0};
    const double halflam[5] = {-120.0 / 64.0, 4.0 / 64.0, 2.0 / 64.0, 1.0 / 64.0, 0.5 / 64.0};
    for (int dag = 0; dag < 2; ++dag)
        for (int dir = 0; dir < 81; ++dir) {
            const int d[4] = {dir % 3 - 1, (dir / 3) % 3 - 1, (dir / 9) % 3 - 1, dir / 27 - 1};
            const int k = (d[0] != 0) + (d[1] != 0) + (d[2] != 0) + (d[3] != 0);
            t.at[dag][dir][0] = static_cast<R>(halflam[k]);
            for (int mu = 0; mu < 4; ++mu) t.at[dag][dir][1 + mu] = static_cast<R>((dag ? -rho[k] : rho[k]) * d[mu]);
        }
    return t;
}
__constant__ SpinTable<float> c_spin_f = make_spin_table<float>();
__constant__ SpinTable<double> c_spin_d = make_spin_table<double>();

template <typename R>
__device__ __forceinline__ const R* spin_table(int dag, int dir);
template <>
__device__ __forceinline__ const float* spin_table<float>(int dag, int dir) {
    return c_spin_f.at[dag][dir];
}
template <>
__device__ __forceinline__ const double* spin_table<double>(int dag, int dir) {
    return c_spin_d.at[dag][dir];
}

// ---------------------------------------------------------------------------
// Apply: one thread per (site, RB right-hand sides); the 80 directions are a runtime loop
// with wave-uniform direction data.
// ---------------------------------------------------------------------------
// o[s] += (sum_mu q_mu g_mu - lh) ch[s] in the chiral basis, one displacement component at a time
// (hx..ht: d_x..d_t non-zero; q_mu = rho_k d_mu, already carrying the adjoint's and the boundary's
// signs, as does lh):
//   g_4: rows (0,1,2,3) <- (2,3,0,1)
//   g_3: rows <- (-i 2, +i 3, +i 0, -i 1)
//   g_2: rows <- (-3, +2, +1, -0)
//   g_1: rows <- (-i 3, -i 2, +i 1, +i 0)
// gamma_<mu>_accumulate: one term alone, o[s] += q (g_mu ch)[s].
template <typename R>
__device__ __forceinline__ void gamma_x_accumulate(cx<R> (&o)[4], const cx<R> (&ch)[4], R q1) {
    o[0].re += q1 * ch[3].im; o[0].im -= q1 * ch[3].re;
    o[1].re += q1 * ch[2].im; o[1].im -= q1 * ch[2].re;
    o[2].re -= q1 * ch[1].im; o[2].im += q1 * ch[1].re;
    o[3].re -= q1 * ch[0].im; o[3].im += q1 * ch[0].re;
}
template <typename R>
__device__ __forceinline__ void gamma_y_accumulate(cx<R> (&o)[4], const cx<R> (&ch)[4], R q2) {
    o[0].re -= q2 * ch[3].re; o[0].im -= q2 * ch[3].im;
    o[1].re += q2 * ch[2].re; o[1].im += q2 * ch[2].im;
    o[2].re += q2 * ch[1].re; o[2].im += q2 * ch[1].im;
    o[3].re -= q2 * ch[0].re; o[3].im -= q2 * ch[0].im;
}
template <typename R>
__device__ __forceinline__ void gamma_z_accumulate(cx<R> (&o)[4], const cx<R> (&ch)[4], R q3) {
    o[0].re += q3 * ch[2].im; o[0].im -= q3 * ch[2].re;
    o[1].re -= q3 * ch[3].im; o[1].im += q3 * ch[3].re;
    o[2].re -= q3 * ch[0].im; o[2].im += q3 * ch[0].re;
    o[3].re += q3 * ch[1].im; o[3].im -= q3 * ch[1].re;
}
template <typename R>
__device__ __forceinline__ void gamma_t_accumulate(cx<R> (&o)[4], const cx<R> (&ch)[4], R q4) {
    o[0].re += q4 * ch[2].re; o[0].im += q4 * ch[2].im;
    o[1].re += q4 * ch[3].re; o[1].im += q4 * ch[3].im;
    o[2].re += q4 * ch[0].re; o[2].im += q4 * ch[0].im;
    o[3].re += q4 * ch[1].re; o[3].im += q4 * ch[1].im;
}

template <typename R>
__device__ __forceinline__ void spin_accumulate(cx<R> (&o)[4], const cx<R> (&ch)[4], R lh, R q1, R q2, R q3, R q4,
                                                bool hx, bool hy, bool hz, bool ht) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        o[s].re -= lh * ch[s].re;
        o[s].im -= lh * ch[s].im;
    }
    if (ht) gamma_t_accumulate(o, ch, q4);
    if (hz) gamma_z_accumulate(o, ch, q3);
    if (hy) gamma_y_accumulate(o, ch, q2);
    if (hx) gamma_x_accumulate(o, ch, q1);
}

// NVC > 0 fixes N_v (= RB) at compile time: the site block is then contiguous in a thread and loaded 16 bytes at a time.
template <int NC, int RB, bool DAG, class P, int NVC>
__global__ __launch_bounds__(256) void brillouin_kernel(const typename P::G* __restrict__ W,
                                                         const typename P::S* __restrict__ in,
                                                         typename P::S* __restrict__ out, typename P::R diag, Geom g,
                                                         int nv, SiteOrder order, const typename P::R* __restrict__ clov,
                                                         int lap) {
    using R = typename P::R;
    using S = typename P::S;
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
    const S* centre = in + site * vs + r0;
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s) acc[k][a][s] = cscale(diag, io<R, S>::ld(centre + (a * 4 + s) * nv + k));
    if (clov) clover_add<NC, RB>(acc, centre, nv, clov + site * clover_reals<NC>());

    // neighbour offsets along each axis for steps -1, 0, +1 (with the periodic wrap) and the
    // fermion sign of the t steps; per direction the neighbour is site + four offsets
    // (site offsets fit in 32 bits: the library limits the volume to < 2^31 sites)
    const int sy = g.nx, sz = g.nx * g.ny, stt = sz * g.nz;
    const int ox[3] = {c.x == 0 ? g.nx - 1 : -1, 0, c.x == g.nx - 1 ? 1 - g.nx : 1};
    const int oy[3] = {(c.y == 0 ? g.ny - 1 : -1) * sy, 0, (c.y == g.ny - 1 ? 1 - g.ny : 1) * sy};
    const int oz[3] = {(c.z == 0 ? g.nz - 1 : -1) * sz, 0, (c.z == g.nz - 1 ? 1 - g.nz : 1) * sz};
    const int ot[3] = {(c.t == 0 ? g.nt - 1 : -1) * stt, 0, (c.t == g.nt - 1 ? 1 - g.nt : 1) * stt};
    const R sgn_t[3] = {(g.apbc && c.t == 0) ? R(-1) : R(1), R(1), (g.apbc && c.t == g.nt - 1) ? R(-1) : R(1)};

    for (int dir = 0; dir < 81; ++dir) {
        if (dir == 40) continue;
        // wave-uniform direction data
        const int ix = dir % 3, iy = (dir / 3) % 3, iz = (dir / 9) % 3, it = dir / 27;
        const int kh = (ix != 1) + (iy != 1) + (iz != 1) + (it != 1);
        // the fermion sign of a t-wrapping hop rides on the spin factor (five scalars)
        const R bsign = sgn_t[it];
        const R rho = bsign * static_cast<R>(DAG ? -c_rho[kh] : c_rho[kh]);
        const R q1 = rho * (ix - 1), q2 = rho * (iy - 1), q3 = rho * (iz - 1), q4 = rho * (it - 1);
        const R lh = bsign * static_cast<R>(c_halflam[kh]);
        const int64_t nb = site + (ox[ix] + oy[iy] + oz[iz] + ot[it]);

        cx<R> l[NC][NC];
        if (dir < 40) {
            const typename P::G* lp = W + (site * 40 + dir) * NC * NC;
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) l[a][b] = io<R, typename P::G>::ld(lp + a * NC + b);
        } else {
            const typename P::G* lp = W + (nb * 40 + (80 - dir)) * NC * NC;
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) l[b][a] = cconj(io<R, typename P::G>::ld(lp + a * NC + b));
        }
        const S* nbp = in + nb * vs + r0;
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            cx<R> p[NC][4];
#pragma unroll
            for (int b = 0; b < NC; ++b)
#pragma unroll
                for (int s = 0; s < 4; ++s) p[b][s] = io<R, S>::ld(nbp + (b * 4 + s) * nv + k);
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                cx<R> ch[4] = {{R(0), R(0)}, {R(0), R(0)}, {R(0), R(0)}, {R(0), R(0)}};
#pragma unroll
                for (int b = 0; b < NC; ++b)
#pragma unroll
                    for (int s = 0; s < 4; ++s) cfma(ch[s], l[a][b], p[b][s]);
                spin_accumulate(acc[k][a], ch, lh, q1, q2, q3, q4, !lap && ix != 1, !lap && iy != 1, !lap && iz != 1,
                                !lap && it != 1);
            }
        }
    }

    S* o = out + site * vs + r0;
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s) io<R, S>::st(o + (a * 4 + s) * nv + k, acc[k][a][s]);
}


// SS: padding units of a (colour, chirality) block of 2 nv one-unit elements, to nv modulo the 16 units of the LDS banks;
// none where it would take more than a fifth of the copy (a few right-hand sides: 1.08 instead of 0.96 ms for N_v = 4
// at 22 x 18 x 14 x 30, the copy leaving room for fewer work-groups)
__host__ __device__ inline uint32_t ss_pad(int nv) {
    const uint32_t p = (16u - static_cast<uint32_t>(nv) % 16u) % 16u;
    return 2u * p <= static_cast<uint32_t>(nv) ? p : 0u;
}

// Row-tiled apply: a work-group owns one x-row (every RHS) and walks the 27 rows at (y, z, t)
// offsets in {-1,0,1}^3 (row copy rc = 9 (d_t+1) + 3 (d_z+1) + (d_y+1)).  Each such row is copied
// into LDS with contiguous 16-byte loads and serves the three directions d_x = -1, 0, +1
// (periodic within the row).  With it comes a window of three consecutive stored links per
// site of one row: for rc < 13 the directions dir0 .. dir0 + 2 (dir0 = 27 it + 9 iz + 3 iy) of the
// own row; for rc > 13 the directions 78 - dir0 .. 80 - dir0 of the neighbour row, whose adjoints
// are the links of the directions 80 - dir (Tab. off-axis); for rc = 13 direction 39 of the own
// row serves d_x = -1 as stored and d_x = +1 as the adjoint at x + 1.  The window holds each link as
// applied: adjoints transposed and conjugated, and the fermion sign of a t step across the boundary
// folded in, so that every hop is the same plain product.  The next row copy is in flight (in
// registers) while the current one is consumed.  The three hops of a row, whose spin factors share
// their gamma_y..gamma_t terms up to fixed ratios, go into one accumulator (15432 instead of 18648
// multiply-adds per site and RHS with N_c = 3, the App. E count unchanged).  Three waves per SIMD
// cap the registers at 168 (FP32 and BF16 fit, the segmented forms spill a few values).
//
// SS (FP64, whose operands take twice the registers): a (site, RHS) has two threads, one per chirality (spins 2 h and
// 2 h + 1).  The link product and the -lambda/2 part stay inside a chirality, and the gamma parts of a thread's c go
// to the other one, so a thread keeps two sums of its size and the partners' are added at the end: the same
// arithmetic and neighbour reads in twice the wavefronts, with half the sums and row copy registers each.  At one
// thread per (site, RHS), two waves per SIMD and a work-group of three, the vector unit was busy a third of the time:
// 1.95 ms at 16^3 x 32 (N_c = 3, N_v = 12), now 1.51, the vector unit 57 % and LDS 55 % busy.
//
// At three waves per SIMD SS alone has no registers for a row copy in flight during the arithmetic (spilling, 16^3 x 32
// took 4 ms); the other work-groups of the CU cover the copies instead.
//
// CS: every colour row has a thread of its own, N_c times the wavefronts with an N_c-th of the work each (and N_c times
// the neighbour reads from LDS).  With SS for launches that would leave most of the chip idle (8^3 x 16, N_v = 4: 59 us
// in FP64, 78 with SS alone; FP32 45 us, 76 with one thread, 99 in the direct kernel) and rows too short for other forms;
// without SS in FP64 where it fills its wavefronts better (10 x 8 x 9 x 12, N_v = 4: 57 us, 90 with SS, 63 with one
// thread at two waves per SIMD).  brillouin_plan.h chooses.
//
// KPS: entries of a window slot that a lane moves at most (1 from about 10 right-hand sides on, N_c = 3).  With a slot
// limited to one entry per lane fewer right-hand sides took the direct kernel (N_v = 4 at 22 x 18 x 14 x 30, FP32: 1.04 ms
// against 0.51).
template <int NC, int RB, bool DAG, class P, int NVC, bool SEG, bool SS, bool CS, int KPS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu((SS && CS) || NC == 4 || (sizeof(typename P::R) == 8 && !SS && !CS && NC == 2) ? 2 : 3))) void brillouin_rows_kernel(const typename P::G* __restrict__ W,
                                                             const typename P::S* __restrict__ in,
                                                             typename P::S* __restrict__ out, typename P::R diag,
                                                             Geom g, int nv, RowTile rt,
                                                             const typename P::R* __restrict__ clov, int lap) {
    using R = typename P::R;
    using S = typename P::S;
    using G = typename P::G;
    static_assert(RB == 1, "the row form takes one RHS per thread");
    constexpr int NS = SS ? 2 : 4;       // spins per thread
    constexpr int NA = CS ? 1 : NC;      // colour rows per thread
    constexpr bool PF = !SS || CS;       // the next row copy is in flight during the arithmetic
    constexpr int SHARE = RowUnits<NC, RB, P>::PER * NS * NA, PER = (SHARE + 4 * NC - 1) / (4 * NC);
    constexpr bool EXACT = SHARE % (4 * NC) == 0;  // otherwise lanes past the row copy's units store nothing
    constexpr bool BLOCKPAD = SS && sizeof(typename P::S) == 16;
    constexpr int L = NC * NC;
    extern __shared__ __align__(16) u32x4 rtile[];
    if constexpr (NVC > 0) nv = NVC;

    const int64_t tix = logical_block();
    if (tix >= rt.ntiles) return;
    const uint32_t nseg = static_cast<uint32_t>(rt.nseg);
    const uint32_t rq = static_cast<uint32_t>(tix) / nseg;
    // first site of the segment (the last one ends with the row: its first sites may be the previous one's as well)
    const int x0 = min(static_cast<int>(static_cast<uint32_t>(tix) - rq * nseg) * rt.S, g.nx - rt.S);
    const uint32_t rho = tile_row(rq, rt, g);
    const uint32_t tid = threadIdx.x;
    const bool active = tid < static_cast<uint32_t>(rt.threads);
    const uint32_t tt = active ? tid : tid - rt.threads;  // padding threads shadow a real one
    const uint32_t j = fast_div(tt, rt.magic_nrg);      // site within the segment
    const int rg = static_cast<int>(tt - j * rt.nrg);  // SS: (colour *) chirality * nv + rhs
    constexpr int NH = SS ? 2 : 1;
    const int ca = CS ? rg / (NH * nv) : 0;                // the thread's first colour row
    const int hs = SS && rg - ca * NH * nv >= nv ? 1 : 0;  // SS: its chirality
    const int col0 = rg - (NH * ca + hs) * nv;             // its right-hand side
    const int x = x0 + static_cast<int>(j);
    int cy, cz, ct;
    {
        const uint32_t q = rho / static_cast<uint32_t>(g.ny);
        cy = static_cast<int>(rho - q * g.ny);
        const uint32_t q2 = q / static_cast<uint32_t>(g.nz);
        cz = static_cast<int>(q - q2 * g.nz);
        ct = static_cast<int>(q2);
    }
    const int64_t own_start = static_cast<int64_t>(rho) * g.nx;
    const u32x4* src = reinterpret_cast<const u32x4*>(in);
    // LDS: with SEG, copy site c = 0 .. S + 1 holds x = x0 - 1 + c (periodic); without, the whole row
    // (c = x, S = n_x, neighbours wrap inside it).  Then the link window.
    constexpr int OFF = SEG ? 1 : 0;  // copy site of the segment's first site
    const int SC = rt.S + 2 * OFF;    // sites per copy
    // the link window, slot-major: lwin[slot][copy site][L], slot = one of the three stored directions
    // Padding after each site, or with SS in FP64 (one unit per element) after each (colour, chirality) block of a site: the runs
    // of right-hand sides that consecutive lanes read (site after site, chirality after chirality) then follow each other
    // around the 64 LDS banks.
    const uint32_t HB = 2u * static_cast<uint32_t>(nv) + (BLOCKPAD ? ss_pad(nv) : 0u);  // SS: elements per block
    const uint32_t PADU =
        BLOCKPAD ? ss_pad(nv) : row_pad(rt.units, static_cast<uint32_t>(nv) * static_cast<uint32_t>(sizeof(S)) / 4u);
    const uint32_t SU = BLOCKPAD ? 2u * NC * HB : rt.units + PADU;  // units per site of the row copy
    auto pad_slot = [&](uint32_t u) __attribute__((always_inline)) { return u + fast_div(u, rt.magic_units) * PADU; };
    // element (colour a, spin s of the thread's) from the thread's first one
    auto el = [&](int a, int s) __attribute__((always_inline)) {
        return SS ? a * 2 * static_cast<int>(HB) + s * nv : (a * 4 + s) * nv;
    };
    G* lwin = reinterpret_cast<G*>(rtile + SC * SU);
    const uint32_t WS = static_cast<uint32_t>(SC) * L;  // elements per slot
    // Each load instruction of the window covers one slot: KPS loads per slot, each lane taking entry
    // q * threads + tt of it (checked at launch: SC * L <= KPS * threads); lanes past the slot repeat its
    // last entry and store nothing.  The slot's transposition, sign and scale are then wave-uniform.
    constexpr int PERL = 3 * KPS;
    uint32_t woff[KPS], wofft[KPS];  // the lane's element in a stored direction block: as stored, transposed
#pragma unroll
    for (int q = 0; q < KPS; ++q) {
        const uint32_t e = min(q * static_cast<uint32_t>(rt.threads) + tt, WS - 1u);
        const uint32_t sx = e / L, ab = e - sx * L;
        const uint32_t xs = SEG ? static_cast<uint32_t>(wrap(x0 - 1 + static_cast<int>(sx), g.nx)) : sx;
        woff[q] = xs * 40u * L + ab;
        wofft[q] = xs * 40u * L + (ab % NC) * NC + ab / NC;
    }
    // main units: the S sites of the segment, copy sites 1 .. S (SS: taken anew per row, for the registers)
    auto slot_of = [&](int k, uint32_t t) __attribute__((always_inline)) {
        const uint32_t u = k * static_cast<uint32_t>(rt.threads) + t;
        return pad_slot(u) + OFF * SU;
    };
    uint32_t slot[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) slot[k] = SS ? 0u : slot_of(k, tt);
    // halo units h = tt and tt + threads (< 2 units) copy the sites x0 - 1 (copy site 0) and x0 + S (copy site S + 1)
    bool halo[2];
    uint32_t hslot[2];
    uint32_t hsrc[2];  // unit index relative to the start of the copied row
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t h = tt + q * static_cast<uint32_t>(rt.threads);
        halo[q] = SEG && h < 2u * rt.units;
        const uint32_t end = h < static_cast<uint32_t>(rt.units) ? 0u : 1u;
        const uint32_t hcu = h - end * rt.units;
        hslot[q] = (end ? rt.S + 1 : 0) * SU + (BLOCKPAD ? pad_slot(hcu) : hcu);
        hsrc[q] = static_cast<uint32_t>(end ? wrap(x0 + rt.S, g.nx) : wrap(x0 - 1, g.nx)) * rt.units + hcu;
    }
    auto row_start = [&](int rc) __attribute__((always_inline)) {
        const int dy = rc % 3 - 1, dz = (rc / 3) % 3 - 1, dt = rc / 9 - 1;
        const int y = wrap(cy + dy, g.ny), z = wrap(cz + dz, g.nz), t = wrap(ct + dt, g.nt);
        return ((static_cast<int64_t>(t) * g.nz + z) * g.ny + y) * g.nx;
    };
    u32x4 pre[PER];
    u32x4 hpre[2];
    G lpre[PERL];
    // row copies and link windows are buffer loads over one lattice row: a scalar base per row, 32-bit
    // offsets per lane (a read past the row returns zero instead of touching memory)
    const uint32_t row_bytes = static_cast<uint32_t>(g.nx) * rt.units * 16u;
    const uint32_t wrow_bytes = static_cast<uint32_t>(g.nx) * 40u * L * static_cast<uint32_t>(sizeof(G));
    auto fetch = [&](int rc) __attribute__((always_inline)) {
        const int64_t start = row_start(rc);
        const auto rrow = raw_buffer(src + start * rt.units, row_bytes);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            pre[k] = buffer_load_unit<u32x4>(rrow, tt * 16u,
                                             (static_cast<uint32_t>(x0) * rt.units + k * static_cast<uint32_t>(rt.threads)) *
                                                 16u);
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (SEG && halo[q]) hpre[q] = buffer_load_unit<u32x4>(rrow, hsrc[q] * 16u, 0u);
        const int dir0 = 9 * (3 * (rc / 9) + (rc / 3) % 3) + 3 * (rc % 3);
        const int64_t lstart = rc <= 13 ? own_start : start;
        const int wb = rc < 13 ? dir0 : (rc == 13 ? 37 : 78 - dir0);
        const auto rw = raw_buffer(W + lstart * 40 * L, wrow_bytes);
        // window slot ws holds W_d(n) as applied: for rc > 13 every slot is the adjoint of the stored
        // link (element (a, b) <- conj of stored (b, a)); for rc = 13 slot 2 holds direction 39 as stored
        // and slot 0 its adjoint
#pragma unroll
        for (int k = 0; k < PERL; ++k) {
            const int ws = k / KPS, q = k % KPS;
            const bool adj = rc > 13 || (rc == 13 && ws == 0);
            const uint32_t from = (adj ? wofft[q] : woff[q]) +
                                  static_cast<uint32_t>(wb + (rc == 13 && ws == 0 ? 2 : ws)) * L;
            lpre[k] = buffer_load_unit<G>(rw, from * static_cast<uint32_t>(sizeof(G)), 0u);
        }
    };
    auto at = [&](int c) __attribute__((always_inline)) {
        return reinterpret_cast<const S*>(rtile + c * SU) + (SS ? hs * static_cast<int>(HB) : 0) + col0;
    };

    cx<R> acc[RB][NA][NS];           // sums of the thread's spins
    cx<R> oth[SS ? NA : 1][NS] = {};  // SS: its part of the other chirality's
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int s = 0; s < NS; ++s) acc[k][a][s] = {R(0), R(0)};
    // acc, oth += (sum_mu q_mu g_mu - lh) c for the listed terms
    const R sg = hs ? R(-1) : R(1);
    auto spin_add = [&](const cx<R> (&c)[NA][NS], R lh, R q1, R q2, R q3, R q4, bool hx, bool hy, bool hz, bool ht)
                        __attribute__((always_inline)) {
        if constexpr (SS) {
            // other[0], other[1] <- q4 (c0, c1), s i q3 (c0, -c1), s q2 (c1, -c0), s i q1 (c1, c0), s = +-1 by chirality
            const R s1 = sg * q1, s2 = sg * q2, s3 = sg * q3;
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const cx<R> c0 = c[a][0], c1 = c[a][1];
                acc[0][a][0].re -= lh * c0.re;
                acc[0][a][0].im -= lh * c0.im;
                acc[0][a][1].re -= lh * c1.re;
                acc[0][a][1].im -= lh * c1.im;
                cx<R>&o0 = oth[a][0], &o1 = oth[a][1];
                if (ht) {
                    o0.re += q4 * c0.re;
                    o0.im += q4 * c0.im;
                    o1.re += q4 * c1.re;
                    o1.im += q4 * c1.im;
                }
                if (hz) {
                    o0.re -= s3 * c0.im;
                    o0.im += s3 * c0.re;
                    o1.re += s3 * c1.im;
                    o1.im -= s3 * c1.re;
                }
                if (hy) {
                    o0.re += s2 * c1.re;
                    o0.im += s2 * c1.im;
                    o1.re -= s2 * c0.re;
                    o1.im -= s2 * c0.im;
                }
                if (hx) {
                    o0.re -= s1 * c1.im;
                    o0.im += s1 * c1.re;
                    o1.re -= s1 * c0.im;
                    o1.im += s1 * c0.re;
                }
            }
        } else {
#pragma unroll
            for (int a = 0; a < NA; ++a) spin_accumulate(acc[0][a], c[a], lh, q1, q2, q3, q4, hx, hy, hz, ht);
        }
    };

    if constexpr (PF) fetch(0);
    for (int rc = 0; rc < 27; ++rc) {
        if constexpr (!PF) fetch(rc);
        __syncthreads();  // the previous row copy has been consumed
        uint32_t ts = tt;
        if constexpr (SS) asm volatile("" : "+v"(ts));  // keeps the slots from being hoisted out of the loop
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (EXACT || k * static_cast<uint32_t>(rt.threads) + tt < static_cast<uint32_t>(rt.S) * rt.units)
                rtile[SS ? slot_of(k, ts) : slot[k]] = pre[k];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (SEG && halo[q]) rtile[hslot[q]] = hpre[q];
        // The window as applied: the adjoint's conjugation, the fermion sign of a t step across the boundary
        // (all three hops of a row take the same t step) and, for the three-hop accumulation below, the
        // d_x = 0 hop times 4 (slot 1 outside the centre row) are factors of the real and imaginary parts,
        // uniform per slot.  They are taken from a copy of rc made opaque here, after the barrier: taken at
        // the loads, they would make the compiler wait for the prefetch there.
        {
            int rs = rc;
            asm volatile("" : "+s"(rs));
            const int its = rs / 9;
            const bool bflip = g.apbc && ((its == 0 && ct == 0) || (its == 2 && ct == g.nt - 1));
#pragma unroll
            for (int k = 0; k < PERL; ++k) {
                const int ws = k / KPS, q = k % KPS;
                const bool adj = rs > 13 || (rs == 13 && ws == 0);
                const R sc = (ws == 1 && rs != 13) ? R(4) : R(1);
                const R fx = bflip ? -sc : sc;
                const R fy = adj != bflip ? -sc : sc;
                const uint32_t u = q * static_cast<uint32_t>(rt.threads) + tt;
                if (u < WS) {
                    G v = lpre[k];
                    v.x *= fx;
                    v.y *= fy;
                    lwin[ws * WS + u] = v;
                }
            }
        }
        __syncthreads();
        // the last pass refetches its own row (a cache hit): an unconditional fetch keeps the prefetched
        // values in the registers they are loaded into
        if constexpr (PF) fetch(rc < 26 ? rc + 1 : 26);
        if (active) {
            const int iy = rc % 3, iz = (rc / 3) % 3, it = rc / 9;
            const int dir0 = 27 * it + 9 * iz + 3 * iy;  // + ix for d_x = ix - 1
            const bool hy = !lap && iy != 1, hz = !lap && iz != 1, ht = !lap && it != 1;
            // c[a] += (W_d u(n + d))_a for d_x = ix - 1, one neighbour colour at a time.  W_d(n) as applied: for
            // rc < 13 (and rc = 13 with d_x = -1) it is stored at the own site, else it is the adjoint of the
            // link stored at n + d, which the window already holds transposed and conjugated
            auto hop_add = [&](int ix, cx<R> (&c)[NA][NS]) __attribute__((always_inline)) {
                const int cn = SEG ? static_cast<int>(j) + ix : wrap(static_cast<int>(j) + ix - 1, g.nx);
                const bool adj = rc > 13 || (rc == 13 && ix == 2);
                const G* lp = lwin + (rc < 13 ? ix : (rc == 13 ? (ix == 2 ? 0 : 2) : 2 - ix)) * WS +
                              (adj ? cn : static_cast<int>(j) + OFF) * L;
                const S* nbp = at(cn);
                if constexpr (SS) {  // one row of the link at a time: the whole link spills
                    cx<R> pb[NC][NS];
#pragma unroll
                    for (int b = 0; b < NC; ++b)
#pragma unroll
                        for (int s = 0; s < NS; ++s) pb[b][s] = io<R, S>::ld(nbp + el(b, s));
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
#pragma unroll
                        for (int b = 0; b < NC; ++b) {
                            const cx<R> l = io<R, G>::ld(lp + ((ca + a) * NC + b));
#pragma unroll
                            for (int s = 0; s < NS; ++s) cfma(c[a][s], l, pb[b][s]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    return;
                }
                cx<R> l[NA][NC];
#pragma unroll
                for (int a = 0; a < NA; ++a)
#pragma unroll
                    for (int b = 0; b < NC; ++b) l[a][b] = io<R, G>::ld(lp + ((ca + a) * NC + b));
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    cx<R> pb[NS];
#pragma unroll
                    for (int s = 0; s < NS; ++s) pb[s] = io<R, S>::ld(nbp + el(b, s));
#pragma unroll
                    for (int a = 0; a < NA; ++a)
#pragma unroll
                        for (int s = 0; s < NS; ++s) cfma(c[a][s], l[a][b], pb[s]);
                }
            };
            if (rc == 13) {  // d_x = 0 is the centre: (m - lambda_0 / 2) u(n), plus the clover term
                const S* nbp = at(static_cast<int>(j) + OFF);
#pragma unroll
                for (int a = 0; a < NA; ++a)
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const cx<R> v = io<R, S>::ld(nbp + el(ca + a, s));
                        acc[0][a][s].re += diag * v.re;
                        acc[0][a][s].im += diag * v.im;
                    }
                if constexpr (NA == NC) {  // the launcher keeps a clover field to whole colour vectors
                    if (clov) {
                        const R* cs = clov + (own_start + x) * clover_reals<NC>();
                        if constexpr (SS)
                            clover_add_half<NC>(acc[0], nbp, 2 * static_cast<int>(HB), nv, cs + hs * 4 * NC * NC);
                        else
                            clover_add<NC, RB>(acc, nbp, nv, cs);
                    }
                }
            }
            const R* sm = spin_table<R>(DAG ? 1 : 0, dir0);
            const R* sp = spin_table<R>(DAG ? 1 : 0, dir0 + 2);
            // The three hops of a row share one accumulator c.  With k the number of non-zero components of
            // d_x = +-1 (and k - 1 for d_x = 0), S_pm = -l + R pm q gamma_x with l = lambda_k / 2 and
            // R = sum over y, z, t of rho_k d_mu gamma_mu; the d_x = 0 hop has S_0 = -2 l + 4 R (rho and
            // lambda fall by 4 and 2 per unit of k).  So S_- chi_- + S_+ chi_+ + S_0 chi_0 =
            //   2 q_- gamma_x chi_- + (q_+ gamma_x - l / 2) (chi_- + chi_+) + (R - l / 2) (chi_- + chi_+ + 4 chi_0),
            // taken as c = chi_-, then c += chi_+, then c += 4 chi_0 (its link is stored times 4).  In the
            // centre row the last step is -l / 2 alone.
            const R lq = R(0.5) * sp[0];
            cx<R> c[NA][NS] = {};
            hop_add(0, c);
            if (!lap) {
                if constexpr (SS) {
                    const R s1 = sg * (R(2) * sm[1]);
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
                        oth[a][0].re -= s1 * c[a][1].im;
                        oth[a][0].im += s1 * c[a][1].re;
                        oth[a][1].re -= s1 * c[a][0].im;
                        oth[a][1].im += s1 * c[a][0].re;
                    }
                } else {
#pragma unroll
                    for (int a = 0; a < NA; ++a) gamma_x_accumulate(acc[0][a], c[a], R(2) * sm[1]);
                }
            }
            hop_add(2, c);
            spin_add(c, lq, sp[1], sp[2], sp[3], sp[4], !lap, false, false, false);
            if (rc != 13) hop_add(1, c);
            spin_add(c, lq, sp[1], sp[2], sp[3], sp[4], false, hy, hz, ht);
        }
    }
    __syncthreads();
    S* o = const_cast<S*>(at(static_cast<int>(j) + OFF));
    // SS: the partner's part of this chirality arrives through the row copy, which is free by now, in the precision of the
    // sums: in place where that is the storage precision, else (BF16) one spin after the other, whose sums take as many
    // bytes as the four spins' elements (8^3 x 16, N_v = 4: 46 us either way)
    if constexpr (SS && sizeof(S) == sizeof(cx<R>)) {
        S* po = o + (hs ? -static_cast<int>(HB) : static_cast<int>(HB));
        if (active)
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int s = 0; s < NS; ++s) io<R, S>::st(po + el(ca + a, s), oth[a][s]);
        __syncthreads();
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int s = 0; s < NS; ++s) acc[0][a][s] = cadd(acc[0][a][s], io<R, S>::ld(o + el(ca + a, s)));
    } else if constexpr (SS) {
        static_assert(2 * sizeof(S) >= sizeof(cx<R>), "a spin's sums fit the row copy");
        cx<R>* const ex = reinterpret_cast<cx<R>*>(rtile);  // [colour row of the thread][thread]
        const uint32_t partner = hs ? tt - nv : tt + nv;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (active)  // a padding thread has no sums
#pragma unroll
                for (int a = 0; a < NA; ++a) ex[a * rt.threads + tt] = oth[a][s];
            __syncthreads();
#pragma unroll
            for (int a = 0; a < NA; ++a) acc[0][a][s] = cadd(acc[0][a][s], ex[a * rt.threads + partner]);
            __syncthreads();
        }
    }
    if (active) {
#pragma unroll
        for (int k = 0; k < RB; ++k)
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int s = 0; s < NS; ++s) io<R, S>::st(o + el(ca + a, s) + k, acc[k][a][s]);
    }
    __syncthreads();
    u32x4* dst = reinterpret_cast<u32x4*>(out) + (own_start + x0) * rt.units;
    const uint32_t total = static_cast<uint32_t>(rt.S) * rt.units;
    for (uint32_t u = tid; u < total; u += blockDim.x) dst[u] = rtile[pad_slot(u) + OFF * SU];
}


// The centre coefficient: m - lambda_0/2 for D_B, m^2/2 - lambda_0/2 for the Laplacian.
double centre_coefficient(const StencilArgs& a) {
    return (a.laplace ? 0.5 * a.mass * a.mass : a.mass) + 120.0 / 64.0;
}

template <int NC, int RB, class P>
bool launch_rows(const StencilArgs& a, hipStream_t st) {
    using S = typename P::S;
    using R = typename P::R;
    const size_t block_bytes = static_cast<size_t>(NC) * 4 * a.nv * sizeof(S);
    if (block_bytes % 16 != 0 || !tile_aligned(a)) return false;
    const int units = static_cast<int>(block_bytes / 16);
    constexpr bool FP64 = sizeof(R) == 8;
    // the kernel addresses a row of the vectors and of the links with 32-bit byte offsets
    constexpr int kLinkBytes = 40 * NC * NC * static_cast<int>(sizeof(typename P::G));
    if (a.g.nx > static_cast<int64_t>(UINT32_MAX) / std::max(units * 16, kLinkBytes)) return false;
    const int64_t rows = a.g.vol / a.g.nx;
    auto lds_of = [&](const RowForm& f, int d) {
        const size_t sc = d + (d != a.g.nx ? 2 : 0);  // sites per copy
        const size_t su = FP64 && f.chirality ? 2 * NC * (2 * a.nv + ss_pad(a.nv))
                                              : units + row_pad(units, a.nv * sizeof(S) / 4);
        return sc * su * 16 + sc * 3 * NC * NC * sizeof(typename P::G);
    };
    const RowPlan plan =
        plan_rows({NC, a.nv, static_cast<int>(sizeof(S)), a.g.nx, rows, a.clover != nullptr}, lds_of);
    if (plan.form < 0) return false;
    const RowForm form = row_form(FP64, plan.form);
    const int seg = plan.seg, kps = plan.entries;
    const int nrg = a.nv * (form.chirality ? 2 : 1) * (form.colour ? NC : 1);
    const size_t lds = lds_of(form, seg);
    const bool segmented = seg != a.g.nx;
    RowTile rt{};
    rt.R = 1;
    rt.S = seg;
    rt.nseg = (a.g.nx + seg - 1) / seg;
    rt.nrg = nrg;
    rt.units = units;
    rt.row_units = a.g.nx * units;
    rt.threads = seg * nrg;
    rt.ntiles = rows * rt.nseg;
    rt.magic_nrg = div_magic(nrg);
    rt.magic_nx = div_magic(a.g.nx);
    rt.magic_units = div_magic(FP64 && form.chirality ? 2 * a.nv : units);  // the padded blocks of a row copy
    rt.magic_row_units = div_magic(rt.row_units);
    if (!row_order(4, a.g, rt)) return false;
    const int block = (rt.threads + 63) / 64 * 64;
    if (!fits_launch(rt.ntiles, block)) return false;  // the direct kernel has fewer threads
    const dim3 grid(static_cast<unsigned>(grid_blocks_x8(rt.ntiles, 1)));
    const R diag = static_cast<R>(centre_coefficient(a));
    auto W = static_cast<const typename P::G*>(a.gauge);
    auto in = static_cast<const S*>(a.in);
    auto out = static_cast<S*>(a.out);
    auto clov = static_cast<const R*>(a.clover);
    const int lap = a.laplace ? 1 : 0;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(block), lds, st, W, in, out, diag, a.g, a.nv, rt, clov, lap);
    };
    auto pick = [&](auto seg_c) {
        constexpr bool SG = decltype(seg_c)::value;
        auto with = [&](auto nvc, auto ss_c, auto cs_c, auto kps_c) {
            constexpr int NVC = decltype(nvc)::value, KPS = decltype(kps_c)::value;
            constexpr bool SS = decltype(ss_c)::value, CS = decltype(cs_c)::value;
            if (a.dagger)
                go(brillouin_rows_kernel<NC, RB, true, P, NVC, SG, SS, CS, KPS>);
            else
                go(brillouin_rows_kernel<NC, RB, false, P, NVC, SG, SS, CS, KPS>);
        };
        const std::integral_constant<int, 0> any;
        const std::integral_constant<int, 1> one;
        const std::integral_constant<int, kMaxWindowEntries> most;
        const std::true_type yes;
        const std::false_type no;
        const std::bool_constant<FP64> ss;
        constexpr int K12 = NC >= 4 && !FP64 ? 2 : 1;
        if (plan.form == 1) {
            if (kps == 1)
                with(any, yes, yes, one);
            else
                with(any, yes, yes, most);
            return;
        }
        if constexpr (FP64) {
            if (plan.form == 2) {
                if (kps == 1)
                    with(any, no, yes, one);
                else
                    with(any, no, yes, most);
                return;
            }
            if constexpr (NC <= 2) {
                if (plan.form == 3) {
                    if (kps == 1)
                        with(any, no, no, one);
                    else
                        with(any, no, no, most);
                    return;
                }
            }
        }
        if (a.nv == 12 && kps <= K12)
            with(std::integral_constant<int, 12>{}, ss, no, std::integral_constant<int, K12>{});
        else if (kps == 1)
            with(any, ss, no, one);
        else
            with(any, ss, no, most);
    };
    if (segmented)
        pick(std::true_type{});
    else
        pick(std::false_type{});
    return true;
}

template <int NC, int RB, class P>
void launch_rb(const StencilArgs& a, hipStream_t st) {
    using R = typename P::R;
    if (a.variant == 4 && launch_rows<NC, RB, P>(a, st)) return;
    const int64_t threads = a.g.vol * (a.nv / RB);
    const int block = direct_block(threads);
    const dim3 grid(static_cast<unsigned>(grid_blocks_x8(threads, block)));
    const R diag = static_cast<R>(centre_coefficient(a));
    auto W = static_cast<const typename P::G*>(a.gauge);
    auto in = static_cast<const typename P::S*>(a.in);
    auto out = static_cast<typename P::S*>(a.out);
    auto clov = static_cast<const R*>(a.clover);
    const int lap = a.laplace ? 1 : 0;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(block), 0, st, W, in, out, diag, a.g, a.nv, make_site_order(a.g), clov, lap);
    };
    if (a.nv == RB) {
        if (a.dagger)
            go(brillouin_kernel<NC, RB, true, P, RB>);
        else
            go(brillouin_kernel<NC, RB, false, P, RB>);
    } else {
        if (a.dagger)
            go(brillouin_kernel<NC, RB, true, P, 0>);
        else
            go(brillouin_kernel<NC, RB, false, P, 0>);
    }
}

template <int NC, class P>
void launch_nc(const StencilArgs& a, hipStream_t st) {
    launch_rb<NC, 1, P>(a, st);
}

template <class P>
int launch_prec(const StencilArgs& a, hipStream_t st) {
    switch (a.nc) {
        case 1: launch_nc<1, P>(a, st); break;
        case 2: launch_nc<2, P>(a, st); break;
        case 3: launch_nc<3, P>(a, st); break;
        case 4: launch_nc<4, P>(a, st); break;
        default: return DIRAC_EUNSUPPORTED;
    }
    return DIRAC_OK;
}

}  // namespace

}  // namespace dirac
