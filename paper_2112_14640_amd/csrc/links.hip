// Hypercube links W of the Brillouin operator (Sec. 6, Tab. off-axis): W_d(n) is the plain average over the |d|!
// orderings of the unit steps of d of the ordered products of V along each path (a step -mu from x uses V_mu(x-mu)^+).
// Directions are numbered dir = 27(d_t+1) + 9(d_z+1) + 3(d_y+1) + (d_x+1); the 40 directions dir < 40 are stored.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace dirac {

namespace {

// ---------------------------------------------------------------------------
// Link construction, level by level.  Grouping the |d|! orderings of the unit steps of d by
// their last step gives
//     W_d(n) = (1/|d|) sum_{mu: d_mu != 0} W_{d - s e_mu}(n) L,   s = d_mu,
// with L = V_mu(n + d - e_mu) for s = +1 and L = V_mu(n + d)^+ for s = -1: the average at
// |d| is built from the averages at |d| - 1 of the same site.  The stored directions and all
// they are built from are dir < 54 (no step +t is ever needed, since level 4 is stored with
// d_t = -1 only), so a site needs 128 products (18 directions of level 2, 20 of level 3, 8 of
// level 4) instead of the 1108 of the separate paths.  A work-group takes S consecutive sites,
// holds the levels of its sites in LDS (in the output precision, products accumulated in FP64),
// and writes each site's 40 stored directions as one contiguous block.
// ---------------------------------------------------------------------------
// A task is one direction of one site.  Its last steps are listed in a packed table (order-templated loops, no
// branch on the direction) and the sites it reads come from a table of offsets in LDS: with the steps as branches and
// the neighbour's index divided out per step, three quarters of the kernel's instructions were neither products nor
// conversions (0.60 ms at 16^3 x 32 in FP32, N_c = 3; then 0.30; loading a wavefront's 64 matrices together, consecutive lanes
// consecutive elements, was slower, 0.52 ms, the exchange through LDS costing more than the addresses).  The 46
// directions that are needed instead of 64, in the tile below: 0.23 ms.  Now the address rate of the link loads bounds
// it (5 loads per matrix and lane, each lane a line of its own, about 0.16 ms), with 0.14 ms of instruction issue, half
// of it FP64 products; fetching a level's links before the barrier of the level below was slower (0.245 ms).
struct LevelTable {
    // bits 0-6 the direction (dir); for its k-th last step, from bit 8 + 10 k: 7 bits the direction one step shorter, 2 bits
    // the axis, 1 bit whether the step is forwards.  Level 2 (18 directions), level 3 (20), level 4 (8)
    uint64_t task[46];
};
constexpr int kLinkDirs = 54;  // directions that are built: dir < 54, without the centre 40
__host__ __device__ constexpr int link_slot(int dir) { return dir < 40 ? dir : dir - 1; }
constexpr int kDirStride[4] = {1, 3, 9, 27};
constexpr LevelTable make_level_table() {
    LevelTable l{};
    int n = 0;
    for (int k = 2; k <= 4; ++k)
        for (int dir = 0; dir < kLinkDirs; ++dir) {
            int nz = 0;
            uint64_t t = static_cast<uint64_t>(dir);
            for (int mu = 0, q = dir; mu < 4; ++mu, q /= 3) {
                const int s = q % 3 - 1;
                if (s == 0) continue;
                const uint64_t prev = static_cast<uint64_t>(dir - s * kDirStride[mu]);
                t |= (prev | static_cast<uint64_t>(mu) << 7 | static_cast<uint64_t>(s > 0) << 9) << (8 + 10 * nz);
                ++nz;
            }
            if (nz == k) l.task[n++] = t;
        }
    return l;
}
__constant__ LevelTable c_levels = make_level_table();

// Sites of a tile: six give each level's tasks (108, 120, 48) nearly full wavefronts, 14 wavefront products for 6 sites
// against 14 for 4 sites (72, 80, 32).  6 x 53 x 9 x 16 B = 45.8 KB of LDS for N_c = 3 in FP64, half in FP32
template <int NC, typename GO>
constexpr int link_tile_sites() {
    return NC <= 3 || sizeof(GO) == 8 ? 6 : 4;
}
constexpr int kLinkThreads = 128;

template <int NC, typename GI, typename GO>
__global__ __launch_bounds__(kLinkThreads) void links_kernel(const GI* __restrict__ U, GO* __restrict__ W, Geom g) {
    constexpr int S = link_tile_sites<NC, GO>();
    constexpr int L = NC * NC;
    using T = std::conditional_t<sizeof(GO) == 8, float, double>;
    __shared__ cx<T> lw[S][kLinkDirs - 1][L];
    __shared__ int disp[S][kLinkDirs];  // site offset of each displacement (32 bits: V < 2^31)
    const int64_t site0 = logical_block() * S;
    if (site0 >= g.vol) return;
    const int ns = static_cast<int>(g.vol - site0 < S ? g.vol - site0 : S);
    const int tid = threadIdx.x;
    __shared__ Coord at[S];
    if (tid < S) at[tid] = site_coord(site0 + (tid < ns ? tid : 0), g);
    __syncthreads();
    for (int u = tid; u < S * kLinkDirs; u += kLinkThreads) {
        const int s = u / kLinkDirs, d = u % kLinkDirs;
        const Coord c = at[s];
        disp[s][d] = static_cast<int>(site_index(wrap(c.x + d % 3 - 1, g.nx), wrap(c.y + (d / 3) % 3 - 1, g.ny),
                                                 wrap(c.z + (d / 9) % 3 - 1, g.nz), wrap(c.t + d / 27 - 1, g.nt), g) -
                                      site0);
    }
    __syncthreads();
    // level 1: W_{+e_mu}(n) = V_mu(n), W_{-e_mu}(n) = V_mu(n - e_mu)^+, in the order -t, -x, +x, -y, +y, -z, +z
    for (int u = tid; u < ns * 7 * L; u += kLinkThreads) {
        const int s = u / (7 * L), j = (u / L) % 7, e = u % L;
        const int mu = j == 0 ? 3 : (j - 1) >> 1, a = e / NC, b = e % NC;
        const int stride = mu == 0 ? 1 : (mu == 1 ? 3 : (mu == 2 ? 9 : 27));
        const bool back = j == 0 || (j & 1);
        const int dir = back ? 40 - stride : 40 + stride;
        const GI* l = U + ((site0 + disp[s][back ? dir : 40]) * 4 + mu) * L;
        const cx<T> v = io<T, GI>::ld(l + (back ? b * NC + a : e));
        lw[s][link_slot(dir)][e] = back ? cconj(v) : v;
    }
    __syncthreads();
    auto level = [&](auto order_c) __attribute__((always_inline)) {
        constexpr int K = decltype(order_c)::value;
        constexpr int FIRST = K == 2 ? 0 : (K == 3 ? 18 : 38), CNT = K == 2 ? 18 : (K == 3 ? 20 : 8);
        for (int u = tid; u < ns * CNT; u += kLinkThreads) {
            const int s = u / CNT;
            const uint64_t task = c_levels.task[FIRST + u % CNT];
            const int dir = static_cast<int>(task) & 127;
            // the links of all last steps are loaded before any product, so their latencies overlap
            GI raw[K][L];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t st = static_cast<uint32_t>(task >> (8 + 10 * k)) & 1023u;
                const GI* lp = U + ((site0 + disp[s][(st >> 9) ? (st & 127u) : dir]) * 4 + ((st >> 7) & 3u)) * L;
#pragma unroll
                for (int e = 0; e < L; ++e) raw[k][e] = lp[e];
            }
            cx<double> acc[NC][NC];
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) acc[a][b] = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t st = static_cast<uint32_t>(task >> (8 + 10 * k)) & 1023u;
                const bool fwd = st >> 9;
                const cx<T>* prev = lw[s][link_slot(static_cast<int>(st & 127u))];
                cx<double> l[NC][NC];
#pragma unroll
                for (int a = 0; a < NC; ++a)
#pragma unroll
                    for (int b = 0; b < NC; ++b) {  // L, or its adjoint for a backward step
                        GI v = raw[k][a * NC + b];
                        if (!fwd) v = raw[k][b * NC + a];
                        if (!fwd) v.y = -v.y;
                        l[a][b] = io<double, GI>::ld(&v);
                    }
#pragma unroll
                for (int a = 0; a < NC; ++a)
#pragma unroll
                    for (int e = 0; e < NC; ++e) {
                        const cx<double> pv{prev[a * NC + e].re, prev[a * NC + e].im};
#pragma unroll
                        for (int b = 0; b < NC; ++b) cfma(acc[a][b], pv, l[e][b]);
                    }
            }
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    const cx<double> v = cscale(1.0 / K, acc[a][b]);
                    lw[s][link_slot(dir)][a * NC + b] = {static_cast<T>(v.re), static_cast<T>(v.im)};
                }
        }
        __syncthreads();
    };
    level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{});
    level(std::integral_constant<int, 4>{});
    // the stored directions 0..39 of the tile's sites are one contiguous block of W
    GO* out = W + site0 * 40 * L;
    for (int u = tid; u < ns * 40 * L; u += kLinkThreads) {
        const int s = u / (40 * L), r = u - s * 40 * L;
        io<T, GO>::st(out + u, lw[s][r / L][r % L]);
    }
}

template <int NC>
void launch_links_nc(dirac_prec prec, const Geom& g, const void* U, void* W, hipStream_t st) {
    auto go = [&](auto v) {
        using G = decltype(v);
        const dim3 grid(static_cast<unsigned>(grid_blocks_x8(g.vol, link_tile_sites<NC, G>())));
        hipLaunchKernelGGL((links_kernel<NC, G, G>), grid, dim3(kLinkThreads), 0, st, static_cast<const G*>(U),
                           static_cast<G*>(W), g);
    };
    if (prec == DIRAC_FP64)
        go(double2{});
    else
        go(float2{});
}

}  // namespace

int launch_brillouin_links(dirac_prec prec, int nc, const Geom& g, const void* U, void* W, hipStream_t st) {
    switch (nc) {
        case 1: launch_links_nc<1>(prec, g, U, W, st); break;
        case 2: launch_links_nc<2>(prec, g, U, W, st); break;
        case 3: launch_links_nc<3>(prec, g, U, W, st); break;
        case 4: launch_links_nc<4>(prec, g, U, W, st); break;
        default: return DIRAC_EUNSUPPORTED;
    }
    return DIRAC_OK;
}

}  // namespace dirac
