// Stout smearing (Sec. 2; Morningstar and Peardon's analytic smearing) and the backward passes that
// carry a link gradient through it and through the Brillouin hypercube links W(V) (Tab. off-axis).
//
// One stout step, for every link at once from the old field:
//   C_mu(n)  = rho sum_{nu != mu} [U_nu(n) U_mu(n+nu) U_nu(n+mu)^+ + U_nu(n-nu)^+ U_mu(n-nu) U_nu(n-nu+mu)]
//   Omega    = C U^+,  Q = (i/2)(Omega^+ - Omega) - (i/(2N)) Tr(Omega^+ - Omega),  U' = exp(i Q) U.
// Gradients follow torch's convention for real losses: G = dL/dRe M + i dL/dIm M, so that
// dL = Re Tr(G^+ dM).  For a product the gradient of a factor is (left part)^+ G (right part)^+; for
// E = exp(X) it is L(X^+, G_E), the Frechet derivative of exp at X^+ in the direction G_E (the adjoint
// of L(X, .) for this inner product), read off the upper right block of exp([[X^+, G_E], [0, X^+]]).
// All arithmetic FP64 (complex128 links and gradients).  The stout gradients are accumulated with atomic adds,
// so the order of the additions (and the last bits of the result) can differ from run to run.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace dirac {

namespace {

template <int N>
struct CM {
    cx<double> e[N][N];
};

template <int N>
__device__ __forceinline__ CM<N> zero() {
    CM<N> r;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) r.e[i][j] = {0.0, 0.0};
    return r;
}

template <int N>
__device__ __forceinline__ CM<N> ident() {
    CM<N> r = zero<N>();
#pragma unroll
    for (int i = 0; i < N; ++i) r.e[i][i] = {1.0, 0.0};
    return r;
}

template <int N>
__device__ __forceinline__ CM<N> mul(const CM<N>& a, const CM<N>& b) {
    CM<N> r;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            cx<double> s{0.0, 0.0};
#pragma unroll
            for (int k = 0; k < N; ++k) cfma(s, a.e[i][k], b.e[k][j]);
            r.e[i][j] = s;
        }
    return r;
}

template <int N>
__device__ __forceinline__ CM<N> adj(const CM<N>& a) {
    CM<N> r;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) r.e[i][j] = cconj(a.e[j][i]);
    return r;
}

template <int N>
__device__ __forceinline__ void add_to(CM<N>& a, const CM<N>& b) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) a.e[i][j] = cadd(a.e[i][j], b.e[i][j]);
}

template <int N>
__device__ __forceinline__ CM<N> scaled(const CM<N>& a, cx<double> s) {
    CM<N> r;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) r.e[i][j] = cmul(s, a.e[i][j]);
    return r;
}

// exp(A) by scaling and squaring: A / 2^s with ||A / 2^s||_1 <= 1/4 (s from `norm_of`, so that a
// block whose off-diagonal part enters linearly can be scaled by its diagonal blocks alone), then an
// 18-term Taylor series, then s squarings.
template <int N>
__device__ CM<N> expm(const CM<N>& A, double norm_of) {
    int s = 0;
    double nrm = norm_of;
    while (nrm > 0.25 && s < 40) {
        nrm *= 0.5;
        ++s;
    }
    const double sc = ldexp(1.0, -s);
    const CM<N> X = scaled(A, cx<double>{sc, 0.0});
    CM<N> term = ident<N>(), sum = ident<N>();
    for (int k = 1; k <= 18; ++k) {
        term = scaled(mul(term, X), cx<double>{1.0 / k, 0.0});
        add_to(sum, term);
    }
    for (int i = 0; i < s; ++i) sum = mul(sum, sum);
    return sum;
}

// max column sum of |entries| of the leading n x n block
template <int N>
__device__ __forceinline__ double norm1(const CM<N>& a, int n) {
    double m = 0.0;
    for (int j = 0; j < n; ++j) {
        double c = 0.0;
        for (int i = 0; i < n; ++i) c += fabs(a.e[i][j].re) + fabs(a.e[i][j].im);
        m = c > m ? c : m;
    }
    return m;
}

template <int NC>
__device__ __forceinline__ CM<NC> load_link(const double2* __restrict__ U, int64_t site, int mu) {
    CM<NC> m;
    const double2* p = U + (site * 4 + mu) * NC * NC;
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            const double2 v = p[a * NC + b];
            m.e[a][b] = {v.x, v.y};
        }
    return m;
}

template <int NC>
__device__ __forceinline__ void atomic_add_link(double2* __restrict__ G, int64_t site, int mu, const CM<NC>& m) {
    double* p = reinterpret_cast<double*>(G + (site * 4 + mu) * NC * NC);
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            atomicAdd(p + 2 * (a * NC + b), m.e[a][b].re);
            atomicAdd(p + 2 * (a * NC + b) + 1, m.e[a][b].im);
        }
}

__device__ __forceinline__ int64_t shifted(const Coord& c, int mu, int s, const Geom& g) {
    int x[4] = {c.x, c.y, c.z, c.t};
    const int ext[4] = {g.nx, g.ny, g.nz, g.nt};
    x[mu] = wrap(x[mu] + s, ext[mu]);
    return site_index(x[0], x[1], x[2], x[3], g);
}

__device__ __forceinline__ int64_t shifted2(const Coord& c, int mu, int s, int nu, int t, const Geom& g) {
    int x[4] = {c.x, c.y, c.z, c.t};
    const int ext[4] = {g.nx, g.ny, g.nz, g.nt};
    x[mu] = wrap(x[mu] + s, ext[mu]);
    x[nu] = wrap(x[nu] + t, ext[nu]);
    return site_index(x[0], x[1], x[2], x[3], g);
}

// C_mu(n) / rho: the six staples
template <int NC>
__device__ CM<NC> staple_sum(const double2* __restrict__ U, int64_t site, const Coord& c, int mu, const Geom& g) {
    CM<NC> acc = zero<NC>();
    for (int nu = 0; nu < 4; ++nu) {
        if (nu == mu) continue;
        const int64_t n_nu = shifted(c, nu, 1, g), n_mu = shifted(c, mu, 1, g);
        add_to(acc, mul(mul(load_link<NC>(U, site, nu), load_link<NC>(U, n_nu, mu)), adj(load_link<NC>(U, n_mu, nu))));
        const int64_t m_nu = shifted(c, nu, -1, g), m_nu_p_mu = shifted2(c, nu, -1, mu, 1, g);
        add_to(acc, mul(mul(adj(load_link<NC>(U, m_nu, nu)), load_link<NC>(U, m_nu, mu)), load_link<NC>(U, m_nu_p_mu, nu)));
    }
    return acc;
}

// X = i Q for the link (mu, n): Q = (i/2)(Omega^+ - Omega) minus its trace, Omega = C U^+
template <int NC>
__device__ __forceinline__ CM<NC> stout_x(const CM<NC>& C, const CM<NC>& Ul) {
    const CM<NC> om = mul(C, adj(Ul));
    CM<NC> a;  // Omega^+ - Omega (anti-hermitian)
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) a.e[i][j] = csub(cconj(om.e[j][i]), om.e[i][j]);
    cx<double> tr{0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NC; ++i) tr = cadd(tr, a.e[i][i]);
#pragma unroll
    for (int i = 0; i < NC; ++i) a.e[i][i] = csub(a.e[i][i], cscale(1.0 / NC, tr));
    // X = i Q = i (i/2) a = -a/2
    return scaled(a, cx<double>{-0.5, 0.0});
}

template <int NC>
__global__ __launch_bounds__(128) void stout_kernel(const double2* __restrict__ U, double2* __restrict__ V, double rho,
                                                    Geom g) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (gid >= 4 * g.vol) return;
    const int64_t site = gid >> 2;
    const int mu = static_cast<int>(gid & 3);
    const Coord c = site_coord(site, g);
    const CM<NC> C = scaled(staple_sum<NC>(U, site, c, mu, g), cx<double>{rho, 0.0});
    const CM<NC> Ul = load_link<NC>(U, site, mu);
    const CM<NC> X = stout_x(C, Ul);
    const CM<NC> Vl = mul(expm(X, norm1(X, NC)), Ul);
    double2* out = V + (site * 4 + mu) * NC * NC;
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) out[a * NC + b] = make_double2(Vl.e[a][b].re, Vl.e[a][b].im);
}

// gU += the gradient with respect to U of L(U'(U)) given gV = dL/dU' (one stout step)
template <int NC>
__global__ __launch_bounds__(64) void stout_backward_kernel(const double2* __restrict__ U,
                                                            const double2* __restrict__ GV,
                                                            double2* __restrict__ GU, double rho, Geom g) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (gid >= 4 * g.vol) return;
    const int64_t site = gid >> 2;
    const int mu = static_cast<int>(gid & 3);
    const Coord c = site_coord(site, g);
    const CM<NC> C = scaled(staple_sum<NC>(U, site, c, mu, g), cx<double>{rho, 0.0});
    const CM<NC> Ul = load_link<NC>(U, site, mu);
    const CM<NC> X = stout_x(C, Ul);
    const double nx = norm1(X, NC);
    const CM<NC> E = expm(X, nx);
    const CM<NC> Gv = load_link<NC>(GV, site, mu);
    // V = E U: direct part E^+ G_V, and G_E = G_V U^+
    CM<NC> gu = mul(adj(E), Gv);
    const CM<NC> GE = mul(Gv, adj(Ul));
    // G_X = L(X^+, G_E) from the block exponential
    constexpr int N2 = 2 * NC;
    CM<N2> M = zero<N2>();
    const CM<NC> Xd = adj(X);
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            M.e[i][j] = Xd.e[i][j];
            M.e[NC + i][NC + j] = Xd.e[i][j];
            M.e[i][NC + j] = GE.e[i][j];
        }
    const CM<N2> EM = expm(M, nx);
    CM<NC> GX;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) GX.e[i][j] = EM.e[i][NC + j];
    // X = i Q -> G_Q = -i G_X; Q = (i/2) A - (i/2N) Tr A -> G_A = (-i/2)(G_Q - Tr(G_Q)/N); A = Om^+ - Om ->
    // G_Om = G_A^+ - G_A; with G_Q = -i G_X: G_A = -(1/2)(G_X - Tr(G_X)/N)
    CM<NC> GA;
    cx<double> trx{0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NC; ++i) trx = cadd(trx, GX.e[i][i]);
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            cx<double> v = GX.e[i][j];
            if (i == j) v = csub(v, cscale(1.0 / NC, trx));
            GA.e[i][j] = cscale(-0.5, v);
        }
    CM<NC> GOm;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) GOm.e[i][j] = csub(cconj(GA.e[j][i]), GA.e[i][j]);
    // Omega = C U^+: G_C = G_Om U, and U gains G_Om^+ C
    add_to(gu, mul(adj(GOm), C));
    atomic_add_link<NC>(GU, site, mu, gu);
    const CM<NC> GP = scaled(mul(GOm, Ul), cx<double>{rho, 0.0});  // gradient of every staple product
    for (int nu = 0; nu < 4; ++nu) {
        if (nu == mu) continue;
        {  // A B D = U_nu(n) U_mu(n+nu) U_nu(n+mu)^+
            const int64_t n_nu = shifted(c, nu, 1, g), n_mu = shifted(c, mu, 1, g);
            const CM<NC> A = load_link<NC>(U, site, nu), B = load_link<NC>(U, n_nu, mu),
                         D = adj(load_link<NC>(U, n_mu, nu));
            atomic_add_link<NC>(GU, site, nu, mul(GP, adj(mul(B, D))));
            atomic_add_link<NC>(GU, n_nu, mu, mul(mul(adj(A), GP), adj(D)));
            atomic_add_link<NC>(GU, n_mu, nu, adj(mul(adj(mul(A, B)), GP)));  // D = U^+: gradient daggered
        }
        {  // A B D = U_nu(n-nu)^+ U_mu(n-nu) U_nu(n-nu+mu)
            const int64_t m_nu = shifted(c, nu, -1, g), m_nu_p_mu = shifted2(c, nu, -1, mu, 1, g);
            const CM<NC> A = adj(load_link<NC>(U, m_nu, nu)), B = load_link<NC>(U, m_nu, mu),
                         D = load_link<NC>(U, m_nu_p_mu, nu);
            atomic_add_link<NC>(GU, m_nu, nu, adj(mul(GP, adj(mul(B, D)))));  // A = U^+
            atomic_add_link<NC>(GU, m_nu, mu, mul(mul(adj(A), GP), adj(D)));
            atomic_add_link<NC>(GU, m_nu_p_mu, nu, mul(adj(mul(A, B)), GP));
        }
    }
}

// ---------------------------------------------------------------------------
// gV += the gradient with respect to V of L(W(V)) given gW = dL/dW for the 40 stored directions.
//
// A path of W_d that uses V_mu(m) forwards splits there into a prefix of displacement a (from n = m - a to m) and a
// suffix of displacement b (from m + mu), d = a + e_mu + b, with a and b in the three other axes and of disjoint
// support.  The paths with the same split are the products W_a(n) V_mu(m) W_b(m + mu), with weight
// |a|! |b|! / |d|!, and W_a(n)^+ = W_{-a}(m), so
//   gV_mu(m) = sum_{a, b} |a|! |b|! / |d|! W_{-a}(m) G_d(m - a) W_b(m + mu)^+
// over the 125 pairs (a, b), where G_d is gW for a stored d and, since W_d(n) = W_{-d}(n + d)^+, the adjoint of
// gW_{-d}(n + d) otherwise (a path that uses V_mu(m) backwards is the reverse of one counted here).  Every output
// is a gather with a fixed order of summation and is added to gV once.
//
// A work-group takes kSplitSites consecutive sites and one mu (blocks of the four mu of a tile are neighbours and
// share the gW lines in L2).  It builds the 26 path averages in the three other axes at m and at m + mu in LDS, level
// by level, one row of a matrix per thread; then a thread owns one column of the output and one of 16 groups of
// pairs, so a product with a pair is a matrix-vector product, and the groups are added across 16 lanes.  The groups
// hold at most 9 pairs each (a = 0 in three groups, |a| = 1 one group each, the rest in seven), which balances them
// to within a tenth.  Bound by the address rate of the gW and V loads (16 bytes a lane, a matrix a few lanes).
// Separate walks along all 1108 paths of a site, with an atomic add per factor, took 7.44 ms at 8^3 x 16 (N_c = 3);
// this takes 0.23 ms.
// ---------------------------------------------------------------------------
constexpr int kSplitSites = 4;
constexpr int kSplitGroups = 16;
constexpr int kSplitPairs = 9;  // the largest group

// Displacements in the three other axes are numbered c = 9 (c_2 + 1) + 3 (c_1 + 1) + c_0 + 1 (13: none; -c: 26 - c).
constexpr int trans_digit(int c, int q) { return (q == 0 ? c : (q == 1 ? c / 3 : c / 9)) % 3 - 1; }
constexpr int trans_order(int c) { return (trans_digit(c, 0) != 0) + (trans_digit(c, 1) != 0) + (trans_digit(c, 2) != 0); }
constexpr int trans_axis(int mu, int q) { return q + (q >= mu); }

// The pairs of one mu, packed, since decoding them with divisions cost more than the products (277 us at 8^3 x 16):
// bits 0-4 26 - a, 5-9 b, 10-15 the stored direction, 16 whether its adjoint is G_d, 17 last pair of this a, 18-21
// 4 |a| + |b|, 22-26 the displacement of the site that holds it (from m, or from m + mu for an adjoint).
struct SplitTable {
    uint32_t pair[4][kSplitGroups][kSplitPairs];
    int count[kSplitGroups];
};
constexpr SplitTable make_split_table() {
    SplitTable t{};
    for (int mu = 0; mu < 4; ++mu) {
        int n0 = 0, n1 = 0, n2 = 0, n3 = 0;
        int cnt[kSplitGroups] = {};
        for (int order = 0; order < 4; ++order)
            for (int a = 0; a < 27; ++a) {
                if (trans_order(a) != order) continue;
                // |a| = 2 (3 pairs each): two to each of groups 9..14; |a| = 3 (1 pair): five to group 15, three more
                const int ga = order == 1 ? 3 + n1 : (order == 2 ? 9 + n2 / 2 : (n3 < 5 ? 15 : 4 + n3));
                int grp = ga;
                for (int b = 0; b < 27; ++b) {
                    int num = 40, stride[4] = {1, 3, 9, 27};
                    bool disjoint = true;
                    num += stride[mu];
                    for (int q = 0; q < 3; ++q) {
                        const int da = trans_digit(a, q), db = trans_digit(b, q);
                        if (da != 0 && db != 0) disjoint = false;
                        num += (da + db) * stride[trans_axis(mu, q)];
                    }
                    if (!disjoint) continue;
                    if (order == 0) grp = n0++ / 9;
                    const bool adj = num > 40;  // -d is stored, at n + d = m + mu + b; else d, at n = m - a
                    t.pair[mu][grp][cnt[grp]++] =
                        static_cast<uint32_t>((26 - a) | b << 5 | (adj ? 80 - num : num) << 10 | (adj ? 1 : 0) << 16 |
                                              (order * 4 + trans_order(b)) << 18 | (adj ? b : 26 - a) << 22);
                }
                n1 += order == 1;
                n2 += order == 2;
                n3 += order == 3;
            }
        for (int grp = 0; grp < kSplitGroups; ++grp) {
            t.count[grp] = cnt[grp];
            for (int e = 0; e < cnt[grp]; ++e)
                if (e + 1 == cnt[grp] || (t.pair[mu][grp][e] & 31u) != (t.pair[mu][grp][e + 1] & 31u))
                    t.pair[mu][grp][e] |= 1u << 17;
        }
    }
    return t;
}
__constant__ SplitTable c_split = make_split_table();
struct TransDirs {
    unsigned char dir[26];  // 6 of order 1, 12 of order 2, 8 of order 3
};
constexpr TransDirs make_trans_dirs() {
    TransDirs t{};
    int n = 0;
    for (int order = 1; order < 4; ++order)
        for (int a = 0; a < 27; ++a)
            if (trans_order(a) == order) t.dir[n++] = static_cast<unsigned char>(a);
    return t;
}
__constant__ TransDirs c_trans = make_trans_dirs();

template <int NC>
__global__ __launch_bounds__(kSplitSites * kSplitGroups * NC) void links_backward_kernel(
    const double2* __restrict__ V, const double2* __restrict__ GW, double2* __restrict__ GV, Geom g) {
    constexpr int S = kSplitSites, L = NC * NC, T = S * kSplitGroups * NC;
    __shared__ cx<double> w[S][2][27][L];  // path averages in the three other axes at m and m + mu (13: identity)
    __shared__ int disp[S][2][27];         // their sites' offsets from m (32 bits: V < 2^31)
    __shared__ uint32_t pairs[kSplitGroups * kSplitPairs];
    const int64_t block = logical_block();
    const int mu = static_cast<int>(block & 3);
    const int64_t site0 = (block >> 2) * S;
    if (site0 >= g.vol) return;
    const int ns = static_cast<int>(g.vol - site0 < S ? g.vol - site0 : S);
    const int tid = threadIdx.x;
    const int ax[3] = {trans_axis(mu, 0), trans_axis(mu, 1), trans_axis(mu, 2)};
    for (int u = tid; u < kSplitGroups * kSplitPairs; u += T) pairs[u] = c_split.pair[mu][0][u];
    for (int u = tid; u < S * 54; u += T) {
        const int s = u / 54, pc = u % 54, c = pc % 27;
        const Coord c0 = site_coord(site0 + (s < ns ? s : 0), g);
        int x[4] = {c0.x, c0.y, c0.z, c0.t};
        const int ext[4] = {g.nx, g.ny, g.nz, g.nt};
#pragma unroll
        for (int nu = 0; nu < 4; ++nu) {
            int v = nu == mu ? pc / 27 : 0;
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (ax[q] == nu) v = trans_digit(c, q);
            x[nu] = wrap(x[nu] + v, ext[nu]);
        }
        disp[s][pc / 27][c] =
            static_cast<int>(site_index(x[0], x[1], x[2], x[3], g) - site0);
    }
    for (int u = tid; u < S * 2 * L; u += T) {
        const int e = u % L;
        w[u / (2 * L)][(u / L) & 1][13][e] = {e % (NC + 1) == 0 ? 1.0 : 0.0, 0.0};
    }
    __syncthreads();

    auto level = [&](auto order_c) __attribute__((always_inline)) {
        constexpr int ORDER = decltype(order_c)::value;
        constexpr int FIRST = ORDER == 1 ? 0 : (ORDER == 2 ? 6 : 18), CNT = ORDER == 1 ? 6 : (ORDER == 2 ? 12 : 8);
        for (int u = tid; u < ns * 2 * CNT * NC; u += T) {
            const int i = u % NC, q = u / NC;
            const int dir = c_trans.dir[FIRST + q % CNT];
            const int p = (q / CNT) & 1, s = q / (2 * CNT);
            const double2* lp[ORDER];
            int prev[ORDER];
            bool fwd[ORDER];
            int n = 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int step = trans_digit(dir, k);
                const int pv = dir - step * (k == 0 ? 1 : (k == 1 ? 3 : 9));  // one step shorter
                // the last step's link: V_nu(n + d - e_nu) forwards, V_nu(n + d)^+ backwards
                const double2* l = V + ((site0 + disp[s][p][step > 0 ? pv : dir]) * 4 + ax[k]) * L;
#pragma unroll
                for (int o = 0; o < ORDER; ++o)
                    if (step != 0 && n == o) {
                        lp[o] = l;
                        prev[o] = pv;
                        fwd[o] = step > 0;
                    }
                n += step != 0;
            }
            cx<double> row[NC];
#pragma unroll
            for (int j = 0; j < NC; ++j) row[j] = {0.0, 0.0};
#pragma unroll
            for (int o = 0; o < ORDER; ++o) {
                const cx<double>* pr = &w[s][p][prev[o]][i * NC];
#pragma unroll
                for (int e = 0; e < NC; ++e)
#pragma unroll
                    for (int j = 0; j < NC; ++j) {
                        const double2 v = lp[o][fwd[o] ? e * NC + j : j * NC + e];
                        cfma(row[j], pr[e], cx<double>{v.x, fwd[o] ? v.y : -v.y});
                    }
            }
#pragma unroll
            for (int j = 0; j < NC; ++j) w[s][p][dir][i * NC + j] = cscale(1.0 / ORDER, row[j]);
        }
        __syncthreads();
    };
    level(std::integral_constant<int, 1>{});
    level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{});

    const int grp = tid % kSplitGroups;
    const int j = (tid / kSplitGroups) % NC;
    const int s = tid / (kSplitGroups * NC);
    if (s >= ns) return;
    cx<double> col[NC], in[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) col[i] = in[i] = {0.0, 0.0};
    const int cnt = c_split.count[grp];
    for (int e = 0; e < cnt; ++e) {
        const uint32_t pk = pairs[grp * kSplitPairs + e];
        const int kab = (pk >> 18) & 15, ka = kab >> 2, kb = kab & 3;
        const bool adj = (pk >> 16) & 1;
        const double fa = ka == 3 ? 6.0 : (ka == 2 ? 2.0 : 1.0), fb = kb == 3 ? 6.0 : (kb == 2 ? 2.0 : 1.0);
        const double wt = fa * fb * (ka + kb == 3 ? 1.0 / 24.0 : (ka + kb == 2 ? 1.0 / 6.0 : (ka + kb == 1 ? 0.5 : 1.0)));
        const double2* gp = GW + ((site0 + disp[s][adj ? 1 : 0][pk >> 22]) * 40 + ((pk >> 10) & 63)) * L;
        const cx<double>* wb = &w[s][1][(pk >> 5) & 31][j * NC];  // column j of W_b(m + mu)^+: row j conjugated
        const int si = adj ? 1 : NC, sk = adj ? NC : 1;
        const double sg = adj ? -1.0 : 1.0;
        double2 z[L];
#pragma unroll
        for (int i = 0; i < NC; ++i)
#pragma unroll
            for (int k = 0; k < NC; ++k) z[i * NC + k] = gp[i * si + k * sk];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const cx<double> v{wt * wb[k].re, -wt * wb[k].im};
#pragma unroll
            for (int i = 0; i < NC; ++i) cfma(in[i], cx<double>{z[i * NC + k].x, sg * z[i * NC + k].y}, v);
        }
        if ((pk >> 17) & 1) {  // the last pair of this a: apply W_{-a}(m)
            const cx<double>* wa = w[s][0][pk & 31];
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
                for (int k = 0; k < NC; ++k) cfma(col[i], wa[i * NC + k], in[k]);
#pragma unroll
            for (int i = 0; i < NC; ++i) in[i] = {0.0, 0.0};
        }
    }
#pragma unroll
    for (int h = 1; h < kSplitGroups; h <<= 1)
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            col[i].re += __shfl_xor(col[i].re, h, kSplitGroups);
            col[i].im += __shfl_xor(col[i].im, h, kSplitGroups);
        }
    if (grp == 0) {
        double* o = reinterpret_cast<double*>(GV + ((site0 + s) * 4 + mu) * L + j);
#pragma unroll
        for (int i = 0; i < NC; ++i) {  // one add per element; atomic, so calls on two streams may share gV
            atomicAdd(o + 2 * i * NC, col[i].re);
            atomicAdd(o + 2 * i * NC + 1, col[i].im);
        }
    }
}

template <int NC>
int launch_nc(int which, const Geom& g, const void* a, const void* b, void* out, double rho, hipStream_t st) {
    auto A = static_cast<const double2*>(a);
    auto B = static_cast<const double2*>(b);
    auto O = static_cast<double2*>(out);
    if (which == 0) {
        const int block = 128;
        hipLaunchKernelGGL((stout_kernel<NC>), dim3(static_cast<unsigned>((4 * g.vol + block - 1) / block)),
                           dim3(block), 0, st, A, O, rho, g);
    } else if (which == 1) {
        const int block = 64;
        hipLaunchKernelGGL((stout_backward_kernel<NC>), dim3(static_cast<unsigned>((4 * g.vol + block - 1) / block)),
                           dim3(block), 0, st, A, B, O, rho, g);
    } else {
        const int64_t blocks = (g.vol + kSplitSites - 1) / kSplitSites * 4;
        hipLaunchKernelGGL((links_backward_kernel<NC>), dim3(static_cast<unsigned>(grid_blocks_x8(blocks, 1))),
                           dim3(kSplitSites * kSplitGroups * NC), 0, st, A, B, O, g);
    }
    return DIRAC_OK;
}

int dispatch(int which, int nc, const Geom& g, const void* a, const void* b, void* out, double rho, hipStream_t st) {
    switch (nc) {
        case 1: return launch_nc<1>(which, g, a, b, out, rho, st);
        case 2: return launch_nc<2>(which, g, a, b, out, rho, st);
        case 3: return launch_nc<3>(which, g, a, b, out, rho, st);
        case 4: return launch_nc<4>(which, g, a, b, out, rho, st);
    }
    return DIRAC_EUNSUPPORTED;
}

}  // namespace

int launch_stout(int nc, const Geom& g, const void* U, void* V, double rho, hipStream_t st) {
    return dispatch(0, nc, g, U, nullptr, V, rho, st);
}

int launch_stout_backward(int nc, const Geom& g, const void* U, const void* gV, void* gU, double rho, hipStream_t st) {
    return dispatch(1, nc, g, U, gV, gU, rho, st);
}

int launch_links_backward(int nc, const Geom& g, const void* V, const void* gW, void* gV, hipStream_t st) {
    return dispatch(2, nc, g, V, gW, gV, 0.0, st);
}

}  // namespace dirac
