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
// All arithmetic FP64 (complex128 links and gradients).  With a workspace the stout gradients are gathered in a fixed
// order (the same bits from run to run); without one they are accumulated with atomic adds, whose order and so the
// last bits of the result can differ.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace dirac {

namespace {

template <int N>
struct CM {
    cx<double> e[N][N];
};

// The row kernels of a smearing step (the backward passes, and the forward pass where stout_link_kernel does not take
// it) give a link N_c threads: thread i owns row i of every matrix, so that a product
// row x matrix needs no exchange and only the right factor is held whole.  Rows meet in LDS where a whole matrix or
// an adjoint's row is needed.  A work-group takes kStoutLinks links; each XCD takes a contiguous range of them, whose
// neighbours its L2 then holds (a gather 38 against 39.7 us, a step's first kernel 26.1 against 27.0, at 8^3 x 16).
constexpr int kStoutLinks = 64;

template <int N>
struct Row {
    cx<double> e[N];
};

// r m
template <int N>
__device__ __forceinline__ Row<N> mul(const Row<N>& r, const CM<N>& m) {
    Row<N> o;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        cx<double> s{0.0, 0.0};
#pragma unroll
        for (int k = 0; k < N; ++k) cfma(s, r.e[k], m.e[k][j]);
        o.e[j] = s;
    }
    return o;
}

// r m^+
template <int N>
__device__ __forceinline__ Row<N> mul_adj(const Row<N>& r, const CM<N>& m) {
    Row<N> o;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        cx<double> s{0.0, 0.0};
#pragma unroll
        for (int k = 0; k < N; ++k) cfma_conj(s, m.e[j][k], r.e[k]);
        o.e[j] = s;
    }
    return o;
}

template <int N>
__device__ __forceinline__ void add_to(Row<N>& a, const Row<N>& b) {
#pragma unroll
    for (int j = 0; j < N; ++j) a.e[j] = cadd(a.e[j], b.e[j]);
}

template <int N>
__device__ __forceinline__ Row<N> scaled(const Row<N>& a, double s) {
    Row<N> r;
#pragma unroll
    for (int j = 0; j < N; ++j) r.e[j] = cscale(s, a.e[j]);
    return r;
}

// Whole matrix, row i and row i of the adjoint of a stored N x N block (of the links, or of rows met in LDS)
template <int N, typename E>
__device__ __forceinline__ CM<N> whole(const E* p) {
    CM<N> m;
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
        for (int b = 0; b < N; ++b) m.e[a][b] = {p[a * N + b].x, p[a * N + b].y};
    return m;
}
template <int N, typename E>
__device__ __forceinline__ Row<N> row_of(const E* p, int i) {
    Row<N> r;
#pragma unroll
    for (int j = 0; j < N; ++j) r.e[j] = {p[i * N + j].x, p[i * N + j].y};
    return r;
}
template <int N, typename E>
__device__ __forceinline__ Row<N> adj_row_of(const E* p, int i) {
    Row<N> r;
#pragma unroll
    for (int j = 0; j < N; ++j) r.e[j] = {p[j * N + i].x, -p[j * N + i].y};
    return r;
}
template <int N>
__device__ __forceinline__ void put_row(double2* p, int i, const Row<N>& r) {
#pragma unroll
    for (int j = 0; j < N; ++j) p[i * N + j] = make_double2(r.e[j].re, r.e[j].im);
}

template <int NC>
__device__ __forceinline__ void atomic_add_row(double2* __restrict__ G, int64_t site, int mu, int i, const Row<NC>& r) {
    double* p = reinterpret_cast<double*>(G + ((site * 4 + mu) * NC + i) * NC);
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        atomicAdd(p + 2 * j, r.e[j].re);
        atomicAdd(p + 2 * j + 1, r.e[j].im);
    }
}

__device__ __forceinline__ int64_t shifted(const Coord& c, int mu, int s, const Geom& g) {
    return site_index(wrap(c.x + (mu == 0 ? s : 0), g.nx), wrap(c.y + (mu == 1 ? s : 0), g.ny),
                      wrap(c.z + (mu == 2 ? s : 0), g.nz), wrap(c.t + (mu == 3 ? s : 0), g.nt), g);
}

__device__ __forceinline__ int64_t shifted2(const Coord& c, int mu, int s, int nu, int t, const Geom& g) {
    return site_index(wrap(c.x + (mu == 0 ? s : (nu == 0 ? t : 0)), g.nx),
                      wrap(c.y + (mu == 1 ? s : (nu == 1 ? t : 0)), g.ny),
                      wrap(c.z + (mu == 2 ? s : (nu == 2 ? t : 0)), g.nz),
                      wrap(c.t + (mu == 3 ? s : (nu == 3 ? t : 0)), g.nt), g);
}

// One thread's place: row i of the link (site, mu).  Threads past the last link shadow it without storing (they
// take part in the barriers).
struct LinkRow {
    int64_t site;
    int mu, i, slot;  // slot: the link's place in the work-group
    bool active;
    Coord c;
};
template <int NC>
__device__ __forceinline__ LinkRow link_row(const Geom& g, int64_t first) {
    LinkRow l;
    l.slot = static_cast<int>(threadIdx.x) / NC;
    l.i = static_cast<int>(threadIdx.x) - l.slot * NC;
    int64_t link = (first + logical_block()) * kStoutLinks + l.slot;
    l.active = link < 4 * g.vol;
    if (!l.active) link = 4 * g.vol - 1;
    l.site = link >> 2;
    l.mu = static_cast<int>(link & 3);
    l.c = site_coord(l.site, g);
    return l;
}

// Row i of C_mu(n) / rho: the six staples
template <int NC>
__device__ __forceinline__ Row<NC> staple_row(const double2* __restrict__ U, const LinkRow& l, const Geom& g) {
    constexpr int L = NC * NC;
    Row<NC> acc;
#pragma unroll
    for (int j = 0; j < NC; ++j) acc.e[j] = {0.0, 0.0};
    const int64_t n_mu = shifted(l.c, l.mu, 1, g);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int nu = k + (k >= l.mu);
        const int64_t n_nu = shifted(l.c, nu, 1, g), m_nu = shifted(l.c, nu, -1, g);
        const int64_t m_nu_p_mu = shifted2(l.c, nu, -1, l.mu, 1, g);
        const Row<NC> up = mul(row_of<NC>(U + (l.site * 4 + nu) * L, l.i), whole<NC>(U + (n_nu * 4 + l.mu) * L));
        add_to(acc, mul_adj(up, whole<NC>(U + (n_mu * 4 + nu) * L)));
        const Row<NC> dn = mul(adj_row_of<NC>(U + (m_nu * 4 + nu) * L, l.i), whole<NC>(U + (m_nu * 4 + l.mu) * L));
        add_to(acc, mul(dn, whole<NC>(U + (m_nu_p_mu * 4 + nu) * L)));
    }
    return acc;
}

// Row i of half the traceless anti-hermitian part of a matrix met in LDS, with the sign of the adjoint:
// (A - Tr A / N) / 2 with A = M - M^+
template <int NC>
__device__ __forceinline__ Row<NC> traceless_row(const double2* m, int i) {
    const Row<NC> r = row_of<NC>(m, i), d = adj_row_of<NC>(m, i);
    double tr = 0.0;  // the trace of M - M^+ is 2 i tr
#pragma unroll
    for (int k = 0; k < NC; ++k) tr += m[k * NC + k].y;
    Row<NC> o;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        o.e[j] = cscale(0.5, csub(r.e[j], d.e[j]));
        if (j == i) o.e[j].im -= tr / NC;
    }
    return o;
}

// max column sum of |entries|
template <int N>
__device__ __forceinline__ double norm1(const CM<N>& a) {
    double m = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double c = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) c += fabs(a.e[i][j].re) + fabs(a.e[i][j].im);
        m = c > m ? c : m;
    }
    return m;
}

// Rows of E = exp(A) and, with FRECHET, of D = L(A, G), the upper right block of exp([[A, G], [0, A]]), by scaling
// and squaring: A and G over 2^s with ||A / 2^s||_1 <= 1/4, a Taylor series of both (T_k = T_{k-1} A / k,
// D_k = (D_{k-1} A + T_{k-1} G) / k; at 1/4 its 14 terms leave 1e-21), then s times E <- E E, D <- E D + D E.
// Carrying the two blocks instead of the 2N x 2N matrix is a quarter of its products.  e, d: LDS for the rows of
// the work-group's links; the squarings of the work-group are counted in `squarings` (LDS, zero on entry).
constexpr int kExpTerms = 14;
template <int NC, bool FRECHET>
__device__ __forceinline__ void exp_rows(CM<NC> A, CM<NC> G, int i, double2* e, double2* d, int* squarings, Row<NC>& E,
                                         Row<NC>& D) {
    int s = 0;
    for (double nrm = norm1(A); nrm > 0.25 && s < 40; nrm *= 0.5) ++s;
    const double sc = ldexp(1.0, -s);
#pragma unroll
    for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            A.e[a][b] = cscale(sc, A.e[a][b]);
            if constexpr (FRECHET) G.e[a][b] = cscale(sc, G.e[a][b]);
        }
    Row<NC> T, Dk;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        T.e[j] = E.e[j] = {j == i ? 1.0 : 0.0, 0.0};
        Dk.e[j] = D.e[j] = {0.0, 0.0};
    }
#pragma unroll 1
    for (int k = 1; k <= kExpTerms; ++k) {
        const double inv = 1.0 / k;
        if constexpr (FRECHET) {
            Dk = mul(Dk, A);
            add_to(Dk, mul(T, G));
            Dk = scaled(Dk, inv);
            add_to(D, Dk);
        }
        T = scaled(mul(T, A), inv);
        add_to(E, T);
    }
    atomicMax(squarings, s);
    __syncthreads();
    const int most = *squarings;
    for (int q = 0; q < most; ++q) {
        put_row<NC>(e, i, E);
        if constexpr (FRECHET) put_row<NC>(d, i, D);
        __syncthreads();
        if (q < s) {
            const CM<NC> W = whole<NC>(e);
            if constexpr (FRECHET) {
                D = mul(D, W);
                add_to(D, mul(E, whole<NC>(d)));
            }
            E = mul(E, W);
        }
        __syncthreads();
    }
}

// V = exp(i Q) U for every link.  i Q = -(A - Tr A / N) / 2 with A = Omega^+ - Omega.
template <int NC>
__global__ __launch_bounds__(kStoutLinks * NC) void stout_kernel(const double2* __restrict__ U, double2* __restrict__ V,
                                                                 double rho, Geom g, int64_t first) {
    constexpr int L = NC * NC;
    __shared__ double2 m0[kStoutLinks][L], m1[kStoutLinks][L];
    __shared__ int squarings;
    if (threadIdx.x == 0) squarings = 0;
    const LinkRow l = link_row<NC>(g, first);
    double2* const b0 = m0[l.slot];
    double2* const b1 = m1[l.slot];
    const double2* up = U + (l.site * 4 + l.mu) * L;
    const Row<NC> C = scaled(staple_row<NC>(U, l, g), rho);
    put_row<NC>(b0, l.i, mul_adj(C, whole<NC>(up)));  // Omega
    __syncthreads();
    put_row<NC>(b1, l.i, traceless_row<NC>(b0, l.i));  // i Q
    __syncthreads();
    const CM<NC> X = whole<NC>(b1);
    Row<NC> E, D;
    exp_rows<NC, false>(X, X, l.i, b0, b1, &squarings, E, D);
    if (l.active) put_row<NC>(V + (l.site * 4 + l.mu) * L, l.i, mul(E, whole<NC>(up)));
}

// The same with one thread per link, which holds whole matrices: the threads of a link otherwise read every right factor
// N_c times.  Faster where the links fill the chip (N_c = 4: 24^4 891 against 1200 us, 8^3 x 16 34 and 34, 4^4 29 against 21;
// N_c = 3: 16^3 x 8 46 against 55, 24^4 418 and 419, 4^4 14 against 11) and for N_c = 1 (18 against 21 us at 16^3 x 32), not
// for N_c = 2 (24^4 167 against 142).
template <int NC>
constexpr int64_t kStoutLinkSites = NC == 1 ? 0 : (NC == 2 ? INT64_MAX : 8192);  // from this volume on
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
__device__ __forceinline__ CM<N> adjoint(const CM<N>& a) {
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
__device__ __forceinline__ CM<N> scaled(const CM<N>& a, double s) {
    CM<N> r;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) r.e[i][j] = cscale(s, a.e[i][j]);
    return r;
}

template <int NC>
__global__ __launch_bounds__(128) void stout_link_kernel(const double2* __restrict__ U, double2* __restrict__ V,
                                                         double rho, Geom g, int64_t first) {
    constexpr int L = NC * NC;
    const int64_t link = (first + logical_block()) * blockDim.x + threadIdx.x;
    if (link >= 4 * g.vol) return;
    const int64_t site = link >> 2;
    const int mu = static_cast<int>(link & 3);
    const Coord c = site_coord(site, g);
    CM<NC> x;  // the staples, then Omega, then i Q
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) x.e[i][j] = {0.0, 0.0};
    const int64_t n_mu = shifted(c, mu, 1, g);
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const int nu = k + (k >= mu);
        const int64_t n_nu = shifted(c, nu, 1, g), m_nu = shifted(c, nu, -1, g), m_nu_p_mu = shifted2(c, nu, -1, mu, 1, g);
        add_to(x, mul(mul(whole<NC>(U + (site * 4 + nu) * L), whole<NC>(U + (n_nu * 4 + mu) * L)),
                      adjoint(whole<NC>(U + (n_mu * 4 + nu) * L))));
        add_to(x, mul(mul(adjoint(whole<NC>(U + (m_nu * 4 + nu) * L)), whole<NC>(U + (m_nu * 4 + mu) * L)),
                      whole<NC>(U + (m_nu_p_mu * 4 + nu) * L)));
    }
    const CM<NC> u = whole<NC>(U + link * L);
    x = mul(scaled(x, rho), adjoint(u));
    double tr = 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) tr += x.e[i][i].im;
    const CM<NC> d = adjoint(x);
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            x.e[i][j] = cscale(0.5, csub(x.e[i][j], d.e[i][j]));
            if (i == j) x.e[i][j].im -= tr / NC;
        }
    int s = 0;  // the series and squarings of exp_rows
    for (double nrm = norm1(x); nrm > 0.25 && s < 40; nrm *= 0.5) ++s;
    x = scaled(x, ldexp(1.0, -s));
    CM<NC> T, E;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) T.e[i][j] = E.e[i][j] = {i == j ? 1.0 : 0.0, 0.0};
#pragma unroll 1
    for (int k = 1; k <= kExpTerms; ++k) {
        T = scaled(mul(T, x), 1.0 / k);
        add_to(E, T);
    }
#pragma unroll 1
    for (int q = 0; q < s; ++q) E = mul(E, E);
    const CM<NC> v = mul(E, u);
    double2* o = V + link * L;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) o[i * NC + j] = make_double2(v.e[i][j].re, v.e[i][j].im);
}

// gU += the gradient with respect to U of L(U'(U)) given gV = dL/dU' (one stout step).  A link passes the gradient of
// its staple products, G_P, on to the 18 links of its staples.  With a workspace (SCATTER false) the link's own part
// and G_P are stored there, two link fields, and stout_gather_kernel collects the 18 parts of every link; without,
// they are added with atomics, 19 matrices a link, which the atomic rate bounds (28 G/s: 437 us at 8^3 x 16 with
// N_c = 3, 587 with a thread per link and the 2N x 2N exponential in scratch memory; gathered: 27 + 40 us).
template <int NC, bool SCATTER>
__global__ __launch_bounds__(kStoutLinks * NC) void stout_backward_kernel(const double2* __restrict__ U,
                                                                          const double2* __restrict__ GV,
                                                                          double2* __restrict__ GU,
                                                                          double2* __restrict__ ws, double rho, Geom g,
                                                                          int64_t first) {
    constexpr int L = NC * NC;
    __shared__ double2 m0[kStoutLinks][L], m1[kStoutLinks][L], m2[kStoutLinks][L];
    __shared__ int squarings;
    if (threadIdx.x == 0) squarings = 0;
    const LinkRow l = link_row<NC>(g, first);
    double2* const b0 = m0[l.slot];
    double2* const b1 = m1[l.slot];
    double2* const b2 = m2[l.slot];
    const double2* up = U + (l.site * 4 + l.mu) * L;
    const double2* gvp = GV + (l.site * 4 + l.mu) * L;
    Row<NC> gu;
    {
        const Row<NC> C = scaled(staple_row<NC>(U, l, g), rho);
        put_row<NC>(b1, l.i, C);
        const CM<NC> Ul = whole<NC>(up);
        put_row<NC>(b0, l.i, mul_adj(C, Ul));                           // Omega
        put_row<NC>(b2, l.i, mul_adj(row_of<NC>(gvp, l.i), Ul));       // V = E U: G_E = G_V U^+
    }
    __syncthreads();
    Row<NC> E, GX;
    {
        // X = i Q is anti-hermitian: A = X^+ = -X, and exp(A) = E^+
        const Row<NC> A = scaled(traceless_row<NC>(b0, l.i), -1.0);
        const CM<NC> GE = whole<NC>(b2);
        __syncthreads();
        put_row<NC>(b0, l.i, A);
        __syncthreads();
        const CM<NC> Am = whole<NC>(b0);
        __syncthreads();
        exp_rows<NC, true>(Am, GE, l.i, b0, b2, &squarings, E, GX);  // G_X = L(X^+, G_E)
    }
    gu = mul(E, whole<NC>(gvp));  // direct part E^+ G_V
    put_row<NC>(b0, l.i, GX);
    __syncthreads();
    // X = i Q -> G_Q = -i G_X; Q = (i/2) A - (i/2N) Tr A -> G_A = -(1/2)(G_X - Tr(G_X)/N) with A = Om^+ - Om ->
    // G_Om = G_A^+ - G_A: the traceless anti-hermitian part of G_X
    const Row<NC> GOm = traceless_row<NC>(b0, l.i);
    // Omega = C U^+: U gains G_Om^+ C = -G_Om C, and G_C = G_Om U
    add_to(gu, scaled(mul(GOm, whole<NC>(b1)), -1.0));
    const Row<NC> gp = scaled(mul(GOm, whole<NC>(up)), rho);  // gradient of every staple product
    if constexpr (!SCATTER) {
        if (l.active) {
            put_row<NC>(ws + (l.site * 4 + l.mu) * L, l.i, gp);
            put_row<NC>(ws + ((g.vol + l.site) * 4 + l.mu) * L, l.i, gu);
        }
        return;
    }
    put_row<NC>(b2, l.i, gp);
    if (l.active) atomic_add_row<NC>(GU, l.site, l.mu, l.i, gu);
    __syncthreads();
    if (!l.active) return;
    const CM<NC> GP = whole<NC>(b2);
    const Row<NC> gpd = adj_row_of<NC>(b2, l.i);
    const int mu = l.mu, i = l.i;
    const int64_t n_mu = shifted(l.c, mu, 1, g);
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const int nu = k + (k >= mu);
        {  // A B D^+ = U_nu(n) U_mu(n+nu) U_nu(n+mu)^+
            const int64_t n_nu = shifted(l.c, nu, 1, g);
            const double2 *a = U + (l.site * 4 + nu) * L, *b = U + (n_nu * 4 + mu) * L, *d = U + (n_mu * 4 + nu) * L;
            const CM<NC> B = whole<NC>(b), D = whole<NC>(d);
            atomic_add_row<NC>(GU, l.site, nu, i, mul_adj(mul(gp, D), B));              // G (B D^+)^+
            atomic_add_row<NC>(GU, n_nu, mu, i, mul(mul(adj_row_of<NC>(a, i), GP), D));  // A^+ G D
            atomic_add_row<NC>(GU, n_mu, nu, i, mul(mul(gpd, whole<NC>(a)), B));         // G^+ A B
        }
        {  // A^+ B D = U_nu(n-nu)^+ U_mu(n-nu) U_nu(n-nu+mu)
            const int64_t m_nu = shifted(l.c, nu, -1, g), m_nu_p_mu = shifted2(l.c, nu, -1, mu, 1, g);
            const double2 *a = U + (m_nu * 4 + nu) * L, *b = U + (m_nu * 4 + mu) * L, *d = U + (m_nu_p_mu * 4 + nu) * L;
            const CM<NC> A = whole<NC>(a), D = whole<NC>(d);
            const Row<NC> bd = mul(row_of<NC>(b, i), D);
            atomic_add_row<NC>(GU, m_nu, nu, i, mul_adj(bd, GP));                       // B D G^+
            atomic_add_row<NC>(GU, m_nu, mu, i, mul_adj(mul(row_of<NC>(a, i), GP), D));  // A G D^+
            atomic_add_row<NC>(GU, m_nu_p_mu, nu, i, mul(mul(adj_row_of<NC>(b, i), A), GP));  // B^+ A G
        }
    }
}

// gU of the link (nu, m) from the workspace of stout_backward_kernel: its own part and, for each other axis la, its
// six places in the staples of other links, G the staple gradient of the link at the site and direction given:
//   staples of links along la:  G(m) U_nu(m+la) U_la(m+nu)^+,  G(m-la)^+ U_nu(m-la) U_la(m-la+nu),
//                               U_la(m) U_nu(m+la) G(m+nu)^+,  U_la(m-la)^+ U_nu(m-la) G(m-la+nu);
//   staples of links along nu:  U_la(m-la)^+ G(m-la) U_la(m-la+nu),  U_la(m) G(m+la) U_la(m+nu)^+.
template <int NC>
__global__ __launch_bounds__(kStoutLinks * NC) __attribute__((amdgpu_waves_per_eu(NC <= 3 ? 2 : 1))) void stout_gather_kernel(const double2* __restrict__ U,
                                                                        const double2* __restrict__ ws,
                                                                        double2* __restrict__ GU, Geom g, int64_t first) {
    constexpr int L = NC * NC;
    const LinkRow l = link_row<NC>(g, first);
    if (!l.active) return;
    const int nu = l.mu, i = l.i;
    Row<NC> acc = row_of<NC>(ws + ((g.vol + l.site) * 4 + nu) * L, i);
    const int64_t m_nu = shifted(l.c, nu, 1, g);
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const int la = k + (k >= nu);
        const int64_t p = shifted(l.c, la, 1, g), q = shifted(l.c, la, -1, g), q_nu = shifted2(l.c, la, -1, nu, 1, g);
        const double2 *ula = U + (l.site * 4 + la) * L, *ula_q = U + (q * 4 + la) * L;
        {
            const CM<NC> u = whole<NC>(U + (p * 4 + nu) * L);
            add_to(acc, mul_adj(mul(row_of<NC>(ws + (l.site * 4 + la) * L, i), u), whole<NC>(U + (m_nu * 4 + la) * L)));
            add_to(acc, mul_adj(mul(row_of<NC>(ula, i), u), whole<NC>(ws + (m_nu * 4 + la) * L)));
        }
        {
            const CM<NC> u = whole<NC>(U + (q * 4 + nu) * L);
            add_to(acc, mul(mul(adj_row_of<NC>(ula_q, i), u), whole<NC>(ws + (q_nu * 4 + la) * L)));
            const CM<NC> v = whole<NC>(U + (q_nu * 4 + la) * L);
            add_to(acc, mul(mul(adj_row_of<NC>(ws + (q * 4 + la) * L, i), u), v));
            add_to(acc, mul(mul(adj_row_of<NC>(ula_q, i), whole<NC>(ws + (q * 4 + nu) * L)), v));
        }
        add_to(acc, mul_adj(mul(row_of<NC>(ula, i), whole<NC>(ws + (p * 4 + nu) * L)), whole<NC>(U + (m_nu * 4 + la) * L)));
    }
    atomic_add_row<NC>(GU, l.site, nu, i, acc);  // one add per element; atomic, so calls on two streams may share gU
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
    const double2* __restrict__ V, const double2* __restrict__ GW, double2* __restrict__ GV, Geom g, int64_t first) {
    constexpr int S = kSplitSites, L = NC * NC, T = S * kSplitGroups * NC;
    __shared__ cx<double> w[S][2][27][L];  // path averages in the three other axes at m and m + mu (13: identity)
    __shared__ int disp[S][2][27];         // their sites' offsets from m (32 bits: V < 2^31)
    __shared__ uint32_t pairs[kSplitGroups * kSplitPairs];
    const int64_t block = first + logical_block();
    const int mu = static_cast<int>(block & 3);
    const int64_t site0 = (block >> 2) * S;
    if (site0 >= g.vol) return;
    const int ns = static_cast<int>(g.vol - site0 < S ? g.vol - site0 : S);
    const int tid = threadIdx.x;
    const int ax[3] = {trans_axis(mu, 0), trans_axis(mu, 1), trans_axis(mu, 2)};
    for (int u = tid; u < kSplitGroups * kSplitPairs; u += T) pairs[u] = c_split.pair[mu][0][u];
    __shared__ Coord at[S];
    if (tid < S) at[tid] = site_coord(site0 + (tid < ns ? tid : 0), g);
    __syncthreads();
    for (int u = tid; u < S * 54; u += T) {
        const int s = u / 54, pc = u % 54, c = pc % 27;
        const Coord c0 = at[s];
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
int launch_nc(int which, const Geom& g, const void* a, const void* b, void* out, double rho, hipStream_t st,
              void* ws) {
    auto A = static_cast<const double2*>(a);
    auto B = static_cast<const double2*>(b);
    auto O = static_cast<double2*>(out);
    auto slices = [&](int64_t blocks, int threads, auto kern, auto... args) {
        launch_slices(blocks, threads, [&](int64_t first, unsigned grid) {
            hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), 0, st, args..., g, first);
        });
    };
    const int64_t groups = (4 * g.vol + kStoutLinks - 1) / kStoutLinks;
    if (which == 0) {
        if constexpr (kStoutLinkSites<NC> != INT64_MAX) {
            if (g.vol >= kStoutLinkSites<NC>) {
                slices((4 * g.vol + 127) / 128, 128, stout_link_kernel<NC>, A, O, rho);
                return DIRAC_OK;
            }
        }
        slices(groups, kStoutLinks * NC, stout_kernel<NC>, A, O, rho);
    } else if (which == 1) {
        auto w = static_cast<double2*>(ws);
        if (w) {
            slices(groups, kStoutLinks * NC, stout_backward_kernel<NC, false>, A, B, O, w, rho);
            slices(groups, kStoutLinks * NC, stout_gather_kernel<NC>, A, static_cast<const double2*>(w), O);
        } else {
            slices(groups, kStoutLinks * NC, stout_backward_kernel<NC, true>, A, B, O, w, rho);
        }
    } else {
        slices((g.vol + kSplitSites - 1) / kSplitSites * 4, kSplitSites * kSplitGroups * NC, links_backward_kernel<NC>,
               A, B, O);
    }
    return DIRAC_OK;
}

int dispatch(int which, int nc, const Geom& g, const void* a, const void* b, void* out, double rho, hipStream_t st,
             void* ws = nullptr) {
    switch (nc) {
        case 1: return launch_nc<1>(which, g, a, b, out, rho, st, ws);
        case 2: return launch_nc<2>(which, g, a, b, out, rho, st, ws);
        case 3: return launch_nc<3>(which, g, a, b, out, rho, st, ws);
        case 4: return launch_nc<4>(which, g, a, b, out, rho, st, ws);
    }
    return DIRAC_EUNSUPPORTED;
}

}  // namespace

int launch_stout(int nc, const Geom& g, const void* U, void* V, double rho, hipStream_t st) {
    return dispatch(0, nc, g, U, nullptr, V, rho, st);
}

int launch_stout_backward(int nc, const Geom& g, const void* U, const void* gV, void* gU, double rho, void* ws,
                          hipStream_t st) {
    return dispatch(1, nc, g, U, gV, gU, rho, st, ws);
}

int launch_links_backward(int nc, const Geom& g, const void* V, const void* gW, void* gV, hipStream_t st) {
    return dispatch(2, nc, g, V, gW, gV, 0.0, st);
}

}  // namespace dirac
