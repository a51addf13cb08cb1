// hmc.hip -- hybrid Monte Carlo around the staggered solver: the simulation
// layer that the paper's backends serve (Sec. 3: HMC, the gauge action and its
// derivatives; the inversion inside it is the dominant cost, Sec. 1).
//
// State in the canonical link layout [4][V][3][3] complex128 (the layout of
// lqs_gauge_create), momenta Q in the same layout (anti-Hermitian traceless).
//   S_g = beta sum_x sum_{mu<nu} (1 - Re tr P_{mu nu}(x) / 3)   (periodic links)
//   K   = -sum_links tr Q^2
//   S_f = phi^dag M^-1 phi,  phi = m eta_e - D_eo eta_o
//   dU/dtau = Q U,  dQ/dtau = -F/2,  F = F_g + F_f with
//   F_g = (beta/3) TA(U V) (V: staple sum), F_f = -TA(U Pi) (force.hip).
// One thread per site (action) or per link (force, update, kinetic energy);
// block partials are summed by one block in index order (deterministic).
#include <chrono>
#include <cmath>

#include "lqs_impl.hpp"

namespace lqs {

typedef Cx<double> Cd;
struct Mat {
    Cd e[3][3];
};

__device__ __forceinline__ Mat mat_load(const double2 *p)
{
    Mat m;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double2 d = p[3 * i + j];
            m.e[i][j] = {d.x, d.y};
        }
    return m;
}

__device__ __forceinline__ void mat_store(double2 *p, const Mat &m)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) p[3 * i + j] = make_double2(m.e[i][j].re, m.e[i][j].im);
}

// a b, a b^dag, a^dag b (each component summed k = 0, 1, 2 in fused multiply-adds)
template <bool DA, bool DB> __device__ __forceinline__ void mat_mac(Mat &c, const Mat &a, const Mat &b)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            Cd s = c.e[i][j];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const Cd x = DA ? Cd{a.e[k][i].re, -a.e[k][i].im} : a.e[i][k];
                const Cd y = DB ? Cd{b.e[j][k].re, -b.e[j][k].im} : b.e[k][j];
                s.re = fused(-x.im, y.im, fused(x.re, y.re, s.re));
                s.im = fused(x.im, y.re, fused(x.re, y.im, s.im));
            }
            c.e[i][j] = s;
        }
}

__device__ __forceinline__ Mat mat_zero()
{
    Mat m;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) m.e[i][j] = {0.0, 0.0};
    return m;
}

template <bool DA, bool DB> __device__ __forceinline__ Mat mat_mul(const Mat &a, const Mat &b)
{
    Mat c = mat_zero();
    mat_mac<DA, DB>(c, a, b);
    return c;
}

// TA(W) = (W - W^dag)/2 - tr(W - W^dag)/6
__device__ __forceinline__ Mat mat_ta(const Mat &w)
{
    Mat t;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) t.e[i][j] = {0.5 * (w.e[i][j].re - w.e[j][i].re), 0.5 * (w.e[i][j].im + w.e[j][i].im)};
    const double tri = (t.e[0][0].im + t.e[1][1].im + t.e[2][2].im) / 3.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) t.e[i][i].im -= tri;
    return t;
}

__device__ __forceinline__ const double2 *link_at(const double2 *U, int vol, int mu, int lex)
{
    return U + 9 * ((int64_t)mu * vol + lex);
}

constexpr int HMC_BLOCK = 256;
constexpr int HMC_MAX_PARTIALS = 4096;

// -sum_links tr Q^2; one partial per block
__global__ void __launch_bounds__(HMC_BLOCK) kinetic_kernel(int64_t nlinks, const double2 *Q, double *partials)
{
    double s = 0.0;
    for (int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; l < nlinks; l += (int64_t)gridDim.x * blockDim.x) {
        const Mat q = mat_load(Q + 9 * l);
        // tr(Q Q) = sum_{ik} q_ik q_ki
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) s -= q.e[i][k].re * q.e[k][i].re - q.e[i][k].im * q.e[k][i].im;
    }
    s = block_sum(s);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// out[slot] = scale * (offset + sum of n partials), in index order
__global__ void __launch_bounds__(1024) hmc_finalize(const double *partials, int n, double offset, double scale,
                                                     double *out, int slot)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) s += partials[i];
    s = block_sum(s);
    if (threadIdx.x == 0) out[slot] = scale * (offset + s);
}

// The force on every link, added to (mode 1) or written over (mode 0) a
// canonical array Q:
//   Q (+)= c TA(U V'),  V' = gb V - Pi
// V: the sum of the six staples of the link; Pi: the fermion's outer products
// (force.hip, with X = Y = chi and psi = D_oe chi), left out without FERM.
// WM: the links are read from their word-major FP64 18-real copy (block
// 2 mu + parity, word k of checkerboard site cb at k Vh + cb), else from the
// canonical array.
//
// One thread per link; the four waves of a block take the four directions of
// the same 64 sites and keep the links U_d(x) and U_d(x-d) in LDS for each
// other (14 link loads per force instead of 19), and blocks follow each other
// plane by plane in runs of time slices (SweepMap), so that what is loaded more
// than once comes from the XCD's L2.  Bound by the vector memory path (TA and
// TD busy 88-92 % of the time); the loads of the next staple are in flight
// while one is multiplied (at 220 VGPRs, two waves per SIMD: more of them with
// the compiler's own order, one or two loads at a time, were slower).  24^4:
// 214 us in a trajectory, canonical Q read and written (the bytes at the card's
// copy rate: 121 us); three threads per link without the LDS share took 437-450.
struct SweepMap {
    int tiles;   // blocks per parity (64 sites each, the last of a chunk may be partly filled)
    int per;     // tiles per XCD
    int chunk;   // sites (of one parity) of one chunk: nz_c z planes of one time slice
    int tpc;     // tiles per chunk
    int nzc;     // chunks per time slice
    int nt, run; // time slices, and how many of them an XCD takes per chunk position
};

// first site and number of sites of tile o in sweep order: runs of time slices,
// inside them the chunks in z order, inside those the slices of the run
__host__ __device__ __forceinline__ int sweep_tile(const SweepMap &m, int o, int &count)
{
    const int c = o / m.tpc, piece = o - c * m.tpc;
    const int rb = c / (m.nzc * m.run), r = c - rb * m.nzc * m.run;
    const int len = m.run < m.nt - rb * m.run ? m.run : m.nt - rb * m.run;
    const int zc = r / len, t = rb * m.run + (r - zc * len);
    const int left = m.chunk - piece * 64;
    count = left < 64 ? left : 64;
    return (t * m.nzc + zc) * m.chunk + piece * 64;
}

static SweepMap sweep_map(const Geom &g, int run)
{
    SweepMap m;
    const int plane = g.n[0] * g.n[1] / 2, nz = g.n[2];
    int k = 1;
    for (int c = 1; c <= 8 && c <= nz; ++c)
        if (nz % c == 0 && (c * plane) % 64 == 0) {
            k = c;
            break;
        }
    if ((k * plane) % 64 != 0)
        for (int c = 1; c <= nz; ++c)  // no exact fit: at least four tiles per chunk, or the slice
            if (nz % c == 0 && (c * plane >= 256 || c == nz)) {
                k = c;
                break;
            }
    m.chunk = k * plane;
    m.tpc = (m.chunk + 63) / 64;
    m.nzc = nz / k;
    m.nt = g.n[3];
    m.run = run < m.nt ? run : m.nt;
    m.tiles = m.tpc * m.nzc * m.nt;
    m.per = (m.tiles + 7) / 8;
    return m;
}

// word-major FP64 18-real matrix of block blk (2 mu + parity, uniform over the
// wave).  The word planes' addresses are scalar and the site is a 32-bit byte
// offset: Vh < 2^28, as the links of a larger lattice (309 GB) exceed the
// device's memory.
__device__ __forceinline__ Mat wm_load(const double2 *a, int vh, int blk, int cb)
{
    const uint32_t off = 16u * (uint32_t)cb;
    // opaque, so that the compiler forms the nine addresses here and does not
    // keep those of every matrix of a kernel in (spilled) scalar registers
    int64_t plane = 16 * (int64_t)vh;
    asm volatile("" : "+s"(plane));
    const char *base = (const char *)a + blk * 9 * plane;
    Mat m;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 d = *(const double2 *)(base + k * plane + off);
        m.e[k / 3][k % 3] = {d.x, d.y};
    }
    return m;
}

template <bool WM>
__device__ __forceinline__ Mat gf_link(const double2 *U, int vh, int mu, int parity, int lex)
{
    if constexpr (WM) return wm_load(U, vh, 2 * mu + parity, lex >> 1);
    else return mat_load(link_at(U, 2 * vh, mu, lex));
}

// The site with checkerboard index cb: its coordinates, and the offsets to its
// forward and backward neighbours in the directions mu ^ k.
struct LinkSite {
    int lex, c[4], fw[4], bw[4];
};
__device__ __forceinline__ void exchange(bool on, int &p, int &r)
{
    const int t = p;
    p = on ? r : p;
    r = on ? t : r;
}
__device__ __forceinline__ LinkSite link_site(const Geom &g, int cb, int par, int mu)
{
    LinkSite s;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    int l = 2 * cb / nx;
    s.c[0] = 2 * cb - l * nx;
    s.c[1] = l % ny;
    l /= ny;
    s.c[2] = l % nz;
    s.c[3] = l / nz;
    const int odd = (s.c[1] + s.c[2] + s.c[3] + par) & 1;
    s.c[0] += odd;
    s.lex = 2 * cb + odd;
    const int w[4] = {1, nx, nx * ny, nx * ny * nz};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        s.fw[d] = s.c[d] == g.n[d] - 1 ? -(g.n[d] - 1) * w[d] : w[d];
        s.bw[d] = s.c[d] == 0 ? (g.n[d] - 1) * w[d] : -w[d];
    }
#pragma unroll
    for (int d = 0; d < 4; d += 2) {
        exchange(mu & 1, s.fw[d], s.fw[d + 1]);
        exchange(mu & 1, s.bw[d], s.bw[d + 1]);
    }
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        exchange(mu & 2, s.fw[d], s.fw[d + 2]);
        exchange(mu & 2, s.bw[d], s.bw[d + 2]);
    }
    return s;
}

// a wave's matrices in LDS, one word of 64 sites after the other
__device__ __forceinline__ void lds_put(double2 *to, int slot, const Mat &m)
{
#pragma unroll
    for (int k = 0; k < 9; ++k)
        to[(slot * 9 + k) * 64 + (threadIdx.x & 63)] = make_double2(m.e[k / 3][k % 3].re, m.e[k / 3][k % 3].im);
}
__device__ __forceinline__ Mat lds_get(const double2 *from, int slot)
{
    Mat m;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 e = from[(slot * 9 + k) * 64 + (threadIdx.x & 63)];
        m.e[k / 3][k % 3] = {e.x, e.y};
    }
    return m;
}

// sum over sites of sum_{mu<nu} Re tr P_{mu nu}(x), one partial per tile and
// parity.  Re tr P = Re tr(a b^dag) with a = U_mu(x) U_nu(x+mu) and
// b = U_nu(x) U_mu(x+nu): the wave of direction mu forms its three products a,
// and the waves of a plane's two directions meet in LDS, so that a site's
// plaquettes take 16 link reads.  24^4: 67 us; one thread per site with its own
// 24 link reads took 94 us.
template <bool WM>
__global__ void __launch_bounds__(256) plaquette_kernel(Geom g, SweepMap sm, const double2 *U, double *partials)
{
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int par = q & 1, o = xcd * sm.per + (q >> 1);
    if (o >= sm.tiles) return;
    int count;
    const int c0 = sweep_tile(sm, o, count);
    __shared__ double2 ex[4 * 9 * 64];
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int cb = c0 + (lane < count ? lane : count - 1);  // idle lanes repeat the last site, not counted
    const LinkSite ls = link_site(g, cb, par, mu);
    const int vh = g.vh, x = ls.lex;
    const Mat u = gf_link<WM>(U, vh, mu, par, x);
    Mat f[3];
#pragma unroll
    for (int k = 1; k < 4; ++k) f[k - 1] = gf_link<WM>(U, vh, mu ^ k, par ^ 1, x + ls.fw[0]);
    double s = 0.0;
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        const Mat a = mat_mul<false, false>(u, f[k - 1]);
        __syncthreads();
        lds_put(ex, mu, a);
        __syncthreads();
        if (mu > (mu ^ k)) continue;
        const Mat b = lds_get(ex, mu ^ k);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) s = fused(a.e[i][j].im, b.e[i][j].im, fused(a.e[i][j].re, b.e[i][j].re, s));
    }
    s = block_sum(lane < count ? s : 0.0);
    if (threadIdx.x == 0) partials[2 * o + par] = s;
}

// Orders the arithmetic behind m before what follows: without it the compiler
// emits products next to their last use and moves the loads in front of them.
__device__ __forceinline__ void pin(Mat &m)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(m.e[k / 3][k % 3].re), "+v"(m.e[k / 3][k % 3].im));
}

__device__ __forceinline__ Cd cfma(Cd a, Cd b, Cd c)
{
    return {fused(-a.im, b.im, fused(a.re, b.re, c.re)), fused(a.im, b.re, fused(a.re, b.im, c.im))};
}

// exp(A) for a 3x3 complex A: A is scaled by 2^-s so that its max-row-sum
// norm is at most 1/4, the Taylor polynomial of degree 16 is evaluated in
// Horner form (truncation below 1e-24), and the result squared s times.
// Every polynomial in A is held as c0 + c1 A + c2 A^2 (Cayley-Hamilton:
// A^3 = t A^2 - w A + d, with t = tr A, w = (t^2 - tr A^2) / 2, d = det A), so
// a Horner step takes three complex products instead of the 27 of a matrix
// product, and the matrix products left are A^2 and the caller's.  Held is
// exp(A) - 1, whose rounding is that of a small number.  Squaring coefficients
// amplifies rounding four times a step where two eigenvalues lie close, squaring
// the matrix twice: the first three squarings (norms up to 2) are of the former
// kind, further ones of the latter.  Relative error against 80-bit sums at norm
// 0.05: 3.2e-17, 0.4: 4.4e-17, 3: 2.9e-16, 1024: 1.0e-13 (the matrix throughout,
// 1 included: 3.2e-17, 1.8e-16, 1.2e-15, 5.3e-13; coefficients throughout, 1
// included: 6.7e-17, 1.8e-16, 1.8e-15, 1.4e-11).
__device__ __forceinline__ Mat mat_exp(const Mat &a0)
{
    double nrm = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double r = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) r += sqrt(a0.e[i][j].re * a0.e[i][j].re + a0.e[i][j].im * a0.e[i][j].im);
        nrm = r > nrm ? r : nrm;
    }
    int s = 0;
    while (nrm > 0.25 && s < 60) {
        nrm *= 0.5;
        ++s;
    }
    const double sc = ldexp(1.0, -s);
    Mat a;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) a.e[i][j] = {a0.e[i][j].re * sc, a0.e[i][j].im * sc};
    const Mat a2 = mat_mul<false, false>(a, a);
    const Cd t = {a.e[0][0].re + a.e[1][1].re + a.e[2][2].re, a.e[0][0].im + a.e[1][1].im + a.e[2][2].im};
    const Cd t2 = {a2.e[0][0].re + a2.e[1][1].re + a2.e[2][2].re, a2.e[0][0].im + a2.e[1][1].im + a2.e[2][2].im};
    const Cd tt = cmul(t, t);
    const Cd nw = {0.5 * (t2.re - tt.re), 0.5 * (t2.im - tt.im)};  // -w
    Cd d = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int j = (i + 1) % 3, k = (i + 2) % 3;
        d = cfma(a.e[0][i], csub(cmul(a.e[1][j], a.e[2][k]), cmul(a.e[1][k], a.e[2][j])), d);
    }
    // Horner: F = a/1 (1 + a/2 (1 + ... (1 + a/16))), exp(a) = 1 + F
    Cd c0 = {0.0, 0.0}, c1 = {0.0, 0.0}, c2 = {0.0, 0.0};
#pragma unroll 4
    for (int k = 16; k >= 1; --k) {
        const double inv = 1.0 / k;
        const Cd n0 = cmul(d, c2), n1 = cfma(nw, c2, Cd{c0.re + 1.0, c0.im}), n2 = cfma(t, c2, c1);
        c0 = {n0.re * inv, n0.im * inv};
        c1 = {n1.re * inv, n1.im * inv};
        c2 = {n2.re * inv, n2.im * inv};
    }
    constexpr int COEFFICIENT_SQUARINGS = 3;
    for (int k = 0; k < s && k < COEFFICIENT_SQUARINGS; ++k) {
        // (1 + F)^2 - 1 = 2 F + F^2, and
        // (c0 + c1 A + c2 A^2)^2 = c0^2 + 2 c0 c1 A + (c1^2 + 2 c0 c2) A^2 + 2 c1 c2 A^3 + c2^2 A^4,
        // reduced by A^4 = t A^3 - w A^2 + d A and then A^3
        const Cd q4 = cmul(c2, c2), h = cmul(c1, c2);
        const Cd q3 = cfma(t, q4, Cd{2.0 * h.re, 2.0 * h.im});
        const Cd c02 = cmul(c0, c2), c01 = cmul(c0, c1);
        const Cd q2 = cfma(nw, q4, cfma(c1, c1, Cd{2.0 * c02.re, 2.0 * c02.im}));
        const Cd q1 = cfma(d, q4, Cd{2.0 * c01.re, 2.0 * c01.im});
        const Cd s0 = cfma(d, q3, cmul(c0, c0)), s1 = cfma(nw, q3, q1), s2 = cfma(t, q3, q2);
        c0 = {fused(2.0, c0.re, s0.re), fused(2.0, c0.im, s0.im)};
        c1 = {fused(2.0, c1.re, s1.re), fused(2.0, c1.im, s1.im)};
        c2 = {fused(2.0, c2.re, s2.re), fused(2.0, c2.im, s2.im)};
    }
    Mat e;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const Cd diag = i == j ? c0 : Cd{0.0, 0.0};
            e.e[i][j] = cfma(c2, a2.e[i][j], cfma(c1, a.e[i][j], diag));
            if (i == j) e.e[i][j].re += 1.0;
        }
    for (int k = COEFFICIENT_SQUARINGS; k < s; ++k) e = mat_mul<false, false>(e, e);
    return e;
}

template <int P, int R> __device__ __forceinline__ void lu_store(const Mat &u, char *out, int blk, int64_t pitch, int cb)
{
    typedef typename RealOf<P>::type T;
    if (!out) return;
    M3<T> v;
#pragma unroll
    for (int k = 0; k < 9; ++k) v.e[k / 3][k % 3] = {(T)u.e[k / 3][k % 3].re, (T)u.e[k / 3][k % 3].im};
    LinkIO<P, R>::store(out + blk * (int64_t)link_block_bytes_per_site(P, R) * pitch, pitch, cb, v);
}

// the link of site cb and block blk in every format a trajectory holds
__device__ __forceinline__ void lu_store_all(const Mat &w, const LinkOut &out, int blk, int64_t vh, int cb)
{
    lu_store<F64, 18>(w, out.fmt[F64][0], blk, vh, cb);
    lu_store<F64, 12>(w, out.fmt[F64][1], blk, vh, cb);
    lu_store<F32, 18>(w, out.fmt[F32][0], blk, vh, cb);
    lu_store<F32, 12>(w, out.fmt[F32][1], blk, vh, cb);
    lu_store<F16, 18>(w, out.fmt[F16][0], blk, vh, cb);
    lu_store<F16, 12>(w, out.fmt[F16][1], blk, vh, cb);
}

template <bool WM, bool FERM, bool UPD>
__global__ void __launch_bounds__(256) link_force_kernel(Geom g, SweepMap sm, const double2 *U, const char *chi,
                                                         const char *psi, double gb, double c, int mode, double2 *Q,
                                                         double eps, LinkOut out)
{
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int par = q & 1, o = xcd * sm.per + (q >> 1);
    if (o >= sm.tiles) return;
    int count;
    const int c0 = sweep_tile(sm, o, count);
    __shared__ double2 own[4 * 9 * 64], back[4 * 9 * 64];
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int cb = c0 + (lane < count ? lane : count - 1);  // idle lanes repeat the last site, without a store
    const int vh = g.vh;
    const LinkSite ls = link_site(g, cb, par, mu);
    const int x = ls.lex, *fw = ls.fw, *bw = ls.bw;
    const int fm = fw[0];
    // Staple s (0..5): nu = mu ^ (s / 2 + 1), so that the waves of a plane's two
    // directions ask for its links together.
    //   even s, upper: (U_nu(x+mu) (U_nu(x) U_mu(x+nu))^dag)
    //   odd s,  lower: ((U_mu(x-nu) U_nu(x+mu-nu))^dag U_nu(x-nu))
    // a, b: the inner product's factors, z: the outer one.  The scheduling
    // barriers keep all 27 loads of a staple in flight while the one before it
    // is multiplied; left alone the compiler waits after every one or two.
    Mat v = mat_zero(), a, b, z;
    // the links U_d(x) and U_d(x-d) of the block's sites, shared by its four waves
    lds_put(own, mu, gf_link<WM>(U, vh, mu, par, x));
    lds_put(back, mu, gf_link<WM>(U, vh, mu, par ^ 1, x + bw[0]));
    auto load_ab = [&](int s) {
        const int k = s / 2 + 1, nu = mu ^ k, d = s & 1 ? bw[k] : fw[k];
        a = s & 1 ? gf_link<WM>(U, vh, mu, par ^ 1, x + d) : lds_get(own, nu);
        b = s & 1 ? gf_link<WM>(U, vh, nu, par, x + fm + d) : gf_link<WM>(U, vh, mu, par ^ 1, x + d);
    };
    auto load_z = [&](int s) {
        const int k = s / 2 + 1;
        z = s & 1 ? lds_get(back, mu ^ k) : gf_link<WM>(U, vh, mu ^ k, par ^ 1, x + fm);
    };
    __syncthreads();
    load_ab(0);
    load_z(0);
    // The records of Q are read and written as the 16-byte pieces j = 64 k + lane
    // of the wave's 64 records (a lane's own record would be 64 separate lines
    // per access): piece j is word j % 9 of the record of lane j / 9.
    double2 prev[9];
    double2 *at[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int j = 64 * k + lane, r = j / 9;
        const int xr = __shfl(x, r, 64);  // by every lane: an idle source lane would hold no value
        at[k] = r < count ? Q + 9 * ((int64_t)mu * 2 * vh + xr) + (j - 9 * r) : nullptr;
    }
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        __builtin_amdgcn_sched_barrier(0);
        Mat ab = mat_mul<false, false>(a, b);
        pin(ab);
        __builtin_amdgcn_sched_barrier(0);
        if (s < 5) {
            load_ab(s + 1);
        } else {  // the link itself and the old records
            a = lds_get(own, mu);
#pragma unroll
            for (int k = 0; k < 9; ++k) prev[k] = mode == 1 && at[k] ? *at[k] : make_double2(0.0, 0.0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s & 1) mat_mac<true, false>(v, ab, z);
        else mat_mac<false, true>(v, z, ab);
        pin(v);
        __builtin_amdgcn_sched_barrier(0);
        if (s < 5) load_z(s + 1);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) v.e[i][j] = {gb * v.e[i][j].re, gb * v.e[i][j].im};
    if constexpr (FERM) {
        // y even: Pi = 2 e psi(y+mu) chi(y)^dag; y odd: Pi = -2 e chi(y+mu) psi(y)^dag
        const int *cc = ls.c;
        const int sg = mu == 0 ? 0 : mu == 1 ? cc[0] : mu == 2 ? cc[0] + cc[1] : cc[0] + cc[1] + cc[2];
        const bool neg = ((sg & 1) != 0) != (mu == 3 && cc[3] == g.n[3] - 1);
        const double e = (neg ? -2.0 : 2.0) * (par == 0 ? 1.0 : -1.0);
        const V3<double> far = SpinorIO<F64>::load(par == 0 ? psi : chi, vh, (x + fm) >> 1);
        const V3<double> own = SpinorIO<F64>::load(par == 0 ? chi : psi, vh, cb);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const Cd a = {e * far.c[i].re, e * far.c[i].im}, b = own.c[j];
                v.e[i][j].re -= fused(a.im, b.im, a.re * b.re);
                v.e[i][j].im -= fused(-a.re, b.im, a.im * b.re);
            }
    }
    const Mat t = mat_ta(mat_mul<false, false>(a, v));
    __syncthreads();  // every wave has read its links: the array takes the result
    double2 *rec = own + mu * 9 * 64;
#pragma unroll
    for (int k = 0; k < 9; ++k) rec[9 * lane + k] = make_double2(t.e[k / 3][k % 3].re, t.e[k / 3][k % 3].im);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 f = rec[64 * k + lane];
        const double2 n = make_double2(fused(c, f.x, prev[k].x), fused(c, f.y, prev[k].y));
        if (at[k]) *at[k] = n;
        if (UPD) rec[64 * k + lane] = n;
    }
    if constexpr (UPD) {
        __syncthreads();
        Mat qn = mat_load(rec + 9 * lane);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) qn.e[i][j] = {eps * qn.e[i][j].re, eps * qn.e[i][j].im};
        const Mat w = mat_mul<false, false>(mat_exp(qn), a);
        if (lane < count) lu_store_all(w, out, 2 * mu + par, vh, cb);
    }
}

// U = exp(eps Q) U on every link.  A block takes 128 consecutive sites of one
// direction (64 of each parity) and moves the canonical records through LDS in
// contiguous runs (see pack.hip).  Bound by memory: 137 us
// at 24^4 for 573 MB without a squaring, 4.2 TB/s; 140 at norms of a trajectory and
// 151 above norm 2 (180 to 217 with a matrix product per Horner step and squaring
// and a lane reading its own 144-byte record).
constexpr int LU_SITES = 128;

__device__ __forceinline__ void lu_stage(double2 *sh, const double2 *src, int n)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int i = threadIdx.x + k * LU_SITES;
        if (i < n) sh[i] = src[i];
    }
    __syncthreads();
}

__global__ void __launch_bounds__(LU_SITES) link_update_kernel(Geom g, double2 *U, const double2 *Q, double eps)
{
    __shared__ double2 sh[9 * LU_SITES];
    const int64_t V = 2 * (int64_t)g.vh, first = (int64_t)blockIdx.x * LU_SITES;
    const int mu = blockIdx.y;
    const int n = 9 * (int)(V - first < LU_SITES ? V - first : LU_SITES);
    const int64_t rec = 9 * (mu * V + first);
    const int parity = threadIdx.x >> 6, cb = (int)(first >> 1) + (threadIdx.x & 63);
    const bool valid = cb < g.vh;
    double2 *own = sh + (valid ? 9 * (lex_of(g, cb, parity) - (int)first) : 0);
    lu_stage(sh, Q + rec, n);
    Mat q = mat_load(own);
    __syncthreads();
    lu_stage(sh, U + rec, n);
    const Mat u = mat_load(own);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) q.e[i][j] = {eps * q.e[i][j].re, eps * q.e[i][j].im};
    const Mat w = mat_mul<false, false>(mat_exp(q), u);
    if (valid) mat_store(own, w);  // own record only: read by this thread alone
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int i = threadIdx.x + k * LU_SITES;
        if (i < n) U[rec + i] = sh[i];
    }
}

// phi = m eta_e - t (FP64 single-parity fields, double2[3][vh])
__global__ void __launch_bounds__(HMC_BLOCK) pseudofermion_kernel(int vh, double m, const double2 *eta_e,
                                                                  const double2 *t, double2 *phi)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 3 * vh) return;
    const double2 a = eta_e[i], b = t[i];
    phi[i] = make_double2(m * a.x - b.x, m * a.y - b.y);
}

// Start of the next solve from the last two solutions (linear extrapolation in
// molecular-dynamics time; successive solves are equally spaced, h/2 apart
// for Omelyan and h for leapfrog): c <- 2c - p, p <- c.
__global__ void __launch_bounds__(HMC_BLOCK) extrapolate_kernel(int64_t n, double2 *c, double2 *p)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 cv = c[i], pv = p[i];
    p[i] = cv;
    c[i] = make_double2(2.0 * cv.x - pv.x, 2.0 * cv.y - pv.y);
}

static int reduce_blocks(int64_t n)
{
    int64_t b = (n + HMC_BLOCK - 1) / HMC_BLOCK;
    return (int)(b > HMC_MAX_PARTIALS ? HMC_MAX_PARTIALS : (b < 1 ? 1 : b));
}

void launch_kinetic(Ctx &ctx, const Geom &g, const double *Q, double *out, int slot, hipStream_t s)
{
    const int64_t nl = 4 * 2 * (int64_t)g.vh;
    double *part = (double *)ctx.workspace("hmc.partials.k", sizeof(double) * HMC_MAX_PARTIALS);
    const int nb = reduce_blocks(nl);
    hipLaunchKernelGGL(kinetic_kernel, dim3(nb), dim3(HMC_BLOCK), 0, s, nl, (const double2 *)Q, part);
    LQS_HIP(hipGetLastError());
    hipLaunchKernelGGL(hmc_finalize, dim3(1), dim3(1024), 0, s, (const double *)part, nb, 0.0, 1.0, out, slot);
    LQS_HIP(hipGetLastError());
}

// Time slices an XCD takes at one chunk position before its next chunk: enough
// that a slice's t neighbours are its own, few enough that what it has read of z
// is still in its L2 at the next position.  Pure-gauge trajectories in ms with
// runs of 1, 2, 3, 4, 6, 8, 24 slices: 24^4 5.45 5.13 4.86 5.04 4.92 5.08 5.09,
// 16^3 x 32 1.67 1.64 1.59 1.63 1.61 1.77 1.91, 32^4 16.7 16.1 16.0 15.5 16.2
// 15.7 17.0, 48^3 x 16 27.0 26.1 27.6 27.3 28.1 28.2 28.0, 32^3 x 8 4.00 3.99 4.12
// 4.06 4.12 4.17 4.16.
constexpr int SWEEP_RUN = 3;

// out[slot] (device) = beta * sum_x sum_{mu<nu} (1 - Re tr P / 3)
template <bool WM>
static void launch_action(Ctx &ctx, const Geom &g, const double *U, double beta, double *out, int slot, hipStream_t s)
{
    const double vol = 2.0 * g.vh;
    const SweepMap sm = sweep_map(g, SWEEP_RUN);
    double *part = (double *)ctx.workspace("hmc.partials.a", sizeof(double) * 2 * (size_t)sm.tiles);
    hipLaunchKernelGGL(plaquette_kernel<WM>, dim3(8u * sm.per * 2), dim3(256), 0, s, g, sm, (const double2 *)U, part);
    LQS_HIP(hipGetLastError());
    // beta * (6 V - sum / 3) = (-beta/3) * (-18 V + sum)
    hipLaunchKernelGGL(hmc_finalize, dim3(1), dim3(1024), 0, s, (const double *)part, 2 * sm.tiles, -18.0 * vol, -beta / 3.0,
                       out, slot);
    LQS_HIP(hipGetLastError());
}

void launch_gauge_action(Ctx &ctx, const Geom &g, const double *U, double beta, double *out, int slot, hipStream_t s)
{
    launch_action<false>(ctx, g, U, beta, out, slot, s);
}

template <bool WM, bool FERM, bool UPD = false>
static void launch_link_force(const Geom &g, const double *U, const double *chi, const double *psi, double gb, double c,
                              int mode, double *Q, hipStream_t s, double eps = 0.0, const LinkOut &out = LinkOut())
{
    const SweepMap sm = sweep_map(g, SWEEP_RUN);
    hipLaunchKernelGGL((link_force_kernel<WM, FERM, UPD>), dim3(8u * sm.per * 2), dim3(256), 0, s, g, sm,
                       (const double2 *)U, (const char *)chi, (const char *)psi, gb, c, mode, (double2 *)Q, eps, out);
    LQS_HIP(hipGetLastError());
}

void launch_gauge_force(const Geom &g, const double *U, double beta, double coeff, int accumulate, double *out,
                        hipStream_t s)
{
    launch_link_force<false, false>(g, U, nullptr, nullptr, 1.0, coeff * beta / 3.0, accumulate ? 1 : 0, out, s);
}

void launch_link_update(const Geom &g, double *U, const double *Q, double eps, hipStream_t s)
{
    const dim3 grid((unsigned)((2 * (int64_t)g.vh + LU_SITES - 1) / LU_SITES), 4);
    hipLaunchKernelGGL(link_update_kernel, grid, dim3(LU_SITES), 0, s, g, (double2 *)U, (const double2 *)Q, eps);
    LQS_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// one trajectory

namespace {

// A gauge object over context workspaces (not freed by ~Gauge).
struct WsGauge {
    lqs_gauge g;
    WsGauge(Ctx &ctx, const Geom &geom, int inner_prec, int inner_recon)
    {
        g.ctx = &ctx;
        g.g = geom;
        g.vh = geom.vh;
        g.temporal = false;
        g.pitch = geom.vh;
        const int rcs[2] = {18, inner_recon};
        const int precs[2] = {F64, inner_prec};
        for (int k = 0; k < 2; ++k) {
            const int rc = rcs[k] == 12 ? 1 : 0;
            if (g.fmt[precs[k]][rc]) continue;
            const size_t bytes = (size_t)link_block_bytes_per_site(precs[k], rcs[k]) * g.pitch * 8;
            g.fmt[precs[k]][rc] = ctx.workspace(std::string("hmc.links.") + std::to_string(precs[k]) + "." +
                                                    std::to_string(rcs[k]),
                                                bytes);
        }
    }
    ~WsGauge()
    {
        for (auto &row : g.fmt)
            for (auto &p : row) p = nullptr;
    }
};

}  // namespace

void hmc_trajectory_impl(Ctx &ctx, const Geom &g, double *links, double *mom, const double *pf, double u,
                         const lqs_hmc_params &prm, lqs_hmc_stats &st, double *proposal, double *phi_out,
                         hipStream_t s)
{
    auto t0 = std::chrono::steady_clock::now();
    const int64_t vol = 2 * (int64_t)g.vh;
    const int64_t f64 = field_bytes(g, F64, 1);
    double *scal = (double *)ctx.workspace("hmc.scalars", sizeof(double) * 16);
    const bool ferm = prm.fermions != 0;
    // the links of the trajectory live in the word-major FP64 18-real format
    // alone (U1), which the force, the link update and the solver's FP64 hops
    // read; the inner format is written along with each link update
    // (the solver's parameters mean nothing without fermions)
    WsGauge wg(ctx, g, ferm ? prm.cg.inner_prec : F64, ferm ? prm.cg.inner_recon : 18);
    Gauge &gauge = wg.g;
    LinkRef L64 = gauge.ref(F64, 18);
    double *U1 = (double *)gauge.fmt[F64][0];
    // where a momentum step that goes on to the link step writes the new links
    double *U2 = (double *)ctx.workspace("hmc.links.next", (size_t)link_block_bytes_per_site(F64, 18) * gauge.pitch * 8);
    LinkOut fmts;
    for (int prec = 0; prec < 3; ++prec)
        for (int rc = 0; rc < 2; ++rc) fmts.fmt[prec][rc] = (char *)gauge.fmt[prec][rc];
    launch_pack_links(g, links, fmts, g.vh, s);
    const LaunchShape sh = default_hop_shape(g, F64, L64, 1);

    double *phi = nullptr, *chi = nullptr, *psx = nullptr, *chi_prev = nullptr;
    int cg_solves = 0, cg_iters = 0, worst = LQS_OK;
    lqs_cg_params cgp = prm.cg;
    cgp.persistent = 0;
    const bool warm = prm.cg.use_x0 != 0;
    if (ferm) {
        phi = (double *)ctx.workspace("hmc.phi", f64);
        chi = (double *)ctx.workspace("hmc.chi", f64);
        chi_prev = (double *)ctx.workspace("hmc.chi_prev", f64);
        psx = (double *)ctx.workspace("hmc.psx", f64);
        LQS_HIP(hipMemsetAsync(chi, 0, f64, s));
        if (prm.fermions == 1) {
            double *eo = (double *)ctx.workspace("hmc.eta_o", f64);
            double *ee = (double *)ctx.workspace("hmc.eta_e", f64);
            launch_field_pack(g, pf, lqs_field{ee, F64, 0, 1}, s);
            launch_field_pack(g, pf, lqs_field{eo, F64, 1, 1}, s);
            // psx (even scratch) = D_eo eta_o
            launch_hop_gated(g, L64, F64, 18, 0, 0, 1, eo, psx, nullptr, 0, sh, s);
            hipLaunchKernelGGL(pseudofermion_kernel, dim3((3 * g.vh + HMC_BLOCK - 1) / HMC_BLOCK), dim3(HMC_BLOCK), 0,
                               s, (int)g.vh, prm.mass, (const double2 *)ee, (const double2 *)psx, (double2 *)phi);
            LQS_HIP(hipGetLastError());
        } else {
            launch_field_pack(g, pf, lqs_field{phi, F64, 0, 1}, s);
        }
        if (phi_out) {
            LQS_HIP(hipMemsetAsync(phi_out, 0, sizeof(double) * 6 * (size_t)vol, s));
            launch_field_unpack(g, lqs_field{phi, F64, 0, 1}, 1.0, phi_out, s);
        }
    }
    // chi = M^-1 phi on the current links (warm start from the previous chi if
    // asked); solves that only feed the force may use the looser force_tol
    int nsol = 0;
    auto solve = [&](bool energy) {
        lqs_problem pb{&wg.g, prm.mass, 1, phi, chi};
        lqs_cg_stats cs{};
        if (!warm) {
            LQS_HIP(hipMemsetAsync(chi, 0, f64, s));
        } else if (nsol == 1) {
            LQS_HIP(hipMemcpyAsync(chi_prev, chi, f64, hipMemcpyDeviceToDevice, s));
        } else if (nsol >= 2) {
            const int64_t n = 3 * (int64_t)g.vh;
            hipLaunchKernelGGL(extrapolate_kernel, dim3((unsigned)((n + HMC_BLOCK - 1) / HMC_BLOCK)), dim3(HMC_BLOCK), 0,
                               s, n, (double2 *)chi, (double2 *)chi_prev);
            LQS_HIP(hipGetLastError());
        }
        ++nsol;
        cgp.use_x0 = warm ? 1 : 0;
        cgp.tol = (energy || prm.force_tol <= 0) ? prm.cg.tol : prm.force_tol;
        cg_solve_one(ctx, pb, cgp, &cs, s);
        ++cg_solves;
        cg_iters += cs.iters;
        if (cs.status != LQS_OK && (worst == LQS_OK || cs.status < worst)) worst = cs.status;
    };
    // mom -= eps F / 2 with F_g = (beta/3) TA(U V) and F_f = -TA(U Pi), the
    // fermion part from chi on the current links; the solve on the final links
    // (last) also gives S_f at the end.  drift > 0: then the links move,
    // U = exp(drift mom) U.
    auto momentum = [&](double eps, bool have_chi, bool last, double drift) {
        if (ferm) {
            if (!have_chi) solve(last);
            launch_hop_gated(g, L64, F64, 18, 0, 1, 1, chi, psx, nullptr, 0, sh, s);
        }
        const double gb = prm.beta / 3.0, c = -0.5 * eps;
        if (drift > 0) {
            LinkOut next = fmts;
            next.fmt[F64][0] = (char *)U2;
            if (ferm) launch_link_force<true, true, true>(g, U1, chi, psx, gb, c, 1, mom, s, drift, next);
            else launch_link_force<true, false, true>(g, U1, nullptr, nullptr, gb, c, 1, mom, s, drift, next);
            std::swap(U1, U2);
            fmts = next;
            gauge.fmt[F64][0] = U1;
            L64 = gauge.ref(F64, 18);
            return;
        }
        if (ferm) launch_link_force<true, true>(g, U1, chi, psx, gb, c, 1, mom, s);
        else launch_link_force<true, false>(g, U1, nullptr, nullptr, gb, c, 1, mom, s);
    };

    // H at the start: scal[0..1] = K0, Sg0 / beta, scal[8] = Sf0
    launch_kinetic(ctx, g, mom, scal, 0, s);
    launch_action<true>(ctx, g, U1, 1.0, scal, 1, s);
    if (ferm) {
        solve(true);
        launch_field_dot(ctx, g, 1, phi, chi, scal + 8, s);
    }

    const double h = prm.tau / prm.nsteps;
    const double lam = prm.lambda > 0 ? prm.lambda : 0.1931833275037836;
    bool have_chi = ferm;  // chi belongs to the current links
    if (prm.integrator == LQS_LEAPFROG) {
        momentum(0.5 * h, have_chi, false, h);
        for (int k = 0; k < prm.nsteps; ++k) {
            const bool last = k == prm.nsteps - 1;
            momentum(last ? 0.5 * h : h, false, last, last ? 0.0 : h);
        }
    } else {
        // consecutive lam*h updates at a step boundary act on the same links: merged
        double pending = lam * h;
        for (int k = 0; k < prm.nsteps; ++k) {
            momentum(pending, k == 0 && have_chi, false, 0.5 * h);
            momentum((1.0 - 2.0 * lam) * h, false, false, 0.5 * h);
            pending = 2.0 * lam * h;
        }
        momentum(lam * h, false, true, 0.0);
    }
    // H at the end: chi is the solve on the final links (last momentum step)
    launch_kinetic(ctx, g, mom, scal, 3, s);
    launch_action<true>(ctx, g, U1, 1.0, scal, 4, s);
    if (ferm) launch_field_dot(ctx, g, 1, phi, chi, scal + 10, s);
    double hs[16];
    LQS_HIP(hipMemcpyAsync(hs, scal, sizeof(hs), hipMemcpyDeviceToHost, s));
    LQS_HIP(hipStreamSynchronize(s));
    st.k0 = hs[0];
    st.sg0 = prm.beta * hs[1];
    st.sf0 = ferm ? hs[8] : 0.0;
    st.k1 = hs[3];
    st.sg1 = prm.beta * hs[4];
    st.sf1 = ferm ? hs[10] : 0.0;
    st.dH = (st.k1 + st.sg1 + st.sf1) - (st.k0 + st.sg0 + st.sf0);
    st.accepted = (std::isfinite(st.dH) && u < std::exp(-st.dH)) ? 1 : 0;
    st.cg_solves = cg_solves;
    st.cg_iters = cg_iters;
    st.status = worst;
    if (proposal) launch_unpack_links(g, U1, proposal, s);
    if (st.accepted) launch_unpack_links(g, U1, links, s);
    // plaquette of the links returned: S_g = beta * 6V (1 - <P>) at beta = 1
    st.plaquette = 1.0 - hs[st.accepted ? 4 : 1] / (6.0 * (double)vol);
    LQS_HIP(hipStreamSynchronize(s));
    st.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
}

}  // namespace lqs
