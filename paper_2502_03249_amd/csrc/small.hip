// small.hip -- independent even-odd CG solves on small lattices, one thread
// block per lattice and one launch for all of them, the links in registers.
//
// Four threads share an even site x, one per direction mu: thread (x, mu) holds
// U_mu(x) and U_mu(x - mu), which for all x and mu is every link of the lattice
// once, signs included, for the whole solve.  D_eo is a gather from t = D_oe p
// in LDS, the quad adding its four parts with DPP moves.  For D_oe the thread
// multiplies p(x) by both links and scatters the products to the odd sites
// x + mu and x - mu in LDS, where they are added in a fixed order.  Thread
// c < 3 of the quad owns colour component c of x, r, p and q.  No vector or
// link is read from memory inside an iteration, and three block barriers are
// its only synchronisation.
//
// The step is the predict-and-recompute form of cg.hip, so <p,q>, <q,q> and
// |r|^2 share one reduction; every wave forms the scalars itself.  Mixed
// precision (FP32 or FP16 links) holds vectors and links in FP32 and takes the
// FP64 residual updates of the other solvers.
//
// Bound by vector issue and by the latency of its dependent phases (LDS round
// trips, the reduction, two divisions), not by bytes.
#include <algorithm>

#include "cg_step.hpp"
#include "hop.hpp"

namespace lqs {

struct SmallLat {
    Geom g;
    LinkRef lo, hi;
    double *x;
    const double *b;
};

template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return bitcast<float>(__builtin_amdgcn_mov_dpp(bitcast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double dpp(double v)
{
    struct I2 { int lo, hi; } w = bitcast<I2>(v);
    w.lo = __builtin_amdgcn_mov_dpp(w.lo, CTRL, 0xf, 0xf, true);
    w.hi = __builtin_amdgcn_mov_dpp(w.hi, CTRL, 0xf, 0xf, true);
    return bitcast<double>(w);
}
// quad_perm controls
constexpr int QP_XOR1 = 0xB1, QP_XOR2 = 0x4E, QP_0 = 0x00, QP_1 = 0x55, QP_2 = 0xAA;

// sum over the four threads of a site, in every one of them
template <typename T> __device__ __forceinline__ T quad_add(T v)
{
    v += dpp<QP_XOR1>(v);
    v += dpp<QP_XOR2>(v);
    return v;
}
template <typename T> __device__ __forceinline__ V3<T> quad_sum(V3<T> v)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        v.c[a].re = quad_add(v.c[a].re);
        v.c[a].im = quad_add(v.c[a].im);
    }
    return v;
}
// component c of v (c = 3: component 2)
template <typename T> __device__ __forceinline__ Cx<T> pick(const V3<T> &v, int c)
{
    return c == 0 ? v.c[0] : c == 1 ? v.c[1] : v.c[2];
}
// the colour vector whose components the quad's threads 0..2 hold
template <typename T> __device__ __forceinline__ V3<T> quad_vector(const Cx<T> &own)
{
    V3<T> v;
    v.c[0] = {dpp<QP_0>(own.re), dpp<QP_0>(own.im)};
    v.c[1] = {dpp<QP_1>(own.re), dpp<QP_1>(own.im)};
    v.c[2] = {dpp<QP_2>(own.re), dpp<QP_2>(own.im)};
    return v;
}
// acc -= U^dag v
template <typename T> __device__ __forceinline__ void sub_mdv(V3<T> &acc, const M3<T> &u, const V3<T> &v)
{
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            acc.c[a].re = fused(-u.e[b][a].im, v.c[b].im, fused(-u.e[b][a].re, v.c[b].re, acc.c[a].re));
            acc.c[a].im = fused(u.e[b][a].im, v.c[b].re, fused(-u.e[b][a].re, v.c[b].im, acc.c[a].im));
        }
}
template <typename T> __device__ __forceinline__ M3<T> signed_link(M3<T> u, bool neg)
{
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) u.e[a][b] = {neg ? -u.e[a][b].re : u.e[a][b].re, neg ? -u.e[a][b].im : u.e[a][b].im};
    return u;
}

struct Nbr {
    int fwd, bwd;     // checkerboard index of x + mu, x - mu
    bool negf, negb;  // signs of links (x, mu), (x - mu, mu)
};
__device__ __forceinline__ Nbr neighbours(const Geom &g, int cb, int parity, int mu)
{
    const Site s = decode(g, cb, parity);
    Nbr n;
    n.fwd = mu == 0 ? s.fwd[0] : mu == 1 ? s.fwd[1] : mu == 2 ? s.fwd[2] : s.fwd[3];
    n.bwd = mu == 0 ? s.bwd[0] : mu == 1 ? s.bwd[1] : mu == 2 ? s.bwd[2] : s.bwd[3];
    n.negf = (s.negf >> mu) & 1;
    n.negb = (s.negb >> mu) & 1;
    return n;
}

// Colour vectors in LDS: [site][3] complex (consecutive sites fall on distinct
// banks).
template <typename T> __device__ __forceinline__ V3<T> lds_vector(const Cx<T> *f, int i)
{
    V3<T> v;
#pragma unroll
    for (int c = 0; c < 3; ++c) v.c[c] = f[3 * i + c];
    return v;
}

// The quad's FP64 sum over mu and both senses of D at site cb of parity `par`:
// links read from memory, one at a time (the hot loop's registers stay held),
// input field in LDS.
__device__ __forceinline__ V3<double> hop_quad64(const Geom &g, const LinkRef &L, int par, int cb, int mu,
                                                 const Cx<double> *in)
{
    typedef LinkIO<F64, 18> LIO;
    const char *lb = (const char *)L.base;
    const Nbr n = neighbours(g, cb, par, mu);
    V3<double> acc = vzero<double>();
    accum(acc, mv(LIO::load(lb + (2 * mu + par) * L.block_bytes, L.pitch, cb), lds_vector(in, n.fwd)), n.negf);
    __builtin_amdgcn_sched_barrier(0);
    accum(acc, mdv(LIO::load(lb + (2 * mu + 1 - par) * L.block_bytes, L.pitch, n.bwd), lds_vector(in, n.bwd)), !n.negb);
    __builtin_amdgcn_sched_barrier(0);
    return quad_sum(acc);
}

// LDS of a block: t and the eight contributions to every odd site (padded to 25
// complex, so that the quads of a wave write to distinct banks), or during an
// FP64 residual x and t64.
constexpr int SCAT = 25;
static size_t small_lds_bytes(int vh, int prec)
{
    return (size_t)vh * std::max((3 + SCAT) * (prec == F64 ? 16 : 8), 2 * 48);
}

struct DppRows {
    template <int N> static __device__ __forceinline__ double by(double v) { return dpp<0x120 + N>(v); }  // row_ror
};

// Sum of v over the threads of the block with the same tid & 3, the same bits in
// every one of them: the loop's control flow and its barriers hang on them (red:
// four rows per wave).
template <int NW> __device__ __forceinline__ double quad_class_sum(double v, double (*red)[4])
{
    const int tid = threadIdx.x;
    v = row_class_sum(v, DppRows());
    if ((tid & 15) < 4) red[tid >> 4][tid & 3] = v;
    __syncthreads();
    const int lane = tid & 63;
    double t = (&red[0][0])[lane];
#pragma unroll
    for (int k = 1; k < NW / 4; ++k) t += (&red[0][0])[64 * k + lane];
    t = row_class_sum(t, DppRows());
    t += __shfl_xor(t, 16, 64);
    t += __shfl_xor(t, 32, 64);
    return t;
}

// A record that every thread holds alike, in scalar registers: the links leave the
// vector registers no room for it, and its branches need no lane masks.
__device__ __forceinline__ CgState uniform_record(const CgState &s)
{
    struct Words { int w[sizeof(CgState) / 4]; } v = bitcast<Words>(s);
#pragma unroll
    for (int &w : v.w) w = __builtin_amdgcn_readfirstlane(w);
    return bitcast<CgState>(v);
}

template <int P, int R, int BS, int S>
__global__ void __launch_bounds__(BS) small_cg_kernel(const SmallLat *lats, CgState *states, int max_trips,
                                                      unsigned long long *clk)
{
    typedef typename RealOf<P>::type T;
    typedef LinkIO<P, R> LIO;
    constexpr bool MIXED = P != F64;
    constexpr int NQ = BS / 4, NW = BS / 64;
    static_assert(NW % 4 == 0, "the final sum reads whole groups of four waves");
    __shared__ SmallLat L;
    __shared__ CgState st;
    __shared__ double red[2][NW * 4][4];  // two buffers: a reduction's reads and the next one's writes need no barrier
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, q0 = tid >> 2, mu = tid & 3;
    if (tid == 0) {
        L = lats[blockIdx.x];
        st = states[blockIdx.x];
        clk[2 * blockIdx.x] = wall_clock64();
    }
    __syncthreads();
    const int vh = L.g.vh;
    Cx<T> *ldsT = (Cx<T> *)lds, *scat = ldsT + 3 * vh;
    const T m2 = (T)st.m2;
    const bool own = mu < 3;

    Cx<T> x[S], r[S], q[S], p[S];  // this thread's component
    M3<T> uf[S], ub[S];            // U_mu(x), U_mu(x - mu), times their phases
    int gf[S], gb[S];              // x + mu, x - mu
    double b2 = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int cb = q0 + s * NQ;
        x[s] = r[s] = q[s] = {T(0), T(0)};
        if (cb < vh) {
            const Nbr n = neighbours(L.g, cb, 0, mu);
            gf[s] = n.fwd;
            gb[s] = n.bwd;
            const char *lb = (const char *)L.lo.base;
            uf[s] = signed_link(LIO::load(lb + (2 * mu) * L.lo.block_bytes, L.lo.pitch, cb), n.negf);
            ub[s] = signed_link(LIO::load(lb + (2 * mu + 1) * L.lo.block_bytes, L.lo.pitch, n.bwd), n.negb);
            if (own) {
                const double2 bv = ((const double2 *)L.b)[mu * (int64_t)vh + cb];
                b2 += bv.x * bv.x + bv.y * bv.y;
                ((double2 *)L.x)[mu * (int64_t)vh + cb] = make_double2(0.0, 0.0);
                r[s] = {(T)bv.x, (T)bv.y};
            }
        }
        p[s] = r[s];
    }
    b2 = quad_class_sum<NW>(quad_add(b2), red[0]);
    if (tid == 0) {
        st.b2 = b2;
        st.stop2 *= b2;
        st.rho = b2;
        st.rho_known = 1;
        st.max_rho = b2;
        st.true_r2 = b2;
        st.phase = b2 == 0.0 ? CG_CONVERGED : (isfinite(b2) ? CG_RUNNING : CG_NONFINITE);
    }
    __syncthreads();
    CgState sc = uniform_record(st);  // the scalars, the same in every thread

    for (int trip = 0;; ++trip) {
        // A solve that stops without its FP64 check (breakdown, non-finite
        // scalar, trip cap) still returns x += x_lo and its measured residual.
        const bool run = sc.phase == CG_RUNNING && trip < max_trips;
        bool measure = !run && sc.phase != CG_CONVERGED && sc.phase != CG_MAXITER;
        if (__builtin_expect(run, 1)) {
            // ---- the products of p that t = D_oe p adds up
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if (q0 + s * NQ >= vh) continue;
                const V3<T> pv = quad_vector(p[s]);
                const V3<T> f = mdv(uf[s], pv), b = mv(ub[s], pv);
                Cx<T> *sf = scat + SCAT * gf[s] + 6 * mu + 3, *sb = scat + SCAT * gb[s] + 6 * mu;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    sf[c] = f.c[c];  // at x + mu: - U^dag p
                    sb[c] = b.c[c];  // at x - mu: + U p
                }
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int cb = q0 + s * NQ;
                if (cb >= vh || !own) continue;
                const Cx<T> *sc0 = scat + SCAT * cb + mu;
                Cx<T> t = csub(sc0[0], sc0[3]);
#pragma unroll
                for (int d = 1; d < 4; ++d) t = csub(cadd(t, sc0[6 * d]), sc0[6 * d + 3]);
                ldsT[3 * cb + mu] = t;
            }
            __syncthreads();
            // ---- q = m^2 p - D_eo t; <p,q>, <q,q>, |r|^2
            double pq = 0.0, qq = 0.0, rr = 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if (q0 + s * NQ >= vh) continue;
                V3<T> acc = mv(uf[s], lds_vector(ldsT, gf[s]));
                sub_mdv(acc, ub[s], lds_vector(ldsT, gb[s]));
                const Cx<T> a = pick(quad_sum(acc), mu);
                if (!own) continue;
                q[s] = {m2 * p[s].re - a.re, m2 * p[s].im - a.im};
                pq += (double)p[s].re * (double)q[s].re + (double)p[s].im * (double)q[s].im;
                qq += (double)q[s].re * (double)q[s].re + (double)q[s].im * (double)q[s].im;
                rr += (double)r[s].re * (double)r[s].re + (double)r[s].im * (double)r[s].im;
            }
            pq = quad_add(pq);
            qq = quad_add(qq);
            rr = quad_add(rr);
            const double sum = quad_class_sum<NW>(mu == 0 ? pq : mu == 1 ? qq : rr, red[trip & 1]);
            cg_step_scalars<false>(sc, lane_value(sum, 0), lane_value(sum, 1), lane_value(sum, 2), 0.0, 1);
            sc = uniform_record(sc);
            measure = !sc.live;
            if (__builtin_expect(sc.live, 1)) {
                // ---- x += alpha p, r -= alpha q, p = r + beta p (left to the residual update when one is due)
                const T alpha = (T)sc.alpha, beta = (T)sc.beta;
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    x[s] = {fused(alpha, p[s].re, x[s].re), fused(alpha, p[s].im, x[s].im)};
                    r[s] = {fused(-alpha, q[s].re, r[s].re), fused(-alpha, q[s].im, r[s].im)};
                    if (!sc.p_due) p[s] = {fused(beta, p[s].re, r[s].re), fused(beta, p[s].im, r[s].im)};
                }
                if (__builtin_expect(!sc.p_due, 1)) continue;
                if (sc.unsettled && !sc.reliable_pending) {
                    rr = 0.0;
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        if (own && q0 + s * NQ < vh)
                            rr += (double)r[s].re * (double)r[s].re + (double)r[s].im * (double)r[s].im;
                    cg_settle(sc, quad_class_sum<NW>(quad_add(rr), red[(trip + 1) & 1]), 1);
                    sc = uniform_record(sc);
                    __syncthreads();  // the sums have been read
                    if (sc.live && !sc.p_due) {
                        const T b = (T)sc.beta;
#pragma unroll
                        for (int s = 0; s < S; ++s) p[s] = {fused(b, p[s].re, r[s].re), fused(b, p[s].im, r[s].im)};
                        continue;
                    }
                }
            }
        }
        const bool due = run && sc.live;
        if (__builtin_expect(due || measure, 0)) {
            // ---- x += x_lo (mixed), t64 = D_oe x, r = b - (m^2 x - D_eo t64)
            Cx<double> *X = (Cx<double> *)lds, *T64 = X + 3 * vh;
            __syncthreads();  // t has been read
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int cb = q0 + s * NQ;
                if (cb >= vh || !own) continue;
                double2 *gx = (double2 *)L.x + mu * (int64_t)vh + cb;
                Cx<double> xv = {(double)x[s].re, (double)x[s].im};
                if (MIXED) {
                    const double2 o = *gx;
                    xv = {o.x + xv.re, o.y + xv.im};
                    x[s] = {T(0), T(0)};
                }
                *gx = make_double2(xv.re, xv.im);
                X[3 * cb + mu] = xv;
            }
            __syncthreads();
#pragma unroll 1
            for (int cb = q0; cb < vh; cb += NQ) {
                const Cx<double> t = pick(hop_quad64(L.g, L.hi, 1, cb, mu, X), mu);
                if (own) T64[3 * cb + mu] = t;
            }
            __syncthreads();
            double r2 = 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int cb = q0 + s * NQ;
                if (cb >= vh) continue;
                const Cx<double> a = pick(hop_quad64(L.g, L.hi, 0, cb, mu, T64), mu);
                if (!own) continue;
                const double2 bv = ((const double2 *)L.b)[mu * (int64_t)vh + cb];
                const Cx<double> xv = X[3 * cb + mu];
                const double re = bv.x - (st.m2 * xv.re - a.re), im = bv.y - (st.m2 * xv.im - a.im);
                r2 += re * re + im * im;
                if (due) r[s] = {(T)re, (T)im};
            }
            r2 = quad_class_sum<NW>(quad_add(r2), red[(trip + 1) & 1]);
            if (due) fin_residual(sc, r2, 0);
            else sc.true_r2 = r2;
            sc = uniform_record(sc);
            if (due && sc.phase == CG_RUNNING) {
                const T beta = (T)sc.beta;
#pragma unroll
                for (int s = 0; s < S; ++s)
                    p[s] = {fused(beta, p[s].re, r[s].re), fused(beta, p[s].im, r[s].im)};
            }
            __syncthreads();  // x, t64 and the sums have been read
        }
        if (!run || measure) break;
    }
    if (tid == 0) {
        states[blockIdx.x] = sc;
        clk[2 * blockIdx.x + 1] = wall_clock64();
    }
}

template <int P, int R, int BS, int S>
static void launch_small(int nlat, int vmax, const SmallLat *lats, CgState *st, int trips, unsigned long long *clk,
                         hipStream_t s)
{
    const void *fn = (const void *)&small_cg_kernel<P, R, BS, S>;
    const size_t lds = small_lds_bytes(vmax, P);
    LQS_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((small_cg_kernel<P, R, BS, S>), dim3(nlat), dim3(BS), lds, s, lats, st, trips, clk);
    LQS_HIP(hipGetLastError());
}

// Sites per parity that one block holds, and the form for a batch whose largest
// lattice has vmax: blocks of 512 threads, whose 256 registers each hold the
// links of up to two sites per quad in FP64 and four in FP32.  Fewer, fuller
// threads win over more waves that all wait at the same barriers and repeat the
// scalars: 4^3 x 6 in FP64 4.4 us per iteration with 512 threads and two sites
// per quad, 4.7 with 768 and one; FP32 arithmetic in 1024 threads of 128
// registers spills, 5.9 against 3.3 (before the scalars left the vector registers:
// now 3.9 and 3.2).
//
// us per iteration, 64 lattices at once, here and in the kernel for lattices
// that several blocks may share (which keeps the larger ones):
//   FP64 18-real   4^4  2.9, 13.1   4^3 x 6  3.9, 14.0   4^3 x 8  4.7, 15.2
//   FP32 12-real   4^4  2.9, 11.7   4^3 x 6  3.2, 11.9   4^2 x 6^2  4.3, 12.8
//                  4^2 x 6 x 8  5.1, 13.2   4 x 8^2 x 4  10.0, 15.6
//   FP16 12-real   4^4  3.0, 12.5   4^2 x 6^2  4.7, 15.8   4 x 8^2 x 4  11.5, 17.8
// A batch with one larger member goes there as a whole: that member's chain of
// group barriers is its time either way (63 of 4^4 and one 6^4 in FP64 3.24 ms,
// the 6^4 alone 3.13).
static int small_max_vh(int prec) { return prec == F64 ? 256 : 512; }

template <int P, int R>
static void launch_small_pr(int vmax, int nlat, const SmallLat *lats, CgState *st, int trips, unsigned long long *clk,
                            hipStream_t s)
{
    if (vmax <= 128) launch_small<P, R, 512, 1>(nlat, vmax, lats, st, trips, clk, s);
    else if (vmax <= 256) launch_small<P, R, 512, 2>(nlat, vmax, lats, st, trips, clk, s);
    else if constexpr (P != F64) {
        if (vmax <= 384) launch_small<P, R, 512, 3>(nlat, vmax, lats, st, trips, clk, s);
        else launch_small<P, R, 512, 4>(nlat, vmax, lats, st, trips, clk, s);
    }
}

bool small_fits(const std::vector<PersistentProblem> &probs, int prec)
{
    for (const PersistentProblem &p : probs)
        if (p.gauge->vh > small_max_vh(prec)) return false;
    return true;
}

// One launch of all problems; the final records and the device clock pairs are
// copied back and waited for.
void small_solve(Ctx &ctx, const std::vector<PersistentProblem> &probs, const lqs_cg_params &prm, const CgState *init,
                 CgState *out, unsigned long long *clk, hipStream_t s)
{
    const int n = (int)probs.size(), prec = prm.inner_prec, recon = prm.inner_recon == 12 ? 12 : 18;
    // descriptors and records in one copy each way: [SmallLat n][CgState n][clock 2n]
    const size_t o_st = (sizeof(SmallLat) * n + 255) & ~size_t(255), o_clk = o_st + ((sizeof(CgState) * n + 255) & ~size_t(255)),
                 bytes = o_clk + 2 * sizeof(unsigned long long) * n;
    char *d = (char *)ctx.workspace("small.io", bytes), *h = (char *)ctx.pinned("small.io", bytes);
    SmallLat *lats = (SmallLat *)h;
    int vmax = 0;
    for (int l = 0; l < n; ++l) {
        const Gauge &g = *probs[l].gauge;
        lats[l] = {g.g, g.ref(prec, recon), g.ref(F64, 18), probs[l].x, probs[l].b};
        CgState &S = ((CgState *)(h + o_st))[l];
        S = *init;
        S.m2 = probs[l].mass * probs[l].mass;
        vmax = std::max(vmax, (int)g.vh);
    }
    LQS_HIP(hipMemcpyAsync(d, h, o_clk, hipMemcpyHostToDevice, s));
    CgState *st = (CgState *)(d + o_st);
    unsigned long long *dclk = (unsigned long long *)(d + o_clk);
    const int trips = prm.max_iter + 8;
    try {
        if (prec == F64 && recon == 18) launch_small_pr<F64, 18>(vmax, n, (const SmallLat *)d, st, trips, dclk, s);
        else if (prec == F64) launch_small_pr<F64, 12>(vmax, n, (const SmallLat *)d, st, trips, dclk, s);
        else if (prec == F32 && recon == 18) launch_small_pr<F32, 18>(vmax, n, (const SmallLat *)d, st, trips, dclk, s);
        else if (prec == F32) launch_small_pr<F32, 12>(vmax, n, (const SmallLat *)d, st, trips, dclk, s);
        else if (recon == 18) launch_small_pr<F16, 18>(vmax, n, (const SmallLat *)d, st, trips, dclk, s);
        else launch_small_pr<F16, 12>(vmax, n, (const SmallLat *)d, st, trips, dclk, s);
        LQS_HIP(hipMemcpyAsync(h + o_st, d + o_st, bytes - o_st, hipMemcpyDeviceToHost, s));
        LQS_HIP(hipStreamSynchronize(s));
    } catch (...) {
        (void)hipStreamSynchronize(s);
        throw;
    }
    std::copy((CgState *)(h + o_st), (CgState *)(h + o_st) + n, out);
    std::copy((unsigned long long *)(h + o_clk), (unsigned long long *)(h + o_clk) + 2 * n, clk);
}

}  // namespace lqs
