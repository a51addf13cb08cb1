// cg.hip -- conjugate gradient on the even-odd normal operator
// M = m^2 - D_eo D_oe (the inversion of Sec. 4.2), in FP64 or with a
// low-precision inner iteration and FP64 residual updates.
//
// Per iteration four kernels run back to back on one stream:
//   1. t = D_oe p                                      (hop)
//   2. q = m^2 p - D_eo t, <p,q> and <q,q>              (hop + fused dots)
//   3. the scalars of the step                          (one block per side)
//   4. x += alpha p, r -= alpha q, p = r + beta p, |r|^2 (one pass)
// beta and the stop decision need the norm of the residual before kernel 4 has
// formed it.  It is predicted from the dots at hand,
//   |r - alpha q|^2 = |r|^2 - 2 alpha <r,q> + alpha^2 <q,q> = alpha^2 <q,q> - |r|^2
// (<r,q> = <p,q> as the directions are conjugate, alpha = |r|^2 / <p,q>; with
// directions in 16 bits corrected for what they are not, see cg_step.hpp), and
// |r|^2 of the next step is the one kernel 4 sums from the residual it stores,
// so the prediction's rounding does not accumulate: the predict-and-recompute
// conjugate gradient of Chen and Carson (SIAM J. Sci. Comput. 42, 2020).
// The x, r and p updates then share one kernel and one read of each vector.
// The dot products are reduced in two fixed-order stages and alpha, beta stay
// on the device; the host only polls the state record.
// The FP64 group
//   x += x_lo, x_lo = 0                                 (mixed precision)
//   t64 = D_oe x, r_hi = b - (m^2 x - D_eo t64), |r_hi|^2, r = r_hi
//   p = r + beta p                                      (kernel 4 left it out)
// is gated on the state.  It decides convergence on the FP64 residual after the
// iterated residual met the target, or the iteration cap; the host queues it
// when it has seen such a state.  In mixed precision it also closes every round
// of eight iterations, for the reliable update (of the mixed-precision solvers
// the paper cites, Clark et al. 2010) that a right-hand side asks for every K
// iterations or when |r| fell below delta * max|r|.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "cg_step.hpp"
#include "hop.hpp"

namespace lqs {

static constexpr int BLAS_BLOCK = 256;

// ---------------------------------------------------------------------------
// The new search direction r + beta p, in the accumulation precision (one
// fused multiply-add per component).

template <int PA>
__device__ __forceinline__ V3<typename RealOf<PA>::type> direction_of(const V3<typename RealOf<PA>::type> &rv,
                                                                      const V3<typename RealOf<PA>::type> &pv,
                                                                      typename RealOf<PA>::type beta)
{
    V3<typename RealOf<PA>::type> o;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o.c[a].re = fused(beta, pv.c[a].re, rv.c[a].re);
        o.c[a].im = fused(beta, pv.c[a].im, rv.c[a].im);
    }
    return o;
}

// Re <a,b> of a site (of vectors in T, for the sums over sites in double)
template <typename T> __device__ __forceinline__ T re_dot(const V3<T> &a, const V3<T> &b)
{
    T s = T(0);
#pragma unroll
    for (int c = 0; c < 3; ++c) s = fused(a.c[c].re, b.c[c].re, fused(a.c[c].im, b.c[c].im, s));
    return s;
}

// ---------------------------------------------------------------------------
// 2. q = m^2 p - D_eo t, <p,q> and <q,q> (output parity even; t odd)

// FP16 storage: left alone the compiler gives the one-vector kernel 120 VGPRs
// (4 waves per SIMD); held to 6 waves it needs 62, without spills, and the
// 64^3x16 launch drops from 89.4 to 86.1 us (FP32/FP64 unchanged or slower).
// Not with LF_PREFETCH, whose words in flight need about 110 VGPRs.
template <int P, int R, int K, int LF>
__global__ void __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu((P == F16 && (LF & LF_PREFETCH) == 0) ? 6 : 1)))
normal_dot_kernel(Geom g, LinkRef L, const char *t, const char *p, char *q, int64_t stride, const CgState *st,
                  double *partials, int max_blocks, int nrhs, int ngroups, TileMap tmap)
{
    typedef typename RealOf<P>::type T;
    int grp;
    const int tile = tile_group(ngroups, tmap, g.n[3], grp);
    if (tile < 0 || tile * (int)blockDim.x >= g.vh) return;  // padding tile (whole block)
    const int cb = tile * blockDim.x + threadIdx.x;
    const bool valid = cb < g.vh;
    const int r0 = grp * K;
    bool blk[K], act[K];
    bool any = false;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        blk[j] = (r0 + j < nrhs) && st[r0 + j].phase == CG_RUNNING;
        act[j] = blk[j] && valid;
        any |= blk[j];
    }
    if (!any) return;  // uniform over the block
    extern __shared__ __align__(16) char win[];
    int w0 = 0, wlen = 0;
    const int wstride = lds_window_stride(g, P);
    if (LF & LF_LDS)
        stage_block_window<P, K>(g, tile * blockDim.x, t + r0 * stride, stride, blk, win, wstride, w0, wlen);
    double dot[2 * K];  // <p,q>, <q,q> of each side
    V3<T> acc[K];
    // LF_PREFETCH with one vector: the site's own p is requested with the hop's words
    constexpr bool PF1 = (LF & LF_PREFETCH) != 0 && K == 1;
    typename SpinorIO<P>::Raw praw{};
    if (PF1 && act[0]) praw = SpinorIO<P>::load_raw(p + r0 * stride, g.vh, cb);
    if (valid) {
        const Site s = decode(g, cb, 0);
        hop_site<P, R, K, LF>(g, L, 0, s, cb, t + r0 * stride, stride, act, acc, win, wstride, w0, wlen);
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        double pq = 0.0, qq = 0.0;
        if (act[j]) {
            const V3<T> pv = PF1 ? SpinorIO<P>::decode(praw) : SpinorIO<P>::load(p + (r0 + j) * stride, g.vh, cb);
            const T m2 = (T)st[r0 + j].m2;
            V3<T> qv;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                qv.c[a].re = m2 * pv.c[a].re - acc[j].c[a].re;
                qv.c[a].im = m2 * pv.c[a].im - acc[j].c[a].im;
                const double pr = pv.c[a].re, pi = pv.c[a].im, qr = qv.c[a].re, qi = qv.c[a].im;
                pq += pr * qr + pi * qi;
                qq += qr * qr + qi * qi;
            }
            SpinorIO<P>::store(q + (r0 + j) * stride, g.vh, cb, qv);
        }
        dot[2 * j] = pq;
        dot[2 * j + 1] = qq;
    }
    __shared__ double red[8][2 * K];
    block_sums<2 * K>(dot, red);
    // thread 2 j + d holds sum d of side j
    const int j = threadIdx.x >> 1;
    if (j < K && r0 + j < nrhs && st[r0 + j].phase == CG_RUNNING)
        partials[(int64_t)(r0 + j) * max_blocks + 2 * tile + (threadIdx.x & 1)] = dot[0];
}

// ---------------------------------------------------------------------------
// 3. the scalars, one block per right-hand side.  (Summing the partials in
// every block of the step kernel instead, with the state record double
// buffered, was slower: 20 us for that kernel at 32^3 x 8 in FP64 against 4.8
// for this one and 9.3 for the step.)
// Bound by its latencies: the record and the first 1024 pairs of partials come in
// one round trip, further ones four at a time, and one wave alone adds the rows
// (64^3 x 16, 8192 pairs: 7.1 -> 5.5 us; 24^4 solves 1 to 2.6 % faster).

template <bool CONJ>
__global__ void __launch_bounds__(1024) step_finalize_kernel(CgState *st, const double *partials,
                                                            const double *rr_partials, int max_blocks, int nblocks,
                                                            int nr_blocks, int last, int32_t *host_phase)
{
    const int r = blockIdx.x;
    const double *pp = partials + (int64_t)r * max_blocks;
    const DotShare first = first_dots<CONJ>(pp, rr_partials + (int64_t)r * max_blocks, nblocks, nr_blocks);
    CgState S = st[r];
    double v[4];
    add_dots(pp, nblocks, nr_blocks, first, v);
    __shared__ double red[16][4];
    if (!block_sums_first<4>(v, red) || threadIdx.x != 0) return;
    // (a step to settle: this iteration's products of the old direction are not used)
    if (S.phase != CG_RUNNING) S.live = 0;
    else if (S.unsettled) cg_settle(S, v[2], last);
    else cg_step_scalars<CONJ>(S, v[0], v[1], v[2], v[3], last);
    st[r] = S;
    publish(host_phase, r, S.phase);
}

// ---------------------------------------------------------------------------
// 4. x += alpha p (x_lo in mixed precision), r -= alpha q, p = r + beta p, and
//    the block partials of |r|^2 (grid-stride, blockIdx.y = rhs)
//
// EARLY (one right-hand side, one site per thread): the site's four vectors are
// requested together with the state record, one memory round trip instead of
// two; otherwise a right-hand side that has converged reads only its record.
// Bound by HBM, or on small lattices by its fixed cost: 7 vectors a site where
// separate r and x/p updates read and wrote 8 in two launches (32^3 x 8, 16
// FP32 vectors: 53 us against 31 + 38; 64^3 x 16 FP16 storage 46 against
// 22 + 32; 32^3 x 8 FP64 9.3 against 6.4 + 6.1).

template <int PA, int PI, bool EARLY>
__global__ void __launch_bounds__(BLAS_BLOCK) step_kernel(int vh, char *x, char *r, char *p, const char *q, int64_t sa,
                                                          int64_t si, const CgState *st, double *rr_partials,
                                                          int max_blocks)
{
    typedef typename RealOf<PA>::type T;
    typedef typename RealOf<PI>::type TI;
    const int rhs = blockIdx.y;
    x += rhs * sa;
    r += rhs * sa;
    p += rhs * si;
    q += rhs * si;
    const int c0 = blockIdx.x * blockDim.x + threadIdx.x;
    typename SpinorIO<PI>::Raw qraw{}, praw{};
    typename SpinorIO<PA>::Raw rraw{}, xraw{};
    if (EARLY) {
        const int cf = c0 < vh ? c0 : vh - 1;  // a valid site for every thread (vh >= 1)
        qraw = SpinorIO<PI>::load_raw(q, vh, cf);
        praw = SpinorIO<PI>::load_raw(p, vh, cf);
        rraw = SpinorIO<PA>::load_raw(r, vh, cf);
        xraw = SpinorIO<PA>::load_raw(x, vh, cf);
    }
    const int live = st[rhs].live;
    const bool pdir = !st[rhs].p_due;
    const T alpha = (T)st[rhs].alpha, beta = (T)st[rhs].beta;
    if (EARLY) {
        issue_here(qraw);
        issue_here(praw);
        issue_here(rraw);
        issue_here(xraw);
    }
    if (!live) return;
    constexpr bool CONJ = corrects_prediction(PI);
    double sums[2] = {0.0, 0.0};  // |r|^2; <q,p> of the new p
    auto site = [&](int cb, const V3<T> &qv, const V3<T> &pv, V3<T> rv, V3<T> xv) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            xv.c[a].re = fused(alpha, pv.c[a].re, xv.c[a].re);
            xv.c[a].im = fused(alpha, pv.c[a].im, xv.c[a].im);
            rv.c[a].re = fused(-alpha, qv.c[a].re, rv.c[a].re);
            rv.c[a].im = fused(-alpha, qv.c[a].im, rv.c[a].im);
            sums[0] += (double)rv.c[a].re * (double)rv.c[a].re + (double)rv.c[a].im * (double)rv.c[a].im;
        }
        SpinorIO<PA>::store(x, vh, cb, xv);
        SpinorIO<PA>::store(r, vh, cb, rv);
        const V3<T> pn = direction_of<PA>(rv, pv, beta);
        if (CONJ) sums[1] += re_dot(qv, pn);
        if (pdir) SpinorIO<PI>::store(p, vh, cb, vcast<TI>(pn));
    };
    if (EARLY) {
        if (c0 < vh)
            site(c0, vcast<T>(SpinorIO<PI>::decode(qraw)), vcast<T>(SpinorIO<PI>::decode(praw)),
                 SpinorIO<PA>::decode(rraw), SpinorIO<PA>::decode(xraw));
    } else {
        for (int cb = c0; cb < vh; cb += gridDim.x * blockDim.x)
            site(cb, vcast<T>(SpinorIO<PI>::load(q, vh, cb)), vcast<T>(SpinorIO<PI>::load(p, vh, cb)),
                 SpinorIO<PA>::load(r, vh, cb), SpinorIO<PA>::load(x, vh, cb));
    }
    rr_partials += (int64_t)rhs * max_blocks + blockIdx.x;
    if constexpr (CONJ) {
        __shared__ double red[BLAS_BLOCK / 64][2];
        block_sums<2>(sums, red);
        if (threadIdx.x < 2) rr_partials[threadIdx.x * PE_PARTIALS] = sums[0];
    } else {
        const double s = block_sum(sums[0]);
        if (threadIdx.x == 0) *rr_partials = s;
    }
}

// FP64 group, last: the direction update the step kernel left out, with the
// residual and beta the group has set.
template <int PA, int PI>
__global__ void __launch_bounds__(BLAS_BLOCK) pdir_kernel(int vh, const char *r, char *p, const char *q, int64_t sa,
                                                          int64_t si, const CgState *st, double *rr_partials,
                                                          int max_blocks, int32_t *host_phase)
{
    typedef typename RealOf<PA>::type T;
    typedef typename RealOf<PI>::type TI;
    const int rhs = blockIdx.y;
    const CgState &S = st[rhs];
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(host_phase, rhs, S.phase);
    if (!S.p_due || S.phase != CG_RUNNING || S.unsettled) return;
    const T beta = (T)S.beta;
    r += rhs * sa;
    p += rhs * si;
    q += rhs * si;
    double pe = 0.0;
    for (int cb = blockIdx.x * blockDim.x + threadIdx.x; cb < vh; cb += gridDim.x * blockDim.x) {
        const V3<T> pn = direction_of<PA>(SpinorIO<PA>::load(r, vh, cb), vcast<T>(SpinorIO<PI>::load(p, vh, cb)), beta);
        SpinorIO<PI>::store(p, vh, cb, vcast<TI>(pn));
        if (corrects_prediction(PI)) pe += re_dot(vcast<T>(SpinorIO<PI>::load(q, vh, cb)), pn);
    }
    if (!corrects_prediction(PI)) return;
    const double s = block_sum(pe);
    if (threadIdx.x == 0) rr_partials[(int64_t)rhs * max_blocks + PE_PARTIALS + blockIdx.x] = s;
}

// ---------------------------------------------------------------------------
// FP64 group: x += x_lo, x_lo = 0   (gate as in gate_state)

template <int PA>
__global__ void __launch_bounds__(BLAS_BLOCK) accumulate_kernel(int vh, double *x, char *xlo, int64_t sa,
                                                                const CgState *st, int gate_mode)
{
    const int rhs = blockIdx.y;
    if (!gate_state(st[rhs], gate_mode)) return;
    char *xd = (char *)x + rhs * spinor_bytes_per_site(F64) * (int64_t)vh;
    xlo += rhs * sa;
    for (int cb = blockIdx.x * blockDim.x + threadIdx.x; cb < vh; cb += gridDim.x * blockDim.x) {
        V3<double> xv = SpinorIO<F64>::load(xd, vh, cb);
        const V3<double> lv = vcast<double>(SpinorIO<PA>::load(xlo, vh, cb));
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            xv.c[a].re += lv.c[a].re;
            xv.c[a].im += lv.c[a].im;
        }
        SpinorIO<F64>::store(xd, vh, cb, xv);
        SpinorIO<PA>::store(xlo, vh, cb, vcast<typename RealOf<PA>::type>(vzero<double>()));
    }
}

// r_hi = b - (m^2 x - D_eo t64) in FP64, |r_hi|^2; r (PA) = r_hi unless mode 2.
// gate_mode as in gate_state (0: all right-hand sides).
template <int R, int PA, int K, int LF>
__global__ void __launch_bounds__(512) residual_kernel(Geom g, LinkRef L, const char *t64, const char *x,
                                                       const char *b, char *r, int64_t sa, CgState *st,
                                                       double *partials, int max_blocks, int nrhs, int gate_mode,
                                                       int mode, int ngroups, TileMap tmap)
{
    const int64_t s64 = spinor_bytes_per_site(F64) * (int64_t)g.vh;
    int grp;
    const int tile = tile_group(ngroups, tmap, g.n[3], grp);
    if (tile < 0 || tile * (int)blockDim.x >= g.vh) return;  // padding tile (whole block)
    const int cb = tile * blockDim.x + threadIdx.x;
    const bool valid = cb < g.vh;
    const int r0 = grp * K;
    bool blk[K], act[K];
    bool any = false;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        blk[j] = (r0 + j < nrhs) && gate_state(st[r0 + j], gate_mode);
        act[j] = blk[j] && valid;
        any |= blk[j];
    }
    if (!any) return;
    V3<double> acc[K];
    double nrm[K];
    if (valid) {
        const Site s = decode(g, cb, 0);
        hop_site<F64, R, K, LF>(g, L, 0, s, cb, t64 + r0 * s64, s64, act, acc);
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        nrm[j] = 0.0;
        if (!act[j]) continue;
        const V3<double> xv = SpinorIO<F64>::load(x + (r0 + j) * s64, g.vh, cb);
        const V3<double> bv = SpinorIO<F64>::load(b + (r0 + j) * s64, g.vh, cb);
        const double m2 = st[r0 + j].m2;
        V3<double> rv;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            rv.c[a].re = bv.c[a].re - (m2 * xv.c[a].re - acc[j].c[a].re);
            rv.c[a].im = bv.c[a].im - (m2 * xv.c[a].im - acc[j].c[a].im);
            nrm[j] += rv.c[a].re * rv.c[a].re + rv.c[a].im * rv.c[a].im;
        }
        if (mode != 2) SpinorIO<PA>::store(r + (r0 + j) * sa, g.vh, cb, vcast<typename RealOf<PA>::type>(rv));
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (!blk[j]) continue;
        const int rr = r0 + j;
        const double s = block_sum(nrm[j]);
        if (threadIdx.x == 0) partials[(int64_t)rr * max_blocks + tile] = s;
    }
}

// |b|^2 per right-hand side; cold start: x = 0, r = b, p = b, x_lo = 0.
template <int PA, int PI>
__global__ void __launch_bounds__(BLAS_BLOCK) init_kernel(int vh, const char *b, double *x, char *r, char *p,
                                                          char *xlo, int64_t sa, int64_t si, CgState *st,
                                                          double *partials, int max_blocks, int cold)
{
    typedef typename RealOf<PA>::type T;
    typedef typename RealOf<PI>::type TI;
    const int rhs = blockIdx.y;
    const int64_t s64 = spinor_bytes_per_site(F64) * (int64_t)vh;
    b += rhs * s64;
    char *xd = (char *)x + rhs * s64;
    double local = 0.0;
    for (int cb = blockIdx.x * blockDim.x + threadIdx.x; cb < vh; cb += gridDim.x * blockDim.x) {
        const V3<double> bv = SpinorIO<F64>::load(b, vh, cb);
#pragma unroll
        for (int a = 0; a < 3; ++a) local += bv.c[a].re * bv.c[a].re + bv.c[a].im * bv.c[a].im;
        if (cold) {
            SpinorIO<F64>::store(xd, vh, cb, vzero<double>());
            SpinorIO<PA>::store(r + rhs * sa, vh, cb, vcast<T>(bv));
            SpinorIO<PI>::store(p + rhs * si, vh, cb, vcast<TI>(bv));
        }
        if (xlo) SpinorIO<PA>::store(xlo + rhs * sa, vh, cb, vzero<T>());
    }
    const double s = block_sum(local);
    if (threadIdx.x == 0) partials[(int64_t)rhs * max_blocks + blockIdx.x] = s;
}

// ---------------------------------------------------------------------------
// Second reduction stage: one block per right-hand side sums the block
// partials of the kernel before it in a fixed order and updates the scalars.
// Running it as its own kernel (rather than in the last block of the
// producer) needs no device-scope fence: the kernel boundary orders the
// partials' stores before these loads.

enum FinMode { FIN_RESID = 0, FIN_INIT = 1 };

__global__ void __launch_bounds__(1024) finalize_kernel(CgState *st, const double *partials, int max_blocks,
                                                       int nblocks, int mode, int gate_mode, int sub)
{
    const int r = blockIdx.x;
    // The state record (into registers) and the partials are requested
    // together, before the gate decides: one memory round trip instead of
    // three (gate, partials, then the fields the bookkeeping reads).  The
    // record is written back whole by thread 0.
    const double *p = partials + (int64_t)r * max_blocks;
    const int i0 = threadIdx.x;
    const double first = p[i0 < nblocks ? i0 : nblocks - 1];  // nblocks >= 1
    CgState S = st[r];
    double acc = 0.0;
    acc += i0 < nblocks ? first : 0.0;
    for (int i = i0 + blockDim.x; i < nblocks; i += blockDim.x) acc += p[i];
    if (mode == FIN_RESID && !gate_state(S, gate_mode)) {
        // sub 4: a direction left to a group before this one has been formed there
        if (sub == 4 && S.phase == CG_RUNNING && threadIdx.x == 0) st[r].p_due = 0;
        return;
    }
    const double v = block_sum(acc);
    if (threadIdx.x != 0) return;
    if (mode == FIN_RESID) {
        fin_residual(S, v, sub);
    } else {  // FIN_INIT, sub = cold start
        S.b2 = v;
        S.stop2 = S.stop2 * v;  // the host stored tol^2 here
        if (sub) {
            S.rho_known = 1;
            S.rho = v;
            S.max_rho = v;
            S.true_r2 = v;
            S.phase = (v == 0.0) ? CG_CONVERGED : (isfinite(v) ? CG_RUNNING : CG_NONFINITE);
        }
    }
    st[r] = S;
}

static void launch_finalize(const CgVectors &v, const double *partials, int nblocks, int mode, int gate_mode, int sub,
                            hipStream_t s)
{
    hipLaunchKernelGGL(finalize_kernel, dim3(v.nrhs), dim3(1024), 0, s, v.state, partials, v.max_blocks, nblocks,
                       mode, gate_mode, sub);
    LQS_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// host side

// Threads per block of the vector kernels: 64 while all sides together leave
// CUs idle (at most 2^16 sites, and so at most 1024 blocks a side).
static int blas_block(int64_t vh, int nrhs) { return vh * nrhs <= (1 << 16) ? 64 : BLAS_BLOCK; }
static int blas_blocks(int64_t vh, int nrhs)
{
    const int block = blas_block(vh, nrhs);
    int64_t b = (vh + block - 1) / block;
    return (int)(b < 1024 ? b : 1024);
}

void cg_fill_rates(lqs_cg_stats &o, const Gauge &gauge, int prec, int recon, int nrhs)
{
    const double t = o.device_seconds > 0 ? o.device_seconds : o.seconds;
    if (!(t > 0) || o.iters <= 0) {
        o.gflops = o.gbytes_per_s = 0.0;
        return;
    }
    const double real = prec == F64 ? 8 : prec == F32 ? 4 : 2;
    const double lps = gauge.temporal ? 6.0 + 2.0 / gauge.g.n[3] : 8.0;
    const double L = lps * real * recon / (nrhs > 0 ? nrhs : 1);
    const double sv = (double)spinor_bytes_per_site(prec), a = (double)spinor_bytes_per_site(prec == F64 ? F64 : F32);
    // t = D_oe p; q = m^2 p - D_eo t; x, r and p updated from one another and q
    const double bytes = (L + 2 * sv) + (L + 3 * sv) + (4 * a + 3 * sv);
    const double n = (double)gauge.vh * o.iters;
    o.gflops = 1140.0 * n / t * 1e-9;
    o.gbytes_per_s = bytes * n / t * 1e-9;
}

template <int P, int R>
static void launch_normal_dot(const Gauge &gauge, const CgVectors &v, LaunchShape sh, hipStream_t s)
{
    const Geom &g = gauge.g;
    const int64_t stride = field_bytes(g, P, 1);
    const LinkRef L = gauge.ref(P, R);
    const int G = (v.nrhs + sh.rhs_per_thread - 1) / sh.rhs_per_thread;
    const TileMap tmap = tile_map(g, sh.block, sh.xcd_slab, time_run(g, sh.block, v.nrhs, P, sh.trun));
    const dim3 grid(tile_map_blocks(g, sh.block, tmap, G));
    const size_t lds = hop_lds_bytes(g, P, sh.rhs_per_thread, sh);
#define LQS_ND(K, LF)                                                                                             \
    hipLaunchKernelGGL((normal_dot_kernel<P, R, K, LF>), grid, dim3(sh.block), lds, s, g, L, (const char *)v.t,   \
                       (const char *)v.p, (char *)v.q, stride, (const CgState *)v.state, v.partials, v.max_blocks, \
                       v.nrhs, G, tmap)
#define LQS_ND_LF(LF)                                                                                            \
    if (sh.rhs_per_thread == 1) LQS_ND(1, LF);                                                                   \
    else if (sh.rhs_per_thread == 2) LQS_ND(2, LF);                                                              \
    else LQS_ND(4, LF)
    const int lf = (L.temporal ? LF_TEMPORAL : 0) | (sh.stream_links ? LF_STREAM : 0) | (lds ? LF_LDS : 0);
    if (sh.prefetch && !lds) {
        switch (lf) {
        case 0: LQS_ND_LF(LF_PREFETCH); break;
        case LF_TEMPORAL: LQS_ND_LF(LF_PREFETCH | LF_TEMPORAL); break;
        case LF_STREAM: LQS_ND_LF(LF_PREFETCH | LF_STREAM); break;
        default: LQS_ND_LF(LF_PREFETCH | LF_TEMPORAL | LF_STREAM); break;
        }
        LQS_HIP(hipGetLastError());
        return;
    }
    switch (lf) {
    case 0: LQS_ND_LF(0); break;
    case LF_TEMPORAL: LQS_ND_LF(LF_TEMPORAL); break;
    case LF_STREAM: LQS_ND_LF(LF_STREAM); break;
    case LF_TEMPORAL | LF_STREAM: LQS_ND_LF(LF_TEMPORAL | LF_STREAM); break;
    case LF_LDS: LQS_ND_LF(LF_LDS); break;
    case LF_LDS | LF_STREAM: LQS_ND_LF(LF_LDS | LF_STREAM); break;
    case LF_LDS | LF_TEMPORAL: LQS_ND_LF(LF_LDS | LF_TEMPORAL); break;
    default: LQS_ND_LF(LF_LDS | LF_TEMPORAL | LF_STREAM); break;
    }
#undef LQS_ND_LF
#undef LQS_ND
    LQS_HIP(hipGetLastError());
}

void launch_normal_dot_shape(const Gauge &gauge, const CgVectors &v, LaunchShape shd, hipStream_t s)
{
    if (v.prec == F64 && v.recon == 18) launch_normal_dot<F64, 18>(gauge, v, shd, s);
    else if (v.prec == F64) launch_normal_dot<F64, 12>(gauge, v, shd, s);
    else if (v.prec == F32 && v.recon == 18) launch_normal_dot<F32, 18>(gauge, v, shd, s);
    else if (v.prec == F32) launch_normal_dot<F32, 12>(gauge, v, shd, s);
    else if (v.recon == 18) launch_normal_dot<F16, 18>(gauge, v, shd, s);
    else launch_normal_dot<F16, 12>(gauge, v, shd, s);
}

// The scalars of a step from the nd_blocks partials of the normal kernel, and
// the step.
template <int PA, int PI>
static void launch_step(const Gauge &gauge, const CgVectors &v, int nd_blocks, int last, int32_t *host_phase,
                        hipStream_t s)
{
    const int vh = (int)gauge.vh;
    const int64_t sa = field_bytes(gauge.g, PA, 1), si = field_bytes(gauge.g, PI, 1);
    const dim3 grid(blas_blocks(vh, v.nrhs), v.nrhs);
    hipLaunchKernelGGL(step_finalize_kernel<corrects_prediction(PI)>, dim3(v.nrhs), dim3(1024), 0, s, v.state, (const double *)v.partials,
                       (const double *)v.partials2, v.max_blocks, nd_blocks, (int)grid.x, last, host_phase);
    const bool early = v.nrhs == 1 && vh <= (int)grid.x * blas_block(vh, v.nrhs);
#define LQS_STEP(EARLY)                                                                                           \
    hipLaunchKernelGGL((step_kernel<PA, PI, EARLY>), grid, dim3(blas_block(vh, v.nrhs)), 0, s, vh, (char *)v.xlo,             \
                       (char *)v.r, (char *)v.p, (const char *)v.q, sa, si, (const CgState *)v.state,             \
                       v.partials2, v.max_blocks)
    if (early) LQS_STEP(true);
    else LQS_STEP(false);
#undef LQS_STEP
    LQS_HIP(hipGetLastError());
}

// The FP64 group's direction update.
template <int PA, int PI>
static void launch_pdir(const Gauge &gauge, const CgVectors &v, int32_t *host_phase, hipStream_t s)
{
    const int vh = (int)gauge.vh;
    const int64_t sa = field_bytes(gauge.g, PA, 1), si = field_bytes(gauge.g, PI, 1);
    hipLaunchKernelGGL((pdir_kernel<PA, PI>), dim3(blas_blocks(vh, v.nrhs), v.nrhs), dim3(blas_block(vh, v.nrhs)), 0, s, vh,
                       (const char *)v.r, (char *)v.p, (const char *)v.q, sa, si, (const CgState *)v.state, v.partials2,
                       v.max_blocks, host_phase);
    LQS_HIP(hipGetLastError());
}

// The hop's default launch for this many right-hand sides (the partials are
// indexed by tile: the sums do not depend on the map or on K).  16
// sides on 32^3 x 8 with 12-real links: 137 us, and 251 with two sides per
// thread in lexicographic order; 8 sides with 18-real links 80 and 175.
template <int PA, int R>
static void launch_residual_k(const Gauge &gauge, const CgVectors &v, int gate_mode, int mode, hipStream_t s)
{
    const Geom &g = gauge.g;
    const LinkRef L = gauge.ref(F64, R);
    const LaunchShape sh = default_hop_shape(g, F64, L, v.nrhs);
    const int block = sh.block, tiles = (g.vh + block - 1) / block;
    const int G = (v.nrhs + sh.rhs_per_thread - 1) / sh.rhs_per_thread;
    const TileMap tmap = tile_map(g, block, sh.xcd_slab, time_run(g, block, v.nrhs, F64, sh.trun));
    const dim3 grid(tile_map_blocks(g, block, tmap, G));
    const int lf =
        (L.temporal ? LF_TEMPORAL : 0) | (sh.stream_links ? LF_STREAM : 0) | (sh.prefetch ? LF_PREFETCH : 0);
    const int64_t sa = field_bytes(g, PA, 1);
    char *r = (char *)(mode == 2 ? nullptr : v.r);
#define LQS_RES(K, LF)                                                                                            \
    hipLaunchKernelGGL((residual_kernel<R, PA, K, LF>), grid, dim3(block), 0, s, g, L, (const char *)v.t64,       \
                       (const char *)v.x, (const char *)v.b, r, sa, v.state, v.partials, v.max_blocks, v.nrhs,    \
                       gate_mode, mode, G, tmap)
#define LQS_RES_K(LF)                                                                                             \
    if (sh.rhs_per_thread == 1) LQS_RES(1, LF);                                                                   \
    else if (sh.rhs_per_thread == 2) LQS_RES(2, LF);                                                              \
    else LQS_RES(4, LF)
    switch (lf) {
    // without prefetch: one side on a large lattice
    case 0: LQS_RES(1, 0); break;
    case LF_TEMPORAL: LQS_RES(1, LF_TEMPORAL); break;
    case LF_STREAM: LQS_RES(1, LF_STREAM); break;
    case LF_TEMPORAL | LF_STREAM: LQS_RES(1, LF_TEMPORAL | LF_STREAM); break;
    case LF_PREFETCH: LQS_RES_K(LF_PREFETCH); break;
    case LF_PREFETCH | LF_TEMPORAL: LQS_RES_K(LF_PREFETCH | LF_TEMPORAL); break;
    case LF_PREFETCH | LF_STREAM: LQS_RES_K(LF_PREFETCH | LF_STREAM); break;
    default: LQS_RES_K(LF_PREFETCH | LF_TEMPORAL | LF_STREAM); break;
    }
#undef LQS_RES_K
#undef LQS_RES
    LQS_HIP(hipGetLastError());
    launch_finalize(v, v.partials, tiles, FIN_RESID, gate_mode, mode, s);
}

// FP64 residual with the R-real FP64 links
static void launch_residual(const Gauge &gauge, const CgVectors &v, int R, int gate_mode, int mode, hipStream_t s)
{
    if (v.acc_prec == F64) {
        if (R == 12) launch_residual_k<F64, 12>(gauge, v, gate_mode, mode, s);
        else launch_residual_k<F64, 18>(gauge, v, gate_mode, mode, s);
    } else {
        if (R == 12) launch_residual_k<F32, 12>(gauge, v, gate_mode, mode, s);
        else launch_residual_k<F32, 18>(gauge, v, gate_mode, mode, s);
    }
}

static void launch_accumulate(const Gauge &gauge, const CgVectors &v, int gate_mode, hipStream_t s)
{
    const int vh = (int)gauge.vh;
    dim3 grid(blas_blocks(vh, v.nrhs), v.nrhs);
    const int64_t sa = field_bytes(gauge.g, v.acc_prec, 1);
    LQS_REQUIRE(v.acc_prec == F32, LQS_EUNSUPPORTED, "accumulate needs an FP32 inner solution");
    hipLaunchKernelGGL((accumulate_kernel<F32>), grid, dim3(blas_block(vh, v.nrhs)), 0, s, vh, v.x, (char *)v.xlo, sa,
                       (const CgState *)v.state, gate_mode);
    LQS_HIP(hipGetLastError());
}

// t64 = D_oe x and the residual kernel with the R-real FP64 links
static void residual_pass(const Gauge &gauge, const CgVectors &v, int R, int gate_mode, int mode, hipStream_t s)
{
    const LinkRef L64 = gauge.ref(F64, R);
    const LaunchShape sh = default_hop_shape(gauge.g, F64, L64, v.nrhs);
    launch_hop_gated(gauge.g, L64, F64, R, 0, 1, v.nrhs, v.x, v.t64, v.state, gate_mode, sh, s);
    launch_residual(gauge, v, R, gate_mode, mode, s);
}

// Stored reals of the FP64 links that a mixed solve's reliable updates use.
static int periodic_links(const Gauge &gauge, const CgVectors &v)
{
    return v.recon == 12 && gauge.fmt[F64][1] ? 12 : 18;
}

// Both at once, for a recurrence that waits for no host: the reliable update,
// and the final check where the iterated residual met the target.
void cg_reliable_group(const Gauge &gauge, const CgVectors &v, hipStream_t s)
{
    launch_accumulate(gauge, v, 2, s);
    if (periodic_links(gauge, v) == 12) {
        residual_pass(gauge, v, 12, 3, 3, s);
        residual_pass(gauge, v, 18, 4, 0, s);
    } else {
        residual_pass(gauge, v, 18, 2, 0, s);
    }
}

// The FP64 residual group: x += x_lo (mixed), t64 = D_oe x, residual kernel,
// with the stored 18-real links.
void cg_residual_group(Ctx &ctx, const Gauge &gauge, const CgVectors &v, int gate_mode, int mode, hipStream_t s)
{
    (void)ctx;
    const bool mixed = v.acc_prec != F64;
    if (mixed && (mode == 0 || mode == 4)) launch_accumulate(gauge, v, gate_mode, s);
    residual_pass(gauge, v, 18, gate_mode, mode, s);
}

void cg_init(Ctx &ctx, const Gauge &gauge, CgVectors &v, bool use_x0, hipStream_t s)
{
    const int vh = (int)gauge.vh;
    dim3 grid(blas_blocks(vh, v.nrhs), v.nrhs);
    const int64_t sa = field_bytes(gauge.g, v.acc_prec, 1), si = field_bytes(gauge.g, v.prec, 1);
    char *xlo = v.acc_prec == F64 ? nullptr : (char *)v.xlo;
    const int cold = use_x0 ? 0 : 1;
#define LQS_INIT(PA, PI)                                                                                          \
    hipLaunchKernelGGL((init_kernel<PA, PI>), grid, dim3(blas_block(vh, v.nrhs)), 0, s, vh, (const char *)v.b, v.x,           \
                       (char *)v.r, (char *)v.p, xlo, sa, si, v.state, v.partials, v.max_blocks, cold)
    if (v.acc_prec == F64) LQS_INIT(F64, F64);
    else if (v.prec == F32) LQS_INIT(F32, F32);
    else LQS_INIT(F32, F16);
#undef LQS_INIT
    LQS_HIP(hipGetLastError());
    launch_finalize(v, v.partials, grid.x, FIN_INIT, 0, cold, s);
    if (use_x0) {
        cg_residual_group(ctx, gauge, v, 0, 1, s);
        launch_convert(gauge.g, v.nrhs, v.acc_prec, v.r, v.prec, v.p, s);
    }
}

// Launch shapes of the CG kernels (tuned, else the default)
static void cg_shapes(Ctx &ctx, const Gauge &gauge, CgVectors &v)
{
    v.hop_shape = v.normal_shape = default_hop_shape(gauge.g, v.prec, gauge.ref(v.prec, v.recon), v.nrhs);
    if (!ctx.tuner) return;
    const bool tg = gauge.temporal;
    ctx.tuner->lookup(tune_key(ctx, tg ? "hop_tg" : "hop", gauge.g, v.prec, v.recon, v.nrhs), v.hop_shape);
    ctx.tuner->lookup(tune_key(ctx, tg ? "normal_dot_tg" : "normal_dot", gauge.g, v.prec, v.recon, v.nrhs),
                      v.normal_shape);
}

template <typename F> static void with_precs(const CgVectors &v, F &&f)
{
    if (v.acc_prec == F64) f(std::integral_constant<int, F64>(), std::integral_constant<int, F64>());
    else if (v.prec == F32) f(std::integral_constant<int, F32>(), std::integral_constant<int, F32>());
    else f(std::integral_constant<int, F32>(), std::integral_constant<int, F16>());
}

// One iteration; `last` of its round: the phases go to the host, in mixed
// precision after the group of the reliable updates.  In a solve on 12-real
// links the updates use the FP64 12-real links (two thirds of the bytes), and
// one that meets the target is handed to the final check; on 18-real links
// the group decides convergence as well.
static void cg_iteration(Ctx &ctx, const Gauge &gauge, CgVectors &v, hipStream_t s, bool last, int32_t *host_phase)
{
    const bool mixed = v.acc_prec != F64;
    // 1. t = D_oe p
    prof_begin(ctx, s);
    launch_hop_gated(gauge.g, gauge.ref(v.prec, v.recon), v.prec, v.recon, 0, 1, v.nrhs, v.p, v.t, v.state, 1,
                     v.hop_shape, s);
    prof_end(ctx, v.prec, v.recon, gauge.vh * v.nrhs, s);
    // 2. q = m^2 p - D_eo t and the dots
    launch_normal_dot_shape(gauge, v, v.normal_shape, s);
    // 3. and 4. the scalars; x, r and p
    const int nd_blocks = (int)((gauge.vh + v.normal_shape.block - 1) / v.normal_shape.block);
    with_precs(v, [&](auto pa, auto pi) {
        launch_step<pa.value, pi.value>(gauge, v, nd_blocks, last && mixed, last && !mixed ? host_phase : nullptr, s);
    });
    if (!last || !mixed) return;
    if (periodic_links(gauge, v) == 12) {
        launch_accumulate(gauge, v, 3, s);
        residual_pass(gauge, v, 12, 3, 3, s);
    } else {
        cg_residual_group(ctx, gauge, v, 2, 0, s);
    }
    with_precs(v, [&](auto pa, auto pi) { launch_pdir<pa.value, pi.value>(gauge, v, host_phase, s); });
}

// The FP64 check of the right-hand sides whose iterated residual met the target
// or that reached the iteration cap, always with the stored 18-real links, so
// the reported residual is that of the operator the caller passed; a side that
// is above the target goes on.  The others are left as they are: one that took a
// reliable update at the end of the round before has its direction already
// (formed a second time, it would no longer belong to the residual).
static void cg_final_check(Ctx &ctx, const Gauge &gauge, CgVectors &v, hipStream_t s, int32_t *host_phase)
{
    cg_residual_group(ctx, gauge, v, 4, 4, s);
    with_precs(v, [&](auto pa, auto pi) { launch_pdir<pa.value, pi.value>(gauge, v, host_phase, s); });
}

// ---------------------------------------------------------------------------
// one problem (nrhs >= 1) with the multi-kernel iteration

static bool final_phase(int32_t ph)
{
    return ph == CG_CONVERGED || ph == CG_BREAKDOWN || ph == CG_NONFINITE || ph == CG_MAXITER;
}

// Initial state records of one problem's right-hand sides.
static void cg_initial_states(const lqs_cg_params &prm, int nrhs, const double *mass, CgState *out)
{
    const bool mixed = prm.inner_prec != F64;
    const int rel_interval = mixed ? (prm.reliable_interval > 0 ? prm.reliable_interval : 100) : 0;
    const double delta =
        mixed ? (prm.reliable_delta > 0 ? prm.reliable_delta : default_reliable_delta(prm.inner_prec)) : 0.0;
    for (int r = 0; r < nrhs; ++r) {
        CgState S{};
        S.stop2 = prm.tol * prm.tol;
        S.delta2 = delta * delta;
        S.rel_interval = rel_interval;
        S.max_iter = prm.max_iter;
        S.phase = CG_RUNNING;
        S.m2 = mass[r] * mass[r];
        out[r] = S;
    }
}

// Device workspace that a problem is charged with against the preallocated
// region of the allocation-free solve (two reduction buffers of one double per
// 64 sites, 1024 at least).  The buffers hold up to twice that (two sums a block
// in the step kernel, and in the normal kernel in blocks of 64 or 128 threads):
// at most NOALLOC_SLACK_BYTES more, which the region holds in addition (a problem
// is charged at least 144 bytes a site and side, so its at most 16 sides have
// fewer than 2^19 sites together).
size_t cg_workspace_bytes(const Gauge &gauge, const lqs_cg_params &prm, int nrhs)
{
    auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
    const bool mixed = prm.inner_prec != F64;
    const size_t fp = field_bytes(gauge.g, prm.inner_prec, nrhs), fa = field_bytes(gauge.g, mixed ? F32 : F64, nrhs),
                 f64 = field_bytes(gauge.g, F64, nrhs);
    const size_t part = sizeof(double) * std::max<size_t>(1024, (size_t)(gauge.vh + 63) / 64) * nrhs;
    size_t n = up(sizeof(CgState) * nrhs) + 2 * up(part) + 3 * up(fp) + up(fa);
    if (mixed) n += up(fa) + up(f64);
    return n;
}

// One problem driven as a small state machine, so that several problems on
// their own streams can be advanced in turn by one host thread.
namespace {

struct CgRun {
    Ctx &ctx;
    lqs_problem pb;
    lqs_cg_params prm;
    lqs_cg_stats *stats;
    hipStream_t s;
    std::string tag;
    std::chrono::steady_clock::time_point t0;
    CgVectors v{};
    bool mixed = false;
    int nrhs = 1;
    size_t sbytes = 0;
    CgState *hs = nullptr;         // host mirror of the records
    int32_t *host_phase = nullptr; // phases as the rounds publish them (null with an arena)
    hipEvent_t ev[2] = {nullptr, nullptr};
    hipEvent_t tev[2] = {nullptr, nullptr};  // timing: first and last kernel of the solve
    int64_t queued = 0, waited = 0;  // rounds and final checks queued, and known to have run
    int64_t check_at = 0;            // `queued` after the last final check (0: none yet)
    int64_t enqueued = 0, cap = 0;   // iterations
    bool done = false;
    bool want_check = false;  // a right-hand side waits for its final check
    bool idle = false;        // none is iterating
    bool use_graph = false;  // s is a side stream and graphs are on
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    // iterations of a round, between polls of the state and in mixed precision
    // between FP64 groups (gated launches that return at once unless a reliable
    // update is pending)
    static constexpr int chunk = 8;

    CgRun(Ctx &c, const lqs_problem &p, const lqs_cg_params &pr, lqs_cg_stats *st, hipStream_t str, std::string tg,
          std::chrono::steady_clock::time_point start)
        : ctx(c), pb(p), prm(pr), stats(st), s(str), tag(std::move(tg)), t0(start)
    {
    }
    ~CgRun()
    {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        for (hipEvent_t e : tev)
            if (e) (void)hipEventDestroy(e);
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
    }

    void round()
    {
        for (int i = 0; i < chunk; ++i) cg_iteration(ctx, gauge(), v, s, i == chunk - 1, host_phase);
    }
    const Gauge &gauge() const { return *pb.gauge; }

    // Buffers come from the context's workspace, or, when `arena` is set,
    // are carved from that preallocated device region (no allocation).
    std::vector<double> masses;  // per right-hand side (empty: pb.mass for all)
    char *arena = nullptr;
    size_t arena_bytes = 0, arena_used = 0;
    CgState *arena_host = nullptr;  // host mirror with an arena
    void *buf(const std::string &slot, size_t bytes)
    {
        if (!arena) return ctx.workspace(slot + tag, bytes);
        const size_t off = (arena_used + 255) & ~size_t(255);
        LQS_REQUIRE(off + bytes <= arena_bytes, LQS_EINVAL, "workspace exceeds the preallocated region");
        arena_used = off + bytes;
        return arena + off;
    }

    void setup()
    {
        const Geom &g = gauge().g;
        nrhs = pb.nrhs;
        mixed = prm.inner_prec != F64;
        v.prec = prm.inner_prec;
        v.acc_prec = mixed ? F32 : F64;
        v.recon = prm.inner_recon == 12 ? 12 : 18;
        v.nrhs = nrhs;
        v.mass = pb.mass;
        (void)gauge().ref(v.prec, v.recon);  // format must exist
        cg_shapes(ctx, gauge(), v);
        v.max_blocks = cg_partials_needed(gauge().vh, v.normal_shape.block);
        sbytes = sizeof(CgState) * nrhs;
        // every size is checked before the first launch
        const size_t need = cg_workspace_bytes(gauge(), prm, nrhs);
        LQS_REQUIRE(!arena || need <= NOALLOC_SCRATCH_BYTES, LQS_EINVAL,
                    "solve needs " + std::to_string(need) + " bytes of workspace, the preallocated region holds " +
                        std::to_string(NOALLOC_SCRATCH_BYTES));
        const int64_t fp = field_bytes(g, v.prec, nrhs), fa = field_bytes(g, v.acc_prec, nrhs),
                      f64 = field_bytes(g, F64, nrhs);
        v.state = (CgState *)buf("cg.state", sbytes);
        v.partials = (double *)buf("cg.partials", sizeof(double) * (size_t)v.max_blocks * nrhs);
        v.partials2 = (double *)buf("cg.partials2", sizeof(double) * (size_t)v.max_blocks * nrhs);
        v.p = buf("cg.p", fp);
        v.q = buf("cg.q", fp);
        v.t = buf("cg.t", fp);
        v.x = pb.x;
        v.b = (double *)pb.b;
        if (mixed) {
            v.r = buf("cg.r", fa);
            v.xlo = buf("cg.xlo", fa);
            v.t64 = buf("cg.t64", f64);
            v.rhi = nullptr;
        } else {
            v.r = buf("cg.r", f64);
            v.xlo = pb.x;
            v.t64 = v.t;
            v.rhi = (double *)v.r;
        }
        if (arena) {
            hs = arena_host;
        } else {
            hs = (CgState *)ctx.pinned("cg.host" + tag, sbytes + sizeof(int32_t) * nrhs);
            host_phase = (int32_t *)(hs + nrhs);
            for (int r = 0; r < nrhs; ++r) host_phase[r] = CG_RUNNING;
        }
        std::vector<double> mass(nrhs, pb.mass);
        if (!masses.empty()) mass = masses;
        LQS_REQUIRE((int)mass.size() == nrhs, LQS_EINVAL, "one mass per right-hand side");
        cg_initial_states(prm, nrhs, mass.data(), hs);
        if (!arena) {
            LQS_HIP(hipEventCreate(&tev[0]));
            LQS_HIP(hipEventCreate(&tev[1]));
            LQS_HIP(hipEventRecord(tev[0], s));
        }
        LQS_HIP(hipMemcpyAsync(v.state, hs, sbytes, hipMemcpyHostToDevice, s));
        cg_init(ctx, gauge(), v, prm.use_x0 != 0, s);
        if (!arena) {
            LQS_HIP(hipEventCreateWithFlags(&ev[0], hipEventDisableTiming));
            LQS_HIP(hipEventCreateWithFlags(&ev[1], hipEventDisableTiming));
        }
        // never reached: an iteration may be followed by one that settles it and by
        // a failed check, behind what is left of its round and two more
        cap = (3 * chunk + 2) * (int64_t)prm.max_iter + 16 * chunk + 64;
    }

    // queue the final check that a right-hand side waits for, or one round of
    // iterations.  With graphs the first round runs eagerly, so that the GPU
    // works while the host captures and instantiates (150-200 us of an idle GPU
    // otherwise, at the start of every solve); the round is then captured once
    // (the kernels read their scalars and gates from the device state, so every
    // replay is the same work) and replayed; the round holds no memset, copy or
    // host synchronisation.
    void enqueue()
    {
        if (want_check) {
            cg_final_check(ctx, gauge(), v, s, host_phase);
            want_check = false;
            check_at = queued + 1;
        } else {
            if (use_graph && enqueued > 0) {
                if (!exec) {
                    LQS_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
                    try {
                        round();
                    } catch (...) {
                        hipGraph_t g = nullptr;
                        (void)hipStreamEndCapture(s, &g);
                        if (g) (void)hipGraphDestroy(g);
                        throw;
                    }
                    LQS_HIP(hipStreamEndCapture(s, &graph));
                    LQS_HIP(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
                }
                LQS_HIP(hipGraphLaunch(exec, s));
            } else {
                round();
            }
            enqueued += chunk;
        }
        if (arena) {
            // no events: wait for the records at once
            fetch();
            waited = ++queued;
            decide();
            return;
        }
        LQS_HIP(hipEventRecord(ev[queued & 1], s));
        ++queued;
    }

    void fetch()
    {
        LQS_HIP(hipMemcpyAsync(hs, v.state, sbytes, hipMemcpyDeviceToHost, s));
        LQS_HIP(hipStreamSynchronize(s));
    }

    int32_t phase_of(int r) const
    {
        return host_phase ? __atomic_load_n(host_phase + r, __ATOMIC_RELAXED) : hs[r].phase;
    }

    // What to queue next, from phases at least as new as entry `waited`.
    void decide()
    {
        bool all = true, waits = false, runs = false;
        for (int r = 0; r < nrhs; ++r) {
            const int32_t ph = phase_of(r);
            all &= final_phase(ph);
            waits |= ph == CG_INNER_DONE;
            runs |= ph == CG_RUNNING;
        }
        // (a check that is still in flight may be about to settle what waits)
        want_check = waits && waited >= check_at;
        idle = waits && !runs;
        if (all || enqueued > cap) done = true;
    }

    // wait for the state the initial residuals left
    void check_initial()
    {
        fetch();
        for (int r = 0; r < nrhs; ++r) host_phase[r] = hs[r].phase;
        decide();
    }

    // Wait for all but the newest entry (so that the GPU has work meanwhile), or
    // for that one too when no side is iterating, and decide.
    void check()
    {
        const int64_t upto = idle ? queued : queued - 1;
        if (upto <= waited) return;
        LQS_HIP(hipEventSynchronize(ev[(upto - 1) & 1]));
        waited = upto;
        decide();
    }

    void finish()
    {
        // right-hand sides that stopped without an FP64 check (breakdown,
        // non-finite, host cap) get x += x_lo and a measured residual
        fetch();
        bool need = false;
        for (int r = 0; r < nrhs; ++r) need |= !(hs[r].phase == CG_CONVERGED || hs[r].phase == CG_MAXITER);
        if (need) {
            if (mixed) launch_accumulate(gauge(), v, 0, s);
            cg_residual_group(ctx, gauge(), v, 0, 2, s);
            fetch();
        }
        float dev_ms = 0.f;
        if (tev[0]) {
            LQS_HIP(hipEventRecord(tev[1], s));
            LQS_HIP(hipEventSynchronize(tev[1]));
            LQS_HIP(hipEventElapsedTime(&dev_ms, tev[0], tev[1]));
        }
        const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        for (int r = 0; r < nrhs; ++r) {
            const CgState &S = hs[r];
            lqs_cg_stats &o = stats[r];
            o.iters = S.iters;
            o.reliable_updates = S.nreliable;
            o.restarts = S.restarts;
            o.true_rel_residual = S.b2 > 0 ? std::sqrt(S.true_r2 / S.b2) : 0.0;
            o.seconds = secs;
            o.device_seconds = 1e-3 * dev_ms;
            cg_fill_rates(o, gauge(), v.prec, v.recon, nrhs);
            switch (S.phase) {
            case CG_CONVERGED: o.status = LQS_OK; break;
            case CG_BREAKDOWN: o.status = LQS_EBREAKDOWN; break;
            case CG_NONFINITE: o.status = LQS_ENONFINITE; break;
            default: o.status = LQS_ENOTCONV; break;
            }
        }
    }
};

}  // namespace

// One problem replays graphs only below this many sites per parity, all sides
// together: between two graph launches the GPU idles for 13 us, and from here
// on a kernel runs longer than the host takes to launch the next.  16^4 FP16
// storage 5.21 ms with graphs, 5.09 launched kernel by kernel; 24^4 trajectory
// with fermions 28.5 and 27.3; 32^3 x 8 FP64 8.65 and 8.52; 8^4 FP64 3.45 and
// 3.51.  (Several problems at once share the host, and graphs win there:
// 16^4, 24^3 x 8 and 32^3 x 8 in FP32 8.6 against 9.1 ms.)
static constexpr int64_t GRAPH_SITES = 1 << 15;

void cg_solve_one(Ctx &ctx, const lqs_problem &pb, const lqs_cg_params &prm, lqs_cg_stats *stats, hipStream_t s,
                  const std::vector<double> *masses)
{
    // The solve runs on a side stream that waits for s (and has nothing left to
    // do when the call returns): the caller's stream may be the null stream,
    // which cannot be captured, and on which every launch would wait for, and
    // hold up, the process's blocking streams.  (The refinement of a multi-shift
    // solve, one mass per column, stays on the stream of its recurrence where it
    // replays no graph: crossing over costs 50 to 100 us.)
    const bool graph = ctx.graphs && !ctx.profiling && pb.gauge->vh * pb.nrhs < GRAPH_SITES;
    const bool side = graph || (ctx.graphs && !ctx.profiling && !masses);
    hipStream_t rs = side ? ctx.side_stream(0) : s;
    struct Event {
        hipEvent_t e = nullptr;
        ~Event()
        {
            if (e) (void)hipEventDestroy(e);
        }
    } fork;
    if (side) {
        LQS_HIP(hipEventCreateWithFlags(&fork.e, hipEventDisableTiming));
        LQS_HIP(hipEventRecord(fork.e, s));
        LQS_HIP(hipStreamWaitEvent(rs, fork.e, 0));
    }
    CgRun run(ctx, pb, prm, stats, rs, "", std::chrono::steady_clock::now());
    run.use_graph = graph;
    if (masses) run.masses = *masses;
    try {
        run.setup();
        // one mass per column: the multi-shift solver's check of solutions
        // that mostly meet the target already; two rounds of gated launches
        // cost more than waiting for the initial residuals
        if (masses && prm.use_x0) run.check_initial();
        while (!run.done) {
            run.enqueue();
            run.check();
        }
        run.finish();
    } catch (...) {
        (void)hipStreamSynchronize(rs);
        throw;
    }
}

// Problems of different sizes each get a side stream (forked from and joined
// back into s with events) and their own workspaces; the host enqueues a
// round of iterations for every unfinished problem before it waits on any
// poll, so the small lattices' kernels fill the gaps of the large ones.
void cg_solve_concurrent(Ctx &ctx, int nprob, const lqs_problem *probs, const lqs_cg_params &prm,
                         lqs_cg_stats *stats, hipStream_t s)
{
    constexpr int MAX_SIDE = 8;
    const auto t0 = std::chrono::steady_clock::now();
    const int nside = nprob < MAX_SIDE ? nprob : MAX_SIDE;
    hipEvent_t fork = nullptr;
    LQS_HIP(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
    std::vector<hipEvent_t> joins;
    std::vector<std::unique_ptr<CgRun>> runs;
    auto cleanup = [&]() {
        for (int k = 0; k < nside; ++k) (void)hipStreamSynchronize(ctx.side_stream(k));
        for (hipEvent_t e : joins) (void)hipEventDestroy(e);
        (void)hipEventDestroy(fork);
    };
    try {
        LQS_HIP(hipEventRecord(fork, s));
        for (int k = 0; k < nside; ++k) LQS_HIP(hipStreamWaitEvent(ctx.side_stream(k), fork, 0));
        int off = 0;
        for (int i = 0; i < nprob; ++i) {
            runs.emplace_back(new CgRun(ctx, probs[i], prm, stats + off, ctx.side_stream(i % nside),
                                        "#" + std::to_string(i), t0));
            runs.back()->use_graph = ctx.graphs && !ctx.profiling;
            off += probs[i].nrhs;
        }
        for (auto &r : runs) r->setup();
        bool any = true;
        while (any) {
            any = false;
            for (auto &r : runs)
                if (!r->done) r->enqueue();
            for (auto &r : runs)
                if (!r->done) {
                    r->check();
                    any |= !r->done;
                }
        }
        for (auto &r : runs) r->finish();
        for (int k = 0; k < nside; ++k) {
            hipEvent_t e = nullptr;
            LQS_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
            joins.push_back(e);
            LQS_HIP(hipEventRecord(e, ctx.side_stream(k)));
            LQS_HIP(hipStreamWaitEvent(s, e, 0));
        }
    } catch (...) {
        cleanup();
        throw;
    }
    cleanup();
}


// ---------------------------------------------------------------------------
// A solve that allocates nothing, for callers that cannot allocate device
// memory.  Its workspace is a file-scope device array (each GPU the library
// runs on holds its own copy until the process ends); host code never uses
// the array's name as an address, only the per-device address fetched once
// with hipGetSymbolAddress.  Every call on one GPU shares that GPU's array:
// calls that overlap on one GPU race.  The solve runs eagerly on the caller's
// stream (no graphs, no events, no pinned host buffers), with the kernels of
// cg_solve and the same launch shapes.

static __device__ __align__(256) char scratch[NOALLOC_SCRATCH_BYTES + NOALLOC_SLACK_BYTES];

static std::mutex scratch_mu;
static void *scratch_ptr[NOALLOC_MAX_DEVICES];

// Device address of this GPU's scratch array; the device must be current.
void *noalloc_scratch(int device)
{
    LQS_REQUIRE(device >= 0 && device < NOALLOC_MAX_DEVICES, LQS_EUNSUPPORTED, "device index too large");
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[device]) {
        void *ptr = nullptr;
        LQS_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        scratch_ptr[device] = ptr;
    }
    return scratch_ptr[device];
}

void cg_solve_noalloc_impl(Ctx &ctx, const lqs_problem &pb, const lqs_cg_params &prm, lqs_cg_stats *stats,
                           hipStream_t s)
{
    LQS_REQUIRE(ctx.noalloc_scratch != nullptr, LQS_EHIP, "scratch address not set up");
    const size_t need = cg_workspace_bytes(*pb.gauge, prm, pb.nrhs);
    LQS_REQUIRE(need <= NOALLOC_SCRATCH_BYTES, LQS_EINVAL,
                "solve needs " + std::to_string(need) + " bytes of workspace, more than the " +
                    std::to_string(NOALLOC_SCRATCH_BYTES) + "-byte scratch array");
    // hop profiling records events it creates on demand: off for this call
    struct ProfOff {
        Ctx &c;
        bool was;
        ~ProfOff() { c.profiling = was; }
    } prof{ctx, ctx.profiling};
    ctx.profiling = false;
    CgState host[16];
    CgRun run(ctx, pb, prm, stats, s, "", std::chrono::steady_clock::now());
    run.arena = (char *)ctx.noalloc_scratch;
    run.arena_bytes = NOALLOC_SCRATCH_BYTES + NOALLOC_SLACK_BYTES;
    run.arena_host = host;
    try {
        run.setup();
        while (!run.done) run.enqueue();
    } catch (...) {
        (void)hipStreamSynchronize(s);
        throw;
    }
    run.finish();
}

}  // namespace lqs
