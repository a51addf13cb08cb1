// multishift.hip -- several masses on one Krylov space (multi-shift CG).
//
// For M_i = m_i^2 - D_eo D_oe all systems share D_eo D_oe; they differ by a
// shift sigma_i = m_i^2 - m_0^2 >= 0 of the smallest mass m_0 (the base).
// CG on the base generates residuals r_k; the residual of shifted system i
// after k steps is zeta_k^i r_k (the Krylov space does not depend on the
// shift).  Writing the CG recurrences as a three-term recurrence for r_k and
// matching it with the shifted one gives, with alpha_k, beta_k of the base,
//   zeta_{k+1} = zeta_k zeta_{k-1} alpha_{k-1} /
//                [zeta_{k-1} alpha_{k-1} (1 + alpha_k sigma) + alpha_k beta_{k-1} (zeta_{k-1} - zeta_k)]
//   alpha^i_k = alpha_k zeta_{k+1} / zeta_k,  beta^i_k = beta_k (zeta_{k+1} / zeta_k)^2
//   x^i += alpha^i_k p^i,  p^i = zeta_{k+1} r_{k+1} + beta^i_k p^i
// (zeta_0 = zeta_{-1} = 1, alpha_{-1} = 1, beta_{-1} = 0).  A shifted system
// stops updating once |zeta| |r| meets the target.  This is the multi-mass
// solve a rational-approximation HMC needs for staggered fermions.
//
// One iteration: the base hop and fused normal operator with its two dots
// (shared with the plain solver), one one-block kernel for every scalar of the
// step (alpha, beta, each zeta, alpha_i, beta_i; |r - alpha q|^2 is predicted
// from the dots, see cg.hip), and one kernel that advances x_0, r, p_0 and every
// x_i, p_i with one read of each.  The recurrence runs in FP64, or with the search
// directions and the operator in FP32 or FP16 storage and the residual and
// the solutions in FP32.  In the mixed recurrence the base system takes the
// reliable updates of the mixed-precision CG: every K iterations, or when
// |r| fell below delta max |r|, every solution is added into the caller's
// FP64 field (its FP32 part restarts from zero), the base residual is
// replaced by b - M_0 x_0 computed in FP64, and beta and every beta_i are
// recomputed from it (the shifted residuals stay zeta_i r, which the
// replacement keeps to the accuracy of the FP64 residual).  Afterwards every
// mass gets an FP64 true-residual check that also refines it with a
// warm-started CG (mixed precision with FP16 storage when the recurrence was
// mixed) if the recurrence left it above tol.
#include <algorithm>
#include <chrono>
#include <cmath>

#include "cg_step.hpp"
#include "hop.hpp"

namespace lqs {

void launch_normal_dot_shape(const Gauge &gauge, const CgVectors &v, LaunchShape sh, hipStream_t s);
void cg_reliable_group(const Gauge &gauge, const CgVectors &v, hipStream_t s);

static constexpr int MS_MAX = 16;
static constexpr int MS_BLOCK = 256;

struct ShiftState {
    double sigma;                    // m_i^2 - m_0^2
    double zeta, zeta_prev;
    double alpha, beta;
    int32_t active;                  // still above the target
    int32_t iters;
    int32_t xupd;                    // alpha was formed this iteration: x_i += alpha p_i is due
};

struct ShiftPtrs {
    char *x[MS_MAX + 1];             // solution of each shifted system (storage PR)
    char *p[MS_MAX + 1];             // search direction of each shifted system (storage PI)
    double *x64[MS_MAX + 1];         // mixed recurrence: the caller's FP64 solution it is added into
                                     // (entry nshift: the base, for the final flush)
};

// What |r|^2 of a step leads to for the base (any: a shift is still active).
__device__ __forceinline__ void ms_decide(CgState &S, double r2, double b, bool any, int last)
{
    S.beta = b;
    S.rho = r2;
    if (r2 > S.max_rho) S.max_rho = r2;
    if ((r2 <= S.stop2 && !any) || S.iters >= S.max_iter) {
        S.phase = CG_INNER_DONE;
        S.p_due = 1;
        // mixed: the FP64 residual of the base decides (and resumes when it is above the target)
        if (S.rel_interval > 0) S.reliable_pending = 1;
        return;
    }
    if (S.rel_interval > 0 && (S.since_rel >= S.rel_interval || r2 < S.delta2 * S.max_rho)) S.reliable_pending = 1;
    if (last && S.reliable_pending) S.p_due = 1;
}

// Settles a step whose |r|^2 could not be predicted (cg_step.hpp) with the one
// that it left, rr: every direction is due, no solution is.
__device__ __forceinline__ void ms_settle(CgState &S, ShiftState &T, bool mine, double rr, int last)
{
    S.unsettled = 0;
    S.live = 0;
    S.p_due = 0;
    const bool on = mine && T.active;
    T.xupd = 0;
    if (!isfinite(rr)) {
        S.phase = CG_NONFINITE;
        return;
    }
    const double b = S.rho_old > 0.0 ? rr / S.rho_old : 0.0;
    if (on) {
        const double ratio = T.zeta / T.zeta_prev;
        T.alpha = 0.0;
        T.beta = b * ratio * ratio;
        T.xupd = 1;
        if (T.zeta * T.zeta * rr <= S.stop2) T.active = 0;
    }
    S.live = 2;
    ms_decide(S, rr, b, __any(mine && T.active), last);
}

// Every scalar of one iteration from the base's <p,q>, <q,q> (partials) and
// |r|^2 as the last step summed it (rr_partials, at most 1024; unused while
// rho holds a measured one; CONJ: <p_old,q> after them).  `last`: the FP64 group follows this iteration.
template <bool CONJ>
__global__ void __launch_bounds__(1024) ms_scalars(CgState *base, ShiftState *sh, int nshift, const double *partials,
                                                   const double *rr_partials, int nblocks, int nr_blocks, int last,
                                                   int32_t *host_phase)
{
    const DotShare first = first_dots<CONJ>(partials, rr_partials, nblocks, nr_blocks);
    CgState S = *base;
    const int phase = S.phase, i = threadIdx.x;
    const bool mine = i < nshift;
    ShiftState T{};
    if (mine) T = sh[i];
    double v[4];
    add_dots(partials, nblocks, nr_blocks, first, v);
    __shared__ double red[16][4];
    if (!block_sums_first<4>(v, red)) return;
    if (__builtin_expect(phase == CG_RUNNING && S.unsettled, 0)) {
        ms_settle(S, T, mine, v[2], last);
        if (mine) sh[i] = T;
        if (i != 0) return;
        *base = S;
        publish(host_phase, 0, S.phase);
        return;
    }
    const double pq = v[0], qq = v[1], rr = S.rho_known ? S.rho : v[2];
    // lane i < nshift advances shift i; lane 0 the base
    const bool ok = phase == CG_RUNNING && isfinite(pq) && pq > 0.0;
    const double a_prev = S.alpha, b_prev = S.beta, a = ok ? rr / pq : 0.0;
    const double r2 = predicted_r2<CONJ>(a, S.beta, qq, rr, v[3]);
    const double b = rr > 0.0 ? r2 / rr : 0.0;
    const bool finite = isfinite(r2), lost = prediction_lost(r2, rr, S.stop2) && S.iters + 1 < S.max_iter;
    T.xupd = 0;
    if (mine && ok && finite && T.active) {
        const double z = T.zeta, zp = T.zeta_prev;
        const double den = zp * a_prev * (1.0 + a * T.sigma) + a * b_prev * (zp - z);
        const double zn = z * zp * a_prev / den, ratio = zn / z;
        T.alpha = a * ratio;
        T.beta = b * ratio * ratio;
        T.zeta_prev = z;
        T.zeta = zn;
        T.iters += 1;
        T.xupd = 1;
        if (zn * zn * r2 <= S.stop2 && !lost) T.active = 0;
    }
    if (mine) sh[i] = T;
    const bool any = __any(mine && T.active);
    if (i != 0) return;
    struct Publish {
        const CgState &S;
        CgState *base;
        int32_t *host;
        __device__ ~Publish()
        {
            *base = S;
            publish(host, 0, S.phase);
        }
    } published{S, base, host_phase};
    S.live = 0;
    if (phase != CG_RUNNING) return;  // (a direction left to the FP64 group stays due until it has run)
    S.p_due = 0;
    if (!ok) {
        S.phase = isfinite(pq) ? CG_BREAKDOWN : CG_NONFINITE;
        return;
    }
    S.rho_known = 0;
    S.iters += 1;
    S.since_rel += 1;
    if (!finite) {
        S.phase = CG_NONFINITE;
        return;
    }
    S.alpha = a;
    S.rho_old = rr;
    S.live = 1;
    if (__builtin_expect(lost, 0)) {
        S.unsettled = 1;
        S.p_due = 1;
        if (S.rel_interval > 0 && S.since_rel >= S.rel_interval) S.reliable_pending = 1;
        return;
    }
    ms_decide(S, r2, b, any, last);
}

// Mixed recurrence, reliable update: add every FP32 solution into its FP64
// field and restart it from zero (gated: the base's update is pending, or
// gated = 0 at the end of the recurrence).
template <int PR>
__global__ void __launch_bounds__(MS_BLOCK) ms_accumulate(int vh, const ShiftPtrs *ptr, int nshift, const CgState *base,
                                                          int gated)
{
    typedef typename RealOf<PR>::type TR;
    if (gated && !base->reliable_pending) return;
    for (int cb = blockIdx.x * blockDim.x + threadIdx.x; cb < vh; cb += gridDim.x * blockDim.x)
        for (int i = 0; i < nshift; ++i) {
            V3<double> xv = SpinorIO<F64>::load(ptr->x64[i], vh, cb);
            const V3<double> lv = vcast<double>(SpinorIO<PR>::load(ptr->x[i], vh, cb));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                xv.c[c].re += lv.c[c].re;
                xv.c[c].im += lv.c[c].im;
            }
            SpinorIO<F64>::store(ptr->x64[i], vh, cb, xv);
            SpinorIO<PR>::store(ptr->x[i], vh, cb, vzero<TR>());
        }
}

// after a reliable update of the base: beta_i = beta (zeta_{k+1} / zeta_k)^2
// with the base's new beta (the same value ms_scalars set otherwise)
__global__ void ms_rebeta(const CgState *base, ShiftState *sh, int nshift)
{
    if (threadIdx.x != 0 || base->phase != CG_RUNNING) return;
    for (int i = 0; i < nshift; ++i) {
        ShiftState &T = sh[i];
        if (!T.active) continue;
        const double ratio = T.zeta / T.zeta_prev;
        T.beta = base->beta * ratio * ratio;
    }
}

// x_0 += alpha p_0, r -= alpha q, p_0 = r + beta p_0 and the block partials of
// |r|^2; for every shift, x_i += alpha_i p_i and p_i = zeta_i r + beta_i p_i.  Vectors are stored as PI
// (p, q) and PR (x, r); the arithmetic is FP64.  DIRS: the directions alone
// (the FP64 group's end, for the updates it was left).  Bound by HBM: 4 vectors
// a site and shift and 7 for the base.  (One block grid per system instead of
// the loop over the shifts measured slower: 0.41 vs 0.37 s for 8 masses on
// 64^3 x 16 in FP64, as every system re-read the residual.)
//
// A lattice of 32^3 x 8 gives each SIMD two waves, so a wave has its own next
// loads in flight: the block keeps the scalars and addresses of the shifts that
// are due in LDS, and x_i, p_i of the next one are requested before the present
// one is advanced (8 masses in FP64: 42.0 -> 34.6 us; 64^3 x 16: solve 357 -> 349 ms;
// 16^3 x 8 with 12 masses, in blocks of 64: 6.4 -> 3.3 ms with the earlier steps).
template <int PI, int PR, bool DIRS>
__global__ void __launch_bounds__(MS_BLOCK) ms_step(int vh, char *x0, char *r, char *p0, const char *q,
                                                    const ShiftPtrs *ptr, int nshift, const CgState *base,
                                                    const ShiftState *sh, double *rr_partials, int32_t *host_phase)
{
    typedef typename RealOf<PI>::type TI;
    typedef typename RealOf<PR>::type TR;
    typedef typename SpinorIO<PI>::Raw RawI;
    typedef typename SpinorIO<PR>::Raw RawR;
    constexpr bool CONJ = corrects_prediction(PI);
    struct Due {
        char *x, *p;
        double alpha, beta, zeta;
        int act;  // p_i too
    };
    __shared__ Due due[MS_MAX];
    __shared__ int ndue;
    const int c0 = blockIdx.x * blockDim.x + threadIdx.x;
    RawI praw, qraw{};
    RawR rraw, xraw{};
    auto load_base = [&](int cb) {
        praw = SpinorIO<PI>::load_raw(p0, vh, cb);
        rraw = SpinorIO<PR>::load_raw(r, vh, cb);
        if (!DIRS || CONJ) qraw = SpinorIO<PI>::load_raw(q, vh, cb);
        if (!DIRS) {
            xraw = SpinorIO<PR>::load_raw(x0, vh, cb);
        }
    };
    // the first site's vectors and the records in one memory round trip
    load_base(c0 < vh ? c0 : vh - 1);
    const int phase = base->phase;
    const int live = base->live;  // 2: x and r stay as they are (alpha 0)
    const bool p_due = base->p_due != 0,
               on = DIRS ? p_due && phase == CG_RUNNING && !base->unsettled : live != 0;
    const double a = live == 2 ? 0.0 : base->alpha, b = base->beta;
    const bool pdir = DIRS || !p_due;
    if (threadIdx.x < 64) {
        const int i = threadIdx.x;
        Due d{};
        bool is = false;
        if (i < nshift) {
            const ShiftState T = sh[i];
            d = {ptr->x[i], ptr->p[i], T.alpha, T.beta, T.zeta, pdir && T.active != 0};
            is = DIRS ? d.act != 0 : T.xupd != 0;  // (an active shift always has an x_i update due)
        }
        const unsigned long long m = __ballot(is);
        if (is) due[__popcll(m & ((1ull << i) - 1))] = d;
        if (i == 0) ndue = __popcll(m);
    }
    issue_here(praw);
    issue_here(rraw);
    if (!DIRS || CONJ) issue_here(qraw);
    if (!DIRS) issue_here(xraw);
    if (DIRS && blockIdx.x == 0 && threadIdx.x == 0) publish(host_phase, 0, phase);
    if (!on) return;
    __syncthreads();
    const int n = ndue;
    double sums[2] = {0.0, 0.0};  // |r|^2; <q,p_0> of the new p_0
    for (int cb = c0; cb < vh; cb += gridDim.x * blockDim.x) {
        if (cb != c0) load_base(cb);
        RawI pnext{};
        RawR xnext{};
        auto load_shift = [&](int i) {
            pnext = SpinorIO<PI>::load_raw(due[i].p, vh, cb);
            if (!DIRS) xnext = SpinorIO<PR>::load_raw(due[i].x, vh, cb);
        };
        if (n > 0) load_shift(0);
        V3<double> pv = vcast<double>(SpinorIO<PI>::decode(praw));
        V3<double> rv = vcast<double>(SpinorIO<PR>::decode(rraw));
        const V3<double> qv = DIRS && !CONJ ? vzero<double>() : vcast<double>(SpinorIO<PI>::decode(qraw));
        if (!DIRS) {
            V3<double> xv = vcast<double>(SpinorIO<PR>::decode(xraw));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                xv.c[c].re += a * pv.c[c].re;
                xv.c[c].im += a * pv.c[c].im;
                rv.c[c].re -= a * qv.c[c].re;
                rv.c[c].im -= a * qv.c[c].im;
            }
            SpinorIO<PR>::store(x0, vh, cb, vcast<TR>(xv));
            const V3<TR> rs = vcast<TR>(rv);
            SpinorIO<PR>::store(r, vh, cb, rs);
            rv = vcast<double>(rs);  // the norm and the directions follow the stored residual
#pragma unroll
            for (int c = 0; c < 3; ++c) sums[0] += rv.c[c].re * rv.c[c].re + rv.c[c].im * rv.c[c].im;
        }
        if (pdir) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                pv.c[c].re = rv.c[c].re + b * pv.c[c].re;
                pv.c[c].im = rv.c[c].im + b * pv.c[c].im;
                if (CONJ) sums[1] += qv.c[c].re * pv.c[c].re + qv.c[c].im * pv.c[c].im;
            }
            SpinorIO<PI>::store(p0, vh, cb, vcast<TI>(pv));
        }
#pragma unroll 1
        for (int i = 0; i < n; ++i) {
            const Due d = due[i];
            V3<double> pi = vcast<double>(SpinorIO<PI>::decode(pnext));
            V3<double> xi = vcast<double>(SpinorIO<PR>::decode(xnext));
            if (i + 1 < n) load_shift(i + 1);
            if (!DIRS) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    xi.c[c].re += d.alpha * pi.c[c].re;
                    xi.c[c].im += d.alpha * pi.c[c].im;
                }
                SpinorIO<PR>::store(d.x, vh, cb, vcast<TR>(xi));
            }
            if (!d.act) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                pi.c[c].re = d.zeta * rv.c[c].re + d.beta * pi.c[c].re;
                pi.c[c].im = d.zeta * rv.c[c].im + d.beta * pi.c[c].im;
            }
            SpinorIO<PI>::store(d.p, vh, cb, vcast<TI>(pi));
        }
    }
    if constexpr (CONJ) {
        __shared__ double red[MS_BLOCK / 64][2];
        block_sums<2>(sums, red);
        // (threads 0 and 1 hold a sum each; the group's |r|^2 is measured elsewhere)
        if (threadIdx.x < 2 && (!DIRS || threadIdx.x == 1))
            rr_partials[threadIdx.x * PE_PARTIALS + blockIdx.x] = sums[0];
    } else if (!DIRS) {
        const double s = block_sum(sums[0]);
        if (threadIdx.x == 0) rr_partials[blockIdx.x] = s;
    }
}

// x_0 = x_i = 0, r = p_0 = p_i = b, |b|^2 (of b in FP64)
template <int PI, int PR>
__global__ void __launch_bounds__(MS_BLOCK) ms_init(int vh, const double *b, char *x0, char *r, char *p0,
                                                    const ShiftPtrs *ptr, int nshift, double *partials)
{
    typedef typename RealOf<PI>::type TI;
    typedef typename RealOf<PR>::type TR;
    double local = 0.0;
    for (int cb = blockIdx.x * blockDim.x + threadIdx.x; cb < vh; cb += gridDim.x * blockDim.x) {
        const V3<double> bv = SpinorIO<F64>::load(b, vh, cb);
#pragma unroll
        for (int c = 0; c < 3; ++c) local += bv.c[c].re * bv.c[c].re + bv.c[c].im * bv.c[c].im;
        SpinorIO<PR>::store(x0, vh, cb, vzero<TR>());
        SpinorIO<PR>::store(r, vh, cb, vcast<TR>(bv));
        SpinorIO<PI>::store(p0, vh, cb, vcast<TI>(bv));
        for (int i = 0; i < nshift; ++i) {
            SpinorIO<PR>::store(ptr->x[i], vh, cb, vzero<TR>());
            SpinorIO<PI>::store(ptr->p[i], vh, cb, vcast<TI>(bv));
        }
    }
    const double s = block_sum(local);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ void __launch_bounds__(1024) ms_finalize_init(CgState *base, const double *partials, int nblocks)
{
    double acc = 0.0;
    for (int i = threadIdx.x; i < nblocks; i += blockDim.x) acc += partials[i];
    const double b2 = block_sum(acc);
    if (threadIdx.x != 0) return;
    CgState &S = *base;
    S.b2 = b2;
    S.stop2 *= b2;
    S.rho = b2;
    S.rho_known = 1;
    S.max_rho = b2;
    S.true_r2 = b2;
    S.alpha = 1.0;  // alpha_{-1}
    S.beta = 0.0;   // beta_{-1}
    S.phase = (b2 == 0.0) ? CG_CONVERGED : (isfinite(b2) ? CG_RUNNING : CG_NONFINITE);
}

void multishift_solve(Ctx &ctx, const Gauge &gauge, int nmass, const double *masses, const double *b, double *const *x,
                      const lqs_cg_params &prm, lqs_cg_stats *stats, hipStream_t s)
{
    auto t0 = std::chrono::steady_clock::now();
    LQS_REQUIRE(nmass >= 1 && nmass <= MS_MAX + 1, LQS_EINVAL, "multi-shift takes 1..17 masses");
    LQS_REQUIRE(prm.inner_prec == F64 || prm.inner_prec == F32 || prm.inner_prec == F16, LQS_EINVAL,
                "inner_prec must be LQS_F64, LQS_F32 or LQS_F16");
    const Geom &g = gauge.g;
    const int vh = (int)gauge.vh;
    int base = 0;
    for (int i = 1; i < nmass; ++i)
        if (masses[i] < masses[base]) base = i;
    std::vector<int> shifts;
    for (int i = 0; i < nmass; ++i)
        if (i != base) shifts.push_back(i);
    const int nshift = (int)shifts.size();

    // precisions of the recurrence: search directions and operator PI, residual PR
    const int PI = prm.inner_prec, PR = PI == F64 ? F64 : F32;
    const int64_t fi = field_bytes(g, PI, 1), fr = field_bytes(g, PR, 1);
    CgVectors v{};
    v.prec = PI;
    v.acc_prec = PR;
    v.recon = prm.inner_recon == 12 ? 12 : 18;
    v.nrhs = 1;
    v.mass = masses[base];
    v.p = ctx.workspace("ms.p", fi);
    v.q = ctx.workspace("ms.q", fi);
    v.t = ctx.workspace("ms.t", fi);
    v.r = ctx.workspace("ms.r", fr);
    // the recurrence's solutions: the caller's FP64 fields, or FP32 workspaces
    std::vector<char *> xr(nmass);
    for (int i = 0; i < nmass; ++i)
        xr[i] = PR == F64 ? (char *)x[i] : (char *)ctx.workspace("ms.x" + std::to_string(i), fr);
    const bool mixed = PR != F64;
    v.x = mixed ? x[base] : (double *)xr[base];
    v.xlo = xr[base];
    v.b = (double *)b;
    v.t64 = mixed ? ctx.workspace("ms.t64", field_bytes(g, F64, 1)) : nullptr;
    const LinkRef L = gauge.ref(PI, v.recon);
    const LaunchShape sh = default_hop_shape(g, PI, L, 1);
    v.max_blocks = cg_partials_needed(gauge.vh, sh.block);
    v.partials = (double *)ctx.workspace("ms.partials", sizeof(double) * (size_t)v.max_blocks);
    v.partials2 = (double *)ctx.workspace("ms.partials2", sizeof(double) * 2 * PE_PARTIALS);
    v.state = (CgState *)ctx.workspace("ms.state", sizeof(CgState));
    ShiftPtrs hp{};
    std::vector<ShiftState> hsh(nshift);
    for (int k = 0; k < nshift; ++k) {
        hp.x[k] = xr[shifts[k]];
        hp.x64[k] = x[shifts[k]];
        hp.p[k] = (char *)ctx.workspace("ms.p" + std::to_string(k), fi);
        ShiftState &T = hsh[k];
        T = ShiftState{};
        T.sigma = masses[shifts[k]] * masses[shifts[k]] - masses[base] * masses[base];
        T.zeta = T.zeta_prev = 1.0;
        T.active = 1;
    }
    ShiftPtrs *dp = (ShiftPtrs *)ctx.workspace("ms.ptrs", sizeof(ShiftPtrs));
    ShiftState *dsh = (ShiftState *)ctx.workspace("ms.shifts", sizeof(ShiftState) * (nshift > 0 ? nshift : 1));
    CgState S{};
    S.m2 = masses[base] * masses[base];
    S.stop2 = prm.tol * prm.tol;
    S.max_iter = prm.max_iter;
    S.phase = CG_RUNNING;
    if (mixed) {
        S.rel_interval = prm.reliable_interval > 0 ? prm.reliable_interval : 100;
        const double delta = prm.reliable_delta > 0 ? prm.reliable_delta : default_reliable_delta(PI);
        S.delta2 = delta * delta;
    }
    // the base as one more entry of the accumulation list (its FP32 and FP64 solutions)
    ShiftPtrs hall = hp;
    hall.x[nshift] = xr[base];
    hall.x64[nshift] = x[base];
    ShiftPtrs *dall = (ShiftPtrs *)ctx.workspace("ms.ptrs_all", sizeof(ShiftPtrs));
    if (mixed) LQS_HIP(hipMemcpyAsync(dall, &hall, sizeof(ShiftPtrs), hipMemcpyHostToDevice, s));
    LQS_HIP(hipMemcpyAsync(dp, &hp, sizeof(ShiftPtrs), hipMemcpyHostToDevice, s));
    if (nshift) LQS_HIP(hipMemcpyAsync(dsh, hsh.data(), sizeof(ShiftState) * nshift, hipMemcpyHostToDevice, s));
    LQS_HIP(hipMemcpyAsync(v.state, &S, sizeof(CgState), hipMemcpyHostToDevice, s));

    if (mixed)
        for (int i = 0; i < nmass; ++i) LQS_HIP(hipMemsetAsync(x[i], 0, field_bytes(g, F64, 1), s));
    // threads per block as in the CG's vector kernels: 64 while 256 leave CUs idle
    const int block = vh <= (1 << 16) ? 64 : MS_BLOCK;
    int blocks = (vh + block - 1) / block;
    if (blocks > 1024) blocks = 1024;
#define LQS_MS_PREC(STMT)                                                                                         \
    if (PI == F64) {                                                                                              \
        constexpr int P_I = F64, P_R = F64;                                                                       \
        STMT;                                                                                                     \
    } else if (PI == F32) {                                                                                       \
        constexpr int P_I = F32, P_R = F32;                                                                       \
        STMT;                                                                                                     \
    } else {                                                                                                      \
        constexpr int P_I = F16, P_R = F32;                                                                       \
        STMT;                                                                                                     \
    }
    LQS_MS_PREC(hipLaunchKernelGGL((ms_init<P_I, P_R>), dim3(blocks), dim3(block), 0, s, vh, b, xr[base], (char *)v.r,
                                   (char *)v.p, (const ShiftPtrs *)dp, nshift, v.partials));
    hipLaunchKernelGGL(ms_finalize_init, dim3(1), dim3(1024), 0, s, v.state, (const double *)v.partials, blocks);
    LQS_HIP(hipGetLastError());

    // Rounds of eight iterations with two polls of the state in flight: the
    // next round is queued before the host waits for this one's poll, so the
    // GPU does not idle between rounds; the kernels of a round queued after the
    // recurrence has ended return at once.
    const int nd_blocks = (vh + sh.block - 1) / sh.block;
    const auto scalars = corrects_prediction(PI) ? ms_scalars<true> : ms_scalars<false>;
    CgState *hs1 = (CgState *)ctx.pinned("ms.host", sizeof(CgState) + sizeof(int32_t));
    int32_t *host_phase = (int32_t *)(hs1 + 1);
    *host_phase = CG_RUNNING;
    struct Events {
        hipEvent_t e[2] = {nullptr, nullptr};
        ~Events()
        {
            for (hipEvent_t x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } ev;
    for (hipEvent_t &e : ev.e) LQS_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    int64_t enqueued = 0;
    const int64_t cap = 8 * (int64_t)prm.max_iter + 64;
    for (int round = 0;; ++round) {
        for (int i = 0; i < 8; ++i) {
            const int group = mixed && (i & 3) == 3;
            int32_t *tell = i == 7 ? host_phase : nullptr;  // by the round's last kernel that settles the phase
            launch_hop_gated(g, L, PI, v.recon, 0, 1, 1, v.p, v.t, v.state, 1, sh, s);
            launch_normal_dot_shape(gauge, v, sh, s);
            hipLaunchKernelGGL(scalars, dim3(1), dim3(1024), 0, s, v.state, dsh, nshift, (const double *)v.partials,
                               (const double *)v.partials2, nd_blocks, blocks, group, mixed ? nullptr : tell);
            LQS_MS_PREC(hipLaunchKernelGGL((ms_step<P_I, P_R, false>), dim3(blocks), dim3(block), 0, s, vh, xr[base],
                                           (char *)v.r, (char *)v.p, (const char *)v.q, (const ShiftPtrs *)dp, nshift,
                                           (const CgState *)v.state, (const ShiftState *)dsh, v.partials2,
                                           (int32_t *)nullptr));
            if (group) {
                // reliable update (gated on the base's pending flag)
                hipLaunchKernelGGL((ms_accumulate<F32>), dim3(blocks), dim3(block), 0, s, vh, (const ShiftPtrs *)dp,
                                   nshift, (const CgState *)v.state, 1);
                cg_reliable_group(gauge, v, s);
                hipLaunchKernelGGL(ms_rebeta, dim3(1), dim3(64), 0, s, (const CgState *)v.state, dsh, nshift);
                LQS_MS_PREC(hipLaunchKernelGGL((ms_step<P_I, P_R, true>), dim3(blocks), dim3(block), 0, s, vh,
                                               xr[base], (char *)v.r, (char *)v.p, (const char *)v.q,
                                               (const ShiftPtrs *)dp, nshift, (const CgState *)v.state,
                                               (const ShiftState *)dsh, v.partials2, tell));
            }
            LQS_HIP(hipGetLastError());
        }
        enqueued += 8;
        LQS_HIP(hipEventRecord(ev.e[round & 1], s));
        if (round == 0) continue;
        LQS_HIP(hipEventSynchronize(ev.e[(round - 1) & 1]));
        if (__atomic_load_n(host_phase, __ATOMIC_RELAXED) != CG_RUNNING || enqueued > cap) break;
    }
    if (nshift) LQS_HIP(hipMemcpyAsync(hsh.data(), dsh, sizeof(ShiftState) * nshift, hipMemcpyDeviceToHost, s));
    LQS_HIP(hipMemcpyAsync(hs1, v.state, sizeof(CgState), hipMemcpyDeviceToHost, s));
    LQS_HIP(hipStreamSynchronize(s));
    const CgState hs = *hs1;

#undef LQS_MS_PREC
    if (mixed) {
        hipLaunchKernelGGL((ms_accumulate<F32>), dim3(blocks), dim3(block), 0, s, vh, (const ShiftPtrs *)dall,
                           nshift + 1, (const CgState *)v.state, 0);
        LQS_HIP(hipGetLastError());
    }
    // every mass: FP64 true residual from its own solution, refined by a
    // warm-started CG (in the recurrence's precision, with reliable updates)
    // when the shared recurrence ended above the target.  The masses are
    // refined together as one block of CGs with one mass per column (up to 16
    // per block), so every hop reads the links once for all masses still
    // refining; a column that starts below the target does no iteration.
    lqs_cg_params rp = prm;
    rp.use_x0 = 1;
    rp.persistent = 0;
    // A refinement starts close to its solution (about 1e-7 relative after an
    // FP32 recurrence), where FP16 storage takes the same iterations as FP32 and
    // each is cheaper: after a mixed recurrence the refinement runs with FP16
    // storage when the gauge holds that format (measured, 64^3 x 16, 8 masses,
    // FP32 recurrence: 41 refinement iterations either way, 57 vs 71 ms).
    if (mixed && gauge.fmt[F16][v.recon == 12 ? 1 : 0]) rp.inner_prec = F16;
    const int64_t f64 = field_bytes(g, F64, 1);
    const int per_block = std::min(nmass, 16);
    char *xb = (char *)ctx.workspace("ms.xblock", f64 * per_block);
    char *bb = (char *)ctx.workspace("ms.bblock", f64 * per_block);
    for (int c0 = 0; c0 < nmass; c0 += per_block) {
        const int n = std::min(per_block, nmass - c0);
        for (int i = 0; i < n; ++i) {
            LQS_HIP(hipMemcpyAsync(xb + i * f64, x[c0 + i], f64, hipMemcpyDeviceToDevice, s));
            LQS_HIP(hipMemcpyAsync(bb + i * f64, b, f64, hipMemcpyDeviceToDevice, s));
        }
        lqs_problem pb{static_cast<const lqs_gauge *>(&gauge), masses[c0], n, (const double *)bb, (double *)xb};
        const std::vector<double> mcol(masses + c0, masses + c0 + n);
        cg_solve_one(ctx, pb, rp, stats + c0, s, &mcol);
        for (int i = 0; i < n; ++i)
            LQS_HIP(hipMemcpyAsync(x[c0 + i], xb + i * f64, f64, hipMemcpyDeviceToDevice, s));
    }
    LQS_HIP(hipStreamSynchronize(s));
    for (int i = 0; i < nmass; ++i) {
        const int shared = (i == base) ? hs.iters : hsh[std::find(shifts.begin(), shifts.end(), i) - shifts.begin()].iters;
        stats[i].restarts += stats[i].iters > 0 ? 1 : 0;
        stats[i].iters += shared;
        if (hs.phase == CG_NONFINITE) stats[i].status = LQS_ENONFINITE;
    }
    const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    for (int i = 0; i < nmass; ++i) {
        stats[i].seconds = secs;
        stats[i].device_seconds = 0.0;
        stats[i].gflops = stats[i].gbytes_per_s = 0.0;
    }
}

}  // namespace lqs
