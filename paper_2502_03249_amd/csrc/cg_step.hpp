// cg_step.hpp -- the scalar bookkeeping of a predict-and-recompute CG step and
// of an FP64 residual update, run by one thread on one right-hand side's record
// (the multi-kernel solver and the one-block solver share it).
#pragma once
#include "lqs_impl.hpp"

namespace lqs {

// The prediction takes <r,q> for <p,q>.  With the directions in 16 bits the two
// differ: <p,q> = <r,q> + beta <p_old,q>, and consecutive directions are
// conjugate only as far as the roundings of p and q, and the jump of r in a
// reliable update, leave them so.  <p_old,q> = <q_old,p> is summed where p is
// formed, which has both at hand.  (Left out, the iterations stay the same and x
// ends 6 to 25 % further from the solution at the same residual: error over
// residual 3.8 on 16^4 with the norm measured as with this, 4.9 without.)
constexpr bool corrects_prediction(int prec) { return prec == F16; }

// |r - alpha q|^2 of a step; beta formed its direction (0: r alone), pe = <p_old,q>.
template <bool CONJ>
__device__ __forceinline__ double predicted_r2(double alpha, double beta, double qq, double rr, double pe)
{
    const double r2 = fma(alpha * alpha, qq, -rr);
    return CONJ && beta != 0.0 ? fma(2.0 * alpha * beta, pe, r2) : r2;
}

// A predicted |r|^2 that says nothing.  It is the difference of two numbers of
// about |r|^2 before the step (rr), each a sum that is good to a few ulp: below
// 16 ulp of rr it is their rounding, unless the target lies above that too.  It
// is negative by more where <r,q> = <p,q> no longer holds.  Either way it neither
// ends a solve nor gives a beta.
__device__ __forceinline__ bool prediction_lost(double r2, double rr, double stop2)
{
    const double noise = 16.0 * 2.220446049250313e-16 * rr;
    if (__builtin_expect(r2 > noise, 1)) return false;
    return r2 < 0.0 || noise > stop2;
}

// The decisions that |r|^2 of a step leads to.
__device__ __forceinline__ void cg_decide(CgState &S, double r2, int last)
{
    S.rho = r2;
    S.beta = S.rho_old > 0.0 ? r2 / S.rho_old : 0.0;
    S.live = 1;
    if (r2 > S.max_rho) S.max_rho = r2;
    if (r2 <= S.stop2 || S.iters >= S.max_iter) {
        S.phase = CG_INNER_DONE;
        S.reliable_pending = 1;
        S.p_due = 1;
        return;
    }
    if (S.rel_interval > 0 && (S.since_rel >= S.rel_interval || r2 < S.delta2 * S.max_rho)) S.reliable_pending = 1;
    if (last && S.reliable_pending) S.p_due = 1;
}

// Settles a step whose prediction was lost with the |r|^2 it left: the direction
// is due, x and r have their updates (alpha 0).
__device__ __forceinline__ void cg_settle(CgState &S, double rr, int last)
{
    S.unsettled = 0;
    S.live = 0;
    S.p_due = 0;
    S.alpha = 0.0;
    if (isfinite(rr)) cg_decide(S, rr, last);
    else S.phase = CG_NONFINITE;
}

// Scalars of one iteration from its dots (rr: |r|^2 as the last step summed it,
// unused while S.rho holds a measured one; pe with CONJ: <p_old,q>).  `live`:
// this iteration's update is due; `p_due`: the direction update is left to the
// FP64 group that closes the round (`last`: the group follows this iteration).
// Where the prediction is lost (`unsettled`) x and r are advanced and the
// direction is not: |r|^2 has to be summed first.
template <bool CONJ>
__device__ __forceinline__ void cg_step_scalars(CgState &S, double pq, double qq, double rr, double pe, int last)
{
    if (S.rho_known) rr = S.rho;
    S.live = 0;
    S.p_due = 0;
    if (!isfinite(pq)) {
        S.phase = CG_NONFINITE;
        return;
    }
    if (!(pq > 0.0)) {
        S.phase = CG_BREAKDOWN;
        return;
    }
    S.alpha = rr / pq;
    const double r2 = predicted_r2<CONJ>(S.alpha, S.beta, qq, rr, pe);
    S.rho_known = 0;
    S.iters += 1;
    S.since_rel += 1;
    if (!isfinite(r2)) {
        S.phase = CG_NONFINITE;
        return;
    }
    S.rho_old = rr;
    if (prediction_lost(r2, rr, S.stop2) && S.iters < S.max_iter) {
        S.unsettled = 1;
        S.live = 1;
        S.p_due = 1;
        if (S.rel_interval > 0 && S.since_rel >= S.rel_interval) S.reliable_pending = 1;
        return;
    }
    cg_decide(S, r2, last);
}

// mode: 0 reliable update inside the iteration, 1 initial residual, 2 measure
// only, 3 periodic update with the reconstructed FP64 links (a residual that
// meets the target is handed on, still pending, to the mode-0 check with the
// stored links instead of ending the solve), 4 as 0, queued by the host after
// a round has ended
__device__ inline void fin_residual(CgState &S, double r2, int mode)
{
    S.true_r2 = r2;
    if (mode == 2) return;
    S.unsettled = 0;
    if (mode == 3 && isfinite(r2) && r2 <= S.stop2) {
        S.phase = CG_INNER_DONE;
        return;
    }
    S.rho_known = 1;  // wherever the iteration goes on, S.rho is set below
    if (mode == 1) {
        S.rho = r2;
        S.max_rho = r2;
        S.phase = isfinite(r2) ? (r2 <= S.stop2 ? CG_CONVERGED : CG_RUNNING) : CG_NONFINITE;
        return;
    }
    S.nreliable += 1;
    S.reliable_pending = 0;
    S.since_rel = 0;
    if (!isfinite(r2)) {
        S.phase = CG_NONFINITE;
    } else if (r2 <= S.stop2) {
        S.phase = CG_CONVERGED;
    } else if (S.iters >= S.max_iter) {
        S.phase = CG_MAXITER;
    } else if (S.rel_interval == 0) {
        // FP64 solver whose iterated residual drifted: restart from r = b - M x
        S.rho = r2;
        S.max_rho = r2;
        S.beta = 0.0;
        S.restarts += 1;
        S.phase = CG_RUNNING;
    } else {
        // mixed precision: continue with the FP64 residual, keep p
        S.beta = S.rho_old > 0.0 ? r2 / S.rho_old : 0.0;
        S.rho = r2;
        S.max_rho = r2;
        S.phase = CG_RUNNING;
    }
}

// A thread's share (of 1024 threads) of the block partials of <p,q> and <q,q>
// (pairs, nblocks >= 1), of |r|^2 (1 <= nr_blocks <= 1024) and, with CONJ, of
// <p_old,q> (PE_PARTIALS after those).  `first` holds what is
// requested before anything is waited for, so that a record loaded between the
// two calls shares the round trip.
struct DotShare {
    double2 pq;
    double rr, pe;
};
template <bool CONJ>
__device__ __forceinline__ DotShare first_dots(const double *partials, const double *rr_partials, int nblocks,
                                               int nr_blocks)
{
    const int i = threadIdx.x, ir = i < nr_blocks ? i : nr_blocks - 1;
    return {((const double2 *)partials)[i < nblocks ? i : nblocks - 1], rr_partials[ir],
            CONJ ? rr_partials[PE_PARTIALS + ir] : 0.0};
}
__device__ __forceinline__ void add_dots(const double *partials, int nblocks, int nr_blocks, const DotShare &first,
                                         double (&v)[4])
{
    const double2 *pp = (const double2 *)partials;
    const int i0 = threadIdx.x;
    v[0] = v[1] = v[2] = v[3] = 0.0;
    if (i0 < nblocks) {
        v[0] = first.pq.x;
        v[1] = first.pq.y;
    }
    if (i0 < nr_blocks) {
        v[2] = first.rr;
        v[3] = first.pe;
    }
    for (int b = 1024; b < nblocks; b += 4 * 1024) {
        double2 a[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = b + 1024 * k + i0;
            a[k] = pp[i < nblocks ? i : nblocks - 1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (b + 1024 * k + i0 < nblocks) {
                v[0] += a[k].x;
                v[1] += a[k].y;
            }
    }
}

// The phase of a right-hand side for the host, in pinned memory (null: not now).
// The host may read it before or after a later kernel has moved the phase on, or
// back from CG_INNER_DONE to CG_RUNNING where a check failed: it then queues a
// round or a check that finds nothing to do, and looks again.  A final phase
// stays.  (A copy of the records on
// the stream instead held the next round back by 12 us.)
__device__ __forceinline__ void publish(int32_t *host_phase, int rhs, int32_t phase)
{
    if (host_phase) __hip_atomic_store(host_phase + rhs, phase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace lqs
