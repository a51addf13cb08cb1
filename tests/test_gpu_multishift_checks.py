"""Mixed multi-shift recurrences whose FP64 check sends them on.

With few reliable updates the iterated residual meets the target before the FP64
one does: the check fails and the recurrence continues from the FP64 residual.
For one mass it is then the mixed-precision CG, with the same rounded vectors,
the same checks and no iteration between a stop and its check: the iterations may
differ by what rounding moves them (5 % and half a round), but not by a direction
that was lost on the way (13 to 40 % at this size).
"""
import pytest

import oracle
import paper_2502_03249_amd as lqs
import synth
from gpu_util import field, gauge, lex_of

pytestmark = pytest.mark.gpu

DIMS, MASS, SEEDS = (8, 8, 8, 8), 0.05, range(12)


@pytest.mark.parametrize("prec,recon,delta", [(lqs.F16, 12, 0.01), (lqs.F32, 12, 1e-5), (lqs.F32, 18, 1e-5)])
def test_recurrence_goes_on_after_a_failed_check(prec, recon, delta):
    ctx = lqs.Context(0)
    kw = dict(tol=1e-10, inner_prec=prec, inner_recon=recon, reliable_interval=1000, reliable_delta=delta)
    slow = []
    for seed in SEEDS:
        U = synth.gauge(DIMS, "smooth", seed=810 + seed, eps=0.3)
        b = synth.source(DIMS, 0, seed=850 + seed)
        g, bf = gauge(ctx, DIMS, U), field(ctx, DIMS, b, 0)
        x = bf.like()
        cg = lqs.cg_solve(ctx, [(g, MASS, bf, x.zero_())], **kw)[0]
        ms = lqs.cg_solve_multishift(ctx, g, [MASS], bf, [x], **kw)[0]
        assert ms["status"] == 0
        assert oracle.true_residual(DIMS, U, MASS, b, lex_of(ctx, x)) <= 1e-10
        if ms["iters"] > 1.05 * cg["iters"] + 4:
            slow.append((seed, ms["iters"], cg["iters"]))
        g.close()
    assert not slow, slow
    ctx.close()
