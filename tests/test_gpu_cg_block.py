"""Columns of a block solve against solves of their own.

On a lattice this small a block runs the kernels of a single solve with the same
launch shapes, so a column's numbers must not depend on the others: same
iterations, same updates and the same bits as its own solve, whichever round the
others stop in, with and without graphs, and in the allocation-free solve.
"""
import numpy as np
import pytest
import torch

import paper_2502_03249_amd as lqs
import synth
from gpu_util import dev, gauge

pytestmark = pytest.mark.gpu

DIMS, MASS, COLS = (8, 8, 8, 8), 0.05, 5


@pytest.mark.parametrize("interval", [8, 20])
@pytest.mark.parametrize("prec,recon", [(lqs.F64, 18), (lqs.F32, 12), (lqs.F16, 12), (lqs.F32, 18), (lqs.F16, 18)])
def test_column_equals_its_own_solve(prec, recon, interval):
    ctx = lqs.Context(0)
    g = gauge(ctx, DIMS, synth.gauge(DIMS, "smooth", seed=71, eps=0.3))
    b = dev(np.stack([synth.source(DIMS, 0, seed=710 + k) for k in range(COLS)]))
    cols = [lqs.Field.from_lex(ctx, b[k], 0) for k in range(COLS)]
    # guesses of falling quality: the columns stop in different rounds
    guesses = []
    for k, c in enumerate(cols):
        x = c.like().zero_()
        lqs.cg_solve(ctx, [(g, MASS, c, x)], tol=10.0 ** -(2 * k + 1))
        guesses.append(x.f64.clone())
    kw = dict(tol=1e-10, inner_prec=prec, inner_recon=recon, reliable_interval=interval, use_x0=True)
    keys = ("status", "iters", "reliable_updates", "restarts", "true_rel_residual")
    own = []
    for c, x0 in zip(cols, guesses):
        x = c.like()
        x.f64.copy_(x0)
        st = lqs.cg_solve(ctx, [(g, MASS, c, x)], **kw)
        own.append((x.f64[0].clone(), [st[0][k] for k in keys]))
    assert len({o[1][1] // 8 for o in own}) >= 3, "the columns stop in the same rounds"
    bf = lqs.Field.from_lex(ctx, b, 0)
    for solve in ("graphs", "plain", "noalloc"):
        ctx.set_graphs(solve == "graphs")
        xf = bf.like()
        xf.f64.copy_(torch.cat(guesses))
        if solve == "noalloc":
            st = lqs.cg_solve_noalloc(ctx, (g, MASS, bf, xf), **kw)
        else:
            st = lqs.cg_solve(ctx, [(g, MASS, bf, xf)], **kw)
        for k in range(COLS):
            assert [st[k][n] for n in keys] == own[k][1], (solve, k)
            assert torch.equal(xf.f64[k], own[k][0]), (solve, k)
    g.close()
    ctx.close()
