"""The CG step kernel (x, r and p in one pass, the residual norm predicted) at the
edges of its launches: fewer sites than one block, a ragged last block, one and
several right-hand sides, solves that end within the dimension of the space, and
multi-shift solves with shifts that stop early.

Every solution has a true residual (recomputed by the oracle) of at most tol and
meets the oracle's within kappa tol, kappa <= (m^2 + 64) / m^2, as in the other
solver tests.
"""
import numpy as np
import pytest

import oracle
import paper_2502_03249_amd as lqs
import synth
from gpu_util import field, gauge, lex_of, rel

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2, 2), (4, 2, 2, 2), (4, 4, 4, 4), (6, 4, 10, 2), (10, 6, 6, 14)]


@pytest.fixture(scope="module")
def ctx():
    c = lqs.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("nrhs", [1, 3, 5])
@pytest.mark.parametrize("dims", DIMS)
def test_step_follows_the_oracle(ctx, dims, nrhs):
    m = 0.2
    U = synth.gauge(dims, "haar", seed=61)
    b = np.stack([synth.source(dims, 0, seed=620 + k) for k in range(nrhs)])
    g = gauge(ctx, dims, U)
    bf = field(ctx, dims, b, 0)
    xf = bf.like().zero_()
    st = lqs.cg_solve(ctx, [(g, m, bf, xf)], tol=1e-10)
    x = lex_of(ctx, xf, squeeze=False)
    for k in range(nrhs):
        xo, _, _, _ = oracle.cg(dims, U, m, b[k])
        assert st[k]["status"] == 0, st[k]
        assert oracle.true_residual(dims, U, m, b[k], x[k]) <= 1e-10
        assert rel(x[k], xo) <= (m * m + 64) / (m * m) * 1e-10


@pytest.mark.parametrize("prec", [lqs.F64, lqs.F32])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 10, 2)])
def test_shifted_steps_follow_the_oracle(ctx, dims, prec):
    masses = [0.2, 0.3, 1.0, 6.0]  # the heaviest stops within a few iterations
    U = synth.gauge(dims, "haar", seed=63)
    b = synth.source(dims, 0, seed=64)
    g = gauge(ctx, dims, U)
    bf = field(ctx, dims, b, 0)
    xs = [bf.like() for _ in masses]
    st = lqs.cg_solve_multishift(ctx, g, masses, bf, xs, tol=1e-10, inner_prec=prec)
    for m, xf, s in zip(masses, xs, st):
        assert s["status"] == 0, s
        x = lex_of(ctx, xf)
        assert oracle.true_residual(dims, U, m, b, x) <= 1e-10
        xo, _, _, _ = oracle.cg(dims, U, m, b)
        assert rel(x, xo) <= (m * m + 64) / (m * m) * 1e-10


@pytest.mark.parametrize("prec", [lqs.F64, lqs.F32])
@pytest.mark.parametrize("dims", [(16, 16, 16, 32), (18, 16, 14, 34), (32, 32, 32, 18)])
def test_shifted_steps_on_each_launch(ctx, dims, prec):
    """2^16 sites per parity (blocks of 64), just above (256, a ragged last block), several sites per thread;
    the shifts stop one after the other."""
    masses = [0.8, 0.5, 5.0, 1.1, 2.0]
    U = synth.gauge(dims, "smooth", seed=65, eps=0.3)
    b = synth.source(dims, 0, seed=66)
    g = gauge(ctx, dims, U)
    bf = field(ctx, dims, b, 0)
    xs = [bf.like() for _ in masses]
    st = lqs.cg_solve_multishift(ctx, g, masses, bf, xs, tol=1e-10, inner_prec=prec)
    for m, xf, s in zip(masses, xs, st):
        assert s["status"] == 0, s
        assert oracle.true_residual(dims, U, m, b, lex_of(ctx, xf)) <= 1e-10
