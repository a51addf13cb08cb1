"""Steps whose residual norm cannot be predicted.

On unit links a plane wave on the even sites is an eigenvector of M, with
eigenvalue m^2 + 4 sum sin^2 p.  A source of one wave and 1e-9 of another loses
nine orders of its residual in the first step: |r|^2 then lies far below the
rounding of the two numbers whose difference predicts it, and may come out
negative.  That is neither convergence nor a beta: FP64 conjugate gradients end
after the second step, with no restart, no shift that stops early and nothing
left to refine.
"""
import numpy as np
import pytest

import oracle
import paper_2502_03249_amd as lqs
from gpu_util import field, gauge, lex_of

pytestmark = pytest.mark.gpu

TOL = 1e-12
MASSES = [0.05 + 0.037 * k for k in range(12)]


def _wave(dims, k, colour):
    nx, ny, nz, nt = dims
    t, z, y, x = np.meshgrid(*[np.arange(n) for n in (nt, nz, ny, nx)], indexing="ij")
    phase = 2 * np.pi * (k[0] * x / nx + k[1] * y / ny + k[2] * z / nz + (k[3] + 0.5) * t / nt)
    w = np.zeros(t.shape + (3,), dtype=np.complex128)
    w[..., colour] = np.where((x + y + z + t) % 2 == 0, np.exp(1j * phase), 0.0)
    return w


def _problem(ctx, dims):
    U = np.zeros((4,) + tuple(reversed(dims)) + (3, 3), dtype=np.complex128)
    U[..., range(3), range(3)] = 1.0
    b = _wave(dims, (1, 0, 0, 0), 0) + 1e-9 * _wave(dims, (0, 1, 1, 1), 1)
    return U, b, gauge(ctx, dims, U), field(ctx, dims, b, 0)


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (8, 6, 4, 10), (16, 16, 16, 16)])
def test_a_lost_prediction_is_not_convergence(dims, persistent):
    ctx = lqs.Context(0)
    U, b, g, bf = _problem(ctx, dims)
    bad = []
    for m in MASSES:
        x = bf.like()
        s = lqs.cg_solve(ctx, [(g, m, bf, x)], tol=TOL, persistent=persistent)[0]
        assert s["status"] == 0
        assert oracle.true_residual(dims, U, m, b, lex_of(ctx, x)) <= TOL
        if (s["iters"], s["restarts"], s["reliable_updates"]) != (2, 0, 1):
            bad.append((m, s["iters"], s["restarts"], s["reliable_updates"]))
    assert not bad, bad
    ctx.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (8, 6, 4, 10)])
def test_a_lost_prediction_does_not_stop_the_shifts(dims):
    ctx = lqs.Context(0)
    U, b, g, bf = _problem(ctx, dims)
    bad = []
    for lo in range(9):
        masses = MASSES[lo:lo + 4]
        xs = [bf.like() for _ in masses]
        st = lqs.cg_solve_multishift(ctx, g, masses, bf, xs, tol=TOL)
        for m, x, s in zip(masses, xs, st):
            assert s["status"] == 0
            assert oracle.true_residual(dims, U, m, b, lex_of(ctx, x)) <= TOL
            if (s["iters"], s["restarts"]) != (2, 0):
                bad.append((m, s["iters"], s["restarts"]))
    assert not bad, bad
    ctx.close()
