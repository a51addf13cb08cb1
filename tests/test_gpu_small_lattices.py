"""Batches of lattices that fit one compute unit (links in registers, one block per
lattice): the smallest lattice, sites per parity below, at and above each step of
the block's sites per quad, temporal-gauge links, a zero source beside others, a
solve cut off by its iteration cap, and the first sizes that the form refuses.

Each solution has a true residual of at most tol, recomputed by the oracle, and
in FP64 meets the oracle's within kappa tol, kappa <= (m^2 + 64) / m^2.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_03249_amd as lqs
import synth
from gpu_util import dev, field, gauge, lex_of, rel

pytestmark = pytest.mark.gpu

# sites per parity: 8, 16, 96, 128 | 144, 192, 256 | 288, 384 | 432, 512 | 576
DIMS = [(2, 2, 2, 2), (4, 2, 2, 2), (6, 4, 2, 4), (4, 4, 4, 4), (6, 6, 2, 4), (4, 4, 4, 6), (4, 4, 4, 8),
        (4, 4, 6, 6), (8, 4, 4, 6), (6, 6, 6, 4), (4, 8, 8, 4), (8, 6, 6, 4)]


@pytest.fixture(scope="module")
def ctx():
    c = lqs.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec,recon", [(lqs.F64, 18), (lqs.F64, 12), (lqs.F32, 18), (lqs.F32, 12), (lqs.F16, 18),
                                        (lqs.F16, 12)])
@pytest.mark.parametrize("largest", range(len(DIMS)))
def test_solutions_at_every_size(ctx, largest, prec, recon):
    """The largest lattice picks the form; a smaller one and a zero source ride along."""
    probs, host = [], []
    for k, j in enumerate((largest, max(0, largest - 3), largest)):
        dims, m = DIMS[j], 0.2 + 0.1 * k
        U = synth.gauge(dims, "smooth", seed=500 + j, eps=0.3)
        b = synth.source(dims, 0, seed=600 + k) * (k < 2)
        bf = field(ctx, dims, b, 0)
        probs.append((gauge(ctx, dims, U), m, bf, bf.like()))
        host.append((dims, U, m, b))
    st = lqs.cg_solve(ctx, probs, tol=1e-10, inner_prec=prec, inner_recon=recon, reliable_interval=100,
                      persistent=True)
    for (_, _, _, xf), (dims, U, m, b), s in zip(probs, host, st):
        x = lex_of(ctx, xf)
        assert s["status"] == 0, s
        if not b.any():
            assert not x.any() and s["iters"] == 0
            continue
        assert oracle.true_residual(dims, U, m, b, x) <= 1e-10
        if prec == lqs.F64:
            assert rel(x, oracle.cg(dims, U, m, b)[0]) <= (m * m + 64) / (m * m) * 1e-10


@pytest.mark.parametrize("prec", [lqs.F64, lqs.F32])
def test_temporal_gauge_links(ctx, prec):
    dims, m = (4, 4, 4, 6), 0.2
    U, _ = lqs.gauge_fix_temporal(ctx, dims, dev(synth.gauge(dims, "haar", seed=71)))
    b = synth.source(dims, 0, seed=72)
    g = lqs.Gauge(ctx, dims, U, lqs.FMT_ALL | lqs.TEMPORAL_GAUGE)
    bf = field(ctx, dims, b, 0)
    xf = bf.like()
    st = lqs.cg_solve(ctx, [(g, m, bf, xf)], tol=1e-10, inner_prec=prec, persistent=True)
    assert st[0]["status"] == 0
    assert oracle.true_residual(dims, U.cpu().numpy(), m, b, lex_of(ctx, xf)) <= 1e-10


@pytest.mark.parametrize("prec", [lqs.F64, lqs.F16])
def test_iteration_cap_returns_the_measured_residual(ctx, prec):
    dims, m = (4, 4, 4, 4), 0.1
    U = synth.gauge(dims, "haar", seed=73)
    b = synth.source(dims, 0, seed=74)
    bf = field(ctx, dims, b, 0)
    xf = bf.like()
    st = lqs.cg_solve(ctx, [(gauge(ctx, dims, U), m, bf, xf)], tol=1e-10, max_iter=7, inner_prec=prec,
                      persistent=True)
    assert st[0]["status"] != 0 and st[0]["iters"] == 7
    r = oracle.true_residual(dims, U, m, b, lex_of(ctx, xf))
    assert r > 1e-3 and abs(st[0]["true_rel_residual"] - r) <= 1e-6 * r
    torch.cuda.synchronize()
    assert np.isfinite(lex_of(ctx, xf)).all()
