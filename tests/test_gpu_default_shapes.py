"""Default launch shapes on both sides of each limit of their rule (sites times
right-hand sides, whole tiles in a z plane): every column of a multi-vector hop
has the bits of the one-vector hop, which meets the oracle at the bounds of the
other hop tests, and a block solve's columns reach the FP64 true residual."""
import numpy as np
import pytest

import oracle
import paper_2502_03249_amd as lqs
import synth
from gpu_util import field, gauge, lex_of, rel

pytestmark = pytest.mark.gpu

# (dims, right-hand sides): one per thread up to 2^16 sites in all, two up to 2^17, then four in
# blocks of 256 or 128 where they tile a z plane, else two (FP16 storage beyond 8 sides: four)
CASES = [((8, 8, 8, 8), 16), ((16, 16, 16, 16), 2), ((16, 16, 16, 16), 3), ((16, 16, 16, 16), 4),
         ((16, 16, 16, 16), 5), ((12, 12, 12, 12), 13), ((12, 12, 12, 14), 16), ((32, 16, 8, 16), 5),
         ((10, 14, 18, 22), 5), ((2, 2, 2, 2), 16)]


@pytest.fixture(scope="module")
def ctx():
    c = lqs.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec,recon,bound", [(lqs.F64, 18, 1e-12), (lqs.F32, 12, 2e-6), (lqs.F16, 12, 4e-3)])
@pytest.mark.parametrize("dims,n", CASES)
def test_columns_have_the_single_vector_bits(ctx, dims, n, prec, recon, bound):
    U = synth.gauge(dims, "smooth", seed=31, eps=0.3)
    src = np.stack([synth.source(dims, 1, seed=320 + k) for k in range(n)])
    g = gauge(ctx, dims, U)
    y = lex_of(ctx, lqs.dslash_apply(ctx, g, field(ctx, dims, src, 1, prec), recon=recon), squeeze=False)
    for k in sorted({0, 1, n // 2, n - 1}):
        one = lex_of(ctx, lqs.dslash_apply(ctx, g, field(ctx, dims, src[k], 1, prec), recon=recon))
        assert np.array_equal(y[k], one)
    assert rel(y[n - 1], oracle.dslash(dims, U, src[n - 1], 0)) <= bound


@pytest.mark.parametrize("prec,recon", [(lqs.F64, 18), (lqs.F16, 12)])
@pytest.mark.parametrize("dims,n", [((8, 8, 8, 8), 16), ((16, 16, 16, 16), 5), ((12, 12, 12, 12), 13)])
def test_block_solves(ctx, dims, n, prec, recon):
    m = 0.3
    U = synth.gauge(dims, "smooth", seed=33, eps=0.3)
    b = np.stack([synth.source(dims, 0, seed=340 + k) for k in range(n)])
    bf = field(ctx, dims, b, 0)
    xf = bf.like()
    st = lqs.cg_solve(ctx, [(gauge(ctx, dims, U), m, bf, xf)], tol=1e-10, inner_prec=prec, inner_recon=recon,
                      reliable_interval=100)
    x = lex_of(ctx, xf, squeeze=False)
    for k in range(n):
        assert st[k]["status"] == 0, st[k]
        assert oracle.true_residual(dims, U, m, b[k], x[k]) <= 1e-10
