"""Plaquette action, staple force, link update and short pure-gauge trajectories
against the oracle on lattices at the edges of the kernels' tiles: fewer sites
than one 64-site tile, z planes that fill tiles exactly, in pairs or never, time
extents below, at and between multiples of the sweep's run of time slices.

Bounds: every output is a sum of at most a few hundred products of numbers of
order one, formed in FP64 on both sides, so the relative 2-norm difference is a
small multiple of 2**-53; 1e-13 leaves a factor of several hundred.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_03249_amd as lqs
import synth
from gpu_util import dev, host, rel

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2, 2), (2, 4, 2, 6), (4, 2, 6, 4), (6, 6, 6, 4), (16, 8, 4, 6), (24, 24, 6, 4), (18, 10, 6, 10)]


@pytest.fixture(scope="module")
def ctx():
    c = lqs.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dims", DIMS)
def test_action_force_and_link_update(ctx, dims):
    U = synth.gauge(dims, "smooth", seed=401, eps=0.6)
    Q = synth.momenta(dims, seed=402)
    beta = 5.6
    want = oracle.plaquette_action(dims, U, beta)
    assert abs(lqs.gauge_action(ctx, dims, dev(U), beta) - want) <= 1e-12 * abs(want)
    Fo = oracle.gauge_force(dims, U, beta, coeff=1.0)
    assert rel(host(lqs.gauge_force(ctx, dims, dev(U), beta)), Fo) <= 1e-13
    out = dev(Q)
    lqs.gauge_force(ctx, dims, dev(U), beta, coeff=-0.5, out=out, accumulate=True)
    assert rel(host(out), Q - 0.5 * Fo) <= 1e-13
    for eps in (0.02, 1.5):
        Ud = dev(U)
        lqs.link_update(ctx, dims, Ud, dev(Q), eps)
        assert rel(host(Ud), oracle.link_update(dims, U, Q, eps)) <= 1e-13


@pytest.mark.parametrize("dims", DIMS)
def test_short_trajectory(ctx, dims):
    U = synth.gauge(dims, "smooth", seed=403, eps=0.3)
    Q = synth.momenta(dims, seed=404)
    Ud, Qd = dev(U), dev(Q)
    prop = torch.empty_like(Ud)
    st = lqs.hmc_trajectory(ctx, dims, Ud, Qd, None, fermions=0, beta=5.5, tau=0.2, nsteps=2,
                            integrator=lqs.OMELYAN, proposal=prop)
    o = oracle.hmc(dims, U, Q, None, 0.1, 5.5, 0.2, 2, integrator="omelyan", fermions=False)
    assert rel(host(prop), o["U1"]) <= 1e-12 and rel(host(Qd), o["Q1"]) <= 1e-12
    e = o["energies"]
    assert abs(st["sg0"] - e[1]) <= 1e-12 * abs(e[1]) and abs(st["sg1"] - e[4]) <= 1e-12 * abs(e[4])
    assert np.array_equal(host(Ud), host(prop) if st["accepted"] else U)


def test_link_update_of_general_matrices(ctx):
    """exp(eps Q) U for Q that is neither traceless nor anti-Hermitian."""
    dims = (4, 6, 4, 2)
    rng = np.random.default_rng(405)
    U = synth.gauge(dims, "haar", seed=406)
    Q = rng.normal(size=U.shape) + 1j * rng.normal(size=U.shape)
    want = oracle.link_update(dims, U, Q, 0.4)
    Ud = dev(U)
    lqs.link_update(ctx, dims, Ud, dev(Q), 0.4)
    # the exponential's own conditioning (norms up to about e^2) times a few roundings
    assert rel(host(Ud), want) <= 1e-13
