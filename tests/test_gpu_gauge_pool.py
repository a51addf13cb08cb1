"""Link storage is pooled per context: a gauge made after another was closed may
stand in its memory.  Every hop must still see its own links, with other sizes
and formats in between, from several threads on their own streams, and a gauge
may outlive its context.  Hops are compared with the oracle at the bounds of the
other hop tests (1e-12 FP64, 2e-6 FP32)."""
import threading

import pytest
import torch

import oracle
import paper_2502_03249_amd as lqs
import synth
from gpu_util import dev, rel

pytestmark = pytest.mark.gpu

BOUND = {lqs.F64: 1e-12, lqs.F32: 2e-6}


def _check(ctx, dims, formats, prec, recon, seed):
    U = synth.gauge(dims, "haar", seed=seed)
    v = synth.source(dims, 1, seed=seed + 1)
    Ud, vd = dev(U), dev(v)
    g = lqs.Gauge(ctx, dims, Ud, formats)
    f = lqs.Field.from_lex(ctx, vd, 1, prec)
    y = lqs.dslash_apply(ctx, g, f, recon=recon).to_lex(ctx)
    torch.cuda.current_stream().synchronize()
    got = y[0].cpu().numpy()
    g.close()
    return rel(got, oracle.dslash(dims, U, v, 0)) <= BOUND[prec]


STEPS = [((4, 4, 4, 4), lqs.FMT_ALL, lqs.F64, 18), ((4, 4, 4, 4), lqs.fmt(lqs.F32, 12), lqs.F32, 12),
         ((8, 6, 4, 6), lqs.FMT_ALL, lqs.F32, 18), ((4, 4, 4, 4), lqs.FMT_ALL, lqs.F64, 12),
         ((8, 6, 4, 6), lqs.fmt(lqs.F64, 12), lqs.F64, 12), ((2, 2, 2, 2), lqs.FMT_ALL, lqs.F64, 18)]


def test_reused_storage_holds_the_new_links():
    ctx = lqs.Context(0)
    for k in range(3):
        for j, (dims, formats, prec, recon) in enumerate(STEPS):
            assert _check(ctx, dims, formats, prec, recon, 700 + 10 * j + k), (k, j)
    ctx.close()


def test_threads_share_the_pool():
    ctx, bad = lqs.Context(0), []

    def work(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            for j, (dims, formats, prec, recon) in enumerate(STEPS):
                if not _check(ctx, dims, formats, prec, recon, 800 + 10 * j + t):
                    bad.append((t, j))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    ctx.close()


def test_gauge_outlives_its_context():
    dims = (4, 4, 4, 4)
    ctx = lqs.Context(0)
    g = lqs.Gauge(ctx, dims, dev(synth.gauge(dims, "haar", seed=900)))
    ctx.close()
    g.close()
