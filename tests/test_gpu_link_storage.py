"""Memory that the link storage of closed gauges may hold: a bounded share of the
device, one pool for all contexts, given back on request and where the package's
own torch allocations run out of memory."""
import pytest
import torch

import paper_2502_03249_amd as lqs

GRANULE = 4 << 20  # of the driver's bookkeeping


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info(0)[0]


def _links(dims):
    nx, ny, nz, nt = dims
    U = torch.zeros((4, nt, nz, ny, nx, 3, 3), dtype=torch.complex128, device="cuda")
    U[..., range(3), range(3)] = 1.0
    return U


@pytest.mark.gpu
def test_storage_of_closed_gauges_is_bounded_and_given_back():
    dims = (64, 64, 64, 16)  # 2.4 GB in FP64
    U = _links(dims)
    ctx = lqs.Context(0)
    lqs.Gauge(ctx, (4, 4, 4, 4), _links((4, 4, 4, 4)), lqs.fmt(lqs.F64, 18)).close()
    lqs.release_cached(0)
    before = _free()
    gauges = [lqs.Gauge(ctx, dims, U, lqs.fmt(lqs.F64, 18)) for _ in range(3)]
    assert before - _free() >= 7_000_000_000
    for g in gauges:
        g.close()
    assert before - _free() <= torch.cuda.get_device_properties(0).total_memory // 64 + GRANULE
    lqs.release_cached(0)
    assert before - _free() <= GRANULE
    ctx.close()


@pytest.mark.gpu
def test_contexts_share_the_storage():
    dims = (32, 32, 32, 8)  # 151 MB in FP64
    U = _links(dims)
    lqs.release_cached(0)
    before = _free()
    a, b = lqs.Context(0), lqs.Context(0)
    lqs.Gauge(a, dims, U, lqs.fmt(lqs.F64, 18)).close()
    held = _free()
    assert before - held >= 140 << 20
    g = lqs.Gauge(b, dims, U, lqs.fmt(lqs.F64, 18))
    assert held - _free() <= GRANULE, "the block of the other context's gauge was not used"
    a.close()
    g.close()
    b.close()
    lqs.release_cached(0)  # (the contexts of other tests may be open)
    assert before - _free() <= GRANULE


@pytest.mark.gpu
def test_release_needs_a_device():
    with pytest.raises(lqs.LqsError):
        lqs.release_cached(-1)


@pytest.mark.parametrize("device", [0, torch.device("cuda", 0)])
def test_allocation_is_tried_again_without_the_storage(monkeypatch, device):
    released = []
    monkeypatch.setattr(lqs, "release_cached", released.append)

    def make():
        if not released:
            raise torch.cuda.OutOfMemoryError("out of memory")
        return "memory"

    assert lqs._allocate(make, device) == "memory" and released == [0]
    released.clear()

    def never():
        raise torch.cuda.OutOfMemoryError("out of memory")

    with pytest.raises(torch.cuda.OutOfMemoryError):
        lqs._allocate(never, device)
    assert released == [0]
