"""Bytes that the model counts for one CG iteration: each kernel's links and vectors once."""
import pytest

from paper_2502_03249_amd import model


@pytest.mark.parametrize("prec,acc", [(model.F64, model.F64), (model.F32, model.F32), (model.F16, model.F32)])
@pytest.mark.parametrize("recon", [18, 12])
def test_iteration_bytes_are_those_of_its_kernels(prec, acc, recon):
    links, s, a = 8 * model.link_bytes(prec, recon), model.spinor_bytes(prec), model.spinor_bytes(acc)
    kernels = {"hop": ([links, s], [s]),                    # p -> t
               "normal": ([links, s, s], [s]),              # t, p -> q
               "step": ([a, a, s, s], [a, a, s])}           # x, r, p, q -> x, r, p
    assert model.cg_iteration_bytes(prec, acc, recon) == sum(sum(r) + sum(w) for r, w in kernels.values())
