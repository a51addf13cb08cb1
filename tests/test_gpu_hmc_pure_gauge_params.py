"""A pure-gauge trajectory does not look at the solver's parameters: whatever stands
in them, links, momenta and energies are the same bits."""
import ctypes

import pytest
import torch

import paper_2502_03249_amd as lqs
import synth
from gpu_util import dev

pytestmark = pytest.mark.gpu


def test_solver_parameters_are_not_read():
    dims = (4, 6, 4, 8)
    U0 = dev(synth.gauge(dims, "smooth", seed=95, eps=0.3))
    q = torch.randn(U0.shape, dtype=torch.complex128, generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    q = q - q.conj().transpose(-1, -2)
    q = q - torch.eye(3, device="cuda") * (q.diagonal(dim1=-2, dim2=-1).sum(-1) / 3)[..., None, None]
    ctx, out = lqs.Context(0), []
    for prec, recon in ((lqs.F64, 18), (lqs.F32, 12), (77, -5)):
        U, Q = U0.clone(), q.clone()
        p = lqs.LqsHmcParams(5.5, 0.0, 0.3, 3, lqs.OMELYAN, 0.0, 0,
                             lqs.LqsCgParams(0.0, 0, prec, recon, 0, 0.0, 0, 0), 0.0)
        st = lqs.LqsHmcStats()
        torch.cuda.synchronize()
        assert lqs.lib().hmc_trajectory(ctx.handle, (ctypes.c_int32 * 4)(*dims), ctypes.c_void_p(U.data_ptr()),
                                        ctypes.c_void_p(Q.data_ptr()), None, 0.0, ctypes.byref(p), ctypes.byref(st),
                                        None, None, None) == lqs.OK
        out.append((U, Q, st.dH, st.plaquette))
    for U, Q, dH, plaq in out[1:]:
        assert torch.equal(U, out[0][0]) and torch.equal(Q, out[0][1])
        assert (dH, plaq) == out[0][2:]
    ctx.close()
