"""The gradient at tight cuts against the oracle's reverse mode.  Bars: twice the
error that the same runs have with every split on the Jacobi sweeps at the
default tolerance (5.3e-12 and 6.3e-11), which the adjoint's divisions by small
singular values make visible."""
import copy

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _inputs(L, chi):
    from paper_1703_00387_amd import api, models
    spec = W.xxz_chain(L, chi, 1.0, 0.5, J_b=W.xxz_grad_couplings(L))
    unit = copy.copy(spec)
    unit.J_b = np.ones(L - 1)
    ch = api.Chain.product(W.initial_vectors(spec), chi, models.bond_hamiltonians(spec))
    return spec, ch, models.bond_hamiltonians(unit), models.sz_operator()


@pytest.mark.parametrize("L,steps,chi,eps,bar", [(12, 10, 16, 1e-10, 1.1e-11), (10, 12, 12, 1e-12, 1.3e-10)])
def test_gradient_at_tight_cuts(L, steps, chi, eps, bar):
    from oracle import grad
    from paper_1703_00387_amd import api
    spec, ch, h0, sz = _inputs(L, chi)
    h = api.Handle(0)
    print(f"[grad] L {L} chi {chi} eps {eps:g}", flush=True)
    _, dJ = api.tebd_grad(h, ch, h0, 0.1, steps, eps, sz, L // 2 - 1, np.kron(sz, sz))
    torch.cuda.synchronize()
    assert h.device_status()[0] == 0
    h.close()
    ref = grad.reverse_gradient(spec, 0.1, steps, chi, eps)[1]
    rel = np.linalg.norm(dJ.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"[grad] relative error {rel:.2e}", flush=True)
    assert rel <= bar, rel
