"""The Lanczos exponential's vector kernels at the edges of their widths: the
Gram-Schmidt passes are compiled for 4, 8, 12, 16, 20 and 32 vectors and deal
the entries to at most 256 workgroups of 512, and the small exponential takes a
Taylor series up to |tau| |T| = 40 and a diagonalisation above.

Reference: exp(-i tau H) x with the dense one-site H_eff in FP64.  Bar: after
n_max vectors the Krylov error is below tol = 1e-12 where the call reports
convergence, the recurrence adds rounding of at most 1e-13 per vector for
|tau H| <= 60 here (FP64 applies, three orthogonalisation passes): 1e-11."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _problem(chi, d, w, key):
    """A Hermitian one-site problem of an MPO with w = 1 or the boson MPO's pairing (w = 4)."""
    def env(k):
        E = np.empty((chi, w, chi), dtype=np.complex128)
        for b in range(w):
            A = W.random_complex((chi, chi), key + (k, b)) / np.sqrt(chi)
            E[:, b, :] = 0.5 * (A + A.conj().T)
        if w == 4:
            E[:, 2, :] = E[:, 1, :].conj().T
        return E
    if w == 4:
        from paper_1703_00387_amd import models
        M = models.mpo(W.bh_chain(4, d - 1, chi))[1]
    else:
        A = W.random_complex((d, d), key + (9,))
        M = (A + A.conj().T).reshape(1, 1, d, d)
    return env(1), M, env(2), W.random_complex((chi, d, chi), key + (3,))


@pytest.mark.parametrize("chi,d,w,tau,n_max", [(1, 2, 1, 0.3, 2), (2, 2, 1, 0.4, 8), (5, 3, 4, 0.05, 12),
                                               (9, 2, 4, 0.3, 16), (9, 5, 4, 0.05, 20), (16, 2, 1, 1.0, 30),
                                               (17, 4, 4, 0.1, 30), (3, 2, 1, 40.0, 18)])
def test_exponential_at_every_width(chi, d, w, tau, n_max):
    from paper_1703_00387_amd import api
    L, M, R, x = _problem(chi, d, w, (401, chi, d, w))
    x /= np.linalg.norm(x)
    Hd = np.einsum("abc,bgst,dge->asdcte", L, M, R).reshape(chi * d * chi, -1)
    assert np.abs(Hd - Hd.conj().T).max() < 1e-12
    e, v = np.linalg.eigh(Hd)
    # one vector count past the invariant subspace ends the recurrence exactly
    ref = (v * np.exp(-1j * tau * e)) @ (v.conj().T @ x.reshape(-1))
    h = api.Handle(0)
    try:
        dev = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in (L, M, R, x)]
        n, err = api.krylov_expm(h, dev[0], dev[1], None, dev[2], dev[3], tau, n_max=n_max, tol=1e-12)
        code, word = h.device_status()
    finally:
        h.close()
    got = dev[3].cpu().numpy().reshape(-1)
    diff = np.linalg.norm(got - ref)
    print(f"[gs] chi={chi} d={d} w={w} |tau H|={abs(tau) * np.abs(e).max():.1f} n={n} err={err:.1e} diff={diff:.1e}",
          flush=True)
    if code == 0:
        assert diff <= 1e-11
    else:           # the vectors ran out: the estimate says by how much
        assert n == n_max and diff <= 100 * err
