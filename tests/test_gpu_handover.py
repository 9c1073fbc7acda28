"""What the direct eigensolver leaves goes on to the Jacobi sweeps: teams that
gave up waiting (theta' untouched), rows that did not pass the check (rotated
already), norms outside its range.  The results are held to the same bars as the
direct ones (test_gpu_eig.py), with a clear status word; the sweeps' own work
counter says that they ran.  And the sweeps' options, which the default path
doesn't reach, on the sweeps alone (an absolute tolerance under 1e-16)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_eig import H, _check, _with_values   # noqa: E402,F401
from test_gpu_tebd import _canonical_bh_chain      # noqa: E402

DEFAULTS = {2: 1e-15, 3: 0, 4: 1, 8: 1, 9: 0, 10: 1e6}


class _Options:
    """Options of the handle for a while, with the kernel timing on."""

    def __init__(self, H, **kw):   # noqa: F811
        self.H, self.kw = H, {int(k[1:]): v for k, v in kw.items()}

    def __enter__(self):
        for k, v in {**self.kw, 3: 1}.items():
            self.H.set_option(k, v)
        self.H.kernel_stats("jac_round", reset=True)
        return self

    def sweep_work(self):
        return self.H.kernel_stats("jac_round", reset=True)[2]

    def __exit__(self, *a):
        for k in {**self.kw, 3: 0}:
            self.H.set_option(k, DEFAULTS[k])


@pytest.mark.parametrize("m,n", [(130, 200), (300, 150), (600, 220), (1100, 150)])
def test_teams_that_give_up(H, m, n):   # noqa: F811
    """One poll a wait (option 10; round launches, which do not wait): every team
    of a stage past 128 rows gives up and the sweeps start from theta' itself."""
    print(f"[handover] give up {m}x{n}", flush=True)
    A = _with_values(m, n, np.geomspace(1.0, 1e-4, min(m, n)), (370, m, n))
    with _Options(H, o10=1, o8=0) as o:
        _check(H, A / np.linalg.norm(A), min(m, n) // 2)
        assert o.sweep_work() > 0


@pytest.mark.parametrize("m,n,kind,tol", [(24, 40, "two", 1e-16), (200, 60, "one", 1e-16)])
def test_rows_that_do_not_pass(H, m, n, kind, tol):   # noqa: F811
    """One value, or two equal ones, far above the rest, under the smallest
    tolerance of the direct path: some of a dozen such matrices have a coupling past
    the check after the rotation, and the sweeps go on from there."""
    print(f"[handover] check {kind} {m}x{n}", flush=True)
    r, ran = min(m, n), 0
    top = 2 if kind == "two" else 1
    s = np.concatenate([np.ones(top), np.geomspace(1e-2, 1e-4, r - top)])
    for key in range(12):
        A = _with_values(m, n, s, (380, m, n, key))
        with _Options(H, o2=tol) as o:
            _check(H, A / np.linalg.norm(A), r // 2)
            ran += o.sweep_work() > 0
    assert ran > 0


@pytest.mark.parametrize("m,n", [(24, 40), (48, 60), (200, 210)])
@pytest.mark.parametrize("scale", [1e-130, 1e130])
def test_norms_outside_the_range(H, m, n, scale):   # noqa: F811
    """|theta|^2 of 1e-260 and 1e260, orthogonal rows (the sweeps' tests, whose
    squares leave the doubles' range there, find nothing to rotate)."""
    print(f"[handover] range {m}x{n} {scale:g}", flush=True)
    V, _ = np.linalg.qr(W.random_complex((n, m), (372, m)))
    s = np.geomspace(1.0, 1e-3, m)
    A = (s[:, None] * V.T)[W.random_complex((m,), (373, m)).real.argsort()] * scale
    k = m // 2
    U, S, Vh, kk, disc, norm2 = H.truncate(torch.from_numpy(np.ascontiguousarray(A)).cuda(), k, 1e-12)
    assert H.device_status()[0] == 0
    S, Vh, U = S.cpu().numpy(), Vh.cpu().numpy(), U.cpu().numpy()
    assert kk == k
    assert np.abs(S / (scale * s[:k]) - 1).max() <= 1e-12
    assert np.abs(np.abs((Vh @ V.conj())[:, :k]) - np.eye(k)).max() <= 1e-10
    assert np.abs(U.conj().T @ U - np.eye(k)).max() <= 1e-10
    assert abs(norm2 / (scale * scale * (s * s).sum()) - 1) <= 1e-12
    assert abs(disc / (scale * scale * (s[k:] ** 2).sum()) - 1) <= 1e-10


@pytest.mark.parametrize("opts", [dict(o10=1, o8=0), dict(o2=1e-16), dict(o2=9e-17), dict(o2=9e-17, o8=0),
                                  dict(o2=9e-17, o9=1), dict(o2=9e-17, o4=3)])
def test_layers_handed_over(H, opts):   # noqa: F811
    """One TEBD2 step of the canonical Bose-Hubbard chain (bonds of 5, 25 and 125
    rows) against the oracle, as test_long_contractions_canonical_chain: teams that
    give up, a check under the direct path's tolerance, and the sweeps alone in
    their schedules and with their options (warm start, inner sweeps)."""
    from oracle import models as om, mps as omps
    from paper_1703_00387_amd import api
    print(f"[handover] layers {opts}", flush=True)
    spec, ch, Bs, lams = _canonical_bh_chain("c128")
    with _Options(H, **opts) as o:
        api.tebd_step(H, [ch], 2, 0.05, 1, 1e-14)
        torch.cuda.synchronize()
        work = o.sweep_work()
    assert H.device_status()[0] == 0
    assert work > 0 or opts == dict(o2=1e-16)
    psi = omps.MPS(Bs, lams, spec.d)
    hs = om.bond_hamiltonians(spec)
    for bonds, tau in omps.strang_layers(spec.L, 0.05):
        for b in bonds:
            omps.apply_bond(psi, b, omps.gate(hs[b], tau), spec.chi_max, 1e-14)
    _, lam1, chi1 = ch.to_host()
    assert list(chi1) == psi.chis()
    assert max(np.abs(lam1[j] - psi.lam[j]).max() for j in range(spec.L + 1)) <= 1e-11
