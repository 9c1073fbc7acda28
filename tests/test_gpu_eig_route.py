"""Which path a truncation takes (the sweeps' own work counter is zero where the
direct eigensolver left nothing), and that either gives the split: narrow
tall matrices, which the sweeps do faster, are left to them.  Bars as in
test_gpu_eig.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_eig import H, _check, _with_values   # noqa: E402,F401


def _sweep_work(H, A, chi):   # noqa: F811
    H.set_option(3, 1)
    try:
        H.kernel_stats("jac_round", reset=True)
        _check(H, A, chi)
        return H.kernel_stats("jac_round", reset=True)[2]
    finally:
        H.set_option(3, 0)


@pytest.mark.parametrize("m,n,direct", [(65, 1, False), (65, 2, False), (65, 3, True), (300, 3, False), (300, 4, True),
                                        (1600, 9, False), (1600, 10, True), (2560, 22, False), (2560, 23, True),
                                        (4096, 16, False)])
def test_narrow_tall_matrices_go_to_the_sweeps(H, m, n, direct):   # noqa: F811
    print(f"[route] {m}x{n}", flush=True)
    A = _with_values(m, n, np.geomspace(1.0, 1e-3, n), (341, m, n))
    work = _sweep_work(H, A / np.linalg.norm(A), max(1, n // 2))
    assert (work == 0) == direct, work


@pytest.mark.parametrize("m,n,direct", [(32, 1281, True), (33, 1280, True), (33, 1281, False), (64, 2000, False)])
def test_wide_panels_go_to_the_sweeps(H, m, n, direct):   # noqa: F811
    print(f"[route] {m}x{n}", flush=True)
    A = _with_values(m, n, np.geomspace(1.0, 1e-3, m), (342, m, n))
    work = _sweep_work(H, A / np.linalg.norm(A), m // 2)
    assert (work == 0) == direct, work


def test_layer_of_a_wide_panel(H):   # noqa: F811
    """A 60 x 1500 bond alone in its layer (the sweep, order 0): one step against
    the oracle's updates, squared values to the split's bar with room."""
    import workloads as W
    from oracle import models as om, mps as omps
    from paper_1703_00387_amd import api
    L, d, cm, prof = 5, 5, 300, [1, 5, 12, 60, 300, 1]
    hs = om.bond_hamiltonians(W.bh_chain(L, 4, cm))
    Bs, lams = [], [np.ones(1)]
    B, lam = np.zeros((L, cm, d, cm), np.complex128), np.zeros((L + 1, cm))
    for i in range(L):
        a, c = prof[i], prof[i + 1]
        Bs.append(W.random_complex((a, d, c), (343, i)) / np.sqrt(c * d))
        s = np.geomspace(1.0, 1e-3, c)
        lams.append(s / np.linalg.norm(s))
        B[i, :a, :, :c], lam[i + 1, :c] = Bs[i], lams[i + 1]
    lam[0, 0] = 1.0
    ch = api.Chain(L, d, cm, torch.from_numpy(B).cuda(), torch.from_numpy(lam).cuda(),
                   torch.tensor(prof, dtype=torch.int32).cuda(), torch.from_numpy(np.ascontiguousarray(hs)).cuda(),
                   torch.zeros(L - 1, dtype=torch.float64).cuda())
    print("[route] wide layer", flush=True)
    api.tebd_step(H, [ch], 0, 0.05, 1, 1e-10)
    torch.cuda.synchronize()
    assert H.device_status()[0] == 0
    psi = omps.MPS([b.copy() for b in Bs], [x.copy() for x in lams], d)
    for b in list(range(L - 1)) + list(range(L - 2, -1, -1)):
        omps.apply_bond(psi, b, omps.gate(hs[b], 0.025), cm, 1e-10)
    _, lam1, chi1 = ch.to_host()
    assert list(chi1) == psi.chis()
    assert max(np.abs(np.asarray(lam1[j]) ** 2 - psi.lam[j] ** 2).max() for j in range(L + 1)) <= 1e-12
