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
