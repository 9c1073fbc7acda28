"""Truncations of matrices whose couplings lie far below their other entries
(test_eig_range.py says what can go wrong there), in every size class of the
direct eigensolver; bars as in test_gpu_eig.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_eig_range import tiny_cases   # noqa: E402
from test_gpu_eig import H, _check      # noqa: E402,F401


@pytest.mark.parametrize("m", [2, 24, 48, 100, 200, 300, 600])
def test_tiny_couplings(H, m):   # noqa: F811
    for name, X in tiny_cases(m, np.random.default_rng(m)):
        print(f"[eig range] {m} {name}", flush=True)
        _check(H, X / np.linalg.norm(X), max(1, m // 2))
