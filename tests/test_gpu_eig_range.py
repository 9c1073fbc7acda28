"""Truncations of matrices whose couplings lie far below their other entries
(test_eig_range.py says what can go wrong there), in every size class of the
direct eigensolver; bars as in test_gpu_eig.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads as W                                    # noqa: E402
from test_eig_range import equal_cases, tiny_cases       # noqa: E402
from test_gpu_eig import H, _check, _with_values         # noqa: E402,F401


@pytest.mark.parametrize("m", [2, 24, 48, 100, 200, 300, 600])
def test_tiny_couplings(H, m):   # noqa: F811
    for name, X in tiny_cases(m, np.random.default_rng(m)):
        print(f"[eig range] {m} {name}", flush=True)
        _check(H, X / np.linalg.norm(X), max(1, m // 2))


@pytest.mark.parametrize("m", [6, 24, 33, 64, 100, 200, 300, 520])
def test_groups_of_equal_values(H, m):   # noqa: F811
    for seed in range(6):
        for name, X in equal_cases(m, np.random.default_rng((m, seed))):
            print(f"[eig range] {m} {name} {seed}", flush=True)
            _check(H, X / np.linalg.norm(X), max(1, m // 2), gap=False)


@pytest.mark.parametrize("m,n", [(200, 300), (500, 520)])
def test_isometries(H, m, n):   # noqa: F811
    for key in range(16):
        print(f"[eig range] isometry {m}x{n} {key}", flush=True)
        A = _with_values(m, n, np.ones(m), (380, m, n, key))
        _check(H, A / np.linalg.norm(A), m // 2, gap=False)


@pytest.mark.parametrize("m,n", [(80, 4), (200, 4), (600, 6), (1025, 8), (1500, 10)])
def test_few_columns(H, m, n):   # noqa: F811
    for key in range(8):
        print(f"[eig range] {m}x{n} {key}", flush=True)
        A = W.random_complex((m, n), (390, m, n, key))
        _check(H, A / np.linalg.norm(A), max(1, n // 2))
