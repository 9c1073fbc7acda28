"""The count rule of the truncated SVD (select_kernel) where a thread holds one
squared value, a few threads hold two, and the cut falls on a thread's, a
wave's and the row's ends; U at a column stride of its own and in tiles that
the count ends inside of.

Bars: squared values are within m 1e-15 + 1e-13 of |X|^2 (the convergence test
that the rotated rows have passed, and rounding); eps is put at the geometric
mean of the two tails around the count, whose ratio is at least 1.01, tails
being 1e-6 |X|^2 or more, so the count itself is exact.  U S Vh is the oracle's
projection to 1e-9 |X| as the cut has a gap."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [65, 256, 257, 1023, 1030])
def test_count_rule_edges(m):
    from paper_1703_00387_amd import api
    print(f"[select] m {m}", flush=True)
    h = api.Handle(0)
    n = m + 3
    s = np.geomspace(1.0, 2e-3, m)
    U, _ = np.linalg.qr(W.random_complex((m, m), (310, m)))
    V, _ = np.linalg.qr(W.random_complex((n, m), (311, m)))
    A = (U * s) @ V.conj().T
    th = torch.from_numpy(A).cuda()
    n2 = float((s * s).sum())
    bar = (m * 1e-15 + 1e-13) * n2
    tail = np.append(np.cumsum((s * s)[::-1])[::-1], 0.0)
    for k in sorted({1, 2, 63, 64, m // 2, m - 1, m} - {0}):
        eps = np.sqrt(tail[k] * tail[k - 1]) / n2 if k < m else 0.0
        Ug, S, Vh, kg, disc, norm2 = h.truncate(th, m, eps)
        assert kg == k
        assert abs(disc - tail[k]) <= bar and abs(norm2 - n2) <= bar
        D = ((Ug * S) @ Vh).cpu().numpy() - (U[:, :k] * s[:k]) @ V[:, :k].conj().T
        assert np.linalg.norm(D) <= 1e-9 * np.sqrt(n2)
    # the capacity below the rule's count
    Ug, S, Vh, kg, disc, norm2 = h.truncate(th, 37, 0.0)
    assert kg == 37 and abs(disc - tail[37]) <= bar
    assert h.device_status()[0] == 0
    h.close()
