"""The direct rotation of the truncated SVD (eig.hip) at the edges of its size
classes and on spectra that its parts treat specially: repeated values and
blocks that do not couple (deflation), a rank below both dimensions, a flat
spectrum, and norms far from one.

Bars, from the split's contract: the rows it returns have passed
|G_pq| <= max(1e-15 |X|^2, 1e-13 sqrt(G_pp G_qq)), so a squared value is off by
at most the sum of a row's couplings, m 1e-15 |X|^2 (and 1e-13 |X|^2 of
rounding for the sizes here), kept right vectors are orthogonal to 1e-10 +
1e-14 |X|^2 / (s_p s_q), and the truncated tensor, a projection of theta onto
their span, is the oracle's to 1e-9 |X| where the cut has a gap."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from paper_1703_00387_amd import api
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    h = api.Handle(0)
    yield h
    h.close()


def _with_values(m, n, s, key):
    U, _ = np.linalg.qr(W.random_complex((m, len(s)), key + (1,)))
    V, _ = np.linalg.qr(W.random_complex((n, len(s)), key + (2,)))
    return (U * s) @ V.conj().T


def _check(H, A, chi, gap=True):
    m, n = A.shape
    n2 = float((np.abs(A) ** 2).sum())
    U, S, Vh, k, disc, norm2 = H.truncate(torch.from_numpy(A).cuda(), chi, 1e-12)
    code, word = H.device_status()
    assert code == 0, word
    u, s, vh = np.linalg.svd(A, full_matrices=False)
    tail = np.cumsum((s * s)[::-1])[::-1]
    want = max(1, min(chi, int((tail > 1e-12 * tail[0]).sum())))
    assert k == want
    S, Vh, U = S.cpu().numpy(), Vh.cpu().numpy(), U.cpu().numpy()
    bar = (m * 1e-15 + 1e-13) * n2
    assert np.abs(S ** 2 - s[:k] ** 2).max() <= bar
    assert abs(norm2 - n2) <= bar and abs(disc - (s[k:] ** 2).sum()) <= bar
    G = np.abs(Vh @ Vh.conj().T - np.eye(k))
    assert (G <= 1e-10 + 1e-14 * n2 / (S[:, None] * S[None, :])).all()
    if gap:
        D = (U * S) @ Vh - (u[:, :k] * s[:k]) @ vh[:k]
        assert np.linalg.norm(D) <= 1e-9 * np.sqrt(n2)


@pytest.mark.parametrize("m,n", [(1, 1), (1, 6), (2, 2), (3, 2), (15, 17), (16, 16), (31, 40), (32, 7), (33, 33),
                                 (47, 64), (63, 100), (64, 64), (64, 9), (65, 70), (96, 33), (127, 200), (128, 128), (129, 129), (130, 64), (192, 191),
                                 (255, 256), (257, 130), (511, 80), (512, 513), (513, 300), (1024, 120), (1025, 64),
                                 (2048, 70), (2049, 90)])
def test_class_edges(H, m, n):
    """Each size class of the tridiagonalisation and of the reflectors, ragged
    leaves and merges (one row over a block), tall and wide."""
    print(f"[eig] {m}x{n}", flush=True)
    A = _with_values(m, n, np.geomspace(1.0, 1e-4, min(m, n)), (301, m, n))
    _check(H, A / np.linalg.norm(A), max(2, min(m, n) // 2))


@pytest.mark.parametrize("m,n", [(200, 150), (60, 48), (30, 24)])
@pytest.mark.parametrize("kind", ["repeated", "low_rank", "flat", "blocks", "tiny", "huge", "one_value"])
def test_special_spectra(H, kind, m, n):
    print(f"[eig] {kind} {m}x{n}", flush=True)
    s = np.geomspace(1.0, 1e-4, n)
    chi = 2 * n // 5
    if kind == "repeated":
        A = _with_values(m, n, np.repeat(np.geomspace(1.0, 1e-3, n // 6), 6), (302, 1))
        _check(H, A, n // 12 * 6)
    elif kind == "low_rank":
        _check(H, _with_values(m, n, s[:n // 4], (302, 2)), n // 2)
    elif kind == "flat":
        _check(H, _with_values(m, n, np.ones(n), (302, 3)), chi, gap=False)
    elif kind == "blocks":
        q = n // 3
        A = np.zeros((m, n), dtype=np.complex128)
        B = _with_values(q, q, np.geomspace(1.0, 1e-3, q), (302, 4))
        for b in range(3):
            A[q * b:q * b + q, q * b:q * b + q] = B
        _check(H, A, q // 2 * 3)
    elif kind == "one_value":
        A = np.zeros((m, n), dtype=np.complex128)
        A[3, 5] = 2.0 - 1.0j
        _check(H, A, 10)
    else:
        _check(H, _with_values(m, n, s, (302, 5)) * (1e-110 if kind == "tiny" else 1e110), chi)


def test_agrees_with_the_sweeps(H):
    """The same tensor by the sweeps alone (an absolute tolerance under 1e-16
    takes them): squared values to the sum of the two bars."""
    A = _with_values(180, 220, np.geomspace(1.0, 1e-5, 180), (303,))
    A /= np.linalg.norm(A)
    x = torch.from_numpy(A).cuda()
    a = H.truncate(x, 90, 1e-12)
    H.set_option(2, 1e-17)
    try:
        b = H.truncate(x, 90, 1e-12)
    finally:
        H.set_option(2, 1e-15)
    assert a[3] == b[3]
    assert (a[1] ** 2 - b[1] ** 2).abs().max().item() <= 2 * (180e-15 + 1e-13)
    ta, tb = (a[0] * a[1]) @ a[2], (b[0] * b[1]) @ b[2]
    assert torch.linalg.vector_norm(ta - tb).item() <= 2e-9


@pytest.mark.parametrize("chi", [70, 140])
def test_team_size_does_not_change_the_bits(H, chi):
    """Up to 8 matrices at once are tridiagonalised by teams of twice the
    workgroups: the sums of a row run in the same order, so a chain of 4 or 5
    bonds a layer ends with the same bits alone and three times in one call."""
    from paper_1703_00387_amd import api
    L, d = 10, 2
    bond = np.array([1, 2, 16, chi, chi, chi, chi, chi, 16, 2, 1], dtype=np.int32)
    B = W.random_complex((L, chi, d, chi), (330, chi)) / np.sqrt(chi * d)
    lam = np.tile(np.geomspace(1.0, 1e-3, chi), (L + 1, 1))
    lam /= np.linalg.norm(lam, axis=1, keepdims=True)
    h = W.random_complex((L - 1, d * d, d * d), (331, chi))
    h = h + h.conj().transpose(0, 2, 1)

    def chain():
        return api.Chain(L, d, chi, torch.from_numpy(B).cuda(), torch.from_numpy(lam).cuda(),
                         torch.from_numpy(bond).cuda(), torch.from_numpy(h).cuda(),
                         torch.zeros(L - 1, dtype=torch.float64).cuda())
    print(f"[eig] teams, chi {chi}", flush=True)
    alone, batch = chain(), [chain() for _ in range(3)]
    api.tebd_step(H, [alone], 2, 0.05, 1, 1e-12)
    api.tebd_step(H, batch, 2, 0.05, 1, 1e-12)
    torch.cuda.synchronize()
    assert H.device_status()[0] == 0
    for c in batch:
        assert torch.equal(alone.chi, c.chi) and torch.equal(alone.lam, c.lam) and torch.equal(alone.B, c.B)
