"""Two-site expectation values where a tile of theta_b ends: 64 / d left and
right bond indices a tile, chunks of 16 of the middle bond, every d, both types,
one operator and one per bond.  Random tensors (the sum needs no canonical
form); the reference sums the same products in float64, so the bar is rounding:
a value is a sum of chi_l chi_r d^4 products of entries of theta, each a sum of
chi_m terms, 1e-13 of the sum of their absolute values."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 5])
def test_bond_values_at_tile_edges(d, dtype):
    from paper_1703_00387_amd import api
    print(f"[observe] d {d} {dtype}", flush=True)
    h = api.Handle(0)
    t = 64 // d
    chi = np.array([1, 2 * t + 1, 1, t, 16, t + 1, 17, 2 * t, 15, 1], dtype=np.int32)
    L, cm, dd = len(chi) - 1, int(chi.max()), d * d
    B = W.random_complex((L, cm, d, cm), (320, d))    # entries past chi must not be read
    lam = 0.5 + np.arange((L + 1) * cm).reshape(L + 1, cm) / ((L + 1) * cm)
    op = W.random_complex((L - 1, dd, dd), (321, d))
    op = op + op.conj().transpose(0, 2, 1)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    Bt = torch.from_numpy(B).to(tdt)
    ch = api.Chain(L, d, cm, Bt.cuda(), torch.from_numpy(lam).cuda(), torch.from_numpy(chi).cuda(),
                   torch.zeros((L - 1, dd, dd), dtype=torch.complex128).cuda(),
                   torch.zeros(L - 1, dtype=torch.float64).cuda())
    B = Bt.to(torch.complex128).numpy()
    for per_bond in (True, False):
        _, got, _ = api.observe(h, ch, None, op if per_bond else op[0], per_bond=per_bond)
        got = got.cpu().numpy()
        for b in range(L - 1):
            l, m, r = chi[b], chi[b + 1], chi[b + 2]
            x, y = B[b, :l, :, :m], B[b + 1, :m, :, :r]
            th = np.einsum("asm,mtr->star", x, y).reshape(dd, l, r) * lam[b, :l][None, :, None]
            ab = np.einsum("asm,mtr->star", abs(x), abs(y)).reshape(dd, l, r) * lam[b, :l][None, :, None]
            O = op[b if per_bond else 0]
            want = np.einsum("par,pq,qar->", th.conj(), O, th).real
            bar = 1e-13 * np.einsum("par,pq,qar->", ab, abs(O), ab)
            assert abs(got[b] - want) <= bar, (b, got[b], want)
    h.close()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("cm", [7, 40])
def test_site_values(cm, d, dtype):
    """Site expectation values for every d, with 256 threads (cm = 7) and 1024:
    sums of chi_l chi_r d^2 products, so 1e-13 of the sum of absolute values."""
    from paper_1703_00387_amd import api
    print(f"[observe] site chi {cm} d {d} {dtype}", flush=True)
    h = api.Handle(0)
    chi = np.array([1, cm, cm - 1, cm, 2, 1], dtype=np.int32)
    L = len(chi) - 1
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    Bt = torch.from_numpy(W.random_complex((L, cm, d, cm), (322, d, cm))).to(tdt)
    lam = 0.5 + np.arange((L + 1) * cm).reshape(L + 1, cm) / ((L + 1) * cm)
    op = W.random_complex((d, d), (323, d))
    op = op + op.conj().T
    ch = api.Chain(L, d, cm, Bt.cuda(), torch.from_numpy(lam).cuda(), torch.from_numpy(chi).cuda(),
                   torch.zeros((L - 1, d * d, d * d), dtype=torch.complex128).cuda(),
                   torch.zeros(L - 1, dtype=torch.float64).cuda())
    got, _, _ = api.observe(h, ch, op)
    got = got.cpu().numpy()
    B = Bt.to(torch.complex128).numpy()
    for i in range(L):
        x = B[i, :chi[i], :, :chi[i + 1]] * lam[i, :chi[i]][:, None, None]
        want = np.einsum("apc,pq,aqc->", x.conj(), op, x).real
        bar = 1e-13 * np.einsum("apc,pq,aqc->", abs(x), abs(op), abs(x))
        assert abs(got[i] - want) <= bar
    h.close()
