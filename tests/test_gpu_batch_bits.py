"""A chain's bits do not depend on what is in its batch nor on the schedule: its
panels of at most 64 rows go through the one-launch split where a layer has
nothing else, through the batched kernels beside larger bonds or where the host
does not know the sizes."""
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


def _canonical(L, chi, key, dtype="c128"):
    """A random state's chain: bonds of 1, 2, 4, ... up to 2^(L/2), so panels of every class."""
    from oracle import mps as omps
    from paper_1703_00387_amd import api, models
    vec = W.random_complex((2 ** L,), (361, key))
    psi = omps.from_vector(vec / np.linalg.norm(vec), L, 2)
    B, lam = np.zeros((L, chi, 2, chi), np.complex128), np.zeros((L + 1, chi))
    for i in range(L):
        B[i, :psi.B[i].shape[0], :, :psi.B[i].shape[2]] = psi.B[i]
    for j in range(L + 1):
        lam[j, :len(psi.lam[j])] = psi.lam[j]
    hb = models.bond_hamiltonians(W.xxz_chain(L, chi, 1.0, 0.5))
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    return api.Chain(L, 2, chi, torch.from_numpy(B).to(tdt).cuda(), torch.from_numpy(lam).cuda(),
                     torch.tensor(psi.chis(), dtype=torch.int32).cuda(), torch.from_numpy(hb).cuda(),
                     torch.zeros(L - 1, dtype=torch.float64).cuda())


def _same(a, b):
    return all(torch.equal(x, y) for x, y in ((a.chi, b.chi), (a.lam, b.lam), (a.B, b.B), (a.disc, b.disc)))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("order", [0, 2])
def test_small_chain_beside_a_larger_one(H, dtype, order):
    from paper_1703_00387_amd import api
    print(f"[bits] beside a larger chain, order {order} {dtype}", flush=True)
    alone, beside = _canonical(10, 32, 1, dtype), _canonical(10, 32, 1, dtype)
    api.tebd_step(H, [alone], order, 0.1, 4, 1e-11)
    api.tebd_step(H, [_canonical(12, 64, 2, dtype), beside], order, 0.1, 4, 1e-11)
    torch.cuda.synchronize()
    assert H.device_status()[0] == 0
    assert int(alone.chi.max()) > 16
    assert _same(alone, beside)


@pytest.mark.parametrize("flags", [0x1, 0x2])
def test_schedules_of_a_chain_below_its_capacity(H, flags):
    from paper_1703_00387_amd import api
    print(f"[bits] flags {flags}", flush=True)
    eager, other = _canonical(10, 80, 3), _canonical(10, 80, 3)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        api.tebd_step(H, [eager], 2, 0.1, 4, 1e-11)
        api.tebd_step(H, [other], 2, 0.1, 4, 1e-11, flags=flags)
    s.synchronize()
    assert H.device_status()[0] == 0
    assert _same(eager, other)
