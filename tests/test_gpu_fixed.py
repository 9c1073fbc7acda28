"""Fixed-sweep steps (MPS_FLAG_FIXED_SWEEPS): what the call promises whatever
path the splits take."""
import time

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIXED = 0x2


@pytest.fixture(scope="module")
def H():
    from paper_1703_00387_amd import api
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    h = api.Handle(0)
    yield h
    h.close()


def test_returns_with_its_work_queued(H):
    """No host wait behind the steps, also where every split has one panel: at
    the return the stream still works off a batch of 40 steps."""
    from paper_1703_00387_amd import api, models
    spec = W.xxz_chain(30, 24, 1.0, 0.5)
    v = W.random_complex((30, 2), (350,))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    hb = models.bond_hamiltonians(spec)
    chains = [api.Chain.product(v, 24, hb) for _ in range(32)]
    api.tebd_step(H, chains, 2, 0.1, 10, 1e-12)      # bonds grown, kernels loaded
    torch.cuda.synchronize()
    print("[fixed] queued steps", flush=True)
    api.tebd_step(H, chains, 2, 0.1, 40, 1e-12, flags=FIXED)
    done = torch.cuda.Event()
    done.record()
    time.sleep(0.002)                                # an idle stream has passed the event by then
    pending = not done.query()
    torch.cuda.synchronize()
    assert H.device_status()[0] == 0
    assert pending


def _chain(chi, key=0):
    """A random chain of 10 sites with bonds of 2 chi rows (it need not be canonical)."""
    from paper_1703_00387_amd import api
    L, d = 10, 2
    bond = np.array([1, 2, 16, chi, chi, chi, chi, chi, 16, 2, 1], dtype=np.int32)
    B = W.random_complex((L, chi, d, chi), (351, chi, key)) / np.sqrt(chi * d)
    lam = np.tile(np.geomspace(1.0, 1e-3, chi), (L + 1, 1))
    lam /= np.linalg.norm(lam, axis=1, keepdims=True)
    h = W.random_complex((L - 1, d * d, d * d), (352, chi))
    h = h + h.conj().transpose(0, 2, 1)
    return api.Chain(L, d, chi, torch.from_numpy(B).cuda(), torch.from_numpy(lam).cuda(),
                     torch.from_numpy(bond).cuda(), torch.from_numpy(h).cuda(),
                     torch.zeros(L - 1, dtype=torch.float64).cuda())


@pytest.mark.parametrize("room_mb", [None, 12, 6])
def test_fixed_and_captured_steps_take_the_eager_path(H, room_mb):
    """The splits' path does not depend on the schedule: a fixed-sweep step and a
    captured one end with the bits of the eager step, on a new handle (None) and
    in a caller's workspace with room for two or one of a layer's four or five
    280-row matrices (5 MiB of scratch each)."""
    from paper_1703_00387_amd import api
    chi = 140
    eager = _chain(chi)
    h0 = api.Handle(0)
    api.tebd_step(h0, [eager], 2, 0.05, 2, 1e-12)
    torch.cuda.synchronize()
    assert h0.device_status()[0] == 0
    plan = h0.workspace_needed()
    h0.close()
    for flags in (FIXED, 0x1):
        print(f"[fixed] room {room_mb} flags {flags}", flush=True)
        ws = None if room_mb is None else torch.empty(plan + (room_mb << 20), dtype=torch.uint8, device="cuda")
        h = api.Handle(0, workspace=ws)
        ch = _chain(chi)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            api.tebd_step(h, [ch], 2, 0.05, 2, 1e-12, flags=flags)
        s.synchronize()
        assert h.device_status()[0] == 0
        h.close()
        assert torch.equal(eager.chi, ch.chi) and torch.equal(eager.lam, ch.lam) and torch.equal(eager.B, ch.B)


def test_batch_past_the_scratch_without_a_second_panel():
    """A caller's workspace with room for one matrix of the capacity, bonds far
    below it: the parts are left out, the bits are the eager step's."""
    from paper_1703_00387_amd import api, models
    L, chi = 10, 140
    v = W.random_complex((L, 2), (353,))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    hb = models.bond_hamiltonians(W.xxz_chain(L, chi, 1.0, 0.5))
    eager, other = api.Chain.product(v, chi, hb), api.Chain.product(v, chi, hb)
    h0 = api.Handle(0)
    api.tebd_step(h0, [eager], 2, 0.1, 6, 1e-10)
    torch.cuda.synchronize()
    plan = h0.workspace_needed()
    h0.close()
    ws = torch.empty(plan + (6 << 20), dtype=torch.uint8, device="cuda")
    h = api.Handle(0, workspace=ws)
    print("[fixed] past the scratch, one panel", flush=True)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        api.tebd_step(h, [other], 2, 0.1, 6, 1e-10, flags=0x1)
    s.synchronize()
    assert h.device_status()[0] == 0
    h.close()
    assert 1 < int(eager.chi.max()) <= 32
    assert torch.equal(eager.chi, other.chi) and torch.equal(eager.lam, other.lam) and torch.equal(eager.B, other.B)
