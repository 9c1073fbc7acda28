"""What a program that evolves matrix product states has this library do, as timed cases.

Every case goes through the public Python entry points (paper_1703_00387_amd.api)
on seeded inputs made on the GPU.  Kinds:

  truncate  the truncated SVD of one two-site tensor (Handle.truncate, truncate_ex)
  tebd      TEBD steps of chains in mid-run, at a given bond dimension (tebd_step)
  quench    TEBD from a random product state, dense or on charge blocks (tebd_step, tebd_step_u1)
  heff      one effective-Hamiltonian apply (heff_apply)
  krylov    one local Lanczos exponential (krylov_expm)
  grad      a TEBD2 run and its gradient (tebd_grad)
  tdvp      two-site TDVP steps of a short boson or spin chain (tdvp2_step)

The tensors of a chain are unique only up to a unitary on every bond, so a
chain is returned as what does not depend on that: its Schmidt values, bond
dimensions, discarded weights, local expectation values, bond energies and
entropies, or (short TDVP chains) its whole state vector; a truncated tensor is
returned as the product of its factors beside the values.  Values of
complex64 chains are returned in single precision, which is what they hold.
Bond dimensions are capped where the discarded weight is well above rounding
(as in a run at its cap), or cut at 1e-8 (short quenches).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads as W
from paper_1703_00387_amd import _lib, api, models

DEV = "cuda"


def _spec_xxz(L, chi, jz):
    return W.xxz_chain(L, chi, 1.0, 0.5, None, jz)


def listed():
    return [
        # a bond near the end of a chain: one call, bound by latency
        {"name": "truncate_24x40", "kind": "truncate", "m": 24, "n": 40, "chi": 12, "dtype": "c128"},
        # an ordinary ragged tensor of a complex64 program
        {"name": "truncate_c64_333x190", "kind": "truncate", "m": 333, "n": 190, "chi": 95, "dtype": "c64"},
        # the two-site tensor of a spin chain at chi = 256
        {"name": "truncate_512", "kind": "truncate", "m": 512, "n": 512, "chi": 256, "dtype": "c128"},
        # the two-site tensor of the Bose-Hubbard chain at chi = 512, d = 5
        {"name": "truncate_2560", "kind": "truncate", "m": 2560, "n": 2560, "chi": 512, "dtype": "c128"},
        # the start of a quench: many steps at small bond dimensions
        {"name": "quench_L16", "kind": "quench", "L": 16, "chi": 32, "order": 2, "steps": 20, "u1": False},
        # the same on a charge-carrying chain
        {"name": "quench_u1_L32", "kind": "quench", "L": 32, "chi": 64, "order": 2, "steps": 30, "u1": True},
        # many chains of mixed lengths advanced together
        {"name": "tebd2_batch48", "kind": "tebd", "chains": 48, "L": 40, "chi": 24, "order": 2, "steps": 2,
         "dtype": "c128", "graph": False},
        # the headline workload: one TEBD4 step of the XXZ chain, L = 64, chi = 256
        {"name": "tebd4_L64_chi256", "kind": "tebd", "chains": 1, "L": 64, "chi": 256, "order": 4, "steps": 1,
         "dtype": "c128", "graph": False},
        # the effective Hamiltonian of the Bose-Hubbard chain at full size
        {"name": "heff_chi512", "kind": "heff", "chi": 512, "d": 5, "two": True, "dtype": "c128"},
        # a local exponential of an ordinary bond, complex64
        {"name": "krylov_c64_chi160", "kind": "krylov", "chi": 160, "d": 5, "two": True, "dtype": "c64"},
        # forward and reverse pass of a short run
        {"name": "grad_L16", "kind": "grad", "L": 16, "chi": 32, "steps": 16},
        # whole TDVP steps, bosons
        {"name": "tdvp_bh_L8", "kind": "tdvp", "model": "bh", "L": 8, "chi": 32, "steps": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["truncate", "truncate", "tebd", "tebd", "quench", "heff", "krylov", "grad", "tdvp"])
    dtype = rng.choice(["c128", "c128", "c64"])
    if kind == "truncate":
        m = _log(rng, 16, 1400)
        n = max(8, min(2000, int(m * 2.0 ** rng.uniform(-1.0, 1.0))))
        return {"kind": kind, "m": m, "n": n, "chi": max(2, min(m, n) // rng.choice([2, 2, 3, 5])), "dtype": dtype}
    if kind == "tebd":
        if rng.random() < 0.4:
            return {"kind": kind, "chains": _log(rng, 2, 64), "L": rng.randint(16, 64), "chi": _log(rng, 8, 32),
                    "order": 2, "steps": 1, "dtype": dtype, "graph": rng.random() < 0.5}
        chi = _log(rng, 16, 256)
        order = rng.choice([0, 2, 2, 4]) if chi <= 96 else 2
        return {"kind": kind, "chains": 1, "L": rng.randint(16, 64), "chi": chi, "order": order, "steps": 1,
                "dtype": dtype, "graph": rng.random() < 0.25}
    if kind == "quench":
        return {"kind": kind, "L": rng.randint(8, 32), "chi": _log(rng, 16, 64), "order": rng.choice([2, 2, 4]),
                "steps": rng.randint(6, 24), "u1": rng.random() < 0.5}
    if kind == "heff":
        return {"kind": kind, "chi": _log(rng, 16, 512), "d": rng.randint(2, 5), "two": rng.random() < 0.7,
                "dtype": dtype}
    if kind == "krylov":
        return {"kind": kind, "chi": _log(rng, 8, 200), "d": rng.randint(2, 5), "two": rng.random() < 0.7,
                "dtype": dtype}
    if kind == "grad":
        return {"kind": kind, "L": rng.randint(8, 18), "chi": _log(rng, 8, 40), "steps": rng.randint(6, 16)}
    model = rng.choice(["bh", "xxz"])
    return {"kind": kind, "model": model, "L": rng.randint(5, 8) if model == "bh" else rng.randint(8, 14),
            "chi": _log(rng, 8, 32), "steps": rng.randint(1, 2)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _cgauss(g, *shape):
    return torch.view_as_complex(torch.randn(*shape, 2, generator=g, device=DEV, dtype=torch.float64))


def _theta(case, seed):
    """A two-site tensor with Schmidt-like gradings of its rows and columns."""
    m, n = case["m"], case["n"]
    g = _gen(seed)
    x = _cgauss(g, m, n)
    lam = 10.0 ** (-3.0 * torch.arange(m, device=DEV, dtype=torch.float64) / m)
    mu = 10.0 ** (-3.0 * torch.arange(n, device=DEV, dtype=torch.float64) / n)
    x = lam[:, None] * x * mu[None, :]
    x = x / torch.linalg.vector_norm(x)
    return x.to(torch.complex64 if case["dtype"] == "c64" else torch.complex128).contiguous()


def _canonical(L, chi, g, d=2):
    """A random chain in Hastings form at bond dimension chi: right-canonical
    tensors B [L][chi][d][chi] and Schmidt values [L+1][chi] that fall by
    several orders of magnitude along every bond."""
    dims = [min(d ** min(i, 30), d ** min(L - i, 30), chi) for i in range(L + 1)]
    w = [10.0 ** (-3.0 * torch.arange(x, device=DEV, dtype=torch.float64) / x) for x in dims]
    groups = {}
    for i in range(L):
        groups.setdefault((dims[i], dims[i + 1]), []).append(i)
    site = [None] * L
    for (a, c), at in sorted(groups.items()):
        wa = 10.0 ** (-3.0 * torch.arange(a, device=DEV, dtype=torch.float64) / a)
        wc = 10.0 ** (-3.0 * torch.arange(c, device=DEV, dtype=torch.float64) / c)
        f = torch.clamp(wc[None, :] / wa[:, None], max=1.0)
        r = (_cgauss(g, len(at), a, d, c) * f[None, :, None, :]).reshape(len(at), a, d * c)
        # rows made orthonormal from the first on (a Gram-Schmidt by Cholesky, twice)
        for _ in range(2):
            ch = torch.linalg.cholesky(torch.matmul(r, r.mH.contiguous()))
            r = torch.linalg.solve_triangular(ch, r, upper=False)
        for k, i in enumerate(at):
            site[i] = r[k].reshape(a, d, c)
    rho = [torch.ones(1, 1, device=DEV, dtype=torch.complex128)]
    for i in range(L):
        a, c = dims[i], dims[i + 1]
        t = torch.matmul(rho[-1], site[i].reshape(a, d * c)).reshape(a * d, c)
        x = torch.matmul(site[i].reshape(a * d, c).mH.contiguous(), t)
        rho.append(0.5 * (x + x.mH))
    groups = {}
    for i in range(L + 1):
        groups.setdefault(dims[i], []).append(i)
    u, lam = [None] * (L + 1), torch.zeros(L + 1, chi, device=DEV, dtype=torch.float64)
    for x, at in groups.items():
        e, v = torch.linalg.eigh(torch.stack([rho[i] for i in at]))
        for k, i in enumerate(at):
            u[i] = v[k].flip(1).contiguous()
            s = e[k].flip(0).clamp(min=0.0).sqrt()
            lam[i, :x] = s / torch.linalg.vector_norm(s)
    B = torch.zeros(L, chi, d, chi, device=DEV, dtype=torch.complex128)
    for i in range(L):
        a, c = dims[i], dims[i + 1]
        t = torch.matmul(u[i].mH.contiguous(), site[i].reshape(a, d * c)).reshape(a * d, c)
        B[i, :a, :, :c] = torch.matmul(t, u[i + 1]).reshape(a, d, c)
    return B, lam, torch.tensor(dims, dtype=torch.int32, device=DEV)


def _rng(seed, *key):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), *key])))


def _product_vectors(L, d, r):
    v = r.normal(size=(L, d)) + 1j * r.normal(size=(L, d))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def _env(chi, w, g, dtype):
    """A Hermitian environment [chi][w][chi] of the boson MPO (channels 1 and 2 are conjugates)."""
    E = torch.empty(chi, w, chi, device=DEV, dtype=torch.complex128)
    for b in range(w):
        A = _cgauss(g, chi, chi) / math.sqrt(chi)
        E[:, b, :] = 0.5 * (A + A.mH)
    E[:, 2, :] = E[:, 1, :].mH
    return E.to(dtype).contiguous()


def _heff_inputs(case, seed):
    chi, d = case["chi"], case["d"]
    dt = torch.complex64 if case["dtype"] == "c64" else torch.complex128
    g = _gen(seed)
    spec = W.bh_chain(4, d - 1, chi)
    Wm = torch.from_numpy(np.ascontiguousarray(models.mpo(spec)[1])).to(dt).to(DEV)
    shape = (chi, d, d, chi) if case["two"] else (chi, d, chi)
    x = _cgauss(g, *shape)
    x = (x / torch.linalg.vector_norm(x)).to(dt).contiguous()
    return {"L": _env(chi, 4, g, dt), "W": Wm, "R": _env(chi, 4, g, dt), "x": x, "two": case["two"]}


def _chain_lengths(case, seed):
    n, L = case["chains"], case["L"]
    if n == 1:
        return [L]
    r = _rng(seed, 3)
    return [L] + [int(x) for x in r.integers(16, L + 1, n - 1)] if L > 16 else [L] * n


def _tebd_inputs(case, seed):
    """(lengths, B, lam, chi, bond terms) of a batch: one canonical chain per length, its own couplings each."""
    lens = _chain_lengths(case, seed)
    n, Lm, chi = len(lens), max(lens), case["chi"]
    B = torch.zeros(n, Lm, chi, 2, chi, device=DEV, dtype=torch.complex128)
    lam = torch.zeros(n, Lm + 1, chi, device=DEV, dtype=torch.float64)
    dims = torch.ones(n, Lm + 1, device=DEV, dtype=torch.int32)
    r, g, hb, made = _rng(seed, 4), _gen(seed), [], {}
    for c, L in enumerate(lens):
        if L not in made:
            made[L] = _canonical(L, chi, g)
        b, l, x = made[L]
        B[c, :L], lam[c, :L + 1], dims[c, :L + 1] = b, l, x
        hb.append(models.bond_hamiltonians(_spec_xxz(L, chi, r.uniform(0.5, 1.5, L - 1))))
    if case["dtype"] == "c64":
        B = B.to(torch.complex64)
    return lens, B, lam, dims, hb


def _quench_inputs(case, seed):
    r, L = _rng(seed, 5), case["L"]
    spec = _spec_xxz(L, case["chi"], r.uniform(0.5, 1.5, L - 1))
    if case.get("u1"):
        v = np.zeros((L, 2), dtype=np.complex128)
        v[np.arange(L), r.permutation(np.arange(L) % 2)] = 1.0
    else:
        v = _product_vectors(L, 2, r)
    return v, models.bond_hamiltonians(spec)


def _tdvp_inputs(case, seed):
    r, L, chi = _rng(seed, 6), case["L"], case["chi"]
    if case["model"] == "bh":
        spec = W.bh_chain(L, 4, chi)
        v = _product_vectors(L, 5, r) * 10.0 ** (-0.25 * np.arange(5))[None, :]
    else:
        spec = _spec_xxz(L, chi, r.uniform(0.5, 1.5, L - 1))
        v = _product_vectors(L, 2, r)
    return v / np.linalg.norm(v, axis=1, keepdims=True), spec


DT = {"tebd": 0.05, "quench": 0.1, "grad": 0.1, "tdvp": 0.1, "krylov": 0.02}
EPS_CAP, EPS_CUT = 1e-12, 1e-8


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case, "h": api.Handle(0)}
    if kind == "truncate":
        st["theta"] = _theta(case, seed)
    elif kind == "tebd":
        lens, B, lam, dims, hb = _tebd_inputs(case, seed)
        n, Lm, chi = len(lens), max(lens), case["chi"]
        st.update(B0=B, lam0=lam, dims0=dims, B=B.clone(), lam=lam.clone(), dims=dims.clone(),
                  disc=torch.zeros(n, Lm - 1, device=DEV, dtype=torch.float64),
                  obs=torch.zeros(case["steps"], n, Lm, device=DEV, dtype=torch.float64),
                  stream=torch.cuda.Stream() if case["graph"] else None)
        st["chains"] = [api.Chain(L, 2, chi, st["B"][c, :L], st["lam"][c, :L + 1], st["dims"][c, :L + 1],
                                  torch.from_numpy(hb[c]).to(DEV), st["disc"][c, :L - 1])
                        for c, L in enumerate(lens)]
    elif kind in ("quench", "grad"):
        v, hb = _quench_inputs(case, seed)
        ch = api.Chain.product(v, case["chi"], hb)
        st.update(chain=ch, B0=ch.B.clone(), lam0=ch.lam.clone(), dims0=ch.chi.clone(), hb=ch.hbond.clone())
        if case.get("u1"):
            st["q"] = api.Charges.product(v, (1, -1), case["chi"])
            st["q0"] = st["q"].qbond.clone()
    elif kind in ("heff", "krylov"):
        st.update(_heff_inputs(case, seed))
    else:
        v, spec = _tdvp_inputs(case, seed)
        ch = api.OCChain.product(v, case["chi"], models.mpo(spec))
        st.update(chain=ch, M0=ch.M.clone(), dims0=ch.chi.clone())
    if kind in ("tebd", "quench", "grad"):
        sz = models.sz_operator()
        st["sz"] = torch.from_numpy(sz).to(DEV)
        st["szz"] = torch.from_numpy(np.kron(sz, sz)).to(DEV)
        st["slot"] = torch.arange(case["chi"], device=DEV, dtype=torch.int32)
    return st


def _live(st, lam, dims):
    """Schmidt values with the unused part of every bond's row at zero."""
    return torch.where(st["slot"] < dims[..., None], lam, 0.0)


def _restore(ch, st):
    ch.B.copy_(st["B0"])
    ch.lam.copy_(st["lam0"])
    ch.chi.copy_(st["dims0"])
    ch.disc.zero_()


def _step_tebd(st):
    case = st["case"]
    st["B"].copy_(st["B0"])
    st["lam"].copy_(st["lam0"])
    st["dims"].copy_(st["dims0"])
    st["disc"].zero_()
    api.tebd_step_ex(st["h"], st["chains"], case["order"], DT["tebd"], case["steps"], EPS_CAP,
                     _lib.MPS_FLAG_GRAPH if case["graph"] else 0, obs_op=st["sz"], obs_log=st["obs"])
    out = {"lam": _live(st, st["lam"], st["dims"]), "chi": st["dims"], "disc": st["disc"], "site": st["obs"]}
    if len(st["chains"]) == 1:
        _, out["bond"], out["entropy"] = api.observe(st["h"], st["chains"][0], None, st["szz"], entropy=True)
    if case["dtype"] == "c64":
        out = {k: v.float() if v.dtype == torch.float64 else v for k, v in out.items()}
    return out


def run(st):
    kind, case, h = st["kind"], st["case"], st["h"]
    if kind == "truncate":
        f = h.truncate if case["dtype"] == "c128" else h.truncate_ex
        U, S, Vh, k, disc, norm2 = f(st["theta"], case["chi"], EPS_CAP)
        return {"S": S, "k": k, "disc": disc, "norm2": norm2, "theta": torch.matmul(U * S.to(U.dtype), Vh)}
    if kind == "tebd":
        if st["stream"] is None:
            return _step_tebd(st)
        st["stream"].wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st["stream"]):
            out = _step_tebd(st)
        torch.cuda.current_stream().wait_stream(st["stream"])
        return out
    if kind == "quench":
        ch = st["chain"]
        _restore(ch, st)
        if "q" in st:
            st["q"].qbond.copy_(st["q0"])
            api.tebd_step_u1(h, [ch], [st["q"]], case["order"], DT["quench"], case["steps"], EPS_CUT)
        else:
            api.tebd_step(h, [ch], case["order"], DT["quench"], case["steps"], EPS_CUT)
        site, bond, ent = api.observe(h, ch, st["sz"], st["szz"], entropy=True)
        out = {"lam": _live(st, ch.lam, ch.chi), "chi": ch.chi, "disc": ch.disc, "site": site, "bond": bond,
               "entropy": ent}
        if "q" in st:
            out["charge"] = torch.where(st["slot"] < ch.chi[:, None], st["q"].qbond, 0)
        return out
    if kind == "grad":
        ch = st["chain"]
        _restore(ch, st)
        loss, dJ = api.tebd_grad(h, ch, st["hb"], DT["grad"], case["steps"], EPS_CUT, st["sz"], case["L"] // 2,
                                 st["szz"])
        return {"loss": loss, "dJ": dJ, "lam": _live(st, ch.lam, ch.chi), "chi": ch.chi}
    if kind == "heff":
        return api.heff_apply(h, st["L"], st["W"], st["W"] if st["two"] else None, st["R"], st["x"])
    if kind == "krylov":
        x = st["x"].clone()
        n_used, _ = api.krylov_expm(h, st["L"], st["W"], st["W"] if st["two"] else None, st["R"], x, DT["krylov"])
        return {"x": x, "n_used": n_used}
    ch = st["chain"]
    ch.M.copy_(st["M0"])
    ch.chi.copy_(st["dims0"])
    ch.disc.zero_()
    api.tdvp2_step(h, ch, DT["tdvp"], case["steps"], EPS_CUT)
    dims = ch.chi.tolist()
    v = torch.ones(1, 1, device=DEV, dtype=ch.M.dtype)
    for i in range(ch.L):
        a, c = dims[i], dims[i + 1]
        v = torch.matmul(v, ch.M[i, :a * ch.d * c].reshape(a, ch.d * c)).reshape(-1, c)
    return {"state": v.reshape(-1), "chi": ch.chi, "disc": ch.disc}


# ---------------------------------------------------------------------------
# work: bytes in and out once, and the operations of the standard algorithms
# (88 m n min(m, n) real operations for a complex SVD, 8 M N K for a product)
# ---------------------------------------------------------------------------
def _svd_flops(m, n):
    return 88.0 * m * n * min(m, n)


def _update_flops(a, b, c, k, d=2):
    m, n = a * d, d * c
    return 8.0 * m * n * b + 8.0 * d ** 4 * a * c + _svd_flops(m, n) + 8.0 * m * n * k


def _layers(order, L):
    if order == 0:
        return [[b] for b in list(range(L - 1)) + list(range(L - 2, -1, -1))]
    odd, even = list(range(0, L - 1, 2)), list(range(1, L - 1, 2))
    return [odd, even, odd] * (1 if order == 2 else 5)


def _full_dims(L, chi, d=2):
    return [min(d ** min(i, 30), d ** min(L - i, 30), chi) for i in range(L + 1)]


def _grown_dims(L, chi, t):
    """Bond dimensions a quench cut at 1e-8 has reached at time t (measured: about 5 at t = 1, 10 at t = 2)."""
    return [min(x, int(2.5 * 2.0 ** min(t, 10.0))) for x in _full_dims(L, chi)]


def work(case):
    kind = case["kind"]
    if kind == "truncate":
        m, n, k = case["m"], case["n"], case["chi"]
        e = 8 if case["dtype"] == "c64" else 16
        return {"bytes": e * (2.0 * m * n + m * k + k * n) + 8.0 * k, "flops": _svd_flops(m, n) + 16.0 * m * n * k}
    if kind in ("heff", "krylov"):
        chi, d, w = case["chi"], case["d"], 4
        e = 8 if case["dtype"] == "c64" else 16
        p = d * d if case["two"] else d
        f = 8.0 * (2.0 * w * p * chi ** 3 + (2 if case["two"] else 1) * w * w * p * d * chi ** 2)
        by = e * (2.0 * w * chi * chi + 2.0 * p * chi * chi)
        # a time step of these environments takes 18 or 19 Lanczos vectors
        return {"bytes": by, "flops": f * (18.0 if kind == "krylov" else 1.0)}
    if kind == "tebd":
        e, f, by = (8 if case["dtype"] == "c64" else 16), 0.0, 0.0
        n, L, chi = case["chains"], case["L"], case["chi"]
        mean = [L] if n == 1 else [(L + 16) // 2] * n if L > 16 else [L] * n
        for x in mean:
            D = _full_dims(x, chi)
            for layer in _layers(case["order"], x):
                f += sum(_update_flops(D[b], D[b + 1], D[b + 2], D[b + 1]) for b in layer) * case["steps"]
            by += 2.0 * e * sum(D[i] * 2 * D[i + 1] for i in range(x))
        return {"bytes": by, "flops": f}
    if kind == "tdvp":
        d, L = (5 if case["model"] == "bh" else 2), case["L"]
        w, f = (4 if case["model"] == "bh" else 5), 0.0
        D = _full_dims(L, case["chi"], d)
        for b in range(L - 1):
            a, c = D[b], D[b + 2]
            f += 2.0 * case["steps"] * (6 * 8.0 * (2 * w * d * d * a * c * max(a, c) + 2 * w * w * d ** 3 * a * c)
                                        + _svd_flops(a * d, d * c))
        return {"bytes": 2.0 * 16 * sum(D[i] * d * D[i + 1] for i in range(L)), "flops": f}
    # quench and grad: from a product state, bond dimensions grow with time
    L, f = case["L"], 0.0
    layers = _layers(case.get("order", 2), L)
    for t in range(case["steps"]):
        D = _grown_dims(L, case["chi"], DT[kind] * t)
        f += sum(_update_flops(D[b], D[b + 1], D[b + 2], D[b + 1]) for layer in layers for b in layer)
    D = _grown_dims(L, case["chi"], DT[kind] * case["steps"])
    by = 2.0 * 16 * sum(D[i] * 2 * D[i + 1] for i in range(L))
    return {"bytes": by, "flops": f * (3.0 if kind == "grad" else 1.0)}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain NumPy and PyTorch
# ---------------------------------------------------------------------------
def _cut(s, chi, eps):
    p = s * s
    tail = np.cumsum(p[::-1])[::-1]       # tail[j] = sum of p[j:]
    k = len(s)
    while k > 1 and tail[k - 1] <= eps * tail[0]:
        k -= 1
    k = max(1, min(k, chi))
    return k, float(tail[k]) if k < len(s) else 0.0


def _expm_herm(h, tau):
    e, v = np.linalg.eigh(h)
    return (v * np.exp(-1j * tau * e)) @ v.conj().T


def _exact_tebd(B, lam, hb, order, dt, steps, eps, chi, site_log):
    """TEBD in the Hastings form on lists of tensors; the outputs of a case."""
    L, d = len(B), B[0].shape[1]
    if order == 4:
        p = 1.0 / (4.0 - 4.0 ** (1.0 / 3.0))
        taus = [t for x in (p, p, 1.0 - 4.0 * p, p, p) for t in (0.5 * x * dt, x * dt, 0.5 * x * dt)]
    elif order == 2:
        taus = [0.5 * dt, dt, 0.5 * dt]
    else:
        taus = [0.5 * dt] * (2 * (L - 1))
    gates = {t: [_expm_herm(h, t) for h in hb] for t in set(taus)}
    disc, log = np.zeros(L - 1), []
    sz = np.diag([0.5, -0.5])
    for _ in range(steps):
        for tau, layer in zip(taus, _layers(order, L)):
            for b in layer:
                a, m, c = B[b].shape[0], B[b].shape[2], B[b + 1].shape[2]
                t = (B[b].reshape(a * d, m) @ B[b + 1].reshape(m, d * c)).reshape(a, d, d, c)
                t = np.einsum("pq,aqc->apc", gates[tau][b], t.reshape(a, d * d, c), optimize=True)
                th = (lam[b][:, None, None] * t).reshape(a * d, d * c)
                s, vh = np.linalg.svd(th, full_matrices=False)[1:]
                k, w = _cut(s, chi, eps)
                nk = math.sqrt(float((s[:k] ** 2).sum()))
                B[b + 1] = vh[:k].reshape(k, d, c)
                B[b] = (t.reshape(a * d, d * c) @ vh[:k].conj().T / nk).reshape(a, d, k)
                lam[b + 1] = s[:k] / nk
                disc[b] += w
        if site_log:
            log.append([_site(lam[i], B[i], sz) for i in range(L)])
    bond = []
    for b in range(L - 1):
        a, c = B[b].shape[0], B[b + 1].shape[2]
        t = lam[b][:, None] * (B[b].reshape(a * d, -1) @ B[b + 1].reshape(B[b].shape[2], -1)).reshape(a, -1)
        t = t.reshape(a, d, d, c)
        z = np.array([0.5, -0.5])
        bond.append(float(np.einsum("astc,s,t->", np.abs(t) ** 2, z, z)) / float((np.abs(t) ** 2).sum()))
    full = np.zeros((L + 1, chi))
    for i in range(L + 1):
        full[i, :len(lam[i])] = lam[i]
    ent = []
    for i in range(1, L):
        q = lam[i] ** 2 / (lam[i] ** 2).sum()
        q = q[q > 0]
        ent.append(float(-(q * np.log(q)).sum()))
    return {"lam": full, "disc": disc, "site": np.array(log) if site_log else
            np.array([_site(lam[i], B[i], sz) for i in range(L)]), "bond": np.array(bond), "entropy": np.array(ent)}


def _site(lam, B, op):
    x = lam[:, None, None] * B
    p = np.einsum("asc,asc->s", x, x.conj()).real
    return float((p * np.diag(op).real).sum() / p.sum())


def _heff_torch(Lenv, W1, W2, Renv, x):
    """y[a', s', t', c'] = L[a', b, a] W1[b, m, s', s] W2[m, e, t', t] R[c', e, c] x[a, s, t, c] in complex128."""
    td = torch.tensordot
    t = td(Lenv, x, dims=([2], [0]))                       # a' b s ... c
    if W2 is not None:
        t = td(t, W1, dims=([1, 2], [0, 3]))               # a' t c m s'
        t = td(t, W2, dims=([3, 1], [0, 3]))               # a' c s' e t'
        return td(t, Renv, dims=([3, 1], [1, 2]))          # a' s' t' c'
    t = td(t, W1, dims=([1, 2], [0, 3]))                   # a' c e s'
    return td(t, Renv, dims=([2, 1], [1, 2]))              # a' s' c'


def exact(case, seed):
    kind = case["kind"]
    if kind == "truncate":
        m, n = case["m"], case["n"]
        if min(m, n) > 1100:
            return None
        th = _theta(case, seed).to(torch.complex128).cpu().numpy()
        u, s, vh = np.linalg.svd(th, full_matrices=False)
        k, w = _cut(s, case["chi"], EPS_CAP)
        return {"S": s[:k], "k": None, "disc": w, "norm2": float((s * s).sum()), "theta": (u[:, :k] * s[:k]) @ vh[:k]}
    if kind in ("heff", "krylov"):
        i = {k: v.to(torch.complex128) if isinstance(v, torch.Tensor) else v
             for k, v in _heff_inputs(case, seed).items()}
        w2 = i["W"] if case["two"] else None
        if kind == "heff":
            return _heff_torch(i["L"], i["W"], w2, i["R"], i["x"])
        y, term = i["x"].clone(), i["x"]
        for j in range(1, 40):
            term = _heff_torch(i["L"], i["W"], w2, i["R"], term) * (-1j * DT["krylov"] / j)
            y = y + term
        return {"x": y, "n_used": None}
    if kind == "tebd":
        updates = sum(len(x) for x in _layers(case["order"], case["L"])) * case["steps"] * case["chains"]
        if updates * (0.002 + 1.2e-9 * (2.0 * case["chi"]) ** 3) > 12.0:
            return None
        lens, B, lam, dims, hb = _tebd_inputs(case, seed)
        B, lam, dims = B.to(torch.complex128).cpu().numpy(), lam.cpu().numpy(), dims.cpu().numpy()
        n, Lm, chi = len(lens), max(lens), case["chi"]
        out = {"lam": np.zeros((n, Lm + 1, chi)), "chi": None, "disc": np.zeros((n, Lm - 1)),
               "site": np.zeros((case["steps"], n, Lm))}
        for c, L in enumerate(lens):
            D = dims[c]
            r = _exact_tebd([B[c, i, :D[i], :, :D[i + 1]] for i in range(L)],
                            [lam[c, i, :D[i]] for i in range(L + 1)], hb[c], case["order"], DT["tebd"],
                            case["steps"], EPS_CAP, chi, True)
            out["lam"][c, :L + 1], out["disc"][c, :L - 1], out["site"][:, c, :L] = r["lam"], r["disc"], r["site"]
        if n == 1:
            out["bond"], out["entropy"] = r["bond"], r["entropy"]
        return out
    if kind == "quench":
        v, hb = _quench_inputs(case, seed)
        L = case["L"]
        r = _exact_tebd([v[i].reshape(1, 2, 1) for i in range(L)], [np.ones(1)] * (L + 1), hb, case["order"],
                        DT["quench"], case["steps"], EPS_CUT, case["chi"], False)
        r["chi"] = None
        if case["u1"]:
            r["charge"] = None
        return r
    return None
