"""Workloads of the library as a user's program runs them, through the Python entry points.

A case names a system (grids, modes, bands, window), an operation and its options.
The systems are seeded stand-ins with the shapes of the repository's own workloads:
a k grid, a q grid that divides it, the states of a cosine band (or two) inside an
energy window, three Debye modes and up to five Einstein modes, and one channel for
every commensurate pair of states and every mode, |g|^2 lognormal and symmetric under
inversion.  With stats "bose" the states are the phonon modes themselves
(phonon-phonon scattering).  A system and its plan depend on the case alone, as a
material does; occupations, baths and loss gradients come from the seed.
"""
import math
import types

import numpy as np
import torch

import paper_2511_03683_amd as E
from paper_2511_03683_amd import autograd as EA

HBAR, KB = 0.6582119569, 8.617333262e-5      # eV fs, eV/K
LATTICE = 5.653                              # Angstrom
DEBYE = (5.0, 3.0, 3.0)                      # km/s
EINSTEIN = (0.020, 0.040, 0.060, 0.030, 0.050)


def _case(name, op, kn, qn, modes=6, keep=0.023, bands=1, dtype="f64", batch=1, baths=False, stats="fermi",
          nsigma=0.0, steps=0):
    c = dict(op=op, kn=kn, qn=qn, modes=modes, keep=keep, bands=bands, dtype=dtype, batch=batch, baths=baths,
             stats=stats, nsigma=nsigma, steps=steps)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the textbook problem: one band on 8^3 k points, every pair a channel; one
        # evaluation inside somebody else's integrator, where the call itself is what costs
        _case("fwd_512k", "fwd", 8, 8, modes=3, keep=1.0),
        # the transport/dynamics grid of the paper's size (100^3 k, 50^3 q, six modes,
        # 2e8 channels): one collision integral
        _case("fwd_100", "fwd", 100, 50),
        # its reverse mode: gradients with respect to occupations and every |g|^2
        _case("vjp_100", "vjp", 100, 50),
        # a mobility: the linearised equation iterated to 1e-8
        _case("transport_100", "transport", 100, 50),
        # occupations of 64 (temperature, field) points evaluated together in one bath
        _case("fwd_b64_100", "fwd", 100, 50, batch=64),
        # real-time dynamics in single precision: RK4 steps replayed from a graph
        _case("rt_100_f32", "rt", 100, 50, dtype="f32", steps=10),
        # a few vectors at once (field directions, finite differences) on a medium grid
        # with an odd number of q points per axis and two bands
        _case("fwd_b5_62", "fwd", 62, 31, bands=2, batch=5),
        # channels selected by energy conservation (three sigma), as the paper's lists are
        _case("fwd_window_74", "fwd", 74, 37, nsigma=3.0),
        # training step through autograd, single precision, a ragged batch
        _case("train_b24_62_f32", "train", 62, 31, dtype="f32", batch=24),
        # each vector with a phonon temperature of its own
        _case("fwd_baths_b20_50", "fwd", 50, 25, batch=20, baths=True),
        # gradients through coupled electron-phonon dynamics
        _case("adjoint_coupled_62", "adjoint_coupled", 62, 31, steps=2),
        # phonon-phonon scattering (2998 modes, 1.3e7 channels): reverse mode
        _case("bose_vjp_10", "vjp", 10, 10, modes=3, keep=1.0, bands=3, stats="bose"),
    ]


def draw(rng):
    op = rng.choice(["fwd", "fwd", "vjp", "vjp", "rt", "transport", "coupled", "adjoint", "adjoint_coupled", "phonon_rate",
                     "train"])
    dtype = rng.choice(["f64", "f64", "f32"])
    batch, baths, steps, nsigma, stats = 1, False, 0, 0.0, "fermi"
    if op in ("fwd", "vjp", "train"):
        batch = rng.choice([1, 1, int(round(math.exp(rng.uniform(0.0, math.log(64.0)))))])
        baths = op != "train" and batch > 1 and rng.random() < 0.25
        nsigma = rng.choice([0.0, 0.0, round(rng.uniform(2.0, 5.0), 1)])
        stats = "bose" if rng.random() < 0.2 else "fermi"
    elif op in ("rt", "coupled"):
        steps = rng.randint(1, 10)
    elif op in ("adjoint", "adjoint_coupled"):
        steps = rng.randint(1, 4)
    if stats == "bose":
        qn = rng.randint(4, 11)
        return _case(None, op, qn, qn, modes=rng.randint(2, 4), keep=1.0, bands=3, dtype=dtype, batch=batch,
                     baths=baths, stats=stats)
    modes = rng.randint(1, 8)
    if rng.random() < 0.3:          # every k point a state, q grid = k grid
        qn = rng.randint(5, 12)
        return _case(None, op, qn, qn, modes=modes, keep=1.0, bands=rng.randint(1, 2), dtype=dtype, batch=batch,
                     baths=baths, nsigma=nsigma, steps=steps)
    top = 48 if modes <= 6 else 44
    if op in ("coupled", "adjoint_coupled", "adjoint", "train") or baths or batch > 16:
        top = 36
    elif op == "rt":
        top = 40
    qn = int(round(math.exp(rng.uniform(math.log(14.0), math.log(float(top))))))
    return _case(None, op, 2 * qn, qn, modes=modes, keep=round(rng.uniform(0.01, 0.023), 4), bands=rng.randint(1, 2),
                 dtype=dtype, batch=batch, baths=baths, nsigma=nsigma, steps=steps)


# ---------------------------------------------------------------- systems
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _coords(n, dev):
    a = torch.arange(n, device=dev)
    return torch.stack(torch.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)


def _hw_table(qn, modes, dev, debye=DEBYE, einstein=EINSTEIN):
    c = _coords(qn, dev)
    m = ((c + qn // 2) % qn - qn // 2).double() / qn * (2.0 * math.pi / LATTICE)
    q = (m * m).sum(1).sqrt()
    na = min(len(debye), max(1, modes // 2 + (modes == 3)))
    cols = [HBAR * v * 1e-2 * q for v in debye[:na]] + [torch.full_like(q, w) for w in einstein[:modes - na]]
    return torch.stack(cols[:modes], 1).contiguous()


def _states(c):
    """Device arrays of the case's states, ordered by coset of the q grid, k, band."""
    dev = _dev()
    kn, qn = c["kn"], c["qn"]
    kc = _coords(kn, dev)
    s = types.SimpleNamespace(dev=dev, r=kn // qn, hw=_hw_table(qn, c["modes"], dev), v=None)
    s.sigma, s.hw_min, s.g2_median = 0.008, 1e-6, 1e-3
    if c["stats"] == "bose":
        w = _hw_table(kn, 3, dev, (4.0, 7.0), (0.030,))
        s.sigma, s.hw_min, s.g2_median = 0.002, 1e-3, 1e-7
        k, b = torch.nonzero(w >= s.hw_min, as_tuple=True)
        eps = w[k, b]
    else:
        th = ((kc + kn // 2) % kn - kn // 2).double() * (2.0 * math.pi / kn)
        base = (1.0 - torch.cos(th)).sum(1) + 0.15 * (1.0 - torch.cos(th[:, 0]) * torch.cos(th[:, 1]) * torch.cos(th[:, 2]))
        e = torch.stack([base * (1.0 + 0.35 * b) + 0.1 * b * base.max() * c["keep"] for b in range(c["bands"])], 1)
        n = max(2, min(e.numel(), int(round(c["keep"] * kn ** 3))))
        edge = torch.sort(e.reshape(-1)).values[n - 1]
        scale = 0.3 / float(edge)
        k, b = torch.nonzero(e <= edge, as_tuple=True)
        eps = e[k, b] * scale
        s.v = torch.sin(th[k]) * (1.0 + 0.35 * b)[:, None] * scale * LATTICE / HBAR * 1e5
    co = kc[k] % s.r
    coset = (co[:, 0] * s.r + co[:, 1]) * s.r + co[:, 2]
    o = torch.argsort((coset * kn ** 3 + k) * 4 + b)
    k, b, s.coset = k[o], b[o], coset[o]
    s.k, s.band, s.eps, s.kc, s.n = k, b, eps[o].contiguous(), kc[k], k.numel()
    if s.v is not None:
        s.v = s.v[o].contiguous()
    neg = (-s.kc) % kn
    s.id = k * 4 + b
    s.inv = ((neg[:, 0] * kn + neg[:, 1]) * kn + neg[:, 2]) * 4 + b
    s.classes = [torch.nonzero(s.coset == x).reshape(-1) for x in torch.unique(s.coset).tolist()]
    return s


def _hash(x):
    """64-bit mixing of integer keys, as a uniform number in (0, 1)."""
    for sh, mul in ((30, -4658895280553007687), (27, -7723592293110705685)):
        x = (x ^ ((x >> sh) & ((1 << (64 - sh)) - 1))) * mul
    x = x ^ ((x >> 31) & ((1 << 33) - 1))
    return (((x >> 12) & ((1 << 52) - 1)).double() + 0.5) * 2.0 ** -52


def _pair_data(c, s, i, j):
    """|g|^2 [..., modes] (0 where there is no channel) and q index of k_j - k_i for state pairs (i, j)."""
    qn = c["qn"]
    d = ((s.kc[j] - s.kc[i]) // s.r) % qn
    q = (d[..., 0] * qn + d[..., 1]) * qn + d[..., 2]
    lo, hi = torch.minimum(s.id[i], s.id[j]), torch.maximum(s.id[i], s.id[j])
    lo2, hi2 = torch.minimum(s.inv[i], s.inv[j]), torch.maximum(s.inv[i], s.inv[j])
    key = torch.minimum((lo << 23) | hi, (lo2 << 23) | hi2)
    g = torch.empty(key.shape + (c["modes"],), dtype=torch.float64, device=s.dev)
    for m in range(c["modes"]):
        k = ((key << 4) | (2 * m)) + 0x2545F491
        g[..., m] = s.g2_median * torch.exp(torch.sqrt(-2.0 * torch.log(_hash(k))) * torch.cos(2.0 * math.pi * _hash(k + 1)))
    ok = (s.hw[q] >= s.hw_min) & (i != j)[..., None]
    return g * ok, q


def _channels(c, s):
    """The channel list (i < j, mode) in lexicographic order, as host arrays."""
    parts = []
    for idx in s.classes:
        n = idx.numel()
        step = max(1, 2_000_000 // max(n, 1))
        for r0 in range(0, n - 1, step):
            rows = torch.arange(r0, min(n - 1, r0 + step), device=s.dev)
            a, b = torch.nonzero(torch.arange(n, device=s.dev)[None, :] > rows[:, None], as_tuple=True)
            i, j = idx[rows[a]], idx[b]
            g, _ = _pair_data(c, s, i, j)
            p, m = torch.nonzero(g, as_tuple=True)
            parts.append((i[p].int().cpu(), j[p].int().cpu(), m.to(torch.int8).cpu(), g[p, m].cpu()))
    if not parts:
        return tuple(np.zeros(0, t) for t in (np.int32, np.int32, np.int8, np.float64))
    return tuple(torch.cat([x[k] for x in parts]).numpy() for k in range(4))


_SYSTEM_KEYS = ("kn", "qn", "modes", "keep", "bands", "stats")
_last = {"system": (None, None), "plan": (None, None)}     # the material at hand and its plan


def _system(c):
    key = tuple(c[k] for k in _SYSTEM_KEYS)
    if _last["system"][0] != key:
        _last["system"] = (None, None)
        s = _states(c)
        ci, cj, cn, g2 = _channels(c, s)
        torch.cuda.empty_cache()
        h = types.SimpleNamespace(
            kgrid=(c["kn"],) * 3, qgrid=(c["qn"],) * 3, n_modes=c["modes"], sigma=s.sigma, n_q_norm=float(c["qn"] ** 3),
            state_k=s.k.int().cpu().numpy(), state_band=s.band.to(torch.int8).cpu().numpy(), eps=s.eps.cpu().numpy(),
            hw=s.hw.cpu().numpy(), ch_i=ci, ch_j=cj, ch_nu=cn, g2=g2, n_states=s.n, n_channels=int(g2.size))
        _last["system"] = (key, (s, h))
    return _last["system"][1]


def _plan(c):
    key = tuple(c[k] for k in _SYSTEM_KEYS) + (c["dtype"], c["nsigma"])
    if _last["plan"][0] != key:
        _last["plan"] = (None, None)
        s, h = _system(c)
        plan = E.build_channels(h, dtype=c["dtype"], device=s.dev.index, energy_nsigma=c["nsigma"], statistics=c["stats"])
        _last["plan"] = (key, plan)
    return _last["plan"][1]


# ---------------------------------------------------------------- inputs
def _inputs(c, s, n_channels, seed):
    """Occupations, baths and loss gradients of the seed, in the plan's type."""
    gen = torch.Generator(device=s.dev).manual_seed(int(seed) * 1000003 + 17)
    rand = lambda *sh: torch.rand(*sh, generator=gen, device=s.dev, dtype=torch.float64)
    randn = lambda *sh: torch.randn(*sh, generator=gen, device=s.dev, dtype=torch.float64)
    dt = torch.float64 if c["dtype"] == "f64" else torch.float32
    B = c["batch"]
    occ = lambda e, mu, T: 0.5 * (1.0 - torch.tanh(0.5 * (e - mu) / (KB * T)))
    bath = lambda T: torch.where(s.hw > 0, 1.0 / torch.expm1(s.hw.clamp_min(1e-300) / (KB * T)), torch.zeros_like(s.hw))
    T = 250.0 + 100.0 * rand(B, 1)
    if c["stats"] == "bose":
        f = (1.0 / torch.expm1(s.eps[None] / (KB * T))) * (0.7 + 0.6 * rand(B, s.n))
    elif c["op"] == "transport":
        f = occ(s.eps[None], -0.1 - 0.05 * rand(1, 1), 300.0)
    elif c["op"] in ("rt", "coupled", "adjoint", "adjoint_coupled"):
        f = occ(s.eps[None], -0.1, 300.0) + 0.1 * torch.exp(-0.5 * ((s.eps[None] - 0.15 - 0.1 * rand(1, 1)) / 0.05) ** 2)
    else:
        f = (occ(s.eps[None], 0.05, T) * (0.8 + 0.4 * rand(B, s.n))).clamp(0.0, 1.0)
    N = torch.stack([bath(float(t)) for t in T.reshape(-1)]) if c["baths"] else bath(300.0 if c["op"] == "transport" else float(T[0, 0]))
    x = types.SimpleNamespace(f=f.to(dt), N=N.to(dt), lam=randn(B, s.n).to(dt), muN=None)
    w = randn(*s.hw.shape)
    neg = (-_coords(c["qn"], s.dev)) % c["qn"]
    qm = (neg[:, 0] * c["qn"] + neg[:, 1]) * c["qn"] + neg[:, 2]
    x.muN, x.qm = (0.5 * (w + w[qm])).to(dt), qm
    if B == 1:
        x.f, x.lam = x.f[0].contiguous(), x.lam[0].contiguous()
    return x


def prepare(case, seed):
    plan = _plan(case)
    s, h = _system(case)
    x = _inputs(case, s, h.n_channels, seed)
    st = types.SimpleNamespace(c=case, plan=plan, f=x.f, N=x.N, lam=x.lam, muN=x.muN)
    op = case["op"]
    if op in ("vjp", "adjoint", "adjoint_coupled"):
        st.gg2 = torch.empty(h.n_channels, dtype=torch.float64, device=s.dev)
    if op in ("rt", "coupled"):
        st.u, st.M = torch.empty_like(st.f), torch.empty_like(st.N)
    if op == "train":
        st.g2 = torch.from_numpy(h.g2).to(s.dev).requires_grad_()
        st.f.requires_grad_()
    if op == "transport":
        st.vel = s.v.to(st.f.dtype)
    return st


def run(st):
    c, plan, op = st.c, st.plan, st.c["op"]
    if op == "fwd":
        return {"I": E.collision_integral(plan, st.f, st.N)}
    if op == "vjp":
        gf, gg2 = E.collision_vjp(plan, st.f, st.N, st.lam, gg2=st.gg2)
        return {"gf": gf, "gg2": gg2}
    if op == "train":
        I = EA.collision(st.f, st.g2, plan, st.N)
        gf, gg2 = torch.autograd.grad(I, [st.f, st.g2], st.lam)
        return {"I": I.detach(), "gf": gf, "gg2": gg2}
    if op == "rt":
        st.u.copy_(st.f)
        return {"f": E.rt_step(plan, st.u, st.N, 1.0, c["steps"], use_graph=True)}
    if op == "coupled":
        st.u.copy_(st.f)
        st.M.copy_(st.N)
        f, N = E.rt_step_coupled(plan, st.u, st.M, 1.0, c["steps"])
        return {"f": f, "N": N}
    if op == "adjoint":
        gf, gg2 = E.rt_adjoint(plan, st.f, st.N, 1.0, c["steps"], 2, st.lam, gg2=st.gg2)
        return {"gf": gf, "gg2": gg2}
    if op == "adjoint_coupled":
        gf, gN, gg2 = E.rt_adjoint_coupled(plan, st.f, st.N, 1.0, c["steps"], 2, st.lam, st.muN, gg2=st.gg2)
        return {"gf": gf, "gN": gN, "gg2": gg2}
    if op == "phonon_rate":
        return {"dN": E.phonon_rate(plan, st.f, st.N)}
    if op == "transport":
        r = E.iterate_transport(plan, st.f, st.vel, 300.0, st.N, tol=1e-8, max_iter=200, want_x=True)
        return {"mu": r["mu"], "x": r["x"]}
    raise ValueError(op)


# ---------------------------------------------------------------- what a pass cannot do without
def _counts(c):
    """(states, pairs, channels) of a case, from its grids."""
    if c["stats"] == "bose":
        n = 3 * c["kn"] ** 3 - 2
        return n, n * (n - 1) / 2.0, n * (n - 1) / 2.0 * c["modes"]
    n = max(2.0, min(float(c["bands"]) * c["kn"] ** 3, round(c["keep"] * c["kn"] ** 3)))
    cos = float((c["kn"] // c["qn"]) ** 3)
    pairs = n * max(n / cos - 1.0, 1.0) / 2.0
    part = 1.0
    if c["nsigma"]:      # pairs and modes near energy conservation, of a 0.3 eV window
        part = min(1.0, 2.0 * 2.0 * c["nsigma"] * 0.008 / 0.3)
    return n, pairs, pairs * c["modes"] * part


def work(case):
    S, pairs, nch = _counts(case)
    es = 8 if case["dtype"] == "f64" else 4
    B, op = case["batch"], case["op"]
    nq = case["qn"] ** 3 * case["modes"]
    one = nch * es + pairs * 4 + nq * es * (B if case["baths"] else 1)   # |g|^2, who pairs with whom, N
    fwd = {"bytes": one + 2 * B * S * es, "flops": 40.0 * nch + 10.0 * pairs * B}
    rev = {"bytes": one + 3 * B * S * es + 8 * nch, "flops": 46.0 * nch + 24.0 * pairs * B}
    if op in ("fwd", "phonon_rate"):
        return fwd
    if op == "vjp":
        return rev
    if op == "train":
        return {k: fwd[k] + rev[k] for k in fwd}
    if op == "transport":      # coefficients once, then a matrix product for three directions an iteration
        return {"bytes": one + 15 * 2 * pairs * es, "flops": 40.0 * nch + 15 * 12.0 * pairs}
    n = case["steps"]
    if op == "rt":
        return {k: 4 * n * v for k, v in fwd.items()}
    if op == "coupled":
        return {k: 8 * n * v for k, v in fwd.items()}
    if op == "adjoint":
        return {k: 4 * n * (fwd[k] + rev[k]) for k in fwd}
    return {k: 8 * n * (fwd[k] + rev[k]) for k in fwd}


# ---------------------------------------------------------------- the same in 64 bits, plain torch
def _gauss(c, s, idx, q):
    x = (s.eps[idx][:, None] - s.eps[idx][None, :])[..., None]
    w = s.hw[q]
    a = -0.5 / (s.sigma * s.sigma)
    return torch.exp(a * (x + w) ** 2), torch.exp(a * (x - w) ** 2)


def _block(c, s, idx):
    """Dense |g|^2, q index and Gaussians of one coset: g, q, Ga, Ge."""
    g, q = _pair_data(c, s, idx[:, None].expand(-1, idx.numel()), idx[None, :].expand(idx.numel(), -1))
    if c["nsigma"]:
        x = (s.eps[idx][:, None] - s.eps[idx][None, :])[..., None]
        g = g * (torch.minimum((x + s.hw[q]).abs(), (x - s.hw[q]).abs()) < c["nsigma"] * s.sigma)
    return (g, q) + _gauss(c, s, idx, q)


def _in_weights(g, q, Ga, Ge, N):
    return torch.nan_to_num(g * (torch.where(g != 0, N[q], 0.0) * (Ga + Ge) + Ga)).sum(-1)


def _pref(c, s, n):
    return 2.0 * math.pi / (HBAR * n) / (s.sigma * math.sqrt(2.0 * math.pi))


def _upper(c, s, idx, val, full):
    """val [n, n, modes] of the coset's channels (i < j) in the caller's order; `full`: before the selection."""
    n = idx.numel()
    g, _ = full
    m = (g != 0) & torch.triu(torch.ones(n, n, dtype=torch.bool, device=s.dev), 1)[..., None]
    return val[m]


def _rhs(B, f, K):
    return K * ((1.0 - f) * (B @ f) - f * (B.T @ (1.0 - f)))


def exact(case, seed):
    c = case
    s = _states(c)
    x = _inputs(c, s, 0, seed)
    f, N, lam, muN = (t.double() for t in (x.f, x.N, x.lam, x.muN))
    K = _pref(c, s, c["qn"] ** 3)
    op = c["op"]
    sg = -1.0 if c["stats"] == "bose" else 1.0
    one = f.dim() == 1
    F, L = (f[None] if one else f) * sg, lam[None] if one else lam
    if op in ("fwd", "vjp", "train"):
        I, gf, gg = torch.zeros_like(F), torch.zeros_like(F), []
        for idx in s.classes:
            g, q, Ga, Ge = _block(c, s, idx)
            u, l = F[:, idx].T, L[:, idx].T
            v = 0.0
            for grp in (range(F.shape[0]) if c["baths"] else [slice(None)]):
                sl = slice(grp, grp + 1) if c["baths"] else grp
                Nb = N[grp] if c["baths"] else N
                Bm = _in_weights(g, q, Ga, Ge, Nb)
                ub, lb = u[:, sl], l[:, sl]
                I[sl, idx] = _rhs(Bm, ub, K).T
                if op != "fwd":
                    gf[sl, idx] = (K * (Bm.T @ (lb * (1 - ub)) - lb * (Bm @ ub) + Bm @ (lb * ub)
                                        - lb * (Bm.T @ (1 - ub)))).T
                    m1 = (lb * (1 - ub)) @ ub.T - (1 - ub) @ (lb * ub).T
                    m2 = (lb * ub) @ (1 - ub).T - ub @ (lb * (1 - ub)).T
                    t = torch.where(g != 0, Nb[q], 0.0) * (Ga + Ge)
                    v = v + torch.where(g != 0, K * (m1[..., None] * (t + Ga) - m2[..., None] * (t + Ge)), 0.0)
            if op != "fwd":
                full = (_pair_data(c, s, idx[:, None].expand(-1, idx.numel()), idx[None, :].expand(idx.numel(), -1))
                        if c["nsigma"] else (g, q))
                gg.append(_upper(c, s, idx, v, full))
        I, gf = (t[0] if one else t for t in (I * sg, gf))
        if op == "fwd":
            return {"I": I}
        r = {"gf": gf, "gg2": sg * torch.cat(gg)}
        return dict(r, I=I) if op == "train" else r
    if op == "phonon_rate":
        return {"dN": _Coupled(c, s, x.qm).rate(f, N)}
    if op in ("adjoint", "coupled", "adjoint_coupled"):
        m = _Coupled(c, s, x.qm)
        if m.cells * c["steps"] > 1.5e8 and op != "coupled":
            return None          # the graph of the steps would not fit the device
        with torch.set_grad_enabled(op != "coupled"):
            u, M = f.clone().requires_grad_(op != "coupled"), N.clone().requires_grad_(op != "coupled")
            g = [b[0].clone().requires_grad_(op != "coupled") for b in m.blocks]
            fT, NT = m.steps(u, M, g, c["steps"], op != "adjoint")
            if op == "coupled":
                return {"f": fT, "N": NT}
            loss = (fT * lam).sum() + ((NT * muN).sum() if op == "adjoint_coupled" else 0.0)
            grads = torch.autograd.grad(loss, [u, M] + g)
        gg = torch.cat([_upper(c, s, idx, d + d.transpose(0, 1), (b[0], None))
                        for d, b, idx in zip(grads[2:], m.blocks, s.classes)])
        r = {"gf": grads[0], "gg2": gg}
        return dict(r, gN=grads[1]) if op == "adjoint_coupled" else r
    Bs = [_in_weights(*_block(c, s, idx), N) for idx in s.classes]
    if op == "rt":
        def rhs(u):
            o = torch.zeros_like(u)
            for idx, Bm in zip(s.classes, Bs):
                o[idx] = _rhs(Bm, u[idx], K)
            return o
        for _ in range(c["steps"]):
            k1 = rhs(f)
            k2 = rhs(f + 0.5 * k1)
            k3 = rhs(f + 0.5 * k2)
            k4 = rhs(f + k3)
            f = f + (k1 + 2 * k2 + 2 * k3 + k4) / 6.0
        return {"f": f}
    vel = s.v.to(x.f.dtype).double()
    rhs = vel * (-f * (1 - f) / (KB * 300.0))[:, None]
    tinv = torch.zeros_like(f)
    for idx, Bm in zip(s.classes, Bs):
        tinv[idx] = K * (Bm.T.sum(1) + (Bm - Bm.T) @ f[idx])
    tau = torch.where(tinv > 0, 1.0 / tinv, 0.0)[:, None]
    xx, mu = tau * rhs, None
    mob = lambda y: -(vel.T @ y) / f.sum() * 1e-11
    mu = mob(xx)
    Ws = [K * (Bm - f[idx][:, None] * (Bm - Bm.T)) for idx, Bm in zip(s.classes, Bs)]
    best, since = math.inf, 0
    for _ in range(200):
        y = torch.zeros_like(xx)
        for idx, W in zip(s.classes, Ws):
            y[idx] = W @ xx[idx]
        xx = tau * (rhs + y)
        new = mob(xx)
        change = float((new - mu).abs().max() / new.abs().max())
        mu = new
        best, since = (change, 0) if change < best else (best, since + 1)
        if change <= 1e-8 or since >= 5:
            break
    # in single precision the last digits decide where the iteration stops
    return {"mu": mu if c["dtype"] == "f64" else None, "x": xx if c["dtype"] == "f64" else None}


class _Coupled:
    """Electron and phonon rates of the whole system as dense blocks, differentiable."""

    def __init__(self, c, s, qm):
        self.c, self.s, self.qm = c, s, qm
        self.blocks = [_block(c, s, idx) for idx in s.classes]
        self.cells = sum(b[0].numel() for b in self.blocks)
        self.K, self.Kp = _pref(c, s, c["qn"] ** 3), _pref(c, s, c["kn"] ** 3)

    def rates(self, u, M, gs, phonons):
        dI, dN = [], torch.zeros_like(M)
        for idx, (g0, q, Ga, Ge), g in zip(self.s.classes, self.blocks, gs):
            ub = u[idx]
            Nq = torch.where(g0 != 0, M[q], 0.0)
            # both weights with N at the row's own q, so that dL/dN falls on that bin
            t = Nq * (Ga + Ge)
            Bm, Am = (g * (t + Ga)).sum(-1), (g * (t + Ge)).sum(-1)
            dI.append(self.K * ((1 - ub) * (Bm @ ub) - ub * (Am @ (1 - ub))))
            if phonons:
                gain, loss = ((1 - ub)[:, None] * ub[None, :])[..., None], (ub[:, None] * (1 - ub)[None, :])[..., None]
                t = g * Ga * ((Nq + 1) * gain - Nq * loss)
                dN = dN.index_add(0, q.reshape(-1), t.reshape(-1, t.shape[-1]))
        return torch.cat(dI), self.Kp * dN

    def rate(self, f, N):
        return self.rates(f, N, [b[0] for b in self.blocks], True)[1]

    def steps(self, u, M, gs, n, phonons):
        even = lambda y: 0.5 * (y + y[self.qm])
        for _ in range(n):
            k1, r1 = self.rates(u, M, gs, phonons)
            k2, r2 = self.rates(u + 0.5 * k1, M + 0.5 * even(r1), gs, phonons)
            k3, r3 = self.rates(u + 0.5 * k2, M + 0.5 * even(r2), gs, phonons)
            k4, r4 = self.rates(u + k3, M + even(r3), gs, phonons)
            u = u + (k1 + 2 * k2 + 2 * k3 + k4) / 6.0
            if phonons:
                M = M + even(r1 + 2 * r2 + 2 * r3 + r4) / 6.0
        return u, M
