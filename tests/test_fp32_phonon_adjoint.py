"""The phonon side's reverse pass in FP32 plans, rounding for rounding.

dL/d|g|^2 is an FP64 output of FP32 plans too, so the FP32 arithmetic behind it is
part of the results: which products are fused into an addition is fixed in the
kernel.  On the CPU the kernel's terms are compared with the same expressions
rounded exactly (rational arithmetic), on the GPU the coupled adjoint with recorded
values.  Both are equalities.
"""
import ctypes
import ctypes.util
import hashlib
import json
import os
from fractions import Fraction

import numpy as np
import pytest

import synth
from test_cpu_build import _out, _run, _write, driver  # noqa: F401

HERE = os.path.dirname(os.path.abspath(__file__))
GOLDEN = os.path.join(HERE, "golden", "coupled_adjoint_f32.json")
HBAR = 0.6582119569
f32 = np.float32


def round32(x):
    """A rational number to the nearest float (ties to even)."""
    c = f32(float(x))
    best = min((np.nextafter(c, f32(-np.inf)), c, np.nextafter(c, f32(np.inf))),
               key=lambda v: (abs(Fraction(float(v)) - x), int(v.view(np.uint32)) & 1))
    return best if best != 0 else f32(0.0)


def fma(a, b, c):
    return round32(Fraction(float(a)) * Fraction(float(b)) + Fraction(float(c)))


@pytest.mark.parametrize("n_modes", [1, 2, 3, 5, 8])
def test_terms_are_fused_as_written(driver, tmp_path, n_modes):  # noqa: F811
    s = synth.random_channel_system(n_states=24, n_channels=60 * n_modes, kn=7, n_modes=n_modes, seed=31, sigma=0.05)
    rng = np.random.default_rng(32 + n_modes)
    S = s.n_states
    r = lambda a: np.asarray(a).astype(f32)
    f, lam = r(rng.uniform(0.05, 0.95, S)), r(rng.normal(size=S))
    N, mu = r(rng.uniform(0.1, 2.0, s.hw.shape)), r(rng.normal(size=s.hw.shape))
    _write(tmp_path, s, dtype="f32", f=f.astype(float), lam=lam.astype(float), nph=N.astype(float), mu=mu.astype(float))
    _run(driver, tmp_path, "phonon_adj")
    gN, gg2 = _out(tmp_path, "gN", s.hw.shape), _out(tmp_path, "gg2")
    eps, hw, g2 = r(s.eps), r(s.hw), r(s.g2)
    libm = ctypes.CDLL(ctypes.util.find_library("m"))
    libm.exp2f.restype, libm.exp2f.argtypes = ctypes.c_float, [ctypes.c_float]
    mc = f32(-1.4426950408889634 / (2.0 * s.sigma * s.sigma))
    gauss = lambda x: f32(libm.exp2f(ctypes.c_float(float(x * x * mc))))
    pref = 2.0 * np.pi / HBAR / (s.sigma * np.sqrt(2.0 * np.pi))
    ke, kp = f32(pref / s.n_q_norm), f32(pref / 7 ** 3)
    chan = {(int(i), int(j), int(m)): c for c, (i, j, m) in enumerate(zip(s.ch_i, s.ch_j, s.ch_nu))}
    checked = 0
    for n, q, qm, a, b in _out(tmp_path, "rec", (-1, 5)).astype(int):
        if n != 1 or q == qm:
            continue
        ofa = f32(1) - f[a]
        p1, p2 = f[b] * ofa, f[a] * (f32(1) - f[b])
        dp = fma(f[b], ofa, -p2)
        x = eps[a] - eps[b]
        for m in range(n_modes):
            c = chan.get((a, b, m), chan.get((b, a, m)))
            if c is None:
                continue
            G, A = gauss(x + hw[q, m]), gauss(x - hw[q, m])
            assert hw[q, m] == hw[qm, m]

            def term(l, w, g):
                t, k = ke * l, kp * w
                return fma(k, g, t * (G + A)) if n_modes == 1 else fma(t, G + A, k * g)

            gd = g2[c] * dp
            # the wave's sum adds zeros of the other lanes: exact
            assert gN[q, m] == round32(Fraction(float(gd)) * Fraction(float(term(lam[a], mu[q, m], G))))
            assert gN[qm, m] == round32(-Fraction(float(gd)) * Fraction(float(term(lam[b], mu[qm, m], A))))
            c2 = mu[qm, m] * A * fma(-N[qm, m], dp, p2)
            assert gg2[c] == kp * fma(mu[q, m] * G, fma(N[q, m], dp, p1), c2)
            checked += 1
    assert checked >= 10


def golden_case(n_modes):
    """Every pair and mode of a 5^3 grid (two batches of records a bin); inputs from
    IEEE arithmetic alone."""
    n = 5
    rng = np.random.Generator(np.random.Philox(1000 + n_modes))
    c = np.stack(np.unravel_index(np.arange(n ** 3), (n,) * 3), 1)
    i, j = np.triu_indices(n ** 3, 1)
    neg = synth.inverse_k(np.arange(n ** 3), (n,) * 3)
    even = lambda x: 0.5 * (x + x[neg])
    s = synth.random_channel_system(n_states=n ** 3, n_channels=1, kn=n, n_modes=n_modes, sigma=0.03, seed=7)
    s.state_k = np.arange(n ** 3, dtype=np.int32)
    s.eps = 0.01 * (c * c).sum(1) + rng.uniform(0.0, 0.05, n ** 3)
    s.hw = even(rng.uniform(0.005, 0.06, (n ** 3, n_modes)))
    s.ch_i = np.repeat(i, n_modes).astype(np.int32)
    s.ch_j = np.repeat(j, n_modes).astype(np.int32)
    s.ch_nu = np.tile(np.arange(n_modes), i.size).astype(np.int8)
    s.g2 = rng.uniform(1e-4, 2e-3, s.ch_i.size)
    return s, dict(f=rng.uniform(0.1, 0.9, n ** 3), N=even(rng.uniform(0.2, 3.0, s.hw.shape)),
                   lam=rng.uniform(-1.0, 1.0, n ** 3), muN=even(rng.uniform(-1.0, 1.0, s.hw.shape)))


def golden_run(E, n_modes, with_mu):
    import torch
    s, x = golden_case(n_modes)
    d = {k: torch.as_tensor(v.astype(f32), device="cuda:0") for k, v in x.items()}
    plan = E.build_channels(s, dtype="f32", device=0)
    gg2 = torch.empty(s.n_channels, dtype=torch.float64, device="cuda:0")
    gf, gN, _ = E.rt_adjoint_coupled(plan, d["f"], d["N"], 1.0, 3, 2, d["lam"], d["muN"] if with_mu else None, gg2=gg2)
    torch.cuda.synchronize()
    out = {k: v.cpu().numpy() for k, v in (("gf", gf), ("gN", gN), ("gg2", gg2))}
    plan.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("with_mu", [True, False])
@pytest.mark.parametrize("n_modes", range(1, 9))
def test_coupled_adjoint_keeps_its_values(n_modes, with_mu):
    pytest.importorskip("torch")
    import paper_2511_03683_amd as E
    with open(GOLDEN) as fh:
        ref = json.load(fh)[f"{n_modes},{int(with_mu)}"]
    got = golden_run(E, n_modes, with_mu)
    assert got["gf"].tobytes().hex()[:64] == ref["gf_head"]
    assert got["gN"].tobytes().hex()[:512] == ref["gN_head"]
    for k in ("gf", "gN", "gg2"):
        assert hashlib.sha256(got[k].tobytes()).hexdigest() == ref[k], k
