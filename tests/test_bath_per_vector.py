"""Vectors with a phonon bath each over q-ordered pair records, on the CPU build
(sanitizers) and on the GPU: odd windows and vector counts, against the oracle
(tolerances as elsewhere, 1e-10 FP64 and 1e-5 FP32, normwise)."""
import copy

import numpy as np
import pytest

import oracle
import synth
from test_cpu_build import _out, _run, _write, driver  # noqa: F401


def full_system(n_states, kn, n_modes=3, seed=5):
    """n_states random states on a kn^3 grid, every pair and mode a channel."""
    s = synth.random_channel_system(n_states=n_states, n_channels=1, kn=kn, n_modes=n_modes, seed=seed)
    i, j = np.triu_indices(s.n_states, 1)
    s.ch_i = np.repeat(i, n_modes).astype(np.int32)
    s.ch_j = np.repeat(j, n_modes).astype(np.int32)
    s.ch_nu = np.tile(np.arange(n_modes), i.size).astype(np.int8)
    s.g2 = synth.lognormal_g2(s.ch_i, s.ch_j, s.ch_nu, seed)
    return s


def inputs(s, B, seed, bose=False):
    rng = np.random.default_rng(seed)
    F = rng.uniform(0.0, 3.0 if bose else 1.0, size=(B, s.n_states))
    NPH = np.stack([s.nph(150.0 + 30.0 * b) for b in range(B)])
    return F, NPH, rng.normal(size=(B, s.n_states))


def nerr(x, ref):
    return float(np.abs(x - ref).max() / max(np.abs(ref).max(), 1e-300))


@pytest.mark.parametrize("S,B", [(63, 7), (65, 3), (21, 3)])
def test_odd_window_and_vector_count(driver, tmp_path, S, B):  # noqa: F811
    s = full_system(S, 6)
    F, NPH, L = inputs(s, B, S)
    _write(tmp_path, s, f=F, lam=L, nph=NPH, B=B, nph_per_batch=1)
    _run(driver, tmp_path, "vjp", fill="random:3")
    gf = _out(tmp_path, "gf", (B, S))
    rg = 0.0
    for b in range(B):
        rf, g = oracle.collision_vjp(s, F[b], NPH[b], L[b])
        assert nerr(gf[b], rf) <= 1e-10, b
        rg = rg + g
    assert nerr(_out(tmp_path, "gg2"), rg) <= 1e-10
