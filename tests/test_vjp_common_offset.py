"""Reverse pass of several vectors over the pair matrix: only differences of the loss
gradients enter, so a constant gives zero exactly and an offset costs no digits."""
import numpy as np
import pytest

import oracle
from test_bath_per_vector import full_system, nerr
from test_cpu_build import _out, _run, _write, driver  # noqa: F401


def inputs(B, S):
    rng = np.random.default_rng(B)
    d = rng.normal(size=(B, S)) * 2.0 ** -20
    lam = 1.0 + np.round(d * 2.0 ** 50) * 2.0 ** -50      # 1 + d, both exact
    lam[2] = -3.7                                          # constants
    lam[3] = 0.0
    lam[4] = 1e6                                           # one state apart from a constant
    lam[4, 7] = 1e6 + 1.0
    lam[5, 0] = 1e12                                       # a value far from the others
    return rng.uniform(size=(B, S)), lam


def check(s, F, nph, lam, gf, gg_const):
    for b in range(len(F)):
        if b in (2, 3):
            assert np.all(gf[b] == 0.0)
            continue
        # the differences are exact, so the oracle sees the same lam without its offset;
        # sums of n = 3 x 129 terms of one sign in FP64: n 2^-53 normwise
        ref = oracle.collision_vjp(s, F[b], nph, lam[b] - lam[b, 50])[0]
        assert nerr(gf[b], ref) <= 1e-13, b
    assert np.all(gg_const == 0.0)


@pytest.mark.parametrize("B", [9])
def test_offset_cpu(driver, tmp_path, B):  # noqa: F811
    s = full_system(130, 6)
    F, lam = inputs(B, 130)
    nph = s.nph(300.0)
    _write(tmp_path, s, f=F, lam=lam, nph=nph, B=B)
    _run(driver, tmp_path, "vjp")
    gf = _out(tmp_path, "gf", F.shape)
    _write(tmp_path, s, f=F, lam=np.full_like(lam, 0.3), nph=nph, B=B)
    _run(driver, tmp_path, "vjp")
    check(s, F, nph, lam, gf, _out(tmp_path, "gg2"))


@pytest.mark.gpu
@pytest.mark.parametrize("B", [7, 9, 70])
def test_offset(B):
    import torch

    import paper_2511_03683_amd as E
    s = full_system(130, 6)
    F, lam = inputs(B, 130)
    nph = s.nph(300.0)
    d = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda:0")
    plan = E.build_channels(s, device=0)
    gf = E.collision_vjp(plan, d(F), d(nph), d(lam), gg2=True)[0].cpu().numpy()
    gg = E.collision_vjp(plan, d(F), d(nph), d(np.full_like(lam, 0.3)), gg2=True)[1].cpu().numpy()
    plan.close()
    check(s, F, nph, lam, gf, gg)
