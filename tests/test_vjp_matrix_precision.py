"""dL/d|g|^2 of several vectors over the pair matrix, FP64, against sums in 80 bits."""
import numpy as np
import pytest

from test_bath_per_vector import full_system
from test_cpu_build import _out, _run, _write, driver  # noqa: F401

# per element about a dozen roundings of the weights and products and a tree over the
# vectors, each 0.3 x 2^-53 rms relative to the terms: 1.2e-16 to 2.5e-16 normwise
TOL = 4e-16


def inputs(s, B):
    rng = np.random.default_rng(B)
    # gradients that vary slowly: lam_d - lam_p is smaller than lam
    L = np.array([np.sin(3 * s.eps / 0.3 + b) + 0.05 * rng.normal(size=s.n_states) for b in range(B)])
    return rng.uniform(size=(B, s.n_states)), s.nph(300.0), L


def ref_gg2(s, F, N, L):
    ld = np.longdouble
    kn = s.kgrid[0]
    k = np.stack(np.unravel_index(s.state_k, s.kgrid), 1)
    i, j, m = s.ch_i, s.ch_j, s.ch_nu
    d = (k[j] - k[i]) % kn
    q = (d[:, 0] * kn + d[:, 1]) * kn + d[:, 2]
    x, hw, sg = s.eps.astype(ld)[i] - s.eps.astype(ld)[j], s.hw.astype(ld)[q, m], ld(s.sigma)
    ga, ge = np.exp(-(x + hw) ** 2 / (2 * sg * sg)), np.exp(-(x - hw) ** 2 / (2 * sg * sg))
    K = 2 * ld(np.pi) / (ld(0.6582119569) * s.n_q_norm) / (sg * np.sqrt(2 * ld(np.pi)))
    t = N.astype(ld)[q, m] * (ga + ge)
    out = np.zeros(i.size, ld)
    for f, l in zip(F.astype(ld), L.astype(ld)):
        out += K * (l[i] - l[j]) * ((t + ga) * f[j] * (1 - f[i]) - (t + ge) * f[i] * (1 - f[j]))
    return out


def nerr(x, r):
    return float(np.linalg.norm(x - r) / np.linalg.norm(r))


def test_gradients_cpu(driver, tmp_path):  # noqa: F811
    s = full_system(130, 6)
    F, N, L = inputs(s, 64)
    _write(tmp_path, s, f=F, lam=L, nph=N, B=64)
    _run(driver, tmp_path, "vjp")
    assert nerr(_out(tmp_path, "gg2"), ref_gg2(s, F, N, L)) <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 24, 40, 64, 80])
def test_gradients(B):
    import torch

    import paper_2511_03683_amd as E
    s = full_system(130, 6)
    F, N, L = inputs(s, B)
    d = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda:0")
    plan = E.build_channels(s, device=0)
    gg = E.collision_vjp(plan, d(F), d(N), d(L), gg2=True)[1].cpu().numpy()
    plan.close()
    assert nerr(gg, ref_gg2(s, F, N, L)) <= TOL
