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


def sparse_system():
    """60 states, one mode, 700 of the 1770 pairs: pair records, and states that are no
    partners of each other."""
    return synth.random_channel_system(n_states=60, n_channels=700, n_modes=1, seed=3)


def touched(s, p):
    t = set(s.ch_j[s.ch_i == p]) | set(s.ch_i[s.ch_j == p]) | {p}
    assert 1 < len(t) < s.n_states
    return np.isin(np.arange(s.n_states), list(t))


class Cpu:
    def __init__(self, driver, folder):  # noqa: F811
        self.driver, self.folder = driver, folder

    def __call__(self, s, dtype, F, NPH, L=None):
        B = len(F)
        kw = dict(f=F, nph=NPH, B=B, nph_per_batch=1)
        if L is None:
            _write(self.folder, s, dtype, **kw)
            _run(self.driver, self.folder, "forward")
            return _out(self.folder, "I", F.shape)
        _write(self.folder, s, dtype, lam=L, **kw)
        _run(self.driver, self.folder, "vjp")
        return _out(self.folder, "gf", F.shape), _out(self.folder, "gg2")


class Gpu:
    def __call__(self, s, dtype, F, NPH, L=None):
        import torch

        import paper_2511_03683_amd as E
        d = lambda a: torch.as_tensor(a, dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda:0")
        h = lambda t: t.cpu().numpy().astype(np.float64)
        plan = E.build_channels(s, dtype=dtype, device=0)
        assert E.plan_info(plan)["pair_records"] > 0
        if L is None:
            r = h(E.collision_integral(plan, d(F), d(NPH)))
        else:
            gf, gg = E.collision_vjp(plan, d(F), d(NPH), d(L), gg2=True)
            r = h(gf), h(gg)
        plan.close()
        return r


@pytest.fixture(params=["cpu", pytest.param("gpu", marks=pytest.mark.gpu)])
def call(request):
    if request.param == "gpu":
        return Gpu()
    return Cpu(request.getfixturevalue("driver"), request.getfixturevalue("tmp_path"))


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("B,dtype", [(9, "f64"), (3, "f64"), (9, "f32")])
def test_non_finite_occupation_reaches_its_partners_only(call, B, dtype, bad):
    s = sparse_system()
    F, NPH, _ = inputs(s, B, 4)
    clean = call(s, dtype, F, NPH)
    F[2, 17] = bad
    got = call(s, dtype, F, NPH)
    t = touched(s, 17)
    assert not np.isfinite(got[2, t]).any()
    assert np.array_equal(got[2, ~t], clean[2, ~t])
    rest = np.arange(B) != 2
    assert np.array_equal(got[rest], clean[rest])


@pytest.mark.parametrize("where", ["f", "lam"])
@pytest.mark.parametrize("B,bad", [(9, np.nan), (9, np.inf), (3, np.nan)])
def test_non_finite_input_of_the_reverse_pass(call, B, bad, where):
    s = sparse_system()
    F, NPH, L = inputs(s, B, 5)
    clean, cg = call(s, "f64", F, NPH, L)
    (F if where == "f" else L)[1, 17] = bad
    got, gg = call(s, "f64", F, NPH, L)
    t = touched(s, 17)
    # a state's own gradient does not contain its own occupation
    own = t & (np.arange(s.n_states) != 17) if where == "f" else t
    assert not np.isfinite(got[1, own]).any()
    assert np.array_equal(got[1, ~t], clean[1, ~t])
    rest = np.arange(B) != 1
    assert np.array_equal(got[rest], clean[rest])
    ch = (s.ch_i == 17) | (s.ch_j == 17)
    assert not np.isfinite(gg[ch]).any()
    assert np.array_equal(gg[~ch], cg[~ch])


@pytest.mark.parametrize("B", [9, 3])
def test_unused_infinite_phonon_occupation(call, B):
    """N = 1 / expm1(0) at q = 0, which no channel uses."""
    s = full_system(40, 4)
    F, NPH, L = inputs(s, B, 6)
    assert not np.any(s.state_k[s.ch_i] == s.state_k[s.ch_j])
    ref, (rf, rg) = call(s, "f64", F, NPH), call(s, "f64", F, NPH, L)
    NPH = NPH.copy()
    NPH[:, 0, :] = np.inf
    got, (gf, gg) = call(s, "f64", F, NPH), call(s, "f64", F, NPH, L)
    for a, b in ((got, ref), (gf, rf), (gg, rg)):
        assert nerr(a, b) <= 1e-10


@pytest.mark.parametrize("scale", [1e3, 1e150])
def test_numbers_of_any_size(call, scale):
    """Occupations of a Fermi plan outside [0, 1], and loss gradients that leave the
    fixed point no scale."""
    s = full_system(40, 4)
    F, NPH, L = inputs(s, 9, 7)
    F[3] = 40.0 * F[3] - 20.0
    F[4, 5] = 1e3
    L[2] *= scale
    L[5] *= 1.0 / scale
    L[6] *= scale * scale
    got, (gf, _) = call(s, "f64", F, NPH), call(s, "f64", F, NPH, L)
    for b in range(9):
        assert nerr(got[b], oracle.collision(s, F[b], NPH[b])) <= 1e-10, b
        assert nerr(gf[b], oracle.collision_vjp(s, F[b], NPH[b], L[b])[0]) <= 1e-10, b


def longdouble_reference(s, F, NPH, L):
    """I and dL/df of each vector in 80-bit arithmetic, every pair and mode a channel."""
    ld = np.longdouble
    S, kn = s.n_states, s.kgrid[0]
    k = np.stack(np.unravel_index(s.state_k, s.kgrid), 1)
    i, j = np.arange(S)[:, None], np.arange(S)[None, :]
    d = (k[j] - k[i]) % kn
    q = (d[..., 0] * kn + d[..., 1]) * kn + d[..., 2]
    g = np.zeros((S, S, s.n_modes), ld)
    g[s.ch_i, s.ch_j, s.ch_nu] = s.g2
    g[s.ch_j, s.ch_i, s.ch_nu] = s.g2
    x = s.eps.astype(ld)[i] - s.eps.astype(ld)[j]
    hw, sg = s.hw.astype(ld)[q], ld(s.sigma)
    G = lambda u: np.exp(-u * u / (2 * sg * sg))
    Ga, Ge = G(x[..., None] + hw), G(x[..., None] - hw)
    K = 2 * ld(np.pi) / (ld(0.6582119569) * s.n_q_norm) / (sg * np.sqrt(2 * ld(np.pi)))
    I, gf = [], []
    for f, nph, lam in zip(F.astype(ld), NPH.astype(ld), L.astype(ld)):
        t = nph[q] * (Ga + Ge)
        a, b = (g * (t + Ge)).sum(-1), (g * (t + Ga)).sum(-1)
        fd, fp = f[:, None], f[None, :]
        I.append(K * (b * fp * (1 - fd) - a * (1 - fp) * fd).sum(1))
        gf.append(K * (-(lam[:, None] - lam[None, :]) * (a * (1 - fp) + b * fp)).sum(1))
    return np.array(I), np.array(gf)


def test_small_elements_keep_their_digits(call):
    """A non-degenerate system: every f is near 1e-9 of the largest it could be, and so
    is I.  Floating-point sums of n terms leave at most n 2^-53 of the gross value, here
    n = 3 x 95, so that the median element (net and gross within a factor of 100) has 12
    digits."""
    s = full_system(96, 6)
    s.sigma = 0.006
    F, NPH, L = inputs(s, 9, 11)
    F *= 1e-9
    got, (gf, _) = call(s, "f64", F, NPH), call(s, "f64", F, NPH, L)
    I, rf = longdouble_reference(s, F, NPH, L)
    for x, ref in ((got, I), (gf, rf)):
        rel = (np.abs(x - ref) / np.abs(ref)).astype(float)
        assert np.median(rel) <= 3e-14 and np.quantile(rel, 0.9) <= 1e-12, np.quantile(rel, [0.5, 0.9, 0.99])


@pytest.mark.gpu
def test_many_vectors_take_the_workspace_of_64():
    import torch

    import paper_2511_03683_amd as E
    s = full_system(48, 6)
    F, NPH, L = inputs(s, 200, 12)
    NPH = NPH * np.linspace(0.5, 1.0, 200)[:, None, None]
    d = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda:0")
    plan = E.build_channels(s, device=0)
    E.collision_integral(plan, d(F[:64]), d(NPH[:64]))
    E.collision_vjp(plan, d(F[:64]), d(NPH[:64]), d(L[:64]), gg2=True)
    held = E.plan_info(plan)["bytes"]
    got = E.collision_integral(plan, d(F), d(NPH)).cpu().numpy()
    gf, gg = (x.cpu().numpy() for x in E.collision_vjp(plan, d(F), d(NPH), d(L), gg2=True))
    assert E.plan_info(plan)["bytes"] == held
    plan.close()
    rg = 0.0
    for b in range(200):
        rf, g = oracle.collision_vjp(s, F[b], NPH[b], L[b])
        rg = rg + g
        if b in (0, 63, 64, 127, 128, 199):
            assert nerr(got[b], oracle.collision(s, F[b], NPH[b])) <= 1e-10, b
            assert nerr(gf[b], rf) <= 1e-10, b
    assert nerr(gg, rg) <= 1e-10
