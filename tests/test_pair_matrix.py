"""The pair matrix (coefficients summed per state pair in 64 x 64 blocks) behind
the forms that apply one bath more than once: RK4 steps, the transport iteration
and several occupation vectors.  Sizes around the block edge, vector counts
around the 16 columns of a matrix instruction and the 64 of a group, states whose
components interleave, and non-finite occupations, against the oracle.

Tolerances are the parity tests' (1e-10 FP64, 1e-5 FP32, normwise): a sum of n
products in FP64 is within n 1.1e-16 of its gross value, and the systems here
have at most a few hundred partners a state.
"""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-10, "f32": 1e-5}
DT = {"f64": torch.float64, "f32": torch.float32}


@pytest.fixture(scope="module")
def E():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2511_03683_amd as lib
    return lib


def dev(a, dtype="f64"):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=DT[dtype], device="cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def full_system(n_states, kn, n_modes=3, seed=5):
    """n_states random states on a kn^3 grid, every pair and mode a channel."""
    s = synth.random_channel_system(n_states=n_states, n_channels=1, kn=kn, n_modes=n_modes, seed=seed)
    i, j = np.triu_indices(s.n_states, 1)
    s.ch_i = np.repeat(i, n_modes).astype(np.int32)
    s.ch_j = np.repeat(j, n_modes).astype(np.int32)
    s.ch_nu = np.tile(np.arange(n_modes), i.size).astype(np.int8)
    s.g2 = synth.lognormal_g2(s.ch_i, s.ch_j, s.ch_nu, seed)
    return s


def two_components(n, kn=6, seed=9):
    """Two all-pairs components whose states alternate in the caller's order."""
    s = full_system(2 * n, kn, seed=seed)
    keep = (s.ch_i % 2) == (s.ch_j % 2)
    s.ch_i, s.ch_j, s.ch_nu, s.g2 = s.ch_i[keep], s.ch_j[keep], s.ch_nu[keep], s.g2[keep]
    return s


def rounded(s, dtype):
    if dtype == "f64":
        return s
    r = copy.copy(s)
    for k in ("eps", "hw", "g2"):
        setattr(r, k, getattr(s, k).astype(np.float32).astype(np.float64))
    return r


def cast(a, dtype):
    return a if dtype == "f64" else a.astype(np.float32).astype(np.float64)


def nerr(x, ref, scale=0.0):
    return float(np.abs(x - ref).max() / max(np.abs(ref).max(), scale))


def gross(r, f, nph):
    return 1e-2 * max(x.max() for x in oracle.collision_inout(r, f, nph))


@pytest.mark.parametrize("S,B,dtype", [(2, 2, "f64"), (63, 7, "f64"), (64, 16, "f64"), (65, 17, "f32"), (129, 33, "f64"),
                                       (200, 48, "f32"), (130, 64, "f64"), (66, 65, "f64"), (128, 130, "f32")])
def test_vectors_through_the_matrix(E, S, B, dtype):
    s = full_system(S, 6)
    rng = np.random.default_rng(S)
    F, nph = cast(rng.uniform(size=(B, S)), dtype), cast(s.nph(300.0), dtype)
    plan = E.build_channels(s, dtype=dtype, device=0)
    out = torch.full((B, S + 3), 7.0, dtype=DT[dtype], device="cuda:0")
    E.collision_integral(plan, dev(F, dtype), dev(nph, dtype), out=out[:, :S])
    got = host(out)
    assert np.all(got[:, S:] == 7.0)
    r = rounded(s, dtype)
    for b in sorted({0, 1, B // 2, B - 1}):
        ref = oracle.collision(r, F[b], nph)
        assert nerr(got[b, :S], ref, gross(r, F[b], nph)) <= TOL[dtype], b
    plan.close()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_interleaved_components(E, dtype):
    """The matrix orders states by component; results come back in the caller's
    order, for vectors, RK4 steps (eager and from a graph) and transport."""
    s = two_components(70)
    S = s.n_states
    rng = np.random.default_rng(3)
    F, nph = cast(rng.uniform(size=(5, S)), dtype), cast(s.nph(300.0), dtype)
    plan = E.build_channels(s, dtype=dtype, device=0)
    r = rounded(s, dtype)
    got = host(E.collision_integral(plan, dev(F, dtype), dev(nph, dtype)))
    for b in range(5):
        assert nerr(got[b], oracle.collision(r, F[b], nph), gross(r, F[b], nph)) <= TOL[dtype]
    ref = F[0].copy()
    for _ in range(3):
        ref = oracle.rk4_step(r, ref, nph, 0.01)
    for graph in (False, True):
        f = dev(F[0], dtype)
        E.rt_step(plan, f, dev(nph, dtype), 0.01, 3, use_graph=graph)
        assert nerr(host(f), ref) <= TOL[dtype]
    f0 = cast(synth.fermi_dirac(s.eps, 0.1, 300.0), dtype)
    vel = cast(rng.normal(size=(S, 3)), dtype)
    out = E.iterate_transport(plan, dev(f0, dtype), dev(vel, dtype), 300.0, dev(nph, dtype), tol=0.0, max_iter=4, want_x=True)
    want = oracle.transport_solve(r, f0, vel, 300.0, nph, max_iter=4, stop_on_tol=False)
    assert nerr(out["mu"], want["mu"]) <= TOL[dtype]
    assert nerr(host(out["x"]), want["x"]) <= TOL[dtype]
    plan.close()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_occupation_reaches_its_partners_only(E, bad):
    """Zero entries of a block do not carry a non-finite value to states that
    have no channel with it."""
    s = synth.random_channel_system(n_states=60, n_channels=700, n_modes=1, seed=3)
    S, B, p = s.n_states, 9, 17
    F = np.random.default_rng(4).uniform(size=(B, S))
    nph = s.nph(300.0)
    plan = E.build_channels(s, device=0)
    assert E.plan_info(plan)["pair_records"] > 0
    clean = host(E.collision_integral(plan, dev(F), dev(nph)))
    F[2, p] = bad
    got = host(E.collision_integral(plan, dev(F), dev(nph)))
    partners = set(s.ch_j[s.ch_i == p]) | set(s.ch_i[s.ch_j == p]) | {p}
    assert 1 < len(partners) < S
    touched = np.isin(np.arange(S), list(partners))
    assert not np.isfinite(got[2, touched]).any()
    assert nerr(got[2, ~touched], clean[2, ~touched], np.abs(clean[2]).max()) <= 1e-14
    rest = np.arange(B) != 2
    assert np.array_equal(got[rest], clean[rest])
    plan.close()


@pytest.mark.parametrize("S,B,modes,dtype", [(2, 2, 1, "f64"), (63, 7, 3, "f64"), (65, 17, 6, "f32"), (129, 33, 3, "f64"),
                                             (130, 50, 4, "f64"), (64, 64, 2, "f32"), (66, 65, 3, "f64"),
                                             (100, 130, 3, "f32")])
def test_reverse_through_the_matrix(E, S, B, modes, dtype):
    """dL/df of every vector and dL/d|g|^2 summed over them, together and each
    alone, overwritten and accumulated."""
    s = full_system(S, 6, n_modes=modes)
    rng = np.random.default_rng(S + B)
    F, nph = cast(rng.uniform(size=(B, S)), dtype), cast(s.nph(300.0), dtype)
    lam = cast(rng.normal(size=(B, S)) + 3.0, dtype)
    plan = E.build_channels(s, dtype=dtype, device=0)
    r = rounded(s, dtype)
    refs = [oracle.collision_vjp(r, F[b], nph, lam[b]) for b in range(B)]
    rg = sum(x[1] for x in refs)
    start = torch.full((s.n_channels,), 0.5, dtype=torch.float64, device="cuda:0")
    args = (plan, dev(F, dtype), dev(nph, dtype), dev(lam, dtype))
    gf, gg = E.collision_vjp(*args, gg2=start.clone())
    gf1, none = E.collision_vjp(*args)
    nogf, gg1 = E.collision_vjp(*args, want_f=False, gg2=start.clone(), accumulate=True)
    assert none is None and nogf is None
    assert np.array_equal(host(gf), host(gf1))
    for b in sorted({0, 1, B // 2, B - 1}):
        assert nerr(host(gf)[b], refs[b][0]) <= TOL[dtype], b
    assert nerr(host(gg), rg) <= TOL[dtype]
    assert nerr(host(gg1) - 0.5, rg) <= TOL[dtype]
    plan.close()


@pytest.mark.parametrize("S,B,modes,dtype,stats", [(2, 2, 1, "f64", "fermi"), (63, 7, 3, "f64", "fermi"),
                                                   (130, 9, 6, "f32", "fermi"), (200, 17, 8, "f64", "fermi"),
                                                   (65, 24, 3, "f64", "bose"), (64, 8, 2, "f32", "bose")])
def test_bath_per_vector_over_pair_records(E, S, B, modes, dtype, stats):
    """Groups of vectors with a phonon table each, forward and reverse (FP64 over
    the pair records; the gradient overwritten and accumulated)."""
    s = full_system(S, 6, n_modes=modes)
    rng = np.random.default_rng(S + B)
    bose = stats == "bose"
    F = cast(rng.uniform(0.0, 3.0 if bose else 1.0, size=(B, S)), dtype)
    NPH = cast(np.stack([s.nph(150.0 + 30.0 * b) for b in range(B)]), dtype)
    lam = cast(rng.normal(size=(B, S)), dtype)
    plan = E.build_channels(s, dtype=dtype, device=0, statistics=stats)
    r = rounded(s, dtype)
    fwd = oracle.collision_bose if bose else oracle.collision
    vjp = oracle.collision_bose_vjp if bose else oracle.collision_vjp
    got = host(E.collision_integral(plan, dev(F, dtype), dev(NPH, dtype)))
    start = torch.full((s.n_channels,), 0.5, dtype=torch.float64, device="cuda:0")
    gf, gg = E.collision_vjp(plan, dev(F, dtype), dev(NPH, dtype), dev(lam, dtype), gg2=start.clone())
    _, ga = E.collision_vjp(plan, dev(F, dtype), dev(NPH, dtype), dev(lam, dtype), want_f=False, gg2=start.clone(),
                            accumulate=True)
    rg = 0.0
    for b in range(B):
        ref = fwd(r, F[b], NPH[b])
        assert nerr(got[b], ref, 0.0 if bose else gross(r, F[b], NPH[b])) <= TOL[dtype], b
        rf, rgb = vjp(r, F[b], NPH[b], lam[b])[:2]
        assert nerr(host(gf)[b], rf) <= TOL[dtype], b
        rg = rg + rgb
    assert nerr(host(gg), rg) <= TOL[dtype]
    assert nerr(host(ga) - 0.5, rg) <= TOL[dtype]
    plan.close()


@pytest.mark.parametrize("n_modes", [1, 2, 3, 5, 6, 8])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_channel_gradients_in_any_channel_order(E, dtype, n_modes):
    """Gradients of records whose channels follow each other (written in channel
    order by the wave) against the same channels shuffled (written by the lane):
    the same products, added to one old value, so they differ by a rounding of the
    FP64 sum at most.  The 37 states leave a remainder in every batch."""
    s = rounded(full_system(37, 4, n_modes=n_modes, seed=21), dtype)
    perm = np.random.default_rng(22).permutation(s.n_channels)
    t = copy.copy(s)
    for k in ("ch_i", "ch_j", "ch_nu", "g2"):
        setattr(t, k, getattr(s, k)[perm])
    rng = np.random.default_rng(23)
    f, lam = rng.uniform(0.1, 0.9, s.n_states), rng.normal(size=s.n_states)
    N, mu = s.nph(300.0), rng.normal(size=s.hw.shape)
    out = []
    for x in (s, t):
        plan = E.build_channels(x, dtype=dtype, device=0)
        a = torch.full((x.n_channels,), 0.25, dtype=torch.float64, device="cuda:0")
        b = a.clone()
        c = a.clone()
        E.collision_vjp(plan, dev(f, dtype), dev(N, dtype), dev(lam, dtype), gg2=a)
        E.collision_vjp(plan, dev(f, dtype), dev(N, dtype), dev(lam, dtype), gg2=b, accumulate=True)
        E.phonon_rate_vjp(plan, dev(f, dtype), dev(N, dtype), dev(mu, dtype), gg2=c, accumulate=True)
        out.append([host(v) for v in (a, b, c)])
    for got, ref in zip(*out):
        assert nerr(ref, got[perm]) <= 4e-16
    assert nerr(out[0][1] - 0.25, out[0][0]) <= 4e-16 * (1 + 0.25 / np.abs(out[0][0]).max())
