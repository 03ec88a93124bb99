"""The batched passes over entries, which plans take that have no pair records (less
than half of the mode slots filled) or whose window holds too few vectors of a bath
each: against the oracle (tolerances as in test_pair_matrix, 1e-10 FP64 and 1e-5 FP32,
normwise)."""
import numpy as np
import pytest

import oracle
import synth
from test_cpu_build import _out, _run, _write, driver  # noqa: F401
from test_pair_matrix import TOL, cast, dev, gross, host, nerr, rounded


def sparse_system(n_states, n_channels, kn=5):
    return synth.random_channel_system(n_states=n_states, n_channels=n_channels, kn=kn, n_modes=3, seed=4)


def inputs(s, B, dtype, own):
    rng = np.random.default_rng(B)
    N = np.stack([s.nph(150.0 + 20.0 * b) for b in range(B)]) if own else s.nph(300.0)
    return [cast(a, dtype) for a in (rng.uniform(size=(B, s.n_states)), rng.normal(size=(B, s.n_states)), N)]


def check(s, dtype, F, L, N, I, gf, gg):
    r, rg = rounded(s, dtype), 0.0
    for b in range(len(F)):
        n = N[b] if N.ndim > s.hw.ndim else N
        if I is not None:
            assert nerr(I[b], oracle.collision(r, F[b], n), gross(r, F[b], n)) <= TOL[dtype], b
        rf, g = oracle.collision_vjp(r, F[b], n, L[b])
        rg = rg + g
        assert nerr(gf[b], rf) <= TOL[dtype], b
    assert nerr(gg, rg) <= TOL[dtype]


@pytest.mark.parametrize("own", [False, True])
def test_reverse_cpu(driver, tmp_path, own):  # noqa: F811
    s = sparse_system(60, 900)
    F, L, N = inputs(s, 9, "f64", own)
    _write(tmp_path, s, f=F, lam=L, nph=N, B=9, nph_per_batch=int(own))
    _run(driver, tmp_path, "vjp", fill="random:3")
    check(s, "f64", F, L, N, None, _out(tmp_path, "gf", F.shape), _out(tmp_path, "gg2"))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("B,own,partners", [(8, False, 0), (33, False, 0), (70, False, 0), (9, True, 0), (17, True, 0),
                                            (16, False, 48), (16, False, 64), (16, False, 96), (16, False, 128),
                                            (16, False, 160)])
def test_no_pair_records(dtype, B, own, partners):
    import paper_2511_03683_amd as E
    s = sparse_system(120, 4000)
    F, L, N = inputs(s, B, dtype, own)
    plan = E.build_channels(s, dtype=dtype, device=0)
    assert E.plan_info(plan)["pair_records"] == 0
    if partners:
        try:
            E.set_tuning(plan, batch_partners=partners)
        except E.EphbteError as e:
            plan.close()
            assert "LDS" in str(e)
            pytest.skip(f"{partners} partners exceed the LDS of a workgroup")
    I = host(E.collision_integral(plan, dev(F, dtype), dev(N, dtype)))
    gf, gg = E.collision_vjp(plan, dev(F, dtype), dev(N, dtype), dev(L, dtype), gg2=True)
    gf, gg = host(gf), host(gg)
    plan.close()
    check(s, dtype, F, L, N, I, gf, gg)


# pair records with windows of all states.  9 vectors: three fit in 160 KB beside 1200
# states (forward also 1700), not beside 2700, where both go by entries; 3 vectors: two
# fit beside 1700 (forward also 2700), else one pass each
@pytest.mark.gpu
@pytest.mark.parametrize("S", [1200, 1700, 2700])
@pytest.mark.parametrize("B", [3, 9])
def test_window_leaves_few_vectors(S, B):
    import paper_2511_03683_amd as E
    s = synth.random_channel_system(n_states=S, n_channels=60000, kn=14, n_modes=1, seed=6)
    F, L, N = inputs(s, B, "f64", True)
    plan = E.build_channels(s, device=0)
    assert E.plan_info(plan)["pair_records"] > 0
    I = host(E.collision_integral(plan, dev(F), dev(N)))
    gf, gg = E.collision_vjp(plan, dev(F), dev(N), dev(L), gg2=True)
    gf, gg = host(gf), host(gg)
    plan.close()
    check(s, "f64", F, L, N, I, gf, gg)
