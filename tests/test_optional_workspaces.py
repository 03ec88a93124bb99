"""Routes that take a workspace others do not: they leave a call that cannot have it
(under the caller's capture, or where memory ran out) as it was without them.  On
the CPU build, whose runtime stand-in counts and limits allocations, and captured on
the GPU; against the oracle (1e-10 FP64, normwise)."""
import numpy as np
import pytest

import oracle
from test_bath_per_vector import full_system, nerr
from test_cpu_build import _out, _run, _write, driver  # noqa: F401


def system_and_inputs(B, per_batch):
    s = full_system(40, 4, n_modes=6)
    rng = np.random.default_rng(B)
    NPH = np.stack([s.nph(150.0 + 30.0 * b) for b in range(B)])
    return s, rng.uniform(size=(B, 40)), NPH if per_batch else NPH[0], rng.normal(size=(B, 40))


@pytest.mark.parametrize("B,per_batch", [(2, 0), (5, 0), (4, 1)])
def test_capture_after_a_single_vector(driver, tmp_path, B, per_batch):  # noqa: F811
    s, F, NPH, L = system_and_inputs(B, per_batch)
    _write(tmp_path, s, f=F, lam=L, nph=NPH, B=B, nph_per_batch=per_batch)
    _run(driver, tmp_path, "capture")
    assert _out(tmp_path, "mallocs")[0] == 0
    I, gf = _out(tmp_path, "I", F.shape), _out(tmp_path, "gf", F.shape)
    for b in range(B):
        nb = NPH[b] if per_batch else NPH
        assert nerr(I[b], oracle.collision(s, F[b], nb)) <= 1e-10
        assert nerr(gf[b], oracle.collision_vjp(s, F[b], nb, L[b])[0]) <= 1e-10


@pytest.mark.gpu
@pytest.mark.parametrize("B,per_batch", [(2, 0), (5, 0), (4, 1)])
def test_capture_after_a_single_vector_gpu(B, per_batch):
    import torch

    import paper_2511_03683_amd as E
    s, F, NPH, L = system_and_inputs(B, per_batch)
    d = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda:0")
    plan = E.build_channels(s, device=0)
    f, N, lam = d(F), d(NPH), d(L)
    out = torch.empty_like(f)
    n0 = N[0] if per_batch else N
    E.collision_integral(plan, f[0], n0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        E.collision_integral(plan, f, N, out=out)
    for k in range(3):
        f.copy_(d(F * (1.0 - 0.1 * k)))
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        for b in range(B):
            assert nerr(got[b], oracle.collision(s, F[b] * (1.0 - 0.1 * k), NPH[b] if per_batch else NPH)) <= 1e-10
    del g
    plan.close()


def islands(n_islands, per, kn, n_modes):
    """Components of `per` states each (all pairs), interleaved in the caller's order."""
    s = full_system(2, kn, n_modes=n_modes)
    S = n_islands * per
    rng = np.random.default_rng(8)
    s.state_k = rng.choice(kn ** 3, size=S, replace=False).astype(np.int32)
    s.state_band = np.zeros(S, np.int8)
    s.eps = rng.uniform(0.0, 0.3, S)
    a, b = np.triu_indices(per, 1)
    i = (a[None, :] * n_islands + np.arange(n_islands)[:, None]).ravel()
    j = (b[None, :] * n_islands + np.arange(n_islands)[:, None]).ravel()
    s.ch_i = np.repeat(i, n_modes).astype(np.int32)
    s.ch_j = np.repeat(j, n_modes).astype(np.int32)
    s.ch_nu = np.tile(np.arange(n_modes), i.size).astype(np.int8)
    s.g2 = rng.uniform(1e-4, 2e-3, s.ch_i.size)
    return s


@pytest.mark.parametrize("room", [0.0, 1.2e6, 1.45e6])
def test_transport_without_room_for_the_matrix(driver, tmp_path, room):  # noqa: F811
    """2112 states in 66 components: the matrix takes 1.08 MB and its partials 0.36, the
    pass over entries 0.52 and both 0.4 for the iterates; with 1.2 MB or 1.45 there is room
    for the latter once the matrix is given back (0: no limit, over the matrix)."""
    s = islands(66, 32, 13, 1)
    S = s.n_states
    rng = np.random.default_rng(10)
    f0, vel, nph = rng.uniform(0.05, 0.4, S), rng.normal(size=(S, 3)), s.nph(300.0)
    _write(tmp_path, s, f=f0, vel=vel, nph=nph, T=300.0, tol=0.0, max_iter=2, room=room)
    _run(driver, tmp_path, "transport")
    want = oracle.transport_solve(s, f0, vel, 300.0, nph, max_iter=2, stop_on_tol=False)
    assert nerr(_out(tmp_path, "mob", (3, 3)), want["mu"]) <= 1e-10
    assert nerr(_out(tmp_path, "x", (S, 3)), want["x"]) <= 1e-10
