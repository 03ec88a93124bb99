"""The transport iteration of FP32 plans against recorded values: the mobility is an
FP64 output of FP32 plans too, so the FP32 sums behind it are part of the results.
Equalities (mobility, iterations, last iterate)."""
import hashlib
import json
import os

import numpy as np
import pytest

from test_fp32_phonon_adjoint import golden_case

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "transport_f32.json")


def golden_run(E, n_modes):
    import torch
    s, x = golden_case(n_modes)
    rng = np.random.Generator(np.random.Philox(2000 + n_modes))
    vel = rng.uniform(-1e5, 1e5, (s.n_states, 3))
    d = lambda a: torch.as_tensor(a.astype(np.float32), device="cuda:0")
    plan = E.build_channels(s, dtype="f32", device=0)
    r = E.iterate_transport(plan, d(0.2 * x["f"]), d(vel), 300.0, d(x["N"]), tol=1e-8, max_iter=60, want_x=True)
    plan.close()
    return dict(mu=[float(v).hex() for v in np.asarray(r["mu"]).ravel()], iters=int(r["iters"]),
                x=hashlib.sha256(np.ascontiguousarray(r["x"].cpu().numpy()).tobytes()).hexdigest())


@pytest.mark.gpu
@pytest.mark.parametrize("n_modes", [1, 3, 4, 6, 8])
def test_mobility_keeps_its_values(n_modes):
    pytest.importorskip("torch")
    import paper_2511_03683_amd as E
    with open(GOLDEN) as fh:
        ref = json.load(fh)[str(n_modes)]
    assert golden_run(E, n_modes) == ref
