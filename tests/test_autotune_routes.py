"""The autotuner times the kernels whose knobs it sets: no call of it goes over the
pair matrix (which would leave the matrix, most of its workspace, with the plan)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from test_pair_matrix import dev, full_system, gross, host, nerr  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [2, 4, 7, 8])
def test_matrix_is_not_timed(batch):
    import paper_2511_03683_amd as E
    s = full_system(500, 8)
    matrix = 8 * 8 * 4096 * 8
    rng = np.random.default_rng(batch)
    F, nph = rng.uniform(size=(batch, 500)), s.nph(300.0)
    plan = E.build_channels(s, device=0)
    E.collision_integral(plan, dev(F[0]), dev(nph))
    b0 = E.plan_info(plan)["bytes"]
    E.autotune(plan, batch)
    assert E.plan_info(plan)["bytes"] - b0 < matrix
    got = host(E.collision_integral(plan, dev(F), dev(nph)))
    assert nerr(got[-1], oracle.collision(s, F[-1], nph), gross(s, F[-1], nph)) <= 1e-10
    if batch > 2:   # the call itself takes it
        assert E.plan_info(plan)["bytes"] - b0 >= matrix
    plan.close()
