"""Single steps of 1D lines of 129 .. 161 nodes (one launch up to 160) equal the same steps of one call, bit for bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [129, 144, 159, 160, 161])
def test_single_steps_equal_one_call(n, precision):
    import torch
    from paper_2005_00322_amd import Plan

    print("line steps", n, precision, flush=True)
    rng = np.random.default_rng(n)
    for with_map, walls in ((False, (0, 1)), (True, (1, 0))):
        c0_map = (1400.0 + 200.0 * rng.random(n)).astype(np.float32) if with_map else None
        c0 = float(c0_map.max()) if with_map else 1500.0
        with Plan((n,), workloads.DX, 0.4 * workloads.DX / c0, c0, (walls,), precision=precision, c0_map=c0_map) as plan:
            p0 = rng.standard_normal(n)
            one, many = plan.init_state(plan.new_state(p0)), plan.init_state(plan.new_state(p0))
            for _ in range(7):
                plan.step(one, 1)
            plan.step(many, 7)
            torch.cuda.synchronize()
            assert torch.equal(one.p, many.p) and torch.equal(one.u[0], many.u[0])
