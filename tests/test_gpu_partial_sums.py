"""How far FP32 contractions sum in FP32 before they go on in FP64.

Two nodes of a line carry powers of two 2^14 apart (products with the operator's entries are exact), everything else is
zero, and the velocity starts at minus the larger product: what is left has to be the smaller product, exactly.  In one
FP32 sum with the larger one its low bits are lost, so the test fails where both nodes lie in one.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _residues(plan, axis, near, far, phase):
    """u + G p along `axis` with p = 2^14 at node `near`, 1 at `far`, u = -2^14 G[:, near]; and G[:, far]."""
    import torch

    G = torch.as_tensor(plan.operator(axis, 0)).to(plan.device, plan.dtype)
    st = plan.new_state()
    st.p.narrow(axis, near, 1).fill_(2.0 ** 14)
    st.p.narrow(axis, far, 1).fill_(1.0)
    line = [-1 if a == axis else 1 for a in range(plan.ndim)]
    st.u[axis].copy_((-2.0 ** 14 * G[:, near]).reshape(line).expand_as(st.u[axis]))
    plan.apply_axis(st, -1 if phase else axis, 0)
    torch.cuda.synchronize()
    return st.u[axis], G[:, far].reshape(line).expand_as(st.u[axis])


@pytest.mark.parametrize("phase", [False, True])
@pytest.mark.parametrize("shape", [(130, 21, 30), (30, 130, 21), (21, 30, 130), (130, 110, 100), (100, 130, 110), (110, 100, 130)])
def test_per_axis_contractions_sum_16_products(shape, phase):
    import torch
    from paper_2005_00322_amd import Plan

    print("partial sums", shape, phase, flush=True)
    axis = shape.index(130)
    with Plan(shape, workloads.DX, 0.2 * workloads.DX / 1500.0, 1500.0, ((0, 0),) * 3) as plan:
        plan.set_path("per_axis")
        for near, far in ((0, 16), (47, 48), (64, 95)):
            got, want = _residues(plan, axis, near, far, phase)
            assert torch.equal(got, want), (near, far)


@pytest.mark.parametrize("shape", [(200, 130), (130, 200), (512, 300), (300, 512), (400, 400)])
def test_fused_phases_sum_8_products(shape):
    import torch
    from paper_2005_00322_amd import Plan

    print("partial sums", shape, flush=True)
    with Plan(shape, workloads.DX, 0.2 * workloads.DX / 1500.0, 1500.0, ((0, 0),) * 2) as plan:
        plan.set_path("fused")
        for axis in range(2):
            for near, far in ((0, 8), (7, 15), (16, 25), (33, 56), (64, 72)):
                got, want = _residues(plan, axis, near, far, True)
                assert torch.equal(got, want), (axis, near, far)
