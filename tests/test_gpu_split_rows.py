"""Split-bf16 contractions whose operator has several row tiles over many lines, against the FP64 oracle.

Axes whose row blocks do not divide evenly among the tiles of up to twelve (25 and 37 of them here), in both layouts, with
enough lines that the tiles stay that long.  Every output row has to be written: the start from rest and the resampling
write into fields of NaN.  Tolerance as in the other split-bf16 tests.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import oracle_problem, rel_l2
from test_gpu_split import TOLERANCE

pytestmark = pytest.mark.gpu

N, D = 0, 1


@pytest.mark.parametrize("shape", [(780, 74, 74), (74, 74, 780), (3, 780, 1830), (1160, 70, 60)])
def test_every_row_is_computed(shape):
    import torch
    from oracle import pstd as opstd
    from paper_2005_00322_amd import STAG_TO_NODES, Plan

    print("split rows", shape, flush=True)
    rng = np.random.default_rng(sum(shape))
    bcs = ((N, D), (D, N), (N, N))
    case = workloads.Case("split_rows", shape, bcs, workloads.DX, 0.25 * workloads.DX / 1500.0, 1500.0, 2,
                          rng.standard_normal(shape), precision="split_bf16")
    p_ref, u_ref = oracle_problem(case).run(case.p0, case.steps)
    with Plan(shape, case.dx, case.dt, case.c0, bcs, precision="split_bf16") as plan:
        plan.set_path("per_axis")
        st = plan.new_state(case.p0)
        for u in st.u:
            u.fill_(float("nan"))
        plan.init_state(st)
        plan.step(st, case.steps)
        torch.cuda.synchronize()
        assert rel_l2(st.p.double().cpu().numpy(), p_ref) < TOLERANCE
        for a in range(3):
            assert rel_l2(st.u[a].double().cpu().numpy(), u_ref[a]) < TOLERANCE
        axis = int(np.argmax(shape))
        out = torch.full(shape, float("nan"), device=plan.device)
        plan.apply_operator(axis, STAG_TO_NODES, st.u[axis], out=out)
        torch.cuda.synchronize()
        A = opstd.make_axis(shape[axis], *bcs[axis], case.dx).resample_matrix(STAG_TO_NODES)
        x = np.moveaxis(st.u[axis].double().cpu().numpy(), axis, 0)
        want = np.moveaxis((A @ x.reshape(x.shape[0], -1)).reshape((A.shape[0],) + x.shape[1:]), 0, axis)
        assert rel_l2(out.double().cpu().numpy(), want) < TOLERANCE
