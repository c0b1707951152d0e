"""1D lines stepped by several workgroups (129 .. 1365 nodes, walls on nodes) against the FP64 oracle.

Sizes at the edges of the kernel's row blocks (16 rows per workgroup) and column tiers (256, 512, 768, 1024
nodes), and its fallback: with no polls allowed a workgroup gives up at the first value that is not there yet
and the steps run in one workgroup instead, from the untouched state.  Tolerances are the ones of the other
parity tests (FP64 1e-10, FP32 1e-5 relative L2).
"""
import ctypes

import numpy as np
import pytest

import workloads
from gpu_helpers import TOL, oracle_problem, rel_l2

pytestmark = pytest.mark.gpu

SIZES = (129, 144, 145, 256, 257, 512, 600, 769, 1024, 1025, 1365)


def _case(n, seed):
    rng = np.random.default_rng(4100 + 7 * n + seed)
    faces = rng.integers(0, 2, size=2)
    c0_map = (1400.0 + 200.0 * rng.random(n)).astype(np.float32) if seed % 2 else None
    c0 = 1500.0 if c0_map is None else float(c0_map.max())
    return workloads.Case("line_%d_%d" % (n, seed), (n,), ((int(faces[0]), int(faces[1])),), workloads.DX,
                          0.4 * workloads.DX / c0, c0, 30, rng.standard_normal(n), c0_map=c0_map)


@pytest.mark.parametrize("spins", [None, 0])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", SIZES)
def test_line_matches_oracle(n, precision, spins):
    import torch
    from paper_2005_00322_amd import Plan, load_library

    for seed in (0, 1):
        case = _case(n, seed)
        print("line", n, precision, "seed", seed, "spins", spins, flush=True)
        p_ref, u_ref = oracle_problem(case).run(case.p0, case.steps)
        with Plan(case.shape, case.dx, case.dt, case.c0, case.bcs, precision=precision, c0_map=case.c0_map) as plan:
            if spins is not None:
                assert load_library().pstd_test_line_spins(plan._h, ctypes.c_uint32(spins)) == 0
            st = plan.init_state(plan.new_state(case.p0))
            for k in (1, 9, case.steps - 10):     # several launches: the exchange's numbering goes on
                plan.step(st, k)
            torch.cuda.synchronize()
            assert rel_l2(st.p.double().cpu().numpy(), p_ref) < TOL[precision]
            assert rel_l2(st.u[0].double().cpu().numpy(), u_ref[0]) < TOL[precision]


def test_captured_line_steps_replay():
    """Replays of a captured step call continue the numbering kept on the device."""
    import torch
    from paper_2005_00322_amd import Plan

    case = _case(300, 0)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with Plan(case.shape, case.dx, case.dt, case.c0, case.bcs, precision="fp64", stream=s) as plan:
            st = plan.init_state(plan.new_state(case.p0))
            ref = plan.init_state(plan.new_state(case.p0))
            plan.step(st, 3)
            plan.step(ref, 3)
            s.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                plan.step(st, 5)
            for _ in range(4):
                g.replay()
                s.synchronize()
                plan.step(ref, 5)
                s.synchronize()
                assert torch.equal(st.p, ref.p) and torch.equal(st.u[0], ref.u[0])
