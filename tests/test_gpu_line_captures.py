"""Step calls of one 1D plan recorded into several graphs: replays on different streams are independent of each other."""
import ctypes

import numpy as np
import pytest

import workloads
from gpu_helpers import TOL, rel_l2

pytestmark = pytest.mark.gpu


def _graph(plan, stream, st, calls):
    import torch

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        for k in calls:
            plan.step(st, k)
    return g


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [300, 1025])
def test_overlapping_replays(n, precision):
    import torch
    from paper_2005_00322_amd import Plan, load_library

    lib = load_library()
    lib.pstd_test_line_captures.argtypes = [ctypes.c_void_p]
    print("line captures", n, precision, flush=True)
    rng = np.random.default_rng(n)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), Plan((n,), workloads.DX, 0.4 * workloads.DX / 1500.0, 1500.0, ((0, 1),), precision=precision,
                                    stream=s) as plan:
        p0 = [rng.standard_normal(n) for _ in range(3)]
        sts = [plan.init_state(plan.new_state(p)) for p in p0]
        refs = [plan.init_state(plan.new_state(p)) for p in p0]
        s.synchronize()
        graphs = [_graph(plan, s, sts[0], (20, 20)), _graph(plan, s, sts[1], (40,))]
        assert lib.pstd_test_line_captures(plan._h) == 2      # one workspace a capture, however many calls
        side = [torch.cuda.Stream(), torch.cuda.Stream()]
        for r in range(4):
            for g, q in zip(graphs, side):
                with torch.cuda.stream(q):
                    g.replay()
            plan.step(sts[2], 40)                              # and the plan's own calls beside them
            torch.cuda.synchronize()
            for st, ref in zip(sts, refs):
                plan.step(ref, 40)
                s.synchronize()
                assert torch.equal(st.p, ref.p) and torch.equal(st.u[0], ref.u[0]), r


def test_captures_beyond_the_workspaces():
    """The eighth capture and later ones step in one workgroup."""
    import torch
    from paper_2005_00322_amd import Plan, load_library

    lib = load_library()
    lib.pstd_test_line_captures.argtypes = [ctypes.c_void_p]
    rng = np.random.default_rng(5)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), Plan((200,), workloads.DX, 0.4 * workloads.DX / 1500.0, 1500.0, ((1, 1),), precision="fp64",
                                    stream=s) as plan:
        p0 = rng.standard_normal(200)
        ref = plan.init_state(plan.new_state(p0))
        plan.step(ref, 6)
        sts = [plan.init_state(plan.new_state(p0)) for _ in range(9)]
        s.synchronize()
        graphs = [_graph(plan, s, st, (6,)) for st in sts]
        assert lib.pstd_test_line_captures(plan._h) == 7
        for g in graphs:
            g.replay()
        torch.cuda.synchronize()
        want = ref.p.cpu().numpy()
        for st in sts:
            assert rel_l2(st.p.cpu().numpy(), want) < TOL["fp64"]
