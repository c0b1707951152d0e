"""Dense contractions (FP32 and FP64) at the edges of their tiles, against the FP64 oracle.

Both tile sizes (64 x 64 from 512 of them on, 32 x 32 before), operator rows and lines that end inside a tile or a wave,
line lengths that end inside a slice or a chunk, columns of several outer blocks in one tile, maps, and every wall
family.  Tolerances are those of the other parity tests (FP64 1e-10, FP32 1e-5 relative L2).  Non-finite values may
reach only the lines they lie on: what a tile reads past a line's end belongs to other lines.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import TOL, oracle_problem, rel_l2, run_gpu

pytestmark = pytest.mark.gpu

N, D, P, NH, DH = 0, 1, 2, 3, 4
CASES = [
    ((3, 3, 3), ((N, D), (D, N), (N, N)), False), ((5, 300, 7), ((D, D), (N, D), (N, N)), True),
    ((65, 200, 170), ((N, N), (D, D), (D, N)), True), ((129, 97, 161), ((P, P), (N, DH), (D, NH)), False),
    ((34, 64, 66), ((N, D), (P, P), (D, D)), True), ((160, 33, 129), ((N, NH), (D, N), (P, P)), False),
    ((600, 70), ((N, D), (D, D)), True),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,bcs,with_map", CASES)
def test_contractions_match_oracle(shape, bcs, with_map, precision):
    print("contractions", shape, bcs, with_map, precision, flush=True)
    rng = np.random.default_rng(sum(shape))
    c0_map = (1400.0 + 200.0 * rng.random(shape)).astype(np.float32) if with_map else None
    c0 = 1500.0 if c0_map is None else float(c0_map.max())
    case = workloads.Case("contract", shape, bcs, workloads.DX, 0.25 * workloads.DX / c0, c0, 3,
                          rng.standard_normal(shape), c0_map=c0_map)
    p_ref, u_ref = oracle_problem(case).run(case.p0, case.steps)
    p, u = run_gpu(case, precision=precision, path="per_axis")
    assert rel_l2(p, p_ref) < TOL[precision]
    for a in range(len(shape)):
        assert rel_l2(u[a], u_ref[a]) < TOL[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(37, 50, 70), (70, 37, 50), (65, 200, 170)])
def test_non_finite_values_stay_on_their_lines(shape, precision):
    import torch
    from paper_2005_00322_amd import Plan

    print("non-finite", shape, precision, flush=True)
    with Plan(shape, workloads.DX, 0.2 * workloads.DX / 1500.0, 1500.0, ((N, N),) * 3, precision=precision) as plan:
        plan.set_path("per_axis")
        for axis in range(3):
            st = plan.new_state(np.ones(shape))
            at = [s // 2 for s in shape]
            at[axis] = 0                     # the first value of its line: the one behind another line's end
            st.p[tuple(at)] = float("nan")
            at2 = [s // 3 for s in shape]
            at2[axis] = shape[axis] - 1
            st.p[tuple(at2)] = float("inf")
            plan.apply_axis(st, axis, 0)
            torch.cuda.synchronize()
            bad = ~torch.isfinite(st.u[axis])
            lines = bad.any(dim=axis)
            want = torch.zeros_like(lines)
            for pos in (at, at2):
                want[tuple(v for i, v in enumerate(pos) if i != axis)] = True
            assert torch.equal(lines, want)
            for pos in (at, at2):            # and there every value is hit (no entry of these operators is zero)
                idx = [v for v in pos]
                idx[axis] = slice(None)
                assert bool(bad[tuple(idx)].all())
