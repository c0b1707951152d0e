"""Split-bf16 contractions at the edges of their tiles, against the FP64 oracle.

Operators of 1 to 12 blocks of 32 rows and beyond 384 rows (waves with three, two, one and no row block), row tiles of
128 rows where lines are few, lines that end inside a tile or a slice, columns of several outer blocks in one tile,
contiguous rows with and without 16-byte alignment, maps, and every wall family.  Non-finite values may reach only the
lines they lie on.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import oracle_problem, rel_l2, run_gpu

pytestmark = pytest.mark.gpu

# hi + lo hold 16 bits of each factor (2^-17 each) and the dropped product is at most 2^-18: 2e-5 a contraction, of
# which the three steps chain up to five (the last step's velocities) on values of one scale
TOLERANCE = 1e-4
N, D, P, NH, DH = 0, 1, 2, 3, 4
CASES = [
    ((3, 3, 3), ((N, D), (D, N), (N, N)), False), ((5, 300, 7), ((D, D), (N, D), (N, N)), True),
    ((33, 65, 97), ((P, P), (N, DH), (D, NH)), False), ((385, 150, 120), ((N, N), (D, D), (D, N)), True),
    ((384, 131, 129), ((N, D), (P, P), (D, D)), False), ((140, 128, 300), ((N, NH), (D, N), (P, P)), True),
    ((600, 70), ((N, D), (D, D)), True), ((257, 1000), ((P, P), (N, D)), False),
]


@pytest.mark.parametrize("shape,bcs,with_map", CASES)
def test_split_contractions_match_oracle(shape, bcs, with_map):
    print("split contractions", shape, bcs, with_map, flush=True)
    rng = np.random.default_rng(sum(shape))
    c0_map = (1400.0 + 200.0 * rng.random(shape)).astype(np.float32) if with_map else None
    c0 = 1500.0 if c0_map is None else float(c0_map.max())
    case = workloads.Case("split", shape, bcs, workloads.DX, 0.25 * workloads.DX / c0, c0, 3,
                          rng.standard_normal(shape), precision="split_bf16", c0_map=c0_map)
    p_ref, u_ref = oracle_problem(case).run(case.p0, case.steps)
    p, u = run_gpu(case, precision="split_bf16", path="per_axis")
    assert rel_l2(p, p_ref) < TOLERANCE
    for a in range(len(shape)):
        assert rel_l2(u[a], u_ref[a]) < TOLERANCE


@pytest.mark.parametrize("shape", [(37, 50, 70), (70, 37, 52), (385, 150, 120)])
def test_split_non_finite_values_stay_on_their_lines(shape):
    import torch
    from paper_2005_00322_amd import Plan

    print("split non-finite", shape, flush=True)
    with Plan(shape, workloads.DX, 0.2 * workloads.DX / 1500.0, 1500.0, ((N, N),) * 3, precision="split_bf16") as plan:
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
            lines = (~torch.isfinite(st.u[axis])).any(dim=axis)
            want = torch.zeros_like(lines)
            for pos in (at, at2):
                want[tuple(v for i, v in enumerate(pos) if i != axis)] = True
            assert torch.equal(lines, want)
