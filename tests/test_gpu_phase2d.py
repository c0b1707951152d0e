"""The fused 2D phases (FP32 and FP64) against the FP64 oracle at the edges of their tiles.

Both tile edges (16 up to 512 tiles, 32 beyond), one to eight chunks of k per wave, shares that end inside a
round, odd rows, and the smallest boxes; walls on nodes, half-step walls and periodic axes, with and without a
sound-speed map, through a plan and (walls on nodes) through a batch of one shape.  Tolerances are those of the
other parity tests (FP64 1e-10, FP32 1e-5 relative L2).
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import TOL, oracle_problem, rel_l2, run_gpu

pytestmark = pytest.mark.gpu

N, D, P, NH, DH = 0, 1, 2, 3, 4
CASES = [
    ((3, 3), ((N, D), (D, N)), False), ((16, 17), ((D, D), (N, N)), True), ((33, 64), ((N, NH), (P, P)), False),
    ((65, 129), ((N, N), (D, N)), True), ((130, 255), ((P, P), (D, DH)), True), ((256, 512), ((D, N), (N, N)), False),
    ((369, 352), ((N, N), (D, D)), True), ((321, 449), ((N, DH), (P, P)), False), ((512, 511), ((D, D), (N, D)), True),
]


def _case(shape, bcs, with_map):
    rng = np.random.default_rng(shape[0] * 1000 + shape[1])
    c0_map = (1400.0 + 200.0 * rng.random(shape)).astype(np.float32) if with_map else None
    c0 = 1500.0 if c0_map is None else float(c0_map.max())
    return workloads.Case("phase_%dx%d" % shape, shape, bcs, workloads.DX, 0.25 * workloads.DX / c0, c0, 6,
                          rng.standard_normal(shape), c0_map=c0_map)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,bcs,with_map", CASES)
def test_phases_match_oracle(shape, bcs, with_map, precision):
    print("phases", shape, bcs, with_map, precision, flush=True)
    case = _case(shape, bcs, with_map)
    p_ref, u_ref = oracle_problem(case).run(case.p0, case.steps)
    p, u = run_gpu(case, precision=precision)
    assert rel_l2(p, p_ref) < TOL[precision]
    for a in range(2):
        assert rel_l2(u[a], u_ref[a]) < TOL[precision]


@pytest.mark.parametrize("shape,count", [((3, 3), 2), ((47, 90), 5), ((130, 257), 3), ((512, 64), 9)])
def test_phases_of_a_batch_match_oracle(shape, count):
    import torch
    from paper_2005_00322_amd import Batch

    print("batch phases", shape, count, flush=True)
    rng = np.random.default_rng(shape[0] + shape[1])
    walls = [((int(a), int(b)), (int(c), int(d))) for a, b, c, d in rng.integers(0, 2, (count, 4))]
    c0s = rng.uniform(1400.0, 1600.0, count)
    p0s = rng.standard_normal((count,) + shape)
    b = Batch([{"shape": shape, "bcs": w, "dx": workloads.DX, "dt": 0.25 * workloads.DX / c, "c0": float(c)}
               for w, c in zip(walls, c0s)])
    b.set_config(tile=16)
    st = b.new_states(list(p0s))
    for x in st:                    # the start of a solve must not depend on what the velocity buffers held
        for v in x.u:
            v.fill_(float("nan"))
    b.init_states(st)
    b.step(st, 6)
    torch.cuda.synchronize()
    for i in range(count):
        case = workloads.Case("b%d" % i, shape, walls[i], workloads.DX, 0.25 * workloads.DX / c0s[i], float(c0s[i]), 6,
                              p0s[i])
        p_ref, u_ref = oracle_problem(case).run(p0s[i], 6)
        assert rel_l2(st[i].p.double().cpu().numpy(), p_ref) < TOL["fp32"]
        for a in range(2):
            assert rel_l2(st[i].u[a].double().cpu().numpy(), u_ref[a]) < TOL["fp32"]
    b.close()
