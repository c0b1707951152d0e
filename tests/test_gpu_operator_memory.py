"""A plan holds each of its operators once: in fragment order, and for the 1D time loops also by rows and by columns."""
import ctypes

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _padded(rows, cols):
    return -(-rows // 128) * 128 * (-(-cols // 64) * 64)


@pytest.mark.parametrize("precision,size", [("fp32", 4), ("fp64", 8)])
@pytest.mark.parametrize("shape,copies", [((100,), 2), ((128,), 2), ((129,), 3), ((1000,), 3), ((300, 241), 1), ((40, 65, 33), 1)])
def test_operators_are_kept_once(shape, copies, precision, size):
    import torch  # noqa: F401  (its HIP runtime is the one that the library has to find)
    from paper_2005_00322_amd import Plan, axis_operator, load_library

    lib = load_library()
    lib.pstd_test_operator_bytes.restype = ctypes.c_int64
    lib.pstd_test_operator_bytes.argtypes = [ctypes.c_void_p]
    print("operator memory", shape, precision, flush=True)
    dt = 0.2 * workloads.DX / 1500.0
    with Plan(shape, workloads.DX, dt, 1500.0, ((0, 1),) * len(shape), precision=precision) as plan:
        assert lib.pstd_test_operator_bytes(plan._h) == copies * size * sum(_padded(n - 1, n) + _padded(n, n - 1) for n in shape)
        for a, n in enumerate(shape):      # and they read back as they were formed
            for which, c in ((0, -dt / 1000.0), (1, -dt * 1000.0 * 1500.0 ** 2)):
                want = c * axis_operator(n, 0, 1, workloads.DX, which)
                got = plan.operator(a, which)
                assert np.abs(got - want).max() <= (1e-15 if size == 8 else 1e-7) * np.abs(want).max()


def test_split_operators_are_kept_once():
    """Also those whose entries are sums of two parts (193 .. 384 rows); path "stored" adds the entries rounded from FP64."""
    import torch
    from paper_2005_00322_amd import STAG_TO_NODES, Plan, load_library

    lib = load_library()
    lib.pstd_test_operator_bytes.restype = ctypes.c_int64
    lib.pstd_test_operator_bytes.argtypes = [ctypes.c_void_p]
    shape = (193, 300, 60)
    print("operator memory", shape, "split", flush=True)
    with Plan(shape, workloads.DX, 0.2 * workloads.DX / 1500.0, 1500.0, ((0, 1), (1, 1), (0, 0)), precision="split_bf16") as plan:
        size = [4 * (_padded(n - 1, n), _padded(n, n - 1))[w] for n in shape for w in (0, 1)]
        held = lambda: lib.pstd_test_operator_bytes(plan._h)  # noqa: E731
        assert held() == sum(size)
        plan.apply_operator(1, STAG_TO_NODES, torch.zeros((193, 299, 60), device=plan.device))
        assert held() == sum(size) + size[3]
        before = [plan.operator(a, w) for a in range(3) for w in (0, 1)]
        plan.set_path("stored")
        # formed: 193 rows of axis 0, both operators of axis 1 and the interpolation
        assert held() == sum(size) + size[1] + size[2] + 3 * size[3]
        for got, want in zip([plan.operator(a, w) for a in range(3) for w in (0, 1)], before):
            assert np.array_equal(got, want)
