"""GPU parity of the surrogate's row-walking channel mixing over the forms of its operand loads.

Modes that are a multiple of 8, of 4 and of 2 only (rows of T in 16-byte loads for bf16 and FP32 storage, for FP32 storage
only, in pairs of values), and channel counts up to 4, 16, 31 and all 32.  With split bf16 products outputs and gradients
match the FP64 reference to 1e-4, the bound of the other split parity tests; with plain products the inference form (bf16
storage) has to give the training form's bits (FP32 storage).
"""
import numpy as np
import pytest

import workloads
from oracle import nop as onop
from test_gpu_nop import _check_parity

pytestmark = pytest.mark.gpu

CASES = [(20, 24, 3, 8, 2), (22, 37, 16, 12, 3), (30, 130, 20, 22, 2), (26, 26, 32, 18, 3), (64, 70, 8, 60, 1)]


@pytest.mark.parametrize("H,W,channels,modes,batch", CASES)
def test_row_mixing_matches_the_reference(H, W, channels, modes, batch):
    import torch
    from paper_2005_00322_amd.surrogate import Surrogate, SurrogateConfig, param_shapes

    print("row mixing", H, W, channels, modes, batch, flush=True)
    scfg = SurrogateConfig(H=H, W=W, channels=channels, modes=modes, layers=2, hidden=24)
    ocfg = onop.Config(H=H, W=W, C=channels, Mm=modes, layers=2, Hp=24)
    theta = workloads.nop_init(param_shapes(scfg), seed=4, gain=1.5).astype(np.float32)
    rng = np.random.default_rng(H + W + channels)
    p0 = rng.standard_normal((batch, H, W)).astype(np.float32)
    c0 = (1400.0 + 200.0 * rng.random((batch, H, W))).astype(np.float32)
    tgt = rng.standard_normal((batch, H, W)).astype(np.float32)
    with Surrogate(scfg, max_batch=batch, split=True) as net:
        net.set_params(theta)
        _check_parity(net, ocfg, theta, p0, c0, tgt, True)
    with Surrogate(scfg, max_batch=batch, split=False) as net:
        net.set_params(theta)
        out = net.forward(p0, c0)
        assert torch.equal(net.infer(p0, c0), out)
