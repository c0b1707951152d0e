"""GPU parity of the surrogate's channel mixing of the modes (and its adjoint) at the edges of its blocks.

Four samples, a pair of kh and up to 48 kw per block: one to three uneven chunks of kw, sample counts that do not fill a
block, fewer channels than the 32 a block holds, the smallest number of modes.  With split bf16 products outputs and
gradients match the FP64 reference to 1e-4, the bound of the other split parity tests.
"""
import numpy as np
import pytest

import workloads
from oracle import nop as onop
from test_gpu_nop import _check_parity

pytestmark = pytest.mark.gpu

CASES = [(60, 56, 32, 50, 5), (40, 40, 7, 2, 3), (128, 100, 32, 96, 1), (20, 20, 16, 20, 9), (110, 108, 5, 98, 2)]


@pytest.mark.parametrize("H,W,channels,modes,batch", CASES)
def test_mode_mixing_matches_the_reference(H, W, channels, modes, batch):
    from paper_2005_00322_amd.surrogate import Surrogate, SurrogateConfig, param_shapes

    print("mode mixing", H, W, channels, modes, batch, flush=True)
    scfg = SurrogateConfig(H=H, W=W, channels=channels, modes=modes, layers=2, hidden=24)
    ocfg = onop.Config(H=H, W=W, C=channels, Mm=modes, layers=2, Hp=24)
    theta = workloads.nop_init(param_shapes(scfg), seed=9, gain=1.5).astype(np.float32)
    rng = np.random.default_rng(H + W + modes)
    p0 = rng.standard_normal((batch, H, W)).astype(np.float32)
    c0 = (1400.0 + 200.0 * rng.random((batch, H, W))).astype(np.float32)
    tgt = rng.standard_normal((batch, H, W)).astype(np.float32)
    with Surrogate(scfg, max_batch=batch, split=True) as net:
        net.set_params(theta)
        _check_parity(net, ocfg, theta, p0, c0, tgt, True)
