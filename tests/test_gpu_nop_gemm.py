"""GPU parity of the surrogate's matrix products at the edges of their tiles and operand layouts.

Tiles of 64 x 64, of 32 x 256 (few rows, 256 columns or more) and of 32 x 32 with four waves along K (weight gradients); rows
that are contiguous in K with and without 16-byte alignment, or contiguous along the rows; a K of one value, one that
ends inside a slice and one of several slices.  With split bf16 products the kernels match the FP64 reference to 1e-4,
the bound of the other split parity tests.
"""
import numpy as np
import pytest

import workloads
from oracle import nop as onop
from test_gpu_nop import _check_parity

pytestmark = pytest.mark.gpu

CASES = [  # H, W, channels, modes, hidden, batch
    (9, 300, 5, 8, 33, 3), (64, 66, 32, 48, 40, 2), (150, 130, 4, 66, 16, 2), (37, 41, 8, 36, 100, 5), (300, 24, 32, 24, 8, 1),
]


@pytest.mark.parametrize("H,W,channels,modes,hidden,batch", CASES)
def test_products_match_the_reference(H, W, channels, modes, hidden, batch):
    from paper_2005_00322_amd.surrogate import Surrogate, SurrogateConfig, param_shapes

    print("products", H, W, channels, modes, hidden, batch, flush=True)
    scfg = SurrogateConfig(H=H, W=W, channels=channels, modes=modes, layers=2, hidden=hidden)
    ocfg = onop.Config(H=H, W=W, C=channels, Mm=modes, layers=2, Hp=hidden)
    theta = workloads.nop_init(param_shapes(scfg), seed=3, gain=1.5).astype(np.float32)
    rng = np.random.default_rng(H + W)
    p0 = rng.standard_normal((batch, H, W)).astype(np.float32)
    c0 = (1400.0 + 200.0 * rng.random((batch, H, W))).astype(np.float32)
    tgt = rng.standard_normal((batch, H, W)).astype(np.float32)
    with Surrogate(scfg, max_batch=batch, split=True) as net:
        net.set_params(theta)
        _check_parity(net, ocfg, theta, p0, c0, tgt, True)
