"""GPU parity of the backward pass through the surrogate's hidden layer at its edges.

One pass over the pre-activations forms dq and sums the gradients of the hidden bias and the output weights over segments
of 4096 positions: one and more of them, a last one that is cut, rows read as 16-byte groups (H W a multiple of
four) or one by one, more hidden rows than a projection pass keeps in registers (128).  With split bf16 products the
gradients match the FP64 reference to 1e-4, the bound of the other split parity tests.
"""
import numpy as np
import pytest

import workloads
from oracle import nop as onop
from test_gpu_nop import _check_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,hidden,batch", [(67, 65, 33, 2), (64, 64, 17, 3), (96, 90, 160, 2)])
def test_hidden_layer_gradients(H, W, hidden, batch):
    from paper_2005_00322_amd.surrogate import Surrogate, SurrogateConfig, param_shapes

    print("hidden layer", H, W, hidden, batch, flush=True)
    scfg = SurrogateConfig(H=H, W=W, channels=6, modes=2, layers=1, hidden=hidden)
    ocfg = onop.Config(H=H, W=W, C=6, Mm=2, layers=1, Hp=hidden)
    theta = workloads.nop_init(param_shapes(scfg), seed=5, gain=1.5).astype(np.float32)
    rng = np.random.default_rng(H * W + hidden)
    p0 = rng.standard_normal((batch, H, W)).astype(np.float32)
    c0 = (1400.0 + 200.0 * rng.random((batch, H, W))).astype(np.float32)
    tgt = rng.standard_normal((batch, H, W)).astype(np.float32)
    with Surrogate(scfg, max_batch=batch, split=True) as net:
        net.set_params(theta)
        _check_parity(net, ocfg, theta, p0, c0, tgt, True)
