"""GPU parity of the surrogate's batch reductions (bias and weight gradients) at their edges.

Each gradient is a sum over samples and positions, taken in two stages: chunks of samples per row (at most 64
of them, so 1, 9 and 130 samples are one, a few and a full set of uneven chunks) over rows read as 16-byte
groups (H W a multiple of four) or one by one (7 x 5).  With split bf16 products the kernels match the FP64
reference to 1e-4, the bound of the other split parity tests; the sums themselves are in double.
"""
import numpy as np
import pytest

import workloads
from oracle import nop as onop
from test_gpu_nop import _check_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 9, 130])
@pytest.mark.parametrize("H,W,channels,hidden", [(7, 5, 3, 33), (8, 12, 32, 16)])
def test_gradients_of_uneven_batches(H, W, channels, hidden, batch):
    from paper_2005_00322_amd.surrogate import Surrogate, SurrogateConfig, param_shapes

    print("batch gradients", H, W, channels, hidden, batch, flush=True)
    scfg = SurrogateConfig(H=H, W=W, channels=channels, modes=4, layers=1, hidden=hidden)
    ocfg = onop.Config(H=H, W=W, C=channels, Mm=4, layers=1, Hp=hidden)
    theta = workloads.nop_init(param_shapes(scfg), seed=3, gain=1.5).astype(np.float32)
    rng = np.random.default_rng(77 + batch)
    p0 = rng.standard_normal((batch, H, W)).astype(np.float32)
    c0 = (1400.0 + 200.0 * rng.random((batch, H, W))).astype(np.float32)
    tgt = rng.standard_normal((batch, H, W)).astype(np.float32)
    with Surrogate(scfg, max_batch=batch, split=True) as net:
        net.set_params(theta)
        _check_parity(net, ocfg, theta, p0, c0, tgt, True)
