"""Batches with new state buffers: starting and stepping them enqueues work and does not wait for the stream."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,tile", [(3, 16), (100, 16), (100, 32), (97, 64)])
def test_new_states_do_not_wait(count, tile):
    import torch
    from paper_2005_00322_amd import Batch

    print("batch states", count, tile, flush=True)
    rng = np.random.default_rng(count)
    dt = 0.2 * workloads.DX / 1600.0
    solves = [dict(shape=(40, 33), bcs=((i % 2, 0), (1, i // 2 % 2)), dx=workloads.DX, dt=dt, c0=1600.0) for i in range(count)]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), Batch(solves, stream=s) as batch:
        batch.set_config(tile=tile)
        p0 = [rng.standard_normal((40, 33)) for _ in range(count)]
        sets = [batch.new_states(p0) for _ in range(4)]

        def run(st):
            batch.init_states(st)
            batch.step(st, 3)

        run(sets[0])                          # loads the kernels and captures the steps
        batch.set_c0_maps([None if i % 3 else torch.full((40, 33), 1450.0 + i, device="cuda") for i in range(count)])
        s.synchronize()
        run(sets[1])
        s.synchronize()
        torch.cuda._sleep(500_000_000)        # work ahead of the calls, and its end
        ahead = torch.cuda.Event()
        ahead.record(s)
        for st in sets[2:]:
            run(st)
        assert not ahead.query()              # the calls came back before that
        s.synchronize()
        for st in sets[2:]:                   # and every set took its own steps
            for a, b in zip(st, sets[1]):
                assert torch.equal(a.p, b.p) and torch.equal(a.u[0], b.u[0]) and torch.equal(a.u[1], b.u[1])
        assert not torch.equal(sets[0][0].p, sets[1][0].p)
