"""Batched steps with a limit on the blocks of a launch: the same results from fewer blocks, which therefore take longer."""
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _states(batch, solves):
    rng = np.random.default_rng(7)
    st = batch.new_states([rng.standard_normal(s["shape"]) for s in solves])
    batch.init_states(st)
    return st


def _solves(shapes):
    return [dict(shape=s, bcs=((0, 1), (1, 0)), dx=workloads.DX, dt=0.2 * workloads.DX / 1500.0, c0=1500.0) for s in shapes]


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("blocks", [1, 5, 8, 19, 40, 100000])
def test_limited_blocks_give_the_same_bits(blocks, tile):
    import torch
    from paper_2005_00322_amd import Batch

    print("batch blocks", blocks, tile, flush=True)
    solves = _solves([(40, 33), (130, 70), (64, 129), (17, 9)])
    with Batch(solves) as batch:
        got = []
        for b in (0, blocks):
            batch.set_config(blocks=b, tile=tile)
            st = _states(batch, solves)
            batch.step(st, 7)
            torch.cuda.synchronize()
            got.append([t.clone() for s in st for t in (s.p, s.u[0], s.u[1])])
        assert all(torch.equal(x, y) for x, y in zip(*got))


def test_the_limit_holds():
    """Eight blocks on 256 CUs: several times as long as one block per tile."""
    import torch
    from paper_2005_00322_amd import Batch

    solves = _solves([(256, 256)] * 16)
    with Batch(solves) as batch:
        times = []
        for b in (0, 8):
            batch.set_config(blocks=b, tile=64)
            st = _states(batch, solves)
            batch.step(st, 5)
            torch.cuda.synchronize()
            t = time.perf_counter()
            batch.step(st, 5)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
    assert times[1] > 4 * times[0], times
