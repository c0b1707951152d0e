"""The autotuner's cache file: entries of other kernels, or of the same solves without their maps, are not taken."""
import json
import struct

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _fnv(data, h=1469598103934665603):
    for b in data:
        h = ((h ^ b) * 1099511628211) % (1 << 64)
    return h


def test_entries_of_other_kernels_and_media_are_not_taken(tmp_path):
    import torch
    from paper_2005_00322_amd import Batch

    shapes = [(40, 33), (52, 70), (64, 24)]
    solves = [dict(shape=s, bcs=((0, 1), (1, 0)), dx=workloads.DX, dt=0.2 * workloads.DX / 1600.0, c0=1600.0) for s in shapes]
    path = str(tmp_path / "tune.json")
    # an entry as the library's first batched kernels wrote it for these solves
    arch = torch.cuda.get_device_properties(0).gcnArchName.encode()
    ints = [len(shapes)] + [s[0] for s in shapes] + [s[1] for s in shapes] + [0, 1, 1, 0] * len(shapes)
    old = "%016x" % _fnv(struct.pack("<%di" % len(ints), *ints) + arch)
    with open(path, "w") as f:
        f.write(json.dumps({"signature": old, "blocks": 512, "order": 1, "tile": 64, "ms_per_step": 1.0}) + "\n")
    with Batch(solves) as b:
        assert not b.autotune(trial_steps=2, cache_path=path)["from_cache"]
        assert b.autotune(trial_steps=2, cache_path=path)["from_cache"]
        b.set_c0_maps([torch.full(shapes[0], 1500.0, device="cuda"), None, None])
        assert not b.autotune(trial_steps=2, cache_path=path)["from_cache"]
        assert b.autotune(trial_steps=2, cache_path=path)["from_cache"]
    assert np.isfinite(json.load(open(path))["ms_per_step"])
