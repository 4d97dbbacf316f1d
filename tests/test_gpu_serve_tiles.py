"""Shots that share a launch on a tile and z-split chosen for all of them:
traces and final fields equal, bit for bit, the ones that each has alone (on
its own tile and split) -- tiny batches on one-plane chunks, narrow and wide
grids in one launch, and a grid deep enough to keep a launch of its own next
to small ones."""

import numpy as np
import pytest

from tests.test_gpu_serve import _run

pytestmark = pytest.mark.gpu

MIXES = {"tiny": [(10, 9, 11, 0), (70, 17, 9, 0), (12, 30, 25, 0)],
         "ragged": [(250, 33, 60, 0), (60, 130, 41, 0), (129, 65, 90, 0), (257, 16, 33, 0)],
         "fp16": [(118, 61, 53, 1), (74, 46, 90, 1), (200, 20, 35, 1)],
         "bf16": [(65, 17, 33, 2), (130, 70, 21, 2)],
         "deep": [(512, 256, 400, 0), (40, 40, 40, 0), (90, 33, 50, 0), (64, 64, 64, 1)]}


@pytest.mark.parametrize("mix", sorted(MIXES))
def test_shared_launch_equals_lone_runs(gpu_lib, mix):
    from paper_2309_04671_amd import lib, serve
    specs = [s + (7 + 2 * i,) for i, s in enumerate(MIXES[mix])]
    _, together = _run(serve, lib, specs, slots=8, chunk=4)
    _, alone = _run(serve, lib, specs, slots=1, chunk=4)
    for k, (a, b) in enumerate(zip(together, alone)):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (mix, k, specs[k])
        assert np.isfinite(a[1]).all()
