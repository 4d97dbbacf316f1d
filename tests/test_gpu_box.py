"""The matrix-core box kernels (3D, radius 2..4) against the FP64 oracle at
the edges of their tiles and z-chunks, and the points an infinity or a NaN
reaches.

Bar: the suite's, |gpu - oracle| <= (n + 2) 2^-24 sum_k |w_k u(p+k)| with n
taps; the integer case is bit-exact (every partial sum below 2^24).
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.test_gpu_suite import _bound, _run

pytestmark = pytest.mark.gpu


# 64 x 32 tiles (x 63..65, y 31..33), 128 x 16 tiles (ny 16, x 127..129), one
# plane, fewer planes than the radius, many short chunks
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 32, 64), (2, 33, 65), (5, 31, 63), (4, 16, 128), (7, 17, 129),
                                   (6, 15, 127), (40, 9, 7), (33, 70, 200)])
@pytest.mark.parametrize("r", [2, 3, 4])
def test_box_at_tile_edges(gpu_lib, r, shape):
    name = "box3d%dr" % r
    rng = np.random.default_rng(17 * r + sum(shape))
    nz, ny, nx = shape
    w = synth.suite_weights(name, seed=r, signed=True)
    u = synth.uniform_field(shape, 5)
    frame = synth.uniform_field((nz + 8, ny + 8, nx + 8), 6)
    got, _ = _run(u, w, "box", 3, frame=frame)
    ref = oracle.stencil_general(u, w, 3, frame=frame)
    assert np.all(np.abs(got - ref) <= _bound(u, w, 3, frame=frame)), np.abs(got - ref).max()
    wi = rng.integers(-3, 4, w.shape).astype(np.float64)
    ui = rng.integers(-100, 101, shape).astype(np.float64)
    got, _ = _run(ui, wi, "box", 3)
    assert np.array_equal(got, oracle.stencil_general(ui, wi, 3))


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("r", [2, 3, 4])
def test_nonfinite_values_reach_their_box_only(gpu_lib, r, value):
    shape = (19, 37, 70)
    w = synth.suite_weights("box3d%dr" % r, seed=r)       # every weight positive
    u = synth.uniform_field(shape, 9)
    pts = [(0, 0, 0), (9, 31, 64), (18, 36, 69), (10, 12, 13)]
    hit = np.zeros(shape, bool)
    for z, y, x in pts:
        u[z, y, x] = value
        hit[max(0, z - r):z + r + 1, max(0, y - r):y + r + 1, max(0, x - r):x + r + 1] = True
    got, _ = _run(u, w, "box", 3)
    assert np.array_equal(~np.isfinite(got), hit)
    if np.isinf(value):
        assert np.all(got[hit] == value)
