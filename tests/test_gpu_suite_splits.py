"""The suite kernels on the tiles and splits that larger grids choose, against
the FP64 oracle: strip and tile edges in x, short and long chunks, the
matrix-core 2D box of radius 4, and the points an infinity reaches.  Bars: the
suite's (see test_gpu_suite)."""

import numpy as np
import pytest

import oracle
import synth
from tests.test_gpu_suite import _bound, _run

pytestmark = pytest.mark.gpu


# 2D: one strip and its neighbours (255..257, 512), rows in chunks of 1 to 6;
# 3D stars and the radius-1 box: 64-, 128- and 256-wide tiles
@pytest.mark.parametrize("name", ["star2d1r", "star2d2r", "star2d3r", "star2d4r", "box2d1r", "box2d3r"])
@pytest.mark.parametrize("shape", [(7, 255), (33, 256), (6, 257), (3, 513), (1500, 260), (9000, 300)])
def test_2d_strips(gpu_lib, name, shape):
    kind, ndim, r = synth.SUITE[name]
    w = synth.suite_weights(name, seed=3, signed=True)
    u = synth.uniform_field((1,) + shape, 5)
    frame = synth.uniform_field((1, shape[0] + 8, shape[1] + 8), 6)
    got, _ = _run(u, w, kind, ndim, flat=True, frame=frame)
    ref = oracle.stencil_general(u, w, ndim, frame=frame)
    assert np.all(np.abs(got - ref) <= _bound(u, w, ndim, frame=frame))


@pytest.mark.parametrize("name", ["star3d1r", "star3d2r", "star3d3r", "star3d4r", "box3d1r"])
@pytest.mark.parametrize("shape", [(5, 17, 65), (21, 95, 129), (64, 64, 300), (150, 200, 190), (40, 770, 1030)])
def test_3d_tiles(gpu_lib, name, shape):
    kind, ndim, r = synth.SUITE[name]
    w = synth.suite_weights(name, seed=4, signed=True)
    u = synth.uniform_field(shape, 7)
    got, _ = _run(u, w, kind, ndim)
    ref = oracle.stencil_general(u, w, ndim)
    assert np.all(np.abs(got - ref) <= _bound(u, w, ndim))


# planes of at least 50000 strip rows take the matrix kernel
@pytest.mark.parametrize("shape", [(1, 50001, 20), (1, 25003, 257), (700, 72, 255)])
def test_2d_box_radius_4_on_matrix_cores(gpu_lib, shape):
    w = synth.suite_weights("box2d4r", seed=5, signed=True)
    u = synth.uniform_field(shape, 8)
    got, _ = _run(u, w, "box", 2, flat=shape[0] == 1)
    ref = oracle.stencil_general(u, w, 2)
    assert np.all(np.abs(got - ref) <= _bound(u, w, 2))
    wi = np.random.default_rng(1).integers(-3, 4, w.shape).astype(np.float64)
    ui = np.random.default_rng(2).integers(-100, 101, shape).astype(np.float64)
    got, _ = _run(ui, wi, "box", 2, flat=shape[0] == 1)
    assert np.array_equal(got, oracle.stencil_general(ui, wi, 2))


@pytest.mark.parametrize("name,shape", [("star2d4r", (40, 600)), ("star2d1r", (40, 600)), ("box2d4r", (50010, 40))])
def test_infinity_reaches_its_stencil_only(gpu_lib, name, shape):
    kind, ndim, r = synth.SUITE[name]
    w = synth.suite_weights(name, seed=6)
    u = synth.uniform_field((1,) + shape, 9)
    ny, nx = shape
    hit = np.zeros((1, ny, nx), bool)
    for y, x in [(0, 0), (20, 31), (ny - 1, nx - 1)] + ([(20, 255), (30, 256)] if nx > 256 else []):
        u[0, y, x] = np.inf
        for dy in range(-r, r + 1):
            for dx in range(-r, r + 1):
                if (kind == "box" or dx == 0 or dy == 0) and 0 <= y + dy < ny and 0 <= x + dx < nx:
                    hit[0, y + dy, x + dx] = True
    got, _ = _run(u, w, kind, ndim, flat=True)
    assert np.array_equal(~np.isfinite(got), hit) and np.all(got[hit] == np.inf)
