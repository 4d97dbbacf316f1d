"""The two-region layer's small-tile shell (64x16 and 32x32 tiles of 4- and
3-plane blocks) against the seven-region map, which runs the same arithmetic
per point in seven launches: equal bit for bit, on layers at the width from
which the small tiles run, x slabs a column past a tile, and slabs that end
inside a block."""

import numpy as np
import pytest

from tests.test_gpu_pml import _multi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(52, 50, 51, 24), (61, 63, 66, 28), (68, 67, 131, 32), (163, 80, 70, 32),
                                   (69, 145, 97, 32), (77, 75, 79, 36), (64, 64, 64, 20)])
def test_small_shell_equals_the_seven_region_map(gpu_lib, shape):
    nx, ny, nz, W = shape
    _, u7, p7, t7 = _multi(1, nx, ny, nz, W, 12)
    _, u2, p2, t2 = _multi(2, nx, ny, nz, W, 12)
    assert np.array_equal(u2, u7) and np.array_equal(p2, p7) and np.array_equal(t2, t7)
    assert np.isfinite(u2).all() and np.abs(u2).max() > 0 and np.abs(p2).max() > 0
