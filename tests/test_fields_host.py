"""Field.interior() is the interior of padded(): same elements, shape and
strides, on every storage type, 3D and 2D grids (CPU buffers)."""

import pytest
import torch

from paper_2309_04671_amd import fields, lib


@pytest.mark.parametrize("dtype", [lib.SP_F32, lib.SP_F16, lib.SP_BF16])
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 3, 2), (33, 32, 31), (70, 9, 4)])
def test_interior_is_the_padded_views_middle(dtype, shape):
    f = fields.Field(lib.grid_init(*shape, dtype), device="cpu")
    f.padded().copy_(torch.arange(f.padded().numel()).reshape(f.padded().shape) % 997)
    want = f.padded()[4:-4, 4:-4, 4:-4]
    got = f.interior()
    assert got.shape == want.shape and got.stride() == want.stride()
    assert got.data_ptr() == want.data_ptr() and torch.equal(got, want)


def test_interior_of_a_2d_grid():
    f = fields.Field(lib.grid_init_2d(37, 21), device="cpu")
    want = f.padded()[0:1, 4:-4, 4:-4]
    got = f.interior()
    assert got.shape == want.shape == (1, 21, 37) and got.data_ptr() == want.data_ptr()
    assert got.stride()[1:] == want.stride()[1:]
