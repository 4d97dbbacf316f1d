"""The energy on the tiles that larger grids get against the 256x16x2 tiles
of smaller ones, at sizes around the rule's line (3 million points) and with
ragged edges.  The same FP64 terms are added in another order: n terms in
partial sums of at most 2^22 and then those, so the sums differ by less than
2^22 eps of the terms' absolute sum, which is at most 8 times the energy for
these states (kinetic term of unit-size differences over m < 1)."""

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(144, 144, 144), (145, 144, 144), (257, 131, 95), (65, 511, 129), (300, 90, 240)])
def test_energy_does_not_depend_on_the_tiles(gpu_lib, n, monkeypatch):
    from paper_2309_04671_amd import fields, lib
    nx, ny, nz = n
    g = lib.grid_init(nx, ny, nz)
    v = synth.layered_velocity(nx, ny, nz, 4)
    dx, dt = 10.0, synth.cfl_dt(v, 10.0)
    V = fields.Field(g).set_interior(v)
    A = fields.Field(g).set_interior(synth.uniform_field((nz, ny, nx), 5))
    B = fields.Field(g).set_interior(synth.uniform_field((nz, ny, nx), 6))
    ws = torch.empty(int(lib.load().sp_energy_ws_bytes(g)) // 8, dtype=torch.float64, device="cuda")
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    res = []
    for tile in (None, "256x16x2"):
        monkeypatch.setenv("SP_TILE", tile) if tile else monkeypatch.delenv("SP_TILE", raising=False)
        lib.sp_energy(g, lib.coeffs(synth.star25_coeffs()), dt, dx, g, V.ptr, A.ptr, B.ptr, out.data_ptr(),
                      ws.data_ptr())
        torch.cuda.synchronize()
        res.append(float(out[0]))
    assert res[0] > 0 and abs(res[0] - res[1]) <= 8 * 2 ** 22 * 2 ** -53 * res[1]
