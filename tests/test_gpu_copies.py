"""The row copies (sp_decode, sp_grad_finish) at the edges of their 8-row
blocks and 64-lane segments, and the energy's sum over many partials."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (2, 7, 63), (3, 8, 64), (17, 9, 65), (33, 40, 257), (2, 3, 300)]


@pytest.mark.parametrize("dtype", [0, 1, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_decode_is_stored_value_times_slab_scale(gpu_lib, shape, dtype):
    from paper_2309_04671_amd import fields, lib
    nz, ny, nx = shape
    g = lib.grid_init(nx, ny, nz, dtype)
    ws = fields.WaveState(g)
    ws.cur().set_padded(torch.tensor(synth.uniform_field((nz + 8, ny + 8, nx + 8), 3) * 1000.0, device="cuda"))
    scale = 2.0 ** torch.arange(ws.nslab, device="cuda", dtype=torch.float32)
    if dtype:
        ws.slot(5)[0].copy_(scale)
    # one float before and after the output stays as it is
    buf = torch.full((nz * ny * nx + 2,), -7.0, device="cuda")
    lib.sp_decode(g, ws.cur().ptr, ws.meta.data_ptr() if dtype else None, 5, buf[1:].data_ptr())
    want = ws.cur().interior().float()
    if dtype:
        want = want * scale.repeat_interleave(16)[:nz].view(nz, 1, 1)
    assert torch.equal(buf[1:-1].view(nz, ny, nx), want)
    assert float(buf[0]) == -7.0 and float(buf[-1]) == -7.0


@pytest.mark.parametrize("shape", SHAPES)
def test_grad_finish_interior_only(gpu_lib, shape):
    from paper_2309_04671_amd import fields, lib
    nz, ny, nx = shape
    g = lib.grid_init(nx, ny, nz)
    rng = np.random.default_rng(1)
    V = fields.Field(g).set_interior(rng.uniform(1500, 4500, shape).astype(np.float32))
    G = torch.tensor(rng.normal(size=int(g.elems)), device="cuda")
    out = fields.Field(g)
    lib.sp_grad_finish(g, V.ptr, G.data_ptr(), out.ptr)
    sy, sz = g.pitch_x, g.pitch_x * g.pitch_y
    gi = torch.as_strided(G, shape, (sz, sy, 1), g.origin)
    assert torch.equal(out.interior(), (2.0 * gi / V.interior().double()).float())
    assert int(torch.count_nonzero(out.buf.view(torch.float32))) == int(torch.count_nonzero(out.interior()))


@pytest.mark.parametrize("zc", [40, 7, 1])
def test_energy_over_many_partials(gpu_lib, zc, monkeypatch):
    # 39 tiles x 1, 6 or 40 chunks: fewer and more partials than the sum's 512 threads
    import oracle
    from paper_2309_04671_amd import fields, lib
    monkeypatch.setenv("SP_TILE", "64x16x1x%d" % zc)
    nz, ny, nx = 40, 200, 130
    p = synth.wave_problem(nx, ny, nz, 1)
    g = lib.grid_init(nx, ny, nz)
    u0, u1 = synth.uniform_field((nz, ny, nx), 1), synth.uniform_field((nz, ny, nx), 2)
    V, F0, F1 = (fields.Field(g).set_interior(a) for a in (p["v"], u0, u1))
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    ws = torch.full((int(lib.load().sp_energy_ws_bytes(g)) // 8,), float("nan"), dtype=torch.float64, device="cuda")
    co = synth.star25_coeffs()
    lib.sp_energy(g, lib.coeffs(co), p["dt"], p["dx"], g, V.ptr, F0.ptr, F1.ptr, out.data_ptr(), ws.data_ptr())
    ref = oracle.energy(co, p["v"], p["dt"], p["dx"], oracle.padded(u0), oracle.padded(u1))
    assert abs(float(out) - ref) <= 1e-6 * abs(ref)       # the energy's bar against the oracle
