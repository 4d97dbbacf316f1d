"""The receiver term of the fused adjoint step (half a wave per receiver)
against the three-launch step, which has kernels of its own for it: odd and
even receiver counts, duplicates, points outside and on every face, a
receiver on a source."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrec", [1, 2, 3, 64, 65, 301])
def test_receiver_term_matches_the_separate_kernels(gpu_lib, nrec, monkeypatch):
    from paper_2309_04671_amd import fields, lib
    nx, ny, nz, steps = 40, 33, 29, 3
    p = synth.wave_problem(nx, ny, nz, steps)
    g = lib.grid_init(nx, ny, nz)
    V = fields.Field(g).set_interior(p["v"])
    r = np.random.default_rng(nrec)
    pts = np.stack([r.integers(-1, n + 1, nrec) for n in (nx, ny, nz)], 1).astype(np.int32)
    pts[0] = p["src"][0]
    if nrec > 64:
        pts[1:7] = [[0, 5, 6], [nx - 1, 5, 6], [7, 0, 6], [7, ny - 1, 6], [7, 5, 0], [7, 5, nz - 1]]
        pts[7] = pts[8] = pts[9]
    rec_d = torch.tensor(pts, device="cuda")
    res = torch.tensor(synth.uniform_field((1, steps, nrec), 3)[0], device="cuda")
    amp = torch.tensor(100.0 + np.arange(steps)[:, None], dtype=torch.float32, device="cuda")
    hist = [fields.Field(g).set_interior(synth.uniform_field((nz, ny, nx), 10 + i)) for i in range(steps)]

    def run(tile):
        monkeypatch.setenv("SP_TILE", tile)
        adj = fields.WaveState(g)
        adj.cur().set_interior(synth.uniform_field((nz, ny, nx), 5))
        adj.st.step = steps
        G = torch.zeros(int(g.elems), dtype=torch.float64, device="cuda")
        lib.sp_wave_adjoint_step(g, lib.coeffs(synth.star25_coeffs()), p["dt"], p["dx"], g, V.ptr, adj.st,
                                 [f.ptr for f in hist], steps, lib.make_sources(p["src"], amp.data_ptr(), 1),
                                 lib.make_receivers(nrec, rec_d.data_ptr(), res.data_ptr(), nrec), G.data_ptr())
        torch.cuda.synchronize()
        return adj.cur().interior().double().cpu().numpy(), G.cpu().numpy()

    (u, G), (u3, G3) = run("64x16x1"), run("256x16x2")     # fused; three launches
    # FP32 star sums of the same 25 terms in another order: a few ulps of the
    # largest term (|c0| max|u| |nu|), products and sums in FP64
    assert np.max(np.abs(u - u3)) <= 1e-5 * np.max(np.abs(u3))
    assert np.max(np.abs(G - G3)) <= 1e-5 * np.max(np.abs(G3))
