"""Receivers recorded by the sweeps' own further blocks: one call of several
steps gives bit for bit the traces of one call per step (which records with a
launch of its own), for receiver counts at the edges of a record block."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

NX, NY, NZ, STEPS = 70, 37, 33, 5
COUNTS = [1, 255, 256, 257, 700]


def _receivers(n):
    r = np.random.default_rng(n)
    # some outside the interior (recorded as zero), some doubled
    p = np.stack([r.integers(-2, NX + 2, n), r.integers(-2, NY + 2, n), r.integers(-2, NZ + 2, n)], 1)
    p[n // 2] = p[0]
    return torch.tensor(p.astype(np.int32), device="cuda")


def _run(entry, dtype, nrec, per_call):
    from paper_2309_04671_amd import fields, lib
    p = synth.wave_problem(NX, NY, NZ, STEPS)
    gv = lib.grid_init(NX, NY, NZ)
    g = lib.grid_init(NX, NY, NZ, dtype)
    V = fields.Field(gv).set_interior(p["v"])
    ws = fields.WaveState(g)
    if dtype == 0:
        ws.cur().set_interior(synth.uniform_field((NZ, NY, NX), 3))
        ws.prev().set_interior(synth.uniform_field((NZ, NY, NX), 4))
    amp = torch.tensor(1e3 * (1.0 + np.arange(STEPS))[:, None], dtype=torch.float32, device="cuda")
    src = lib.make_sources(p["src"], amp.data_ptr(), 1)
    co = lib.coeffs(synth.star25_coeffs())
    rec_d = _receivers(nrec)
    tr = torch.full((STEPS, nrec + 3), -5.0, device="cuda")      # a row stride wider than the row
    E, PSI = fields.Field(gv), fields.Field(gv)
    if entry.startswith("pml"):
        lib.sp_pml_profile(gv, 4, synth.pml_eta_max(4500.0, 4, 10.0), E.ptr)
    states = [ws.prev().ptr, ws.cur().ptr] + [f.ptr for f in (fields.Field(g) for _ in range(STEPS))]
    keep = [fields.Field(g) for _ in range(STEPS)]
    states[2:] = [f.ptr for f in keep]
    n = 0
    while n < STEPS:
        k = min(per_call, STEPS - n)
        rec = lib.make_receivers(nrec, rec_d.data_ptr(), tr[n:].data_ptr(), nrec + 3)
        if entry == "wave":
            lib.sp_wave_step(g, co, p["dt"], p["dx"], gv, V.ptr, ws.st, k, src=src, rec=rec)
        elif entry == "states":
            lib.sp_wave_run_states(g, co, p["dt"], p["dx"], gv, V.ptr, states[n:n + k + 2], n, k, src=src, rec=rec)
        else:
            pml = lib.make_pml(4, E.ptr, PSI.ptr, 47.0, int(entry[3:]))
            lib.sp_wave_step_pml(g, co, p["dt"], p["dx"], gv, V.ptr, ws.st, k, pml, src=src, rec=rec)
        n += k
    torch.cuda.synchronize()
    assert torch.all(tr[:, nrec:] == -5.0)
    return tr[:, :nrec].clone()


@pytest.mark.parametrize("nrec", COUNTS)
@pytest.mark.parametrize("entry,dtype", [("wave", 0), ("wave", 1), ("wave", 2), ("states", 0), ("pml0", 0),
                                         ("pml1", 0), ("pml2", 0)])
def test_traces_of_one_call_equal_those_of_single_steps(gpu_lib, entry, dtype, nrec):
    one = _run(entry, dtype, nrec, 1)
    assert float(one.abs().max()) > 0
    for per_call in (2, STEPS):
        assert torch.equal(_run(entry, dtype, nrec, per_call), one)


@pytest.mark.parametrize("nrec", COUNTS)
def test_queued_traces_equal_a_direct_run(gpu_lib, nrec):
    from paper_2309_04671_amd import fields, lib, serve
    p = synth.wave_problem(NX, NY, NZ, 7)
    co = synth.star25_coeffs()
    rec = _receivers(nrec).cpu().numpy()
    for chunk in (1, 3, 16):
        cl = serve.ServeClient(arena_bytes=256 << 20, chunk_steps=chunk)
        shots = [serve.Shot(p["v"], p["dt"], p["dx"], 7, co, p["src"], p["amp"], rec=rec, dtype=d) for d in (0, 1)]
        for s in shots:
            cl.submit(s)
        cl.drain()
        cl.close()
        for s, d in zip(shots, (0, 1)):
            gv, g = lib.grid_init(NX, NY, NZ), lib.grid_init(NX, NY, NZ, d)
            V = fields.Field(gv).set_interior(p["v"])
            ws = fields.WaveState(g)
            tr = torch.zeros((7, nrec), device="cuda")
            for n in range(7):
                r = lib.make_receivers(nrec, s.rec_d.data_ptr(), tr[n:].data_ptr(), nrec)
                lib.sp_wave_step(g, lib.coeffs(co), p["dt"], p["dx"], gv, V.ptr, ws.st, 1,
                                 src=lib.make_sources(p["src"], s.amp.data_ptr(), 1), rec=r)
            torch.cuda.synchronize()
            assert torch.equal(s.traces, tr)
