"""Gradient from kept forward states against the checkpointed one.

Both run the same sweeps on the same states, so traces and gradient are equal
bit for bit; also where the memory is refused, on a second backward of one
graph, and without receivers or steps to keep.
"""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _run(n, steps, nrec, ckpt, twice=False):
    from paper_2309_04671_amd.adjoint import WaveOp, WaveProblem
    nx, ny, nz = n
    v = synth.layered_velocity(nx, ny, nz, 3)
    dt = synth.cfl_dt(v, 10.0)
    src = np.array([[nx // 2, ny // 2, nz // 2], [0, 0, 0]], np.int32)
    amp = (np.stack([synth.ricker(steps, dt, 40.0)] * 2, 1) * 1e4).astype(np.float32)
    rec = np.array([[(nx // 2 + 3 * i) % nx, (ny // 2 + i) % ny, nz // 2] for i in range(nrec)], np.int32)
    prob = WaveProblem(nx, ny, nz, synth.star25_coeffs(), dt, 10.0, steps, src, amp, rec.reshape(-1, 3), ckpt=ckpt)
    vt = torch.tensor(v, device="cuda", requires_grad=True)
    tr = WaveOp.apply(vt, prob)
    if not nrec:
        return prob, tr.detach(), None
    J = 0.5 * (tr * tr).sum()
    J.backward(retain_graph=twice)
    g = vt.grad.clone()
    if twice:
        vt.grad = None
        J.backward()
        assert torch.equal(vt.grad, g)
    return prob, tr.detach(), g


@pytest.mark.parametrize("n,steps,nrec", [((40, 24, 20), 1, 5), ((65, 17, 9), 2, 5), ((72, 33, 21), 23, 70),
                                          ((40, 24, 20), 6, 0)])
def test_kept_states_equal_checkpoints(gpu_lib, monkeypatch, n, steps, nrec):
    from paper_2309_04671_amd import adjoint
    kept = _run(n, steps, nrec, None, twice=True)
    assert kept[0].keep_all and kept[0].ckpt == max(1, int(np.ceil(np.sqrt(steps))))
    other = [_run(n, steps, nrec, max(1, int(np.ceil(np.sqrt(steps)))))]
    assert not other[0][0].keep_all
    monkeypatch.setattr(adjoint.WaveProblem, "kept_states", lambda self: (None, None))
    other.append(_run(n, steps, nrec, None))
    monkeypatch.setattr(adjoint, "KEEP_BYTES", 0)
    other.append(_run(n, steps, nrec, None))
    assert not other[2][0].keep_all
    for prob, tr, g in other:
        assert torch.equal(tr, kept[1])
        assert (g is None) == (kept[2] is None) and (g is None or torch.equal(g, kept[2]))
    assert nrec == 0 or float(kept[1].abs().max()) > 0 or steps == 1
