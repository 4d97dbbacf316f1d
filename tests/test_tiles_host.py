"""The launch configuration a grid gets, without a GPU: every shape and
storage type has one that is compiled in for the direct call and for the
queue, its z-chunks cover the grid, and a 16-bit chunk fits the staged slab
records (a call of 0 steps validates and chooses, and launches nothing)."""

import ctypes
import random
import re
import subprocess
import sys

import pytest

from paper_2309_04671_amd import lib
from tests.test_queue_host import FAKE_ARENA, desc, make_queue, submit

SHAPES = [(1, 1, 1), (1, 1, 5000), (5000, 3, 1), (3, 5000, 2), (64, 64, 64), (63, 17, 16), (65, 15, 17), (128, 120, 96),
          (257, 33, 31), (300, 280, 200), (512, 512, 512), (750, 994, 300), (1024, 1024, 512), (20, 20, 20000)]
_r = random.Random(5)
SHAPES += [tuple(_r.randint(1, 700) for _ in range(3)) for _ in range(40)]


def _chosen(shapes):
    code = """
import ctypes, sys
sys.path.insert(0, '.')
from paper_2309_04671_amd import lib
L, c, r = lib.load(), lib.sp_coeffs(), ctypes.c_int()
for shp in %r:
    for dt in (0, 1, 2):
        g, gv = lib.grid_init(*shp, dt), lib.grid_init(*shp)
        st = lib.sp_wave_state(1 << 44, 1 << 45, (1 << 46) if dt else None, 0)
        lib.check(L.sp_wave_step(ctypes.byref(g), ctypes.byref(c), 1e-3, 10.0, ctypes.byref(gv), 1 << 47,
                                 ctypes.byref(st), 0, None, None, None))
    lib.check(L.sp_stencil_apply(ctypes.byref(gv), ctypes.byref(c), 0, 1 << 44, 1 << 45, ctypes.byref(r), None))
""" % (shapes,)
    import os
    env = dict(os.environ, SP_LOG="1")
    env.pop("SP_TILE", None)
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, env=env, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    pat = re.compile(r"(\w+): (\d+)x(\d+)x(\d+) dtype (\d) mode (\d) -> tile (\d+)x(\d+)x(\d+), z-chunk (\d+), (\d+) blocks")
    return [(m[1],) + tuple(int(x) for x in m.groups()[1:]) for m in pat.finditer(p.stderr)]


def test_every_shape_has_a_compiled_configuration_that_covers_it():
    got = _chosen(SHAPES)
    assert len(got) == 4 * len(SHAPES)
    for name, nx, ny, nz, dt, mode, tx, ty, ry, zc, blocks in got:
        assert 1 <= zc <= nz and (dt == 0 or zc <= 1024)
        chunks = -(-nz // zc)
        assert blocks == -(-nx // tx) * -(-ny // ty) * chunks
        assert (chunks - 1) * zc < nz
        # no more blocks than one per plane and narrowest tile
        assert blocks <= -(-nx // 64) * -(-ny // 16) * nz


@pytest.mark.parametrize("dtype", [lib.SP_F32, lib.SP_F16, lib.SP_BF16])
def test_queue_accepts_every_shape(dtype):
    q = make_queue(1 << 40)
    try:
        for nx, ny, nz in SHAPES:
            d = desc(1, 1, dtype)
            d.nx, d.ny, d.nz = nx, ny, nz
            d.src_xyz[0][0] = d.src_xyz[0][1] = d.src_xyz[0][2] = 0
            rc, _ = submit(q, d)
            assert rc == lib.SP_OK, (nx, ny, nz, lib.last_error())
        lib.check(lib.load().sp_queue_drain(q))
    finally:
        lib.check(lib.load().sp_queue_destroy(q))
    assert FAKE_ARENA > 0
