"""Interpolation at a uniform grid (both passes in one kernel) where its split
can go wrong: output rows closer than a cell and further apart than the
kernel's width, row counts around the rows of a workgroup, one row or one
column, off-centre grids touching the window's edge; against the FP64 oracle
at the same points."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import check_close, dev, geometry, host, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUND = {1e-2: 2e-2, 1e-3: 2e-3, 1e-6: 1e-5, 1e-9: 2e-6, 1e-12: 2e-6}
G = 4e-6


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


# N = 64: the window is 64 pixels (128 cells); pitch in pixels
@pytest.mark.parametrize("nx,ny,pitch,cx,cy,tol", [
    (1, 1, 1.0, 0.0, 0.0, 1e-6),
    (64, 1, 1.0, 0.0, 3.3, 1e-6),
    (1, 63, 1.0, 5.2, 0.0, 1e-6),
    (65, 41, 0.5, 10.0, -7.0, 1e-6),     # one cell apart, one column past a wave
    (130, 129, 0.25, 0.1, 0.2, 1e-6),
    (200, 640, 0.03, 20.0, -20.0, 1e-6),  # many rows a cell: 64 rows a workgroup
    (17, 17, 3.4999, 0.0, 0.0, 1e-6),    # 6.9998 cells: just below the width 7
    (17, 17, 3.5, 0.0, 0.0, 1e-6),       # at the width: rows kept apart
    (7, 13, 4.7, 1.0, -1.0, 1e-6),
    (33, 35, 1.7, 2.0, 1.0, 1e-2),       # width 3
    (12, 21, 2.9, 0.0, 0.0, 1e-9),       # width 10
    (9, 9, 6.4, 0.0, 0.0, 1e-12),        # width 13, 12.8 cells
    (64, 64, 1.0, 0.5, 0.5, 1e-3),       # last sample half a pixel inside the edge
    (129, 129, 0.5, 0.0, 0.0, 1e-6),     # both edges of the closed window
])
def test_grid_interpolation_matches_oracle(P, nx, ny, pitch, cx, cy, tol):
    geo = geometry(N=64, g=G, lam=633e-9, z=0.01, tf="asm", band="full")
    u1 = synth.unit_phase(np.random.default_rng(nx * 1000 + ny), (64, 64))
    plan = make_plan(P, geo, 2, tol=tol)
    plan.set_grid_points(nx, ny, pitch * G, cx * G, cy * G)
    got = host(plan.execute(dev(torch, u1)))
    xs = cx * G + (np.arange(nx) - nx // 2) * pitch * G
    ys = cy * G + (np.arange(ny) - ny // 2) * pitch * G
    y, x = (a.ravel() for a in np.meshgrid(ys, xs, indexing="ij"))
    check_close(got, O.nuasm2(geo, u1, x, y), BOUND[tol])
