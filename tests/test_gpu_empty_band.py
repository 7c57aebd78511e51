"""An explicit band that is empty along one axis holds no mode, however wide it
is along the other: every operator and adjoint gives zeros, also where the
other axis' extent lies outside the small spectral grid such a plan gets."""
import numpy as np
import pytest

import synth
from gpu_util import dev, geometry, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, M, M2 = 64, 700, 300


@pytest.mark.parametrize("full", [False, True], ids=["band-grid", "full-grid"])
@pytest.mark.parametrize("centre", [-60.0, 0.0, 62.0])
@pytest.mark.parametrize("width", [0.0, 8.0, 128.0])
@pytest.mark.parametrize("axis", ["x", "y"])
def test_band_empty_along_one_axis_gives_zero(axis, width, centre, full):
    import paper_1308_6644_amd as P
    e, w = (0.5, 0.0), (centre, width)  # no whole number in [0.5, 0.5]
    bx, by = (e, w) if axis == "x" else (w, e)
    geo = geometry(N=N, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="explicit", band_c=(bx[0], by[0]),
                   band_w=(bx[1], by[1]))
    rng = np.random.default_rng(5)
    x, y = (dev(torch, a) for a in synth.uniform_box(rng, M, N * geo.g))
    x2, y2 = (dev(torch, a) for a in synth.uniform_box(rng, M2, N * geo.g))
    c, u1, v = (dev(torch, synth.unit_phase(rng, s)) for s in (M, (N, N), (2 * N, 2 * N)))
    w2 = dev(torch, synth.unit_phase(rng, M2))
    p1, p2 = (make_plan(P, geo, t, full_fine_grid=full).set_points(x, y) for t in (1, 2))
    p3 = make_plan(P, geo, 3, full_fine_grid=full).set_points(x, y).set_dest_points(x2, y2)
    pc = make_plan(P, geo, 1, full_fine_grid=full, crop=True).set_points(x, y)
    outs = [p1.execute(c), p1.adjoint(v), p2.execute(u1), p2.adjoint(c), p3.execute(c), p3.adjoint(w2), pc.execute(c)]
    for i, o in enumerate(outs):
        assert not o.abs().any(), i
