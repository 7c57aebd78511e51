"""Column passes over the strips of columns that meet the band: bands of one
column, at either end of the spectrum, ending inside a strip, and empty along
one axis, for the three operator types and the adjoints, against the FP64
oracle."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import check_close, dev, geometry, host, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BANDS = [  # (centre, width) along x and y in index units, N' = 128
    ((63.0, 0.0), (0.0, 128.0)),     # the last column alone
    ((-64.0, 0.0), (0.0, 128.0)),    # the first column alone
    ((-40.0, 47.0), (3.0, 60.0)),    # from the left edge to the middle of a strip
    ((17.0, 2.0), (-5.0, 1.0)),      # three columns inside one strip, one row
    ((15.5, 1.0), (0.0, 30.0)),      # two columns astride two strips
]


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


@pytest.mark.parametrize("full", [False, True], ids=["band-grid", "full-grid"])
@pytest.mark.parametrize("bx,by", BANDS)
def test_band_strips_match_oracle(P, bx, by, full):
    geo = geometry(N=64, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="explicit", band_c=(bx[0], by[0]),
                   band_w=(bx[1], by[1]))
    rng = np.random.default_rng(11)
    M, M2 = 900, 700
    x, y = synth.uniform_box(rng, M, geo.N * geo.g)
    x2, y2 = synth.uniform_box(rng, M2, geo.N * geo.g)
    c, u1 = synth.unit_phase(rng, M), synth.unit_phase(rng, (geo.N, geo.N))
    w = synth.unit_phase(rng, M)
    d = [dev(torch, a) for a in (x, y, x2, y2)]
    p1 = make_plan(P, geo, 1, full_fine_grid=full).set_points(d[0], d[1])
    p2 = make_plan(P, geo, 2, full_fine_grid=full).set_points(d[0], d[1])
    p3 = make_plan(P, geo, 3, full_fine_grid=full).set_points(d[0], d[1]).set_dest_points(d[2], d[3])
    check_close(host(p1.execute(dev(torch, c))), O.nuasm1(geo, x, y, c), 1e-5, "type 1")
    check_close(host(p2.execute(dev(torch, u1))), O.nuasm2(geo, u1, x, y), 1e-5, "type 2")
    check_close(host(p2.adjoint(dev(torch, w))), O.nuasm2_adjoint(geo, w, x, y), 1e-5, "type 2 adjoint")
    check_close(host(p3.execute(dev(torch, c))), O.nuasm3(geo, x, y, c, x2, y2), 1e-5, "type 3")


@pytest.mark.parametrize("bx,by", [((0.5, 0.0), (0.0, 60.0)), ((200.0, 4.0), (0.0, 60.0))])
def test_band_without_columns_gives_zero(P, bx, by):
    geo = geometry(N=64, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="explicit", band_c=(bx[0], by[0]),
                   band_w=(bx[1], by[1]))
    rng = np.random.default_rng(12)
    x, y = (dev(torch, a) for a in synth.uniform_box(rng, 500, geo.N * geo.g))
    p1 = make_plan(P, geo, 1).set_points(x, y)
    p2 = make_plan(P, geo, 2).set_points(x, y)
    assert not p1.execute(dev(torch, synth.unit_phase(rng, 500))).abs().any()
    assert not p2.execute(dev(torch, synth.unit_phase(rng, (64, 64)))).abs().any()
