"""Type-2 column pass with narrow bands: the forward transform whole (up to
N' = 2048) and by half-length transforms (beyond), every ratio of the spectral
grid to N', against the full fine grid, and the oracle where that is quick.
Outputs differ from the full grid's by two results' float32 rounding, from the
oracle's by the operator bar."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import check_close, dev, geometry, host, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (the spectral grid has at least 32 modes)
@pytest.mark.parametrize("N,ratio", [(N, r) for N in (32, 64, 256, 512, 1024, 2048) for r in (2, 4, 8) if 2 * N // r >= 32])
def test_narrow_band_columns(N, ratio):
    import paper_1308_6644_amd as P
    npf = 2 * N // ratio
    geo = geometry(N=N, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="explicit", band_c=(0.0, 1.0),
                   band_w=(npf - 2.0, npf - 4.0))
    rng = np.random.default_rng(N + ratio)
    M = 1500
    x, y = synth.uniform_box(rng, M, N * geo.g)
    u1, w = synth.unit_phase(rng, (N, N)), synth.unit_phase(rng, M)
    out = []
    for full in (False, True):
        p = make_plan(P, geo, 2, full_fine_grid=full).set_points(dev(torch, x), dev(torch, y))
        assert p.info["Npf"] == (2 * N if full else npf)
        out.append((host(p.execute(dev(torch, u1))), host(p.adjoint(dev(torch, w)))))
    for a, b, what in zip(*out, ("execute", "adjoint")):
        check_close(a, b, 3e-6, what=what)
    if N <= 256:
        check_close(out[0][0], O.nuasm2(geo, u1, x, y), 1e-5, what="oracle")
