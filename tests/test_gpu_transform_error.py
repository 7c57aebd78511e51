"""Rounding of the grid passes: Fresnel planes far away, whose spectrum is a few
modes, so that errors of the transforms' twiddles add up instead of averaging
out.  Bound: the error that full-length transforms with the twiddles as
separate factors had on these inputs, the mean of five seeds."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import dev, geometry, host, make_plan, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUND = {256: 8.42e-7, 512: 1.20e-6}


@pytest.mark.parametrize("N", sorted(BOUND))
def test_error_of_a_far_plane(N):
    import paper_1308_6644_amd as P
    geo = geometry(N=N, g=4e-6, lam=633e-9, z=0.425 * N / 256, tf="fresnel")
    err = []
    for seed in range(5):
        rng = np.random.default_rng(seed)
        x, y = synth.uniform_box(rng, 20000, N * geo.g)
        u1 = synth.unit_phase(rng, (N, N))
        plan = make_plan(P, geo, 2, tol=1e-9).set_points(dev(torch, x), dev(torch, y))
        got = host(plan.execute(dev(torch, u1)))
        s = slice(0, 20000, 40)
        err.append(rel_l2(got[s], O.nuasm2(geo, u1, x[s], y[s])))
    assert np.mean(err) <= BOUND[N]
