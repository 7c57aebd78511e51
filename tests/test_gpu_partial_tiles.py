"""Partial tiles of split bins: once a plan has spread, another set of points
within its capacity allocates nothing when it is executed, so that the execute
can be captured, whatever the chunk sizes of the new count are."""
import numpy as np
import pytest

import synth
from gpu_util import check_close, dev, geometry, host, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GEO = dict(N=256, g=4e-6, lam=633e-9, z=0.02, tf="asm", band="limited")


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


def _set(rng, geo, M, dense):
    x, y = synth.clustered_box(rng, M, geo.N * geo.g)
    if dense:  # all in a few cells: every bin they touch is split
        x, y = (rng.uniform(-2 * geo.g, 2 * geo.g, M) for _ in range(2))
    return dev(torch, x), dev(torch, y), dev(torch, synth.unit_phase(rng, M))


# counts on either side of the steps of the chunk sizes: 512 up to 8192 points, then 256, 512 from 65505 on, ...
@pytest.mark.parametrize("counts", [(8192, 4001), (30000, 8193, 8192), (66000, 65504, 60000), (300007, 262000, 65504)])
@pytest.mark.parametrize("defer", [False, True], ids=["checked", "deferred"])
def test_execute_of_another_set_allocates_nothing(P, counts, defer):
    geo = geometry(**GEO)
    rng = np.random.default_rng(counts[0])
    p = make_plan(P, geo, 1, defer_range_check=defer)
    x, y, c = _set(rng, geo, counts[0], False)
    p.set_points(x, y).execute(c)
    after_first = p.info["device_bytes"]
    for M in counts[1:]:
        x, y, c = _set(rng, geo, M, True)
        p.set_points(x, y)
        bound = p.info["device_bytes"]
        assert not defer or bound == after_first
        p.execute(c)
        assert p.info["device_bytes"] == bound, M


@pytest.mark.parametrize("defer", [False, True], ids=["checked", "deferred"])
def test_captured_execute_after_a_smaller_denser_set(P, defer):
    geo = geometry(**GEO)
    rng = np.random.default_rng(1)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        p = make_plan(P, geo, 1, defer_range_check=defer)
        x, y, c = _set(rng, geo, 66000, False)
        p.set_points(x, y).execute(c)
        x, y, c = _set(rng, geo, 60000, True)
        p.set_points(x, y)
        out = torch.empty((2 * geo.N, 2 * geo.N), dtype=torch.complex64, device="cuda")
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            p.execute(c, out)
        for _ in range(3):
            c.copy_(dev(torch, synth.unit_phase(rng, 60000)))
            out.fill_(float("nan"))
            g.replay()
            got = host(out)
            check_close(got, host(p.execute(c)), 1e-6)
