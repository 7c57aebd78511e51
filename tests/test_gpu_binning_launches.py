"""The binning in one launch (small sets) and in three, against the four
separately timed launches: the same records in every bin, the same counts, the
same operator outputs, rejected points included."""
import numpy as np
import pytest

import synth
from gpu_util import dev, geometry, host, make_plan, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


def _records(plan):
    recs, counts = plan.debug_records()
    recs, counts = recs.cpu().numpy(), counts.cpu().numpy()
    b = np.repeat(np.arange(counts.size), counts)
    assert b.size == recs.shape[0]
    return counts, recs[np.lexsort((recs[:, 0], recs[:, 3], b))]


# 25, 81, 4225 (five rounds of 1024), 1089 bins, 16641 (too many for the LDS cursors)
@pytest.mark.parametrize("N,tile,full", [(64, 32, True), (128, 32, True), (1024, 32, True), (1024, 64, True),
                                         (2048, 32, True)])
@pytest.mark.parametrize("M", [1, 1023, 4096, 4097, 70001])
def test_fused_binning_equals_separate_launches(P, N, tile, full, M):
    geo = geometry(N=N, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="full")
    rng = np.random.default_rng(M + N)
    x, y = synth.clustered_box(rng, M, N * geo.g)
    bad = rng.choice(M, size=M // 50, replace=False)
    x[bad] = 2.0 * N * geo.g
    xd, yd = dev(torch, x), dev(torch, y)
    c = dev(torch, synth.unit_phase(rng, M))
    w = dev(torch, synth.unit_phase(rng, (2 * N, 2 * N)))
    got = []
    for timing in (False, True):
        p = make_plan(P, geo, 1, defer_range_check=True, full_fine_grid=full)
        if tile != 32:
            p.set_tuning(bin_tile=tile)
        p.set_timing(timing)
        p.set_points(xd, yd)
        got.append((_records(p), host(p.execute(c)), p.adjoint(w)))
        assert (p.read_timing()["bin_scan"][1] > 0) == timing
    (ca, ra), ua, ga = got[0]
    (cb, rb), ub, gb = got[1]
    assert np.array_equal(ca, cb) and np.array_equal(ra, rb)
    assert rel_l2(ua, ub) <= 1e-6  # float32 sums in another order
    assert torch.equal(torch.view_as_real(ga).nan_to_num(7.0), torch.view_as_real(gb).nan_to_num(7.0))
    assert int(torch.isnan(ga.real).sum()) == bad.size


def test_forward_only_small_set(P):
    geo = geometry(N=64, g=4e-6, lam=633e-9, z=0.01, tf="fresnel", band="full")
    rng = np.random.default_rng(3)
    u1 = dev(torch, synth.unit_phase(rng, (64, 64)))
    for M in (500, 4096, 6000):
        x, y = (dev(torch, a) for a in synth.uniform_box(rng, M, 64 * geo.g))
        a = make_plan(P, geo, 2, forward_only=True).set_points(x, y).execute(u1)
        b = make_plan(P, geo, 2).set_points(x, y).execute(u1)
        assert torch.equal(a, b)
