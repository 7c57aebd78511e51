"""The stable scatter of deterministic mode: the records of every bin in point
order, the same ones as the default scatter's, for counts around a range of
1024 points, all points in one bin, rejected points among them, both bin
sides, and supports up to the most bins (whose counters take 132 KB of LDS)."""
import numpy as np
import pytest

import synth
from gpu_util import dev, geometry, make_plan

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
    return recs, np.repeat(np.arange(counts.size), counts)


@pytest.mark.parametrize("N,tile,M,kind", [
    (32, 32, 1, "uniform"), (32, 32, 1023, "uniform"), (32, 32, 1024, "one bin"), (32, 32, 1025, "one bin"),
    (64, 64, 3000, "clustered"), (128, 32, 5000, "one bin"), (1024, 32, 20000, "clustered"),
    (2048, 32, 4097, "uniform"), (4096, 32, 3000, "clustered"),
])
def test_bins_in_point_order(P, N, tile, M, kind):
    geo = geometry(N=N, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="full")
    rng = np.random.default_rng(M)
    if kind == "one bin":
        x, y = (rng.uniform(0.2, 3.0, M) * geo.g for _ in range(2))
    else:
        x, y = synth.make_points(kind, rng, M, N, geo.g)
    bad = rng.choice(M, size=M // 40, replace=False)
    y[bad] = np.nan
    xd, yd = dev(torch, x), dev(torch, y)
    got = []
    for det in (True, False):
        p = make_plan(P, geo, 1, defer_range_check=True, deterministic=det)
        if tile != 32:
            p.set_tuning(bin_tile=tile)
        got.append(_records(p.set_points(xd, yd)))
        p.close()
    (rd, bd), (rn, bn) = got
    key = bd.astype(np.int64) * M + rd[:, 3]
    assert np.all(np.diff(key) > 0)  # by bin, then by point
    order = np.lexsort((rn[:, 3], bn))
    assert np.array_equal(bd, bn[order]) and np.array_equal(rd, rn[order])


@pytest.mark.parametrize("N,M,kind", [(64, 70, "one bin"), (64, 71, "one bin"), (64, 72, "one bin"),
                                      (32, 61113, "uniform"), (64, 20000, "uniform"), (256, 9000, "three_clusters")])
def test_long_runs_in_point_order(P, N, M, kind):
    """Runs of a range around the length from which a run is ranked by bits,
    and many long runs that begin at any position."""
    geo = geometry(N=N, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="full")
    rng = np.random.default_rng(M)
    if kind == "one bin":
        x, y = (rng.uniform(0.2, 3.0, M) * geo.g for _ in range(2))
    elif kind == "uniform":
        x, y = (rng.uniform(-0.5, 0.5, M) * N * geo.g for _ in range(2))
    else:
        c = rng.integers(0, 3, M)
        x, y = (rng.normal(np.array([-0.3, 0.0, 0.25])[c], 0.02).clip(-0.5, 0.5) * N * geo.g for _ in range(2))
    xd, yd = dev(torch, x), dev(torch, y)
    got = []
    for det in (True, False):
        p = make_plan(P, geo, 1, deterministic=det)
        got.append(_records(p.set_points(xd, yd)))
        p.close()
    (rd, bd), (rn, bn) = got
    order = np.lexsort((rn[:, 3], bn))
    assert np.array_equal(bd, bn[order]) and np.array_equal(rd, rn[order])
