"""Interpolation with its batches sorted in LDS: record counts around the sort
threshold, a batch and a chunk, dense and thin bins, both bin sides, odd and
even kernel widths, sets with and without the records of neighbouring bins;
against the FP64 oracle, and bitwise between the record sets."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import check_close, dev, geometry, host, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUND = {1e-3: 2e-3, 1e-6: 1e-5, 1e-7: 3e-6, 1e-9: 2e-6}


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("tol", [1e-3, 1e-6, 1e-7, 1e-9])
@pytest.mark.parametrize("M", [383, 384, 385, 1024, 1025, 1408, 1409, 2048, 2049, 5000])
def test_one_bin(P, M, tol, tile):
    """All points inside one bin of the support."""
    geo = geometry(N=32, g=4e-6, lam=633e-9, z=0.004, tf="asm", band="full")
    rng = np.random.default_rng(M + tile)
    x, y = (rng.uniform(-0.5, 9.0, M) * geo.g for _ in range(2))
    u1 = synth.unit_phase(rng, (32, 32))
    xd, yd, ud = dev(torch, x), dev(torch, y), dev(torch, u1)
    outs = []
    for fo in (False, True):
        p = make_plan(P, geo, 2, tol=tol, forward_only=fo)
        p.set_tuning(interp_chunk=2048, bin_tile=tile)
        outs.append(p.set_points(xd, yd).execute(ud))
    assert torch.equal(outs[0], outs[1])
    check_close(host(outs[0]), O.nuasm2(geo, u1, x, y), BOUND[tol])


def test_batches_after_the_first(P):
    """A chunk of many batches, the last one below the sort threshold."""
    geo = geometry(N=32, g=4e-6, lam=633e-9, z=0.004, tf="fresnel", band="full")
    rng = np.random.default_rng(5)
    x, y = (rng.uniform(0.0, 5.0, 7300) * geo.g for _ in range(2))
    u1 = synth.unit_phase(rng, (32, 32))
    p = make_plan(P, geo, 2)
    p.set_tuning(interp_chunk=65536)
    got = p.set_points(dev(torch, x), dev(torch, y)).execute(dev(torch, u1))
    check_close(host(got), O.nuasm2(geo, u1, x, y), 1e-5)


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("tol", [1e-3, 1e-5, 1e-6, 1e-9])
@pytest.mark.parametrize("M", [319 * 1100, 319 * 1100 + 1, 320 * 1100 + 385, 400 * 1100])
def test_chunk_count_rule(P, M, tol, tile):
    """Around the number of chunks from which batches are sorted: bitwise the
    outputs of a launch of few chunks, which sorts nothing, and those against
    the oracle at some points."""
    geo = geometry(N=32, g=4e-6, lam=633e-9, z=0.004, tf="asm", band="full")
    rng = np.random.default_rng(M + tile)
    x, y = (rng.uniform(-0.5, 9.0, M) * geo.g for _ in range(2))
    u1 = synth.unit_phase(rng, (32, 32))
    xd, yd, ud = dev(torch, x), dev(torch, y), dev(torch, u1)
    outs = []
    for chunk in (1100, 65536):
        p = make_plan(P, geo, 2, tol=tol, forward_only=True)
        p.set_tuning(interp_chunk=chunk, bin_tile=tile)
        outs.append(p.set_points(xd, yd).execute(ud))
    assert torch.equal(outs[0], outs[1])
    pick = rng.choice(M, size=200, replace=False)
    check_close(host(outs[0])[pick], O.nuasm2(geo, u1, x[pick], y[pick]), BOUND.get(tol, 10 * tol))
