"""Chunk sizes that follow the point count: bins split into one-sub-batch
chunks, counts on either side of a size step, and the bound of the
allocation-free execute, against the FP64 oracle and the tuned fixed sizes."""
import ctypes

import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import check_close, dev, geometry, host, make_plan, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GEO = dict(N=32, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="full")


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


@pytest.mark.parametrize("M", [1, 255, 256, 257, 2047, 4097])
def test_dense_bin_matches_oracle(P, M):
    """Every point within a few cells: one bin split into M / 256 chunks."""
    geo = geometry(**GEO)
    rng = np.random.default_rng(M)
    x, y = (rng.uniform(0.0, 3.0 * geo.g, M) for _ in range(2))
    c, u1 = synth.unit_phase(rng, M), synth.unit_phase(rng, (geo.N, geo.N))
    xd, yd = dev(torch, x), dev(torch, y)
    p1, p2 = make_plan(P, geo, 1).set_points(xd, yd), make_plan(P, geo, 2).set_points(xd, yd)
    check_close(host(p1.execute(dev(torch, c))), O.nuasm1(geo, x, y, c), 1e-5, "type 1")
    check_close(host(p2.execute(dev(torch, u1))), O.nuasm2(geo, u1, x, y), 1e-5, "type 2")


@pytest.mark.parametrize("M", [65504, 65505, 131009, 300007, 458000, 458753])
@pytest.mark.parametrize("defer", [False, True])
def test_chunk_sizes_agree_with_fixed_size(P, M, defer):
    """Around the steps of the rule: the same sums as with the tuned fixed
    sizes, in either range-check mode, and accepted by the allocation-free
    execute as far as the fixed size is (8 M / 1792 + 1 <= 2048 tiles)."""
    geo = geometry(**GEO)
    rng = np.random.default_rng(7)
    x, y = synth.clustered_box(rng, M, geo.N * geo.g)
    xd, yd, c = dev(torch, x), dev(torch, y), dev(torch, synth.unit_phase(rng, M))
    auto = make_plan(P, geo, 1, defer_range_check=defer).set_points(xd, yd)
    fixed = make_plan(P, geo, 1, defer_range_check=defer)
    fixed.set_tuning(spread_chunk=1792, interp_chunk=2048).set_points(xd, yd)
    a, b = auto.execute(c), fixed.execute(c)
    # float32 sums in another order: a few rounding units of the largest sums
    assert rel_l2(host(a), host(b)) <= 1e-6
    out = torch.empty_like(a)
    if 8 * M // 1792 + 1 <= 2048:
        st = P.load().nuasm_execute_noalloc(auto._h, ctypes.c_void_p(c.data_ptr()), ctypes.c_void_p(out.data_ptr()))
        assert st == 0
        torch.cuda.synchronize()
        assert rel_l2(host(out), host(b)) <= 1e-6
    w = dev(torch, synth.unit_phase(rng, (2 * geo.N, 2 * geo.N)))
    assert torch.equal(auto.adjoint(w), fixed.adjoint(w))


def test_smaller_set_after_larger(P):
    """A plan whose buffers were sized for many points takes few, in smaller chunks."""
    geo = geometry(**GEO)
    rng = np.random.default_rng(9)
    p = make_plan(P, geo, 1, defer_range_check=True)
    for M in (300007, 70001, 3001):
        x, y = synth.clustered_box(rng, M, geo.N * geo.g)
        c = synth.unit_phase(rng, M)
        p.set_points(dev(torch, x), dev(torch, y))
        got = host(p.execute(dev(torch, c)))
        if M < 5000:
            check_close(got, O.nuasm1(geo, x, y, c), 1e-5)
