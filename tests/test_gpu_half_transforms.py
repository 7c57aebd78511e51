"""The half-length transforms and strip layouts of the grid passes at every
transform length and band reduction they are built for, and planes aligned to
one element only, against the FP64 oracle."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import check_close, dev, geometry, host, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


def _geo(N, reduce):
    # band width N' / 2^reduce (less two modes), so that N'' = N' / 2^reduce
    # where that is at least 32; off-centre by one mode
    if reduce == 0:
        return geometry(N=N, g=4e-6, lam=633e-9, z=0.003, tf="asm", band="full")
    w = 2.0 * N / 2 ** reduce - 4
    return geometry(N=N, g=4e-6, lam=633e-9, z=0.003, tf="asm", band="explicit", band_c=(1.0, -1.0), band_w=(w, w))


@pytest.mark.parametrize("reduce", [0, 1, 2, 3])
@pytest.mark.parametrize("N", [16, 32, 64, 128, 256, 512])
def test_operators_at_every_length(P, N, reduce):
    geo = _geo(N, reduce)
    rng = np.random.default_rng(N + reduce)
    M, M2 = 300, 211
    x, y = synth.uniform_box(rng, M, N * geo.g)
    x2, y2 = synth.uniform_box(rng, M2, N * geo.g)
    # the corners of the closed window: their taps reach the support's margin
    h = N * geo.g / 2
    x[:4], y[:4] = (-h, h, -h, h), (-h, -h, h, h)
    c, u1 = synth.unit_phase(rng, M), synth.unit_phase(rng, (N, N))
    w, v = synth.unit_phase(rng, M), synth.unit_phase(rng, (2 * N, 2 * N))
    d = [dev(torch, a) for a in (x, y, x2, y2)]
    p1 = make_plan(P, geo, 1).set_points(d[0], d[1])
    p2 = make_plan(P, geo, 2).set_points(d[0], d[1])
    p3 = make_plan(P, geo, 3).set_points(d[0], d[1]).set_dest_points(d[2], d[3])
    assert p1.info["Npf"] == max(32, 2 * N >> reduce, 2 * N >> 3)
    check_close(host(p1.execute(dev(torch, c))), O.nuasm1(geo, x, y, c), 1e-5, "type 1")
    check_close(host(p1.adjoint(dev(torch, v))), O.nuasm1_adjoint(geo, v, x, y), 1e-5, "type 1 adjoint")
    check_close(host(p2.execute(dev(torch, u1))), O.nuasm2(geo, u1, x, y), 1e-5, "type 2")
    check_close(host(p2.adjoint(dev(torch, w))), O.nuasm2_adjoint(geo, w, x, y), 1e-5, "type 2 adjoint")
    check_close(host(p3.execute(dev(torch, c))), O.nuasm3(geo, x, y, c, x2, y2), 1e-5, "type 3")


@pytest.mark.parametrize("N", [16, 64, 256])
def test_planes_aligned_to_one_element(P, N):
    """Inputs and outputs that start 8 bytes past a 16-byte boundary."""
    geo = _geo(N, 0)
    rng = np.random.default_rng(N)
    M = 500
    x, y = synth.uniform_box(rng, M, N * geo.g)
    xd, yd = dev(torch, x), dev(torch, y)

    def odd(a):  # a copy of a, one element past an aligned start
        b = torch.empty(a.numel() + 1, dtype=a.dtype, device=a.device)
        t = b[1:].view(a.shape)
        t.copy_(a)
        assert t.data_ptr() % 16 == 8
        return t
    for kind, plan, inp in (("crop", make_plan(P, geo, 1, crop=True), synth.unit_phase(rng, M)),
                            ("plane", make_plan(P, geo, 1), synth.unit_phase(rng, M)),
                            ("type 2", make_plan(P, geo, 2), synth.unit_phase(rng, (N, N)))):
        plan.set_points(xd, yd)
        i = dev(torch, inp)
        want = plan.execute(i)
        got = plan.execute(odd(i), odd(torch.zeros_like(want)))
        assert float((got - want).abs().max()) <= 2e-6 * float(want.abs().max()), kind
        v = dev(torch, synth.unit_phase(rng, tuple(want.shape)))
        if kind == "crop":
            continue
        want = plan.adjoint(v)
        got = plan.adjoint(odd(v), odd(torch.zeros_like(want)))
        assert float((got - want).abs().max()) <= 2e-6 * float(want.abs().max()), kind
