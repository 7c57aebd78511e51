"""Rayleigh-Sommerfeld summation on both sides of the distance at which the
form of its phase changes (|z| / lambda = 1e5), near and far, both signs of z,
counts around a wave, a source group and a float32 partial sum, against the
FP64 oracle."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import dev, host, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LAM = 500e-9


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


@pytest.mark.parametrize("zl", [20.0, 1.6e4, 0.99999e5, 1e5, 1.00001e5, 2e6, 2e8])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("M1,M2", [(1, 1), (7, 65), (513, 64), (1024, 130)])
def test_phase_forms_match_oracle(P, zl, sign, M1, M2):
    z = sign * zl * LAM
    rng = np.random.default_rng(M1)
    W = 1e-3
    x1, y1 = synth.uniform_box(rng, M1, W)
    x2, y2 = synth.uniform_box(rng, M2, W)
    c = synth.unit_phase(rng, M1)
    got = host(P.rs_direct(dev(torch, x1), dev(torch, y1), dev(torch, c), dev(torch, x2), dev(torch, y2), lam=LAM, z=z,
                           ox=1.3e-4, oy=-2e-5))
    ref = O.rayleigh_sommerfeld_points(x1, y1, c, x2, y2, LAM, z, 1.3e-4, -2e-5)
    # the float32 argument of the sine and cosine (2^-25 cycles), their own
    # 1.3e-7, the amplitude's few roundings, the float32 sums of 64 terms
    assert rel_l2(got, ref) <= 1e-6
