"""A grid bound to a forward-only plan needs no buffer for spreading: it takes
no device memory, interpolates as an ordinary plan does, and the testing entry
that spreads from it still does."""
import numpy as np
import pytest

import synth
from gpu_util import dev, geometry, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_forward_only_grid_takes_no_memory():
    import paper_1308_6644_amd as P
    geo = geometry(N=128, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="limited")
    rng = np.random.default_rng(3)
    u1, v = dev(torch, synth.unit_phase(rng, (128, 128))), dev(torch, synth.unit_phase(rng, 100 * 90))
    fwd, both = make_plan(P, geo, 2, forward_only=True), make_plan(P, geo, 2)
    before = fwd.info["device_bytes"], both.info["device_bytes"]
    for p in (fwd, both):
        p.set_grid_points(100, 90, 4e-6)
    rows = 8 * 90 * both.info["L"]
    assert (fwd.info["device_bytes"] - before[0], both.info["device_bytes"] - before[1]) == (0, rows)
    assert torch.equal(fwd.execute(u1), both.execute(u1))
    assert torch.equal(fwd.debug_spread(v), both.debug_spread(v))
    assert fwd.info["device_bytes"] - before[0] == rows
