"""nuasm_debug_interp takes a support grid aligned to one complex element: the
values are those of the same grid at a 16-byte boundary, bit for bit."""
import numpy as np
import pytest

import synth
from gpu_util import dev, geometry, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tol", [1e-3, 1e-6])
def test_grid_aligned_to_one_element(tol):
    import paper_1308_6644_amd as P
    geo = geometry(N=64, g=4e-6, lam=633e-9, z=0.01, tf="asm", band="full")
    rng = np.random.default_rng(2)
    p = make_plan(P, geo, 2, tol=tol)
    p.set_points(*(dev(torch, a) for a in synth.uniform_box(rng, 3000, geo.N * geo.g)))
    L = p.info["L"]
    buf = torch.empty(L * L + 1, dtype=torch.complex64, device="cuda")
    grid = dev(torch, synth.unit_phase(rng, (L, L)))
    buf[1:] = grid.reshape(-1)
    odd = buf[1:].reshape(L, L)
    assert odd.data_ptr() % 16 == 8 and grid.data_ptr() % 16 == 0
    assert torch.equal(p.debug_interp(odd), p.debug_interp(grid))
