"""The three recorded graphs of a batch (one-shot run, binning, operators)
share their planes' buffers.  When one of them has moved a buffer, the others
are not replayed as they are: their arguments are collected again."""
import numpy as np
import pytest

import synth
from gpu_util import check_close, dev, host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, G = 512, 4e-6


@pytest.fixture(scope="module")
def P():
    import paper_1308_6644_amd as P
    P.load()
    return P


def _set(rng, M):
    x, y = synth.clustered_box(rng, M, N * G)
    return [dev(torch, x)], [dev(torch, y)], [dev(torch, synth.unit_phase(rng, M))]


@pytest.mark.parametrize("grouped", [True, False], ids=["grouped", "branches"])
# more points (records and chunk tables move), fewer (more partial tiles: 8 M / chunk)
@pytest.mark.parametrize("first,other", [(20000, 40000), (66000, 60000)])
def test_run_after_other_graphs_moved_buffers(P, first, other, grouped):
    spec = dict(N=N, type=1, lam=633e-9, z=0.05, g=G, tf="asm", band="limited", tol=1e-6)
    rng = np.random.default_rng(first)
    a, o = _set(rng, first), _set(rng, other)
    out, out2 = ([torch.empty((2 * N, 2 * N), dtype=torch.complex64, device="cuda")] for _ in range(2))

    def plain(s):
        return host(P.Plan(**spec).set_points(s[0][0], s[1][0]).execute(s[2][0]))

    b = P.Batch([spec])
    b.set_grouped(grouped)
    b.run(*a, out)
    b.set_points(o[0], o[1])
    b.execute(o[2], out2)
    check_close(host(out2[0]), plain(o), 1e-6, what="other points")
    before = b.debug_graphs()
    out[0].fill_(float("nan"))
    b.run(*a, out)
    check_close(host(out[0]), plain(a), 1e-6, what="the first points again")
    if other > first:
        r, f = (n - m for n, m in zip(b.debug_graphs(), before))
        assert (r, f) == ((0, 1) if grouped else (1, 0))
    b.close()
