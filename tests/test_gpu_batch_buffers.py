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


@pytest.mark.parametrize("grouped", [True, False], ids=["grouped", "branches"])
@pytest.mark.parametrize("t", [1, 2])
def test_operator_after_replay_uses_the_replayed_points(P, t, grouped):
    """A replayed one-shot run binds its points again, on the host too: the
    operators that follow take their launch grids from its point count, not
    from the smaller set bound in between."""
    spec = dict(N=N, type=t, lam=633e-9, z=0.05, g=G, tf="asm", band="limited", tol=1e-6)
    rng = np.random.default_rng(3)
    a, o = _set(rng, 20000), _set(rng, 500)
    if t == 2:
        a = a[:2] + ([dev(torch, synth.unit_phase(rng, (N, N)))],)
    n = (2 * N, 2 * N) if t == 1 else (20000,)
    out, out2 = ([torch.full(n, float("nan"), dtype=torch.complex64, device="cuda")] for _ in range(2))
    ref = host(P.Plan(**spec).set_points(a[0][0], a[1][0]).execute(a[2][0]))
    b = P.Batch([spec])
    b.set_grouped(grouped)
    b.run(*a, out)
    b.set_points(o[0], o[1])
    graphs = b.debug_graphs()
    b.run(*a, out)
    assert b.debug_graphs() == graphs  # replayed
    b.execute(a[2], out2)
    check_close(host(out[0]), ref, 1e-6, what="run")
    check_close(host(out2[0]), ref, 1e-6, what="execute")
    b.close()
