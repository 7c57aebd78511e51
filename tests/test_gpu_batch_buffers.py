"""When a batch replays a recorded graph, and when not.  Its three graphs
(one-shot run, binning, operators) share their planes' buffers: once one of them
has moved a buffer, the others are not replayed as they are.  Arguments that a
graph was not recorded with get new tables (grouped form, same counts) or run
plainly, and are recorded when they come a second time in a row."""
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
        assert (r, f) == ((0, 1) if grouped else (0, 0))
    out[0].fill_(float("nan"))
    b.run(*a, out)
    check_close(host(out[0]), plain(a), 1e-6, what="once more")
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


def _batch(rng, specs, counts):
    xs, ys, ins = [], [], []
    for sp, M in zip(specs, counts):
        x, y = synth.clustered_box(rng, M, sp["N"] * sp["g"])
        xs.append(dev(torch, x))
        ys.append(dev(torch, y))
        ins.append(dev(torch, synth.unit_phase(rng, M if sp["type"] == 1 else (sp["N"], sp["N"]))))
    return xs, ys, ins


SPECS = [dict(N=n, type=t, lam=633e-9, z=0.02, g=G, tf=tf, band="limited" if tf == "asm" else "full", tol=1e-6)
         for n, t, tf in ((64, 1, "asm"), (128, 2, "fresnel"), (256, 1, "fresnel"), (64, 2, "asm"))]


def _outs(counts):
    return [torch.full((2 * s["N"], 2 * s["N"]) if s["type"] == 1 else (M,), float("nan"), dtype=torch.complex64,
                       device="cuda") for s, M in zip(SPECS, counts)]


def _plain(P, data):
    return [host(P.Plan(**s).set_points(x, y).execute(i)) for s, x, y, i in zip(SPECS, *data)]


def _check(outs, refs, what):
    for p, (o, r) in enumerate(zip(outs, refs)):
        check_close(host(o), r, 1e-6, what=f"{what}, plane {p}")


def test_grouped_graph_takes_new_buffers(P):
    """Other buffers, same counts: the grouped graphs are kept, their tables rewritten."""
    rng = np.random.default_rng(31)
    counts = [3000, 20000, 7000, 500]
    a, c = _batch(rng, SPECS, counts), _batch(rng, SPECS, counts)
    ra, rc = _plain(P, a), _plain(P, c)
    b = P.Batch(SPECS)
    oa, oc, oa2 = _outs(counts), _outs(counts), _outs(counts)
    for n, (d, o) in enumerate(((a, oa), (c, oc), (a, oa2))):
        b.run(*d, o)
        assert b.debug_graphs() == (1, n)
    _check(oa, ra, "first buffers")
    _check(oc, rc, "other buffers")
    _check(oa2, ra, "first buffers again")
    b.set_points(*a[:2])
    graphs = b.debug_graphs()
    e1, e2 = _outs(counts), _outs(counts)
    b.execute(a[2], e1)
    b.execute(a[2], e2)
    assert b.debug_graphs() == (graphs[0] + 1, graphs[1] + 1)
    _check(e1, ra, "execute")
    _check(e2, ra, "execute, other outputs")
    b.close()


@pytest.mark.parametrize("grouped", [True, False], ids=["grouped", "branches"])
def test_changed_arguments_run_plainly_until_they_repeat(P, grouped):
    """Counts changed (either form) and buffers changed (per-plane form)."""
    rng = np.random.default_rng(32)
    ca = [3000, 20000, 7000, 500]
    cc = [1000, 30000, 7000, 500] if grouped else ca
    a, c = _batch(rng, SPECS, ca), _batch(rng, SPECS, cc)
    ra, rc = _plain(P, a), _plain(P, c)
    b = P.Batch(SPECS)
    b.set_grouped(grouped)
    oa, oc = _outs(ca), _outs(cc)
    b.run(*a, oa)
    b.run(*c, oc)  # right behind the graph: plain
    assert b.debug_graphs() == (1, 0)
    t = b.plane_times()
    assert t == sorted(t) and t[0] > 0
    _check(oa, ra, "recorded")
    _check(oc, rc, "plain")
    for o in oa + oc:
        o.fill_(float("nan"))
    b.run(*a, oa)  # (grouped: a larger count has moved buffers, new tables)
    b.run(*c, oc)
    _check(oa, ra, "the graph again")
    _check(oc, rc, "plain again")
    assert b.debug_graphs() == (1, 1 if grouped else 0)
    for o in oc:
        o.fill_(float("nan"))
    b.run(*c, oc)  # a second time in a row: recorded
    _check(oc, rc, "recorded in its place")
    for o in oc:
        o.fill_(float("nan"))
    b.run(*c, oc)
    _check(oc, rc, "replayed")
    assert b.debug_graphs() == (2, 1 if grouped else 0)
    assert all(v > 0 for v in b.plane_times())
    b.close()
