"""nuasm_plan_info reports the chunk sizes that the bound points run with."""
import pytest

from gpu_util import geometry, make_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _chunks(p):
    return p.info["spread_chunk"], p.info["interp_chunk"]


def test_info_reports_the_bound_sets_chunks():
    import paper_1308_6644_amd as P
    geo = geometry(N=256, g=4e-6, lam=633e-9, z=0.02, tf="asm", band="limited")
    x = torch.linspace(-4e-4, 4e-4, 500000, dtype=torch.float64, device="cuda")

    def bind(p, M, dest=False):
        return (p.set_dest_points if dest else p.set_points)(x[:M].contiguous(), x[:M].flip(0).contiguous())

    p = make_plan(P, geo, 1)
    assert _chunks(p) == (1792, 2048)
    # 8 M / chunk < 2048 tiles and 4 M / chunk <= 1024 workgroups, in steps of 256
    for M, want in ((4000, (512, 512)), (60000, (256, 512)), (66000, (512, 512)), (262000, (1024, 1024)),
                    (500000, (1792, 2048))):
        bind(p, M)
        assert _chunks(p) == want, M
        assert 8 * M // p.info["spread_chunk"] < 2048 or M == 500000
    bind(p, 60000)
    p.set_tuning(interp_chunk=1024)  # the points have to be bound again
    assert _chunks(p) == (1792, 1024)
    bind(p, 60000)
    assert _chunks(p) == (256, 1024)
    d = make_plan(P, geo, 1, deterministic=True)
    bind(d, 60000)
    assert _chunks(d) == (1792, 2048)
    t3 = make_plan(P, geo, 3)
    bind(t3, 60000)
    bind(t3, 262000, dest=True)
    assert _chunks(t3) == (256, 1024)
