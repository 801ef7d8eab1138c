"""What a plan launches can be read back: a plan asked for that form and tile
gives the same grids and residuals, bit for bit, under every tuning, and reports
itself."""
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KW = {"heat3d7": dict(coef=(0.4, 0.1)), "poisson19": dict(omega=0.8), "wave25": dict(coef=synth.WAVE25_COEF)}


@pytest.mark.parametrize("kind", ["heat3d7", "poisson19", "wave25"])
@pytest.mark.parametrize("tune", ["fixed", "exhaustive", "model"])
@pytest.mark.parametrize("n", [(70, 41, 33), (20, 150, 90)])
def test_a_plan_of_the_launch(kind, tune, n):
    from paper_2306_13002_amd.stencil import Plan
    dt = torch.float32 if kind == "poisson19" else torch.float64
    r = 4 if kind == "wave25" else 1
    gen = torch.Generator(device="cuda").manual_seed(6)
    rand = lambda: torch.rand([e + 2 * r for e in reversed(n)], dtype=dt, device="cuda", generator=gen)  # noqa: E731
    u, c = rand(), [0.05 * rand() for _ in range({"poisson19": 12, "wave25": 1}.get(kind, 0))] or None
    with Plan(kind, n, tune=tune, **KW[kind]) as p:
        for T in (1, 6):
            how = p.launch(T)
            with Plan(kind, n, variant=how["variant"], tile=how["tile"], tile_map=p.config()["tile_map"], **KW[kind]) as q:
                assert q.launch(T) == how and q.config()["tile"] == how["tile"]
                a, b = [u.clone(), u.clone()], [u.clone(), u.clone()]
                p.run(a, c, iterations=T)
                q.run(b, c, iterations=T)
                assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
                assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual()


def test_marching_launches():
    from paper_2306_13002_amd.stencil import Plan
    with Plan("heat2d5", (300, 200), coef=(0.6, 0.1)) as p:
        assert p.launch(1) == {"variant": "plain", "tile": (64, 4, 1), "sweeps": 1}
        assert p.launch(2)["sweeps"] == 1
        for T, k in ((10, 5), (16, 8), (17, 5), (100, 8)):
            how = p.launch(T)
            assert how["variant"] == "plain" and how["sweeps"] == k == how["tile"][2]
            assert how["tile"][0] == 64 - 2 * k


def test_refused():
    from paper_2306_13002_amd import stencil as S
    with S.BatchPlan([(10, 10, 10)]) as b, S.Plan("heat3d7", (10, 10, 10), coef=(0.4, 0.1)) as p:
        assert S.lib().stencil_plan_launch(b._h, 1, None, None, None, None, None) == S.E_UNSUPPORTED
        assert S.lib().stencil_plan_launch(p._h, 0, None, None, None, None, None) == S.E_INVAL
        assert S.lib().stencil_plan_launch(None, 1, None, None, None, None, None) == S.E_INVAL
