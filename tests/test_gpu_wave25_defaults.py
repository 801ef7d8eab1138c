"""WAVE25 saturated plans of open shape pick tile and z-block by the grid: bit
for bit the same steps as a given tile, residuals to rounding, for sizes around
the tiles, both shapes of the rule, captured replays and the allocation-free
run; what the plan reports stays 64 x 32."""
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["auto", "saturated"])
@pytest.mark.parametrize("n", [(1, 1, 1), (17, 9, 3), (33, 31, 70), (64, 65, 66), (5, 4, 700), (250, 250, 250)])
def test_defaults_equal_given_tile(variant, n):
    from paper_2306_13002_amd.stencil import Plan
    a, b, v = (torch.tensor(x, device="cuda") for x in synth.wave25_inputs(*n, seed=7))
    kw = dict(coef=synth.WAVE25_COEF)
    with Plan("wave25", n, variant=variant, **kw) as p, Plan("wave25", n, variant="saturated", tile=(32, 16, 8), **kw) as q:
        assert p.config()["variant"] == "saturated" and tuple(p.config()["tile"]) == (64, 32, min(n[2], 256))
        f, h = [a.clone(), b.clone()], [a.clone(), b.clone()]
        p.use_graphs()
        for T in (1, 2, 2, 2, 2, 3):
            p.run(f, [v], iterations=T)
            q.run(h, [v], iterations=T)
            assert torch.equal(f[0], h[0]) and torch.equal(f[1], h[1]), T
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual() + 1e-300
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        p.run_noalloc(f, [v], iterations=3, residual=r)
        q.run(h, [v], iterations=3)
        assert torch.equal(f[0], h[0]) and torch.equal(f[1], h[1])
        assert abs(r.item() - q.residual()) <= 1e-12 * q.residual() + 1e-300
