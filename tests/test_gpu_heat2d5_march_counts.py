"""Marching HEAT2D5 runs of any sweep count: bit for bit the one-sweep launches'
grid, in an even number of launches of at most eight sweeps that share the
count evenly, so that the result is not copied back -- the scratch grid then
holds the state before the last launch."""
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [3, 15, 16, 17, 31, 33, 49, 50, 97, 100, 113, 120, 121])
def test_counts(T):
    from paper_2306_13002_amd.stencil import Plan
    n = (150, 70)
    u0 = torch.tensor(synth.heat2d5_input(n[0], ny=n[1]), device="cuda")
    launches = 2 * -(-T // 16)
    last = T // launches  # the first T % launches launches do one sweep more
    with Plan("heat2d5", n, coef=(0.6, 0.1)) as p, Plan("heat2d5", n, coef=(0.6, 0.1), variant="plain",
                                                        tile=(64, 4, 1)) as q:
        f, h, before = ([u0.clone(), torch.full_like(u0, float("nan"))] for _ in range(3))
        p.run(f, iterations=T)
        got = p.residual()
        q.run(before, iterations=T - last)
        q.run(h, iterations=T)
        assert torch.equal(f[0], h[0])
        assert abs(got - q.residual()) <= 1e-12 * q.residual()
        assert torch.equal(f[1], before[0])
        p.use_graphs()
        for _ in range(3):
            f[0].copy_(u0)
            p.run(f, iterations=T)
            assert torch.equal(f[0], h[0]) and torch.equal(f[1], before[0])
