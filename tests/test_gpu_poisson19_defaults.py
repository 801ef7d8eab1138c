"""POISSON19 plans of open shape pick tile and z-block by size and AUTO makes
two sweeps per pass: bit for bit the single saturated sweeps of a given tile,
for sweep counts around the pass, sizes around the tiles, captured replays and
the allocation-free run; what the plan reports stays its form's shape."""
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant,shape", [("auto", ("saturated", (128, 4))), ("saturated", ("saturated", (128, 4))),
                                           ("saturated_t2", ("saturated_t2", (64, 8)))])
@pytest.mark.parametrize("n", [(1, 1, 1), (31, 31, 31), (33, 9, 5), (64, 60, 70), (130, 17, 40)])
def test_defaults_equal_single_sweeps(variant, shape, n):
    from paper_2306_13002_amd.stencil import Plan
    p0, cf = synth.poisson19_random_inputs(tuple(e + 2 for e in reversed(n)), seed=5)
    cs = [torch.tensor(c, device="cuda") for c in cf]
    with Plan("poisson19", n, variant=variant, omega=0.8) as p, Plan("poisson19", n, variant="saturated", omega=0.8,
                                                                     tile=(32, 4, 4)) as q:
        assert p.config()["variant"] == shape[0] and tuple(p.config()["tile"][:2]) == shape[1]
        f, h = ([torch.tensor(p0, device="cuda"), torch.full(p0.shape, float("nan"), device="cuda")] for _ in range(2))
        p.use_graphs()
        for T in (1, 2, 3, 3, 3, 3, 4, 1):
            p.run(f, cs, iterations=T)
            q.run(h, cs, iterations=T)
            assert torch.equal(f[0], h[0]), T
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual() + 1e-300
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        for T in (1, 5):
            p.run_noalloc(f, cs, iterations=T, residual=r)
            q.run(h, cs, iterations=T)
            assert torch.equal(f[0], h[0])
            assert abs(r.item() - q.residual()) <= 1e-12 * q.residual() + 1e-300
