"""Flat and thin grids whose default launch would exceed the allocation-free
run's 2^17 residual partials run in the reported shape instead: accepted, and
the grid a plan of given tile produces, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    ("heat3d7", (1, 3_600_000, 1), "saturated_t3", (28, 28, 1), dict(coef=(0.4, 0.1)), 3),
    ("wave25", (1, 1_300_000, 1), "saturated", (64, 32, 1), dict(coef=(-2.8, 1.6, -0.2, 0.025, -0.0018)), 2),
]


@pytest.mark.parametrize("kind,n,variant,tile,kw,T", CASES, ids=[c[0] for c in CASES])
def test_noalloc_accepts_what_the_reported_shape_fits(kind, n, variant, tile, kw, T):
    from paper_2306_13002_amd.stencil import Plan
    r = 1 if kind == "heat3d7" else 4
    shape = [e + 2 * r for e in reversed(n)]
    u = torch.rand(shape, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    with Plan(kind, n, variant=variant, **kw) as p, Plan(kind, n, variant=variant, tile=tile, **kw) as q:
        got, want = [u, u.clone()], [u.clone(), u.clone()]
        cs = [torch.full(shape, 0.02, dtype=torch.float64, device="cuda")] if kind == "wave25" else None
        res = torch.zeros(1, dtype=torch.float64, device="cuda")
        p.run_noalloc(got, cs, iterations=T, residual=res)
        q.run(want, cs, iterations=T)
        assert torch.equal(got[0], want[0])
        assert abs(res.item() - q.residual()) <= 1e-12 * q.residual()
