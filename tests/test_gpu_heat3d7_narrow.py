"""HEAT3D7 plans of open shape on narrow and flat grids, where the default is
the LDS tile in place of a register tile: the grids of a plan of given tile,
bit for bit, the scratch grid's halo, the allocation-free run, replays, a batch
and both boundary conditions."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rand(n, seed):
    return torch.rand([e + 2 for e in reversed(n)], dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(seed))


@pytest.mark.parametrize("variant,n,bc", [("saturated", (20, 300, 300), "dirichlet"), ("saturated", (64, 150, 200), "periodic"),
                                          ("saturated", (1, 400, 300), "periodic"), ("saturated_t2", (3, 3, 4000), "dirichlet"),
                                          ("saturated_t2", (64, 3, 2000), "dirichlet"), ("auto", (20, 300, 300), "dirichlet")])
def test_narrow_grids(variant, n, bc):
    from paper_2306_13002_amd.stencil import Plan
    u0 = rand(n, 3)
    halo = torch.ones(u0.shape, dtype=torch.bool, device="cuda")
    halo[1:-1, 1:-1, 1:-1] = False
    with Plan("heat3d7", n, variant=variant, coef=(0.4, 0.1), bc=bc) as p, \
            Plan("heat3d7", n, variant="saturated", coef=(0.4, 0.1), bc=bc, tile=(32, 8, 4)) as q:
        p.use_graphs()
        for T in (1, 2, 3, 4, 4, 4):
            a, b = ([u0.clone(), torch.full_like(u0, float("nan"))] for _ in range(2))
            p.run(a, iterations=T)
            q.run(b, iterations=T)
            assert torch.equal(a[0], b[0]), T
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual()
            assert bc == "periodic" or torch.equal(a[1][halo], u0[halo])
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        a = [u0.clone(), torch.full_like(u0, float("nan"))]
        p.run_noalloc(a, iterations=4, residual=r)
        assert torch.equal(a[0], b[0]) and abs(r.item() - q.residual()) <= 1e-12 * q.residual()


@pytest.mark.parametrize("variant", ["saturated", "saturated_t2"])
def test_narrow_batch(variant):
    from paper_2306_13002_amd.stencil import BatchPlan, Plan
    sizes = [(4, 120, 120)] * 40 + [(9, 100, 97), (1, 98, 128)]
    us = [rand(n, i) for i, n in enumerate(sizes)]
    fs = [(u.clone(), torch.full_like(u, float("nan"))) for u in us]
    with BatchPlan(sizes, variant=variant) as b:
        for _ in range(2):
            for (x, _), u in zip(fs, us):
                x.copy_(u)
            b.run(fs, iterations=3)
    for n, u, (x, _) in zip(sizes, us, fs):
        with Plan("heat3d7", n, variant="saturated", coef=(0.4, 0.1), tile=(32, 8, 4)) as q:
            w = [u.clone(), u.clone()]
            q.run(w, iterations=3)
        assert torch.equal(x, w[0])
