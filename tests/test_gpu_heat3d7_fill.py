"""The first launch of a HEAT3D7 run in register tiles stores the scratch grid's
halo: every cell of it is the input's (corners too), nothing else outside the
interior is written, and the grid equals single sweeps of a given tile, bit for
bit, for one tile and several per axis, ragged last tiles, halo values of any
kind, pitched rows, replays and the allocation-free run."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["auto", "saturated", "saturated_t2", "saturated_t3"])
@pytest.mark.parametrize("n", [(1, 1, 1), (58, 26, 16), (59, 10, 3), (62, 14, 8), (63, 43, 17), (125, 29, 5)])
def test_first_launch_stores_the_halo(variant, n):
    from paper_2306_13002_amd.stencil import Plan
    nx, ny, nz = n
    py = nx + 2 + 3
    pz = py * (ny + 2) + 5
    u0 = torch.rand((nz + 2) * pz, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
    idx = torch.arange((nz + 2) * pz, device="cuda")
    z, rest = idx // pz, idx % pz
    y, x = rest // py, rest % py
    own = (y < ny + 2) & (x < nx + 2)
    inner = own & (z >= 1) & (z <= nz) & (y >= 1) & (y <= ny) & (x >= 1) & (x <= nx)
    halo = own & ~inner
    u0[halo & (idx % 7 == 0)] = -0.0
    with Plan("heat3d7", n, variant=variant, coef=(0.4, 0.1), pitch=(py, pz)) as p, \
            Plan("heat3d7", n, variant="saturated", coef=(0.4, 0.1), pitch=(py, pz), tile=(32, 8, 4)) as q:
        p.use_graphs()
        for T in (1, 2, 3, 4, 4, 4, 4, 7):
            a, b = [u0.clone(), torch.full_like(u0, float("nan"))], [u0.clone(), torch.full_like(u0, float("nan"))]
            p.run(a, iterations=T)
            q.run(b, iterations=T)
            assert torch.equal(a[0], b[0]), T
            assert torch.equal(a[1][halo].view(torch.int64), u0[halo].view(torch.int64)), T
            assert bool(a[1][~own].isnan().all()) and torch.equal(a[0][~inner], u0[~inner]), T
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual() + 1e-300
        f = [u0.clone(), torch.full_like(u0, float("nan"))]
        for T in (4, 4, 4, 4):  # the same buffers: replayed
            f[0].copy_(u0)
            f[1].fill_(float("nan"))
            p.run(f, iterations=T)
            want = [u0.clone(), torch.full_like(u0, float("nan"))]
            q.run(want, iterations=T)
            assert torch.equal(f[0], want[0]) and torch.equal(f[1][halo], u0[halo])
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        f = [u0.clone(), torch.full_like(u0, float("nan"))]
        p.run_noalloc(f, iterations=4, residual=r)
        assert torch.equal(f[0], want[0]) and torch.equal(f[1][halo], u0[halo])
        assert abs(r.item() - q.residual()) <= 1e-12 * q.residual() + 1e-300


@pytest.mark.parametrize("variant", ["auto", "saturated_t2", "saturated_t3"])
@pytest.mark.parametrize("T", [1, 3, 4, 5])
def test_batch_first_launch_stores_the_halos(variant, T):
    from paper_2306_13002_amd.stencil import BatchPlan, Plan
    sizes = [(1, 1, 1), (59, 27, 9), (40, 90, 33), (130, 20, 64), (7, 100, 5)]
    gen = torch.Generator(device="cuda").manual_seed(4)
    ins = [torch.rand([e + 2 for e in reversed(n)], dtype=torch.float64, device="cuda", generator=gen) for n in sizes]
    fields = [(u.clone(), torch.full_like(u, float("nan"))) for u in ins]
    with BatchPlan(sizes, coef=(0.4, 0.1), variant=variant) as p:
        for rep in range(3):
            for (a, s), u in zip(fields, ins):
                a.copy_(u)
                s.fill_(float("nan"))
            p.run(fields, iterations=T)
            for n, (a, s), u in zip(sizes, fields, ins):
                h = torch.ones(u.shape, dtype=torch.bool, device="cuda")
                h[1:-1, 1:-1, 1:-1] = False
                with Plan("heat3d7", n, variant="saturated", coef=(0.4, 0.1), tile=(32, 8, 4)) as q:
                    w = [u.clone(), torch.empty_like(u)]
                    q.run(w, iterations=T)
                assert torch.equal(a, w[0]) and torch.equal(s[h], u[h]), (rep, n)
