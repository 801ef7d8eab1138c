"""The scratch grid's halo where rows are long enough to be cut into pieces:
the input's halo, cell for cell, and nothing outside the grid, in two and three
dimensions, single plans and batches."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(u, v, nx, ny, r, three):
    """u: padded input (z, y, pitch) before the run, v: the scratch grid after."""
    own = torch.zeros(u.shape, dtype=torch.bool, device="cuda")
    own[:, : ny + 2 * r, : nx + 2 * r] = True
    inner = torch.zeros_like(own)
    z = slice(r, u.shape[0] - r) if three else slice(0, 1)
    inner[z, r : ny + r, r : nx + r] = True
    assert torch.equal(v[own & ~inner], u[own & ~inner])
    assert bool((v[~own] == -7.0).all())


@pytest.mark.parametrize("nx", [1016, 1022, 1023, 1278, 1279, 3000])
@pytest.mark.parametrize("kind,ny,nz,r", [("heat2d5", 3, 1, 1), ("generic", 2, 3, 1), ("generic", 3, 1, 4)])
def test_long_rows(kind, ny, nz, r, nx):
    from paper_2306_13002_amd.stencil import Plan
    py = nx + 2 * r + 3
    shape = (1 if kind == "heat2d5" else nz + 2 * r, ny + 2 * r, py)
    u = torch.rand(shape, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(nx))
    v = torch.full_like(u, -7.0)
    a = u.clone()
    if kind == "heat2d5":
        plan = Plan(kind, (nx, ny), coef=(0.6, 0.1), variant="plain", tile=(64, 4, 1), pitch=(py, 0))
    else:
        plan = Plan(kind, (nx, ny, nz), dtype="f64", radius=r, taps=[(0, 0, 0), (r, 0, 0), (0, -r, 0), (0, 0, r)],
                    cids=[0, 1, 1, 1], coef=[0.5, 0.1], pitch=(py, py * (ny + 2 * r)))
    with plan as p:
        p.run([u.view(-1), v.view(-1)], iterations=2)
    check(a, v, nx, ny, r, kind != "heat2d5")


def test_long_rows_of_a_batch():
    from paper_2306_13002_amd.stencil import BatchPlan
    sizes = [(1500, 2, 3), (1510, 3, 2), (1500, 1, 1)]
    us = [torch.rand([e + 2 for e in reversed(n)], dtype=torch.float64, device="cuda") for n in sizes]
    fs = [(u.clone(), torch.full_like(u, -7.0)) for u in us]
    with BatchPlan(sizes, variant="saturated", tile=(32, 8, 4)) as b:
        b.run(fs, iterations=2)
    for n, u, (_, v) in zip(sizes, us, fs):
        check(u, v, n[0], n[1], 1, True)
