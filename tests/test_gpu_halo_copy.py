"""The scratch grid's halo after a run: the input's halo, cell for cell, for
every halo width, with rows shorter and longer than a wave's four chunks,
pitched rows and planes, both element types; nothing outside it and the
interior is written."""
import pytest


torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1, 1, 1), (255, 3, 2), (300, 5, 4), (61, 70, 9)])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_halo_of_scratch_is_the_inputs(n, r, dtype):
    from paper_2306_13002_amd.stencil import Plan
    nx, ny, nz = n
    py, pz = nx + 2 * r + 5, (nx + 2 * r + 5) * (ny + 2 * r + 2)
    taps = [(0, 0, 0), (r, 0, 0), (0, -r, 0), (0, 0, r)]
    t = torch.float64 if dtype == "f64" else torch.float32
    u = torch.arange(1, pz * (nz + 2 * r) + 1, dtype=t, device="cuda").reshape(nz + 2 * r, -1)
    v = torch.full_like(u, -7.0)
    views = [w[:, : (ny + 2 * r + 2) * py].reshape(nz + 2 * r, ny + 2 * r + 2, py) for w in (u, v)]
    with Plan("generic", n, dtype=dtype, radius=r, taps=taps, cids=[0, 1, 1, 1], coef=[0.5, 0.1],
              pitch=(py, pz)) as p:
        a = views[0].clone()
        p.run([u, v], iterations=2)  # two sweeps end in u and leave the scratch as the first left it
    own = torch.zeros(views[0].shape, dtype=torch.bool, device="cuda")
    own[:, : ny + 2 * r, : nx + 2 * r] = True
    inner = torch.zeros_like(own)
    inner[r : nz + r, r : ny + r, r : nx + r] = True
    assert torch.equal(views[1][own & ~inner], a[own & ~inner])
    assert bool((views[1][~own] == -7.0).all()) and torch.equal(views[0][~inner], a[~inner])
