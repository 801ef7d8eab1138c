"""Flat GENERIC grids whose default tile would leave more than 2^17 residual
partials: the allocation-free run (the table-driven kernel's) takes them, and
gives the grid of a plan of given tile."""
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [((1, 60_000, 60), "f64"), ((68_813, 67, 65), "f32"), ((603_251, 51, 16), "f64")])
@pytest.mark.parametrize("shape", ["star", "box"])
def test_flat_grid_runs_without_allocation(monkeypatch, n, dtype, shape):
    from paper_2306_13002_amd.stencil import Plan
    monkeypatch.setenv("STENCIL_GENERIC_TABLE", "1")
    taps = synth.star_taps(1) if shape == "star" else synth.box_taps(1)
    kw = dict(dtype=dtype, radius=1, taps=taps, cids=list(range(len(taps))),
              coef=[1.0 / len(taps)] * len(taps), variant="saturated")
    u = torch.rand([e + 2 for e in reversed(n)], dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda",
                   generator=torch.Generator(device="cuda").manual_seed(4))
    got, want = [u.clone(), u.clone()], [u.clone(), u.clone()]
    res = torch.zeros(1, dtype=torch.float64, device="cuda")
    with Plan("generic", n, **kw) as p, Plan("generic", n, tile=(64, 4, 16), **kw) as q:
        p.run_noalloc(got, iterations=2, residual=res)
        q.run(want, iterations=2)
        assert torch.equal(got[0], want[0])
        assert abs(res.item() - q.residual()) <= 1e-12 * q.residual()
