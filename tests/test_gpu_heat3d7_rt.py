"""HEAT3D7 register tiles: every form and tile equals single saturated sweeps
of the LDS tile (32 x 8) bit for bit, on grids at the edges of the tiles, the
waves and the z-blocks; a batch equals its problems' single plans; cells that
are not finite stay what they are."""
import numpy as np
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILES = {"saturated": [(62, 6), (62, 14), (60, 12), (60, 28), (60, 44)],
         "saturated_t2": [(60, 12), (60, 28), (60, 44)],
         "saturated_t3": [(58, 10), (58, 26), (58, 42)]}
CASES = [(v, t) for v in TILES for t in TILES[v]]
GRIDS = [((1, 1, 1), 1), ((58, 26, 5), 2), ((59, 27, 9), 3), ((62, 14, 8), 8), ((63, 15, 33), 16), ((130, 85, 21), 4)]


def run(u0, n, T, **kw):
    from paper_2306_13002_amd.stencil import Plan
    with Plan("heat3d7", n, coef=(0.4, 0.1), **kw) as p:
        f = [torch.tensor(u0, device="cuda"), torch.full(u0.shape, float("nan"), dtype=torch.float64, device="cuda")]
        p.run(f, iterations=T)
        return f[0].cpu().numpy(), p.residual(), p.config()


@pytest.mark.parametrize("variant,tile", CASES)
@pytest.mark.parametrize("n,zb", GRIDS)
def test_equals_single_sweeps(variant, tile, n, zb):
    u0 = synth.uniform_f64(4, 900 + n[0], tuple(e + 2 for e in reversed(n)))  # a boundary that is not 0
    for T in (1, 2, 3, 5):
        want, wr, _ = run(u0, n, T, variant="saturated", tile=(32, 8, 4))
        got, gr, cfg = run(u0, n, T, variant=variant, tile=(tile[0], tile[1], zb))
        assert cfg["tile"] == (tile[0], tile[1], zb)
        assert np.array_equal(got, want)
        assert abs(gr - wr) <= 1e-12 * wr  # the same squares, summed in another order


@pytest.mark.parametrize("variant", ["auto", "saturated", "saturated_t2", "saturated_t3"])
def test_defaults_pitched_and_odd_values(variant):
    """The default tile, rows and planes with gaps, and inf and NaN cells in
    the grid and on the boundary."""
    from paper_2306_13002_amd.stencil import Plan
    n, py, pz = (70, 33, 20), 75, 75 * 35 + 11
    u0 = synth.uniform_f64(4, 77, (22, 35, 72))
    u0[5, 1, 1], u0[9, 30, 60], u0[0, 3, 3], u0[12, 0, 71] = np.inf, np.nan, -np.inf, np.nan
    want, _, _ = run(u0, n, 4, variant="saturated", tile=(32, 8, 4))
    size = 21 * pz + 34 * py + 72
    host = np.full(size, -7.0)
    at = (np.arange(22)[:, None, None] * pz + np.arange(35)[None, :, None] * py + np.arange(72)).reshape(-1)
    host[at] = u0.reshape(-1)
    f = [torch.tensor(host, device="cuda"), torch.full((size,), -7.0, dtype=torch.float64, device="cuda")]
    with Plan("heat3d7", n, coef=(0.4, 0.1), variant=variant, pitch=(py, pz)) as p:
        p.run(f, iterations=4)
    got = f[0].cpu().numpy()
    assert np.array_equal(got[at].reshape(u0.shape), want, equal_nan=True)
    gap = np.ones(size, bool)
    gap[at] = False
    assert (got[gap] == -7.0).all() and (f[1].cpu().numpy()[gap] == -7.0).all()


@pytest.mark.parametrize("variant", ["auto", "saturated", "saturated_t2", "saturated_t3"])
@pytest.mark.parametrize("T", [1, 3, 4])
def test_batch_defaults(variant, T):
    from paper_2306_13002_amd.stencil import BatchPlan
    sizes = [(33, 20, 17), (64, 64, 64), (70, 41, 23), (96, 5, 90), (130, 120, 9)]
    us = [synth.heat3d7_input(*n, stream=60 + i) for i, n in enumerate(sizes)]
    fs = [(torch.tensor(u, device="cuda"), torch.zeros(u.shape, dtype=torch.float64, device="cuda")) for u in us]
    with BatchPlan(sizes, variant=variant) as bp:
        bp.run(fs, iterations=T)
        res = bp.residuals()
    for i, n in enumerate(sizes):
        want, wr, _ = run(us[i], n, T, variant="saturated", tile=(32, 8, 4))
        assert np.array_equal(fs[i][0].cpu().numpy(), want)
        assert abs(res[i] - wr) <= 1e-12 * wr


def test_auto_runs_between_sweep_counts():
    """Runs of one sweep and of several on one plan (other launches, other
    residual partials), the allocation-free run and captured replays."""
    from paper_2306_13002_amd.stencil import Plan
    n = (70, 33, 20)
    u0 = synth.heat3d7_input(*n, stream=71)
    with Plan("heat3d7", n, coef=(0.4, 0.1)) as p, Plan("heat3d7", n, coef=(0.4, 0.1), variant="saturated",
                                                        tile=(32, 8, 4)) as q:
        assert p.config()["variant"] == "saturated" and p.config()["tile"] == (32, 8, 8)
        f, h = ([torch.tensor(u0, device="cuda"), torch.zeros(u0.shape, dtype=torch.float64, device="cuda")]
                for _ in range(2))
        p.use_graphs()
        for T in (4, 1, 3, 3, 3, 3, 1, 1, 1, 2, 6):
            p.run(f, iterations=T)
            q.run(h, iterations=T)
            assert torch.equal(f[0], h[0])
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual()
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        for T in (1, 5):
            p.run_noalloc(f, iterations=T, residual=r)
            q.run(h, iterations=T)
            assert torch.equal(f[0], h[0])
            assert abs(r.item() - q.residual()) <= 1e-12 * q.residual()
