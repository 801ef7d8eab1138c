"""HEAT2D5 plans of open shape march several sweeps per launch: bit for bit
the one-sweep launches' grid (boundary ring included), at widths around the
strips (64 minus twice the sweeps per launch), heights around the row blocks
and sweep counts around the launches; not-finite cells, pitched rows, the
allocation-free run and captured replays."""
import numpy as np
import pytest

import oracle
from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def plans(n, **kw):
    from paper_2306_13002_amd.stencil import Plan
    return Plan("heat2d5", n, coef=(0.6, 0.1), **kw), Plan("heat2d5", n, coef=(0.6, 0.1), variant="plain",
                                                           tile=(64, 4, 1), **kw)


def fields(u0):
    return [torch.tensor(u0, device="cuda"), torch.full(u0.shape, float("nan"), dtype=torch.float64, device="cuda")]


@pytest.mark.parametrize("nx", [1, 47, 48, 49, 54, 55, 62, 108, 193, 249])
@pytest.mark.parametrize("ny", [1, 4, 5, 33, 200])
def test_equals_single_sweeps(nx, ny):
    u0 = synth.uniform_f64(1, 300 + nx, (ny + 2, nx + 2))
    p, q = plans((nx, ny))
    with p, q:
        assert p.config()["variant"] == "plain" and p.config()["tile"] == (64, 4, 1)
        for T in (1, 2, 3, 5, 8, 10, 13, 16, 17, 33):
            f, h = fields(u0), fields(u0)
            p.run(f, iterations=T)
            q.run(h, iterations=T)
            assert torch.equal(f[0], h[0]), T
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual()


def test_matches_oracle():
    u0 = synth.heat2d5_input(173, ny=91)
    p, q = plans((173, 91))
    with p, q:
        f = fields(u0)
        p.run(f, iterations=10)
        want, wr = oracle.heat(u0, 10, 0.6, 0.1)
        assert np.array_equal(f[0].cpu().numpy(), want)
        assert abs(p.residual() - wr) <= 1e-10 * wr


def test_pitched_and_not_finite():
    n, py = (130, 45), 140
    u0 = synth.uniform_f64(1, 5, (47, 132))
    u0[1, 1], u0[20, 131], u0[45, 60], u0[0, 7] = np.inf, np.nan, -np.inf, np.nan
    host = np.full(46 * py + 132, -7.0)
    at = (np.arange(47)[:, None] * py + np.arange(132)).reshape(-1)
    host[at] = u0.reshape(-1)
    p, q = plans(n, pitch=(py, 0))
    with p, q:
        f, h = ([torch.tensor(host, device="cuda"), torch.full((host.size,), -7.0, dtype=torch.float64, device="cuda")]
                for _ in range(2))
        p.run(f, iterations=7)
        q.run(h, iterations=7)
    got = [x.cpu().numpy() for x in f]
    assert np.array_equal(got[0], h[0].cpu().numpy(), equal_nan=True)
    gap = np.ones(host.size, bool)
    gap[at] = False
    assert (got[0][gap] == -7.0).all() and (got[1][gap] == -7.0).all()


def test_replays_and_noalloc():
    u0 = synth.heat2d5_input(150, ny=70)
    p, q = plans((150, 70))
    with p, q:
        f, h = fields(u0), fields(u0)
        p.use_graphs()
        for T in (10, 10, 10, 1, 10, 6, 6, 6):
            p.run(f, iterations=T)
            q.run(h, iterations=T)
            assert torch.equal(f[0], h[0])
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual()
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        for T in (1, 9):
            p.run_noalloc(f, iterations=T, residual=r)
            q.run(h, iterations=T)
            assert torch.equal(f[0], h[0])
            assert abs(r.item() - q.residual()) <= 1e-12 * q.residual()
