"""Plans whose launch shape a tuner picked: they produce the grids of the form
they report, under both boundary conditions."""
import numpy as np
import pytest

import oracle
from paper_2306_13002_amd import synth
from gpu_util import inner, maxrel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def run(u0, n, T, kind="heat3d7", coef=(0.4, 0.1), **kw):
    from paper_2306_13002_amd.stencil import Plan
    with Plan(kind, n, coef=coef, **kw) as p:
        f = [torch.tensor(u0, device="cuda"), torch.full(u0.shape, float("nan"), dtype=torch.float64, device="cuda")]
        p.run(f, iterations=T)
        return f[0].cpu().numpy(), p.residual(), p.config()


@pytest.mark.parametrize("tune", ["exhaustive", "model"])
@pytest.mark.parametrize("n", [(96, 96, 96), (160, 70, 64), (8, 9, 10)])
@pytest.mark.parametrize("T", [2, 5])
def test_tuned_periodic_plans_match_the_oracle(tune, n, T):
    u0 = synth.uniform_f64(4, 60 + n[0], tuple(e + 2 for e in reversed(n)))
    got, gr, cfg = run(u0, n, T, tune=tune, bc="periodic")
    assert cfg["variant"] in ("plain", "saturated")
    want, wr = oracle.heat(u0, T, 0.4, 0.1, periodic=True)
    assert maxrel(inner(got, 1), inner(want, 1)) <= 1e-12
    assert abs(gr - wr) <= 1e-10 * wr


@pytest.mark.parametrize("bc", ["dirichlet", "periodic"])
@pytest.mark.parametrize("n", [(8, 9, 10), (30, 12, 20), (96, 50, 40)])
def test_exhaustive_plans_give_the_reported_form(n, bc):
    """Bit for bit the grids of a plan of the reported form and shape."""
    u0 = synth.uniform_f64(4, 80 + n[0], tuple(e + 2 for e in reversed(n)))
    got, gr, cfg = run(u0, n, 4, tune="exhaustive", bc=bc)
    want, wr, _ = run(u0, n, 4, bc=bc, **cfg)
    assert np.array_equal(got, want)
    assert abs(gr - wr) <= 1e-12 * wr


@pytest.mark.parametrize("n", [(256, 200), (31, 17)])
def test_exhaustive_heat2d5_gives_the_plain_grid(n):
    u0 = synth.heat2d5_input(n[0], ny=n[1])
    got, _, cfg = run(u0, n, 9, kind="heat2d5", coef=(0.6, 0.1), tune="exhaustive")
    assert cfg["variant"] == "plain"
    want, _ = oracle.heat(u0, 9, 0.6, 0.1)
    assert np.array_equal(got, want)
