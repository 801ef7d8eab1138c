"""Plans whose launch shape a tuner picked: they produce the grids of the form
they report, under both boundary conditions."""
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
