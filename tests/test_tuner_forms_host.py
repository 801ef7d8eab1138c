"""The forms the tuners may pick (no GPU needed): several sweeps per launch
only where the boundary is fixed, since a periodic halo is filled again before
every sweep."""
import pytest

from paper_2306_13002_amd import stencil as S


@pytest.mark.parametrize("kind,n,coef", [("heat2d5", (70, 70), (0.6, 0.1)), ("heat3d7", (70, 70, 70), (0.4, 0.1))])
def test_periodic_candidates_are_single_sweeps(kind, n, coef):
    fixed = S.candidates(kind, n, coef=coef)
    per = S.candidates(kind, n, coef=coef, bc="periodic")
    assert per and {v for v, _, _ in per} <= {"plain", "saturated"}
    assert set(per) <= set(fixed)
    assert kind == "heat2d5" or {v for v, _, _ in fixed} == {"plain", "saturated", "saturated_t2", "saturated_t3"}
