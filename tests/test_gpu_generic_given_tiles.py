"""GENERIC plans of given tile, with one row per thread (few blocks) or the
tile's own rows (many): every tile of a stencil gives the same grid, bit for
bit, within the rounding of the oracle's (see test_gpu_generic_rows); narrow
and wide pitches of one stencil do not take each other's kernels."""
import numpy as np
import pytest

import oracle
from gpu_util import inner, maxrel
from test_gpu_generic_rows import TOL, shared, stencil

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILES = [(32, 4), (32, 8), (64, 2), (64, 4), (128, 2), (32, 16), (32, 32), (64, 16)]


def run(st, T=2, **kw):
    from paper_2306_13002_amd.stencil import Plan
    with Plan("generic", st["n"], dtype=st["dtype"], radius=st["radius"], coef=st["coef"], taps=st["taps"],
              cids=st["cids"], variant="saturated", **kw) as p:
        f = [torch.tensor(st["u0"], device="cuda"), torch.tensor(st["u0"], device="cuda")]
        p.run(f, iterations=T)
        return f[0].cpu().numpy(), p.residual()


@pytest.mark.parametrize("n,zb", [((37, 22, 13), 4), ((37, 22, 13), 64), ((130, 131, 120), 2)])
@pytest.mark.parametrize("r,shape,pattern,dtype", [(2, "box", "partition", "f64"), (4, "star", "reflection", "f64"),
                                                   (1, "box", "symmetric", "f64"), (3, "box", "symmetric", "f32"),
                                                   (2, "box", "distinct", "f32"), (1, "star", "symmetric", "f64")])
def test_every_tile_gives_the_same_grid(n, zb, r, shape, pattern, dtype):
    taps, cids = shared(r, shape, pattern)
    st = stencil(r, taps, cids, dtype, n)
    first, res = run(st)  # the default tile
    want, _ = oracle.generic(st["u0"], r, taps, cids, st["coef"], 2)
    assert maxrel(inner(first, r), inner(want, r)) <= TOL[dtype]
    for tile in TILES:
        got, gr = run(st, tile=(*tile, zb))
        assert np.array_equal(got, first), tile
        assert abs(gr - res) <= 1e-12 * res


def test_narrow_and_wide_pitches_in_turn():
    from paper_2306_13002_amd.stencil import Plan
    taps, cids = shared(1, "box", "reflection")
    st = stencil(1, taps, cids, "f64", (70, 2, 2), seed=5)
    want, _ = oracle.generic(st["u0"], 1, taps, cids, st["coef"], 1)
    for py in (72, 24_000_000, 80):  # 18 rows of 24e6 doubles span 3.5 GB, of the 32-row tile 6.5 GB
        at = (torch.arange(4)[:, None, None] * (4 * py) + torch.arange(4)[None, :, None] * py
              + torch.arange(72)[None, None, :]).reshape(-1).cuda()
        f = [torch.zeros(15 * py + 72, dtype=torch.float64, device="cuda") for _ in range(2)]
        f[0][at] = torch.tensor(st["u0"], device="cuda").reshape(-1)
        for tile in ((32, 32, 2), (64, 4, 1)):
            g = [x.clone() for x in f]
            with Plan("generic", st["n"], dtype="f64", radius=1, coef=st["coef"], taps=taps, cids=cids,
                      variant="saturated", pitch=(py, 4 * py), tile=tile) as p:
                p.run(g, iterations=1)
            got = g[0][at].cpu().numpy().reshape(st["u0"].shape)
            assert maxrel(inner(got, 1), inner(want, 1)) <= TOL["f64"], (py, tile)
