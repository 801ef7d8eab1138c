"""GENERIC plans over grids that stream from memory (F64, radius 1 and 2; their
own default tiles): the grid of a plan of given tile, bit for bit, the residual
and the untouched halo, at sizes on both sides of the rules."""
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tile", [((200, 190, 160), None), ((257, 190, 160), (64, 4, 8)), ((63, 400, 300), None),
                                    ((301, 270, 261), (64, 4, 16))])
@pytest.mark.parametrize("r,shape", [(1, "star"), (2, "star")])
def test_streaming_defaults(n, tile, r, shape):
    from paper_2306_13002_amd.stencil import Plan
    taps = synth.star_taps(r) if shape == "star" else synth.box_taps(r)
    kw = dict(dtype="f64", radius=r, taps=taps, cids=[0] + [1] * (len(taps) - 1), variant="saturated",
              coef=[0.4, 0.6 / (len(taps) - 1)])
    u = torch.rand([e + 2 * r for e in reversed(n)], dtype=torch.float64, device="cuda",
                   generator=torch.Generator(device="cuda").manual_seed(7))
    with Plan("generic", n, **kw) as p, Plan("generic", n, tile=(32, 32, 16), **kw) as q:
        if r == 1 and tile:
            assert p.config()["tile"] == tile
        for T in (1, 2):
            a, b = [u.clone(), torch.full_like(u, float("nan"))], [u.clone(), torch.full_like(u, float("nan"))]
            p.run(a, iterations=T)
            q.run(b, iterations=T)
            assert torch.equal(a[0], b[0])
            assert abs(p.residual() - q.residual()) <= 1e-12 * q.residual()
        inner = tuple(slice(r, -r) for _ in range(3))
        a[0][inner] = u[inner]
        assert torch.equal(a[0], u)
