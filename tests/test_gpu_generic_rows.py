"""GPU parity of the generated GENERIC kernels with several rows per thread
against the CPU oracle, where a tile, a block in z or an emitted sum can go
wrong.

The kernels add the same products in another order than the oracle.  Both are
sums of N positive FP64 terms per point (coefficients sum to 1), so each is
within (N + 1) 2^-53 of the exact one in any order and the two within
2 (N + 1) 2^-53 <= 1.7e-13 for N <= 729, per sweep; two sweeps: 4e-13.  F32
storage rounds the result once per sweep (2^-24 each on both sides, and the
first sweep's difference carries over): 2e-7."""
import numpy as np
import pytest

import oracle
from paper_2306_13002_amd import synth
from gpu_util import inner, maxrel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 4e-13, "f32": 2e-7}


def stencil(r, taps, cids, dtype, n, seed=0):
    u = iter(synth.uniform_f64(9, 300 + seed, (1024,)))
    vals = [0.1 + 0.9 * next(u) for _ in range(max(cids) + 1)]
    tot = sum(vals[c] for c in cids)
    return dict(radius=r, taps=taps, cids=cids, coef=[v / tot for v in vals], dtype=dtype, n=n,
                u0=synth.generic_input(n, r, dtype, seed=9, stream=40 + seed))


def shared(r, shape, pattern):
    taps = synth.box_taps(r) if shape == "box" else synth.star_taps(r)
    cids, _ = synth.sharing_ids(taps, pattern, iter(synth.uniform_f64(9, 77 + r, (4096,))))
    return taps, cids


def check(st, T=2, **kw):
    from paper_2306_13002_amd.stencil import Plan
    tdt = torch.float32 if st["dtype"] == "f32" else torch.float64
    with Plan("generic", st["n"], dtype=st["dtype"], radius=st["radius"], coef=st["coef"], taps=st["taps"],
              cids=st["cids"], variant="saturated", **kw) as p:
        f = [torch.tensor(st["u0"], device="cuda"), torch.full(st["u0"].shape, float("nan"), dtype=tdt, device="cuda")]
        p.run(f, iterations=T)
        got, gr, cfg = f[0].cpu().numpy(), p.residual(), p.config()
    w, _ = oracle.generic(st["u0"], st["radius"], st["taps"], st["cids"], st["coef"], T)
    _, wr = oracle.generic(st["u0"], st["radius"], st["taps"], st["cids"], st["coef"], T,
                           mode="F32STORE" if st["dtype"] == "f32" else "F64")
    r = st["radius"]
    assert maxrel(inner(got, r), inner(w, r)) <= TOL[st["dtype"]]
    assert np.array_equal(got[:r], st["u0"][:r]) and np.array_equal(got[:, :, -r:], st["u0"][:, :, -r:])
    assert abs(gr - wr) <= (1e-5 if st["dtype"] == "f32" else 1e-10) * wr
    return cfg


@pytest.mark.parametrize("tile", [(32, 16), (64, 16), (32, 32)])
@pytest.mark.parametrize("n,zb", [((1, 1, 1), 1), ((33, 17, 9), 4), ((64, 16, 8), 8), ((130, 35, 11), 3),
                                  ((65, 47, 21), 64)])
@pytest.mark.parametrize("r,shape,pattern,dtype", [(3, "box", "symmetric", "f64"), (2, "box", "distinct", "f32"),
                                                   (4, "star", "reflection", "f32"), (1, "box", "partition", "f64")])
def test_rows_tiles_and_blocks(tile, n, zb, r, shape, pattern, dtype):
    taps, cids = shared(r, shape, pattern)
    check(stencil(r, taps, cids, dtype, n), tile=(tile[0], tile[1], zb))


ODD = {
    "one corner tap": (2, [(2, -2, 1)], [0]),
    "one plane": (2, [(x, y, 0) for y in (-2, 0, 1) for x in (-1, 0, 2)], [0, 1, 2, 0, 1, 2, 0, 1, 2]),
    "column only": (4, [(0, 0, z) for z in range(-4, 5)], [0, 1, 2, 3, 4, 3, 2, 1, 0]),
    "a tap named twice": (1, [(1, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 0, 1), (0, 0, 1)], [0, 0, 0, 1, 2]),
    "mirrored rows, one side longer": (3, [(x, y, z) for z in (-3, 3) for y in (-3, 3) for x in (-2, 2)] +
                                       [(1, 3, 3), (0, 0, 0)], [0] * 8 + [0, 1]),
    "shared shape, other coefficients": (1, synth.box_taps(1), [0] * 9 + [1] * 9 + [2] * 9),
    "large box, not unrolled": (4, synth.box_taps(4), list(range(729))),
}


@pytest.mark.parametrize("name", sorted(ODD))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_rows_odd_stencils(name, dtype):
    r, taps, cids = ODD[name]
    check(stencil(r, taps, cids, dtype, (37, 22, 13)))


@pytest.mark.parametrize("n", [(64, 64, 64), (70, 33, 130), (257, 5, 6)])
def test_default_tile_is_offered_and_fits(n):
    for r, shape, pattern in ((1, "star", "distinct"), (3, "box", "symmetric"), (2, "box", "distinct")):
        taps, cids = shared(r, shape, pattern)
        cfg = check(stencil(r, taps, cids, "f32", n), T=1)
        assert cfg["variant"] == "saturated" and cfg["tile"][1] in (4, 8, 16, 32) and cfg["tile"][2] in (2, 4, 8, 16, 32, 64)


@pytest.mark.parametrize("kw,tile", [(dict(tile=(32, 0, 0)), (32, 4, 16)), (dict(tile=(0, 2, 0)), (64, 2, 16)),
                                     (dict(tile=(0, 0, 5)), None)])
def test_partly_given_tiles(kw, tile):
    taps, cids = shared(1, "box", "distinct")
    cfg = check(stencil(1, taps, cids, "f64", (45, 20, 18)), **kw)
    assert cfg["tile"] == tile if tile else cfg["tile"][2] == 5


def test_rows_of_a_tile_beyond_4_gib():
    """A row pitch whose tile needs 64-bit lane offsets (18 rows x 24e6 x 8 B)."""
    from paper_2306_13002_amd.stencil import Plan
    taps, cids = shared(1, "box", "reflection")
    st = stencil(1, taps, cids, "f64", (70, 2, 2))
    py = 24_000_000
    at = (torch.arange(4)[:, None, None] * (4 * py) + torch.arange(4)[None, :, None] * py
          + torch.arange(72)[None, None, :]).reshape(-1).cuda()
    f = [torch.zeros(15 * py + 72, dtype=torch.float64, device="cuda") for _ in range(2)]
    f[0][at] = torch.tensor(st["u0"], device="cuda").reshape(-1)
    with Plan("generic", st["n"], dtype="f64", radius=1, coef=st["coef"], taps=taps, cids=cids, variant="saturated",
              pitch=(py, 4 * py)) as p:
        p.run(f, iterations=1)
    got = f[0][at].cpu().numpy().reshape(st["u0"].shape)
    w, _ = oracle.generic(st["u0"], 1, taps, cids, st["coef"], 1)
    assert maxrel(inner(got, 1), inner(w, 1)) <= TOL["f64"]
