"""Rounding of the saturated GENERIC kernels where coefficients repeat: a
coefficient's taps are summed before they are multiplied, whatever way a kernel
is emitted.

The error of a sweep against long double is compared with that of the plain
statement of that order in FP64 on the host: per plane and coefficient id a
balanced tree over the taps and one FMA into the running sum.  A kernel's trees
may pair the taps otherwise, which leaves the number and the size of the
roundings as they are; the rms over some 20000 points then agrees within a few
per cent, and 15 % are allowed.  (One FMA per tap of the whole stencil is 1.8 to
2.8 times off; one per tap of a plane, added once, is below 1.)"""
import numpy as np
import pytest

from paper_2306_13002_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
LD = np.longdouble


def tree(v):
    if len(v) == 1:
        return v[0]
    m = (len(v) + 1) // 2
    return tree(v[:m]) + tree(v[m:])


def stencil(r, n_ids, shape="box", seed=3):
    taps = synth.box_taps(r) if shape == "box" else synth.star_taps(r)
    rng = np.random.RandomState(seed)
    if n_ids:
        ids = [int(i) for i in np.unique(rng.randint(0, n_ids, len(taps)), return_inverse=True)[1]]
    else:  # one per distance
        ids = [int(np.abs(t).sum()) for t in taps]
    c = 0.1 + 0.9 * rng.random_sample(max(ids) + 1)
    return taps, ids, [float(v) for v in c / c[ids].sum()]


def host(u, r, taps, ids, coef):
    """(exact sweep in long double, the grouped sums in FP64)"""
    cut = lambda a, d: a[tuple(slice(r + e, s - r + e) for s, e in zip(u.shape, (d[2], d[1], d[0])))]  # noqa: E731
    exact = sum(LD(coef[i]) * cut(u, d).astype(LD) for d, i in zip(taps, ids))
    acc = np.zeros_like(cut(u, (0, 0, 0)))
    for dz in range(-r, r + 1):
        for i in range(len(coef)):
            v = [cut(u, d) for d, k in sorted(zip(taps, ids), key=lambda e: e[0][::-1]) if k == i and d[2] == dz]
            if v:
                acc = (LD(coef[i]) * tree(v).astype(LD) + acc.astype(LD)).astype(np.float64)
    return exact, acc


@pytest.mark.parametrize("tile", [(0, 0, 0), (32, 8, 8)])
@pytest.mark.parametrize("shape,r,n_ids", [("box", 1, 3), ("box", 2, 3), ("box", 2, 10), ("box", 2, 40), ("box", 3, 10),
                                           ("box", 3, 100), ("box", 4, 10), ("box", 4, 240), ("star", 1, 0),
                                           ("star", 2, 0), ("star", 3, 0), ("star", 4, 0), ("star", 4, 10)])
def test_no_more_rounding_than_grouped_sums(shape, r, n_ids, tile):
    from paper_2306_13002_amd.stencil import Plan
    taps, ids, coef = stencil(r, n_ids, shape)
    n = (40, 30, 16)
    u = synth.uniform_f64(4, 900 + r, tuple(e + 2 * r for e in reversed(n)))
    with Plan("generic", n, dtype="f64", radius=r, taps=taps, cids=ids, coef=coef, variant="saturated", tile=tile) as p:
        f = [torch.tensor(u, device="cuda"), torch.tensor(u, device="cuda")]
        p.run(f, iterations=1)
        got = f[0].cpu().numpy()[r:-r, r:-r, r:-r]
    exact, grouped = host(u, r, taps, ids, coef)
    rms = lambda a: float(np.sqrt(np.mean(((a.astype(LD) - exact) / exact) ** 2)))  # noqa: E731
    print(shape, r, n_ids, tile, rms(got) / rms(grouped))
    assert rms(got) <= 1.15 * rms(grouped)
