"""Rounding of the table-driven GENERIC kernel: a group's taps go, eight at a
time, into four partial sums before the one FMA.

Its error of a sweep against long double is compared with that order stated in
FP64 on the host: the same roundings, so the rms over some 20000 points may
differ by the host's FMA only (a long double product, 2^-11 of a rounding);
5 % are allowed.  (Two partial sums: 1.2 to 1.6 times off in one plane.)"""
import numpy as np
import pytest

from paper_2306_13002_amd import synth
from test_gpu_generic_rounding import LD, stencil

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def four_sums(v):
    p = [np.zeros_like(v[0]) for _ in range(4)]
    k = 0
    while k + 8 <= len(v):
        for q in range(4):
            p[q] = p[q] + (v[k + q] + v[k + q + 4])
        k += 8
    for x in v[k:]:
        p[0] = p[0] + x
    return (p[0] + p[1]) + (p[2] + p[3])


@pytest.mark.parametrize("r,n_ids,plane", [(2, 1, True), (3, 1, True), (4, 1, True), (4, 2, True), (4, 2, False),
                                           (4, 10, False), (1, 3, False)])
def test_four_partial_sums(monkeypatch, r, n_ids, plane):
    from paper_2306_13002_amd.stencil import Plan
    monkeypatch.setenv("STENCIL_GENERIC_TABLE", "1")
    taps, ids, coef = stencil(r, n_ids)
    if plane:  # one plane's taps: the error is mostly its groups'
        taps, ids = zip(*[(t, i) for t, i in zip(taps, ids) if t[2] == 0])
    n = (40, 30, 16)
    u = synth.uniform_f64(4, 950 + r, tuple(e + 2 * r for e in reversed(n)))
    with Plan("generic", n, dtype="f64", radius=r, taps=taps, cids=ids, coef=coef, variant="saturated") as p:
        f = [torch.tensor(u, device="cuda"), torch.tensor(u, device="cuda")]
        p.run_noalloc(f, iterations=1)  # (only the table-driven kernel runs so)
        got = f[0].cpu().numpy()[r:-r, r:-r, r:-r]
    cut = lambda d: u[tuple(slice(r + e, s - r + e) for s, e in zip(u.shape, (d[2], d[1], d[0])))]  # noqa: E731
    exact = sum(LD(coef[i]) * cut(d).astype(LD) for d, i in zip(taps, ids))
    acc = np.zeros_like(cut((0, 0, 0)))
    for dz in range(-r, r + 1):
        for i in range(len(coef)):
            v = [cut(d) for d, k in sorted(zip(taps, ids), key=lambda e: e[0][::-1]) if k == i and d[2] == dz]
            if v:
                acc = (LD(coef[i]) * four_sums(v).astype(LD) + acc.astype(LD)).astype(np.float64)
    rms = lambda a: float(np.sqrt(np.mean(((a.astype(LD) - exact) / exact) ** 2)))  # noqa: E731
    print(r, n_ids, plane, rms(got) / rms(acc))
    assert rms(got) <= 1.05 * rms(acc)
