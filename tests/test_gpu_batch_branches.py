"""Batch graphs: where the copies of several classes stand (before the fork, in
the branches, after the join), for odd and even launch counts, against single
plans."""
import pytest
import torch

from paper_2306_13002_amd.stencil import BatchPlan, Plan

pytestmark = pytest.mark.gpu

SMALL = [(26, 4, 101), (219, 17, 11), (14, 15, 245)]     # 200 halo blocks
LARGE = [(160, 160, 160), (150, 160, 140), (120, 120, 120), (40, 40, 40)]  # halos more than 256, copies back more than 8192
MIXED = [(8, 8, 8)] * 3 + [(70, 9, 20)]


def _grids(sizes, seed):
    g = torch.Generator().manual_seed(seed)
    out = []
    for nx, ny, nz in sizes:
        u = torch.rand((nz + 2, ny + 2, nx + 2), generator=g, dtype=torch.float64).cuda()
        out.append((u, torch.zeros_like(u)))
    return out


@pytest.mark.parametrize("sizes", [SMALL, LARGE, MIXED], ids=["small", "large", "mixed"])
@pytest.mark.parametrize("variant,tile", [("plain", None), ("saturated", (32, 8, 8)), ("saturated_t2", (32, 8, 8)),
                                          ("saturated_t3", None)])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 7])
def test_batch_equals_single_plans(sizes, variant, tile, T):
    kw = dict(variant=variant) if tile is None else dict(variant=variant, tile=tile)
    got, want = _grids(sizes, T), _grids(sizes, T)
    with BatchPlan(sizes, coef=(0.4, 0.1), **kw) as p:
        for _ in range(3):  # captured, then replayed
            p.run(got, iterations=T)
        torch.cuda.synchronize()
    for n, a, b in zip(sizes, got, want):
        with Plan("heat3d7", n, coef=(0.4, 0.1), **kw) as q:
            for _ in range(3):
                q.run(list(b), iterations=T)
        torch.cuda.synchronize()
        assert torch.equal(a[0], b[0])
