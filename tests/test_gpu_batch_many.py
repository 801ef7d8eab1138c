"""A batch of 2^17 tiny problems with one larger grid among them: copy launches
of many blocks per problem would exceed what one launch holds.  Every problem
equals its own single plan."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(variant="saturated_t3"), dict(variant="saturated", tile=(32, 8, 4))])
def test_many_problems_one_large(kw):
    from paper_2306_13002_amd import stencil as S
    big, tiny, m = (64, 64, 64), (3, 2, 1), 1 << 17
    descs = (S.StencilDesc * (m + 1))()
    keep = []
    for i, n in ((0, big), (1, tiny)):
        descs[i], k = S.make_desc("heat3d7", n, coef=(0.4, 0.1), **kw)
        keep.append(k)
    for i in range(2, m + 1):
        descs[i] = descs[1]
    h = ctypes.c_void_p()
    S._check(S.lib().stencil_plan_batch(descs, m + 1, ctypes.byref(h)))
    sb, st = [e + 2 for e in reversed(big)], [e + 2 for e in reversed(tiny)]
    gen = torch.Generator(device="cuda").manual_seed(8)
    ub = torch.rand(sb, dtype=torch.float64, device="cuda", generator=gen)
    ut = torch.rand([m] + st, dtype=torch.float64, device="cuda", generator=gen)
    fb, ft = [ub.clone(), torch.zeros_like(ub)], [ut.clone(), torch.zeros_like(ut)]
    step = ut[0].numel() * 8
    ptrs = (ctypes.c_void_p * (2 * (m + 1)))()
    ptrs[0], ptrs[1] = fb[0].data_ptr(), fb[1].data_ptr()
    for i in range(m):
        ptrs[2 * i + 2], ptrs[2 * i + 3] = ft[0].data_ptr() + i * step, ft[1].data_ptr() + i * step
    try:
        S._check(S.lib().stencil_run(h, ptrs, None, 1, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        torch.cuda.synchronize()
    finally:
        S.lib().stencil_destroy(h)
    for n, u, got in [(big, ub, fb[0])] + [(tiny, ut[i], ft[0][i]) for i in (0, 1, m // 2, m - 1)]:
        with S.Plan("heat3d7", n, coef=(0.4, 0.1), variant="saturated", tile=(32, 8, 4)) as q:
            want = [u.clone(), u.clone()]
            q.run(want, iterations=1)
        assert torch.equal(got, want[0])
    d = (ft[0] - ut).abs().amax(dim=(1, 2, 3))
    assert bool((d > 0).all())  # every problem moved
