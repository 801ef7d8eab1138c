"""AUTO HEAT3D7 runs of two sweeps, in two launches where the grids are small:
the scratch grid then holds the state after the first sweep (it is not copied
back from), and the result is that of single sweeps of a given tile, bit for
bit, on both sides of the rule."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1, 1, 1), (70, 33, 20), (128, 128, 128), (254, 254, 254), (254, 254, 258)])
def test_two_sweeps(n):
    from paper_2306_13002_amd.stencil import Plan
    u0 = torch.rand([e + 2 for e in reversed(n)], dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(2))
    small = 2 * u0.numel() * 8 <= 256 << 20
    assert small == (n[2] <= 254)  # 256^3 doubles twice: exactly the cache
    with Plan("heat3d7", n, coef=(0.4, 0.1)) as p, Plan("heat3d7", n, variant="saturated", coef=(0.4, 0.1),
                                                        tile=(32, 8, 4)) as q:
        p.use_graphs()
        for T in (2, 3, 2, 2, 2):
            a, b, one = ([u0.clone(), torch.full_like(u0, float("nan"))] for _ in range(3))
            p.run(a, iterations=T)
            q.run(b, iterations=T)
            q.run(one, iterations=1)
            assert torch.equal(a[0], b[0])
            if T == 2:
                assert torch.equal(a[1], one[0] if small else b[0])
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        a = [u0.clone(), torch.full_like(u0, float("nan"))]
        p.run_noalloc(a, iterations=2, residual=r)
        b = [u0.clone(), u0.clone()]
        q.run(b, iterations=2)
        assert torch.equal(a[0], b[0]) and abs(r.item() - q.residual()) <= 1e-12 * q.residual()
