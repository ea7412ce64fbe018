"""Periodic solves of a constant right-hand side, whose mean-free part is zero: x = 0 after no cycle, on the
grids solved in one workgroup as on the next larger ones."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n", [(2, 4), (2, 8), (2, 16), (2, 32), (2, 64), (2, 128), (3, 8), (3, 16), (3, 32)])
def test_constant_rhs(d, n):
    import torch
    from paper_2402_17913_amd import binding as B
    print("constant rhs", d, n, flush=True)
    values = [0.1, 1.0 / 3.0, -2.7] + torch.randn(13, generator=torch.Generator().manual_seed(n), dtype=torch.float64).tolist()
    for v in values:
        f = torch.full((n,) * d, v, dtype=torch.float64, device="cuda")
        for kw in (dict(), dict(smooth_prec=B.FP32), dict(smooth_prec=B.BF16), dict(warm_start=2), dict(static=True)):
            kw = dict(kw)
            solve = B.mg_poisson_solve_noalloc if kw.pop("static", False) else B.mg_poisson_solve
            x = torch.full_like(f, 1.0)
            st, s = solve(f, x, 1.0 / n, 1, tol=1e-10, check=False, **kw)
            assert st == 0 and s["cycles"] == 0 and s["rel_res"] == 0.0, (v, kw, st, s["cycles"])
            assert not x.any(), (v, kw)
