"""The legs of 256^2 and 128^2 in one kernel against a kernel per level and leg: the
same arithmetic in the same order, so iterates and residual histories agree bit for
bit (the finest level and its partials are not touched)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("n", [512, 1024])
def test_paired_levels(n, bc):
    import torch
    from paper_2402_17913_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n + bc)
    f = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g)
    f -= f.mean()
    print("paired levels", n, bc, flush=True)

    def poisson(**kw):
        x = torch.zeros_like(f)
        st, s = B.mg_poisson_solve(f, x, 1.0 / n, bc, tol=1e-9, check=False, **kw)
        return x, st, list(s["hist"])

    def ad(scheme, a):
        x = f.clone()
        st, s = B.np_ad_implicit_solve(f, x, 1.0, bc, B.ad_op(20.0, 2.0, a, scheme), tol=1e-10, check=False)
        return x, st, list(s["hist"])

    runs = [lambda: poisson(fixed_cycles=1), lambda: poisson(), lambda: poisson(smooth_prec=B.FP32),
            lambda: poisson(smooth_prec=B.BF16), lambda: ad(0, [1.0, -0.5]), lambda: ad(1, [0.2, 0.1])]
    got = {}
    try:
        for pair in (0, 1):
            B.np_set_tuning("pair", pair)
            got[pair] = [r() for r in runs]
    finally:
        B.np_set_tuning("pair", 1)
    for k, (u, v) in enumerate(zip(got[0], got[1])):
        assert u[1:] == v[1:], k
        assert torch.equal(u[0], v[0]), k
