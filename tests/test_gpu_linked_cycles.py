"""Linked V-cycles on 2D finest levels (the up-leg of a cycle and the down-leg of the
next in one pass) against the separate legs: the same arithmetic in the same order, so
the iterates agree bit for bit; the residual norms are summed over other partials and
agree to rounding (n^2 <= 2^18 positive terms in FP64: 1e-12 relative is generous)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture()
def B():
    from paper_2402_17913_amd import binding as B
    B.np_set_tuning("w2min", 8)
    yield B
    B.np_set_tuning("w2min", 10)
    B.np_set_tuning("link", 11)
    B.np_release_all()


def same(B, run, linked):
    import torch
    got = []
    for link in (15, linked):  # 15: never linked
        B.np_set_tuning("link", link)
        got.append(run())
    (x0, st0, h0), (x1, st1, h1) = got
    assert st0 == st1 and len(h0) == len(h1)
    assert all(abs(a - b) <= 1e-12 * abs(a) for a, b in zip(h0, h1))
    assert torch.equal(x0, x1)


def field(n, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    f = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g)
    return f - f.mean()


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("n", [256, 512])
def test_poisson(B, n, bc):
    import torch
    f, h = field(n, n + bc), 1.0 / n
    print("linked poisson", n, bc, flush=True)
    for kw in (dict(tol=1e-9), dict(tol=1e-9, fixed_cycles=1), dict(tol=1e-9, fixed_cycles=2),
               dict(tol=1e-9, fixed_cycles=11), dict(tol=1e-14, max_cycles=3), dict(tol=1e-9, warm_start=2)):
        def run():
            x = f * 1e-3 if kw.get("warm_start") else torch.full_like(f, float("nan"))
            st, s = B.mg_poisson_solve(f, x, h, bc, check=False, **kw)
            return x, st, s["hist"]
        same(B, run, 8)
    for inner in (1, 2, 3, 4):  # refinement: the FP32 cycles of a step
        def run():
            x = torch.zeros_like(f)
            st, s = B.mg_poisson_solve(f, x, h, bc, tol=1e-9, check=False, smooth_prec=B.FP32, inner_cycles=inner)
            return x, st, s["hist"]
        same(B, run, 8)


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("scheme,a", [(0, [1.0, -0.5]), (1, [0.2, 0.1])])
def test_advection_diffusion(B, bc, scheme, a):
    f = field(256, 7 + bc)
    op = B.ad_op(20.0, 2.0, a, scheme)
    print("linked ad", bc, scheme, flush=True)
    for kw in (dict(tol=1e-10), dict(tol=1e-10, fixed_cycles=3)):
        def run():
            x = f.clone()
            st, s = B.np_ad_implicit_solve(f, x, 1.0, bc, op, check=False, **kw)
            return x, st, s["hist"]
        same(B, run, 8)


def test_unaligned_fields_and_a_zero_or_nan_rhs(B):
    """Fields that the paired accesses cannot take, f = 0 and f with a NaN."""
    import torch
    n = 256
    base = torch.empty(2 * n * n + 2, dtype=torch.float64, device="cuda")
    f, h = base[1:1 + n * n].view(n, n), 1.0 / n
    for fill in (field(n, 3), torch.zeros(n, n, dtype=torch.float64, device="cuda")):
        f.copy_(fill)

        def run():
            x = torch.full_like(fill, 1.0)
            st, s = B.mg_poisson_solve(f, x, h, 0, tol=1e-9, check=False)
            return x, st, s["hist"]
        same(B, run, 8)
    g = field(n, 4)
    g[3, 5] = float("nan")
    B.np_set_tuning("link", 8)
    x = torch.zeros_like(g)
    st, _ = B.mg_poisson_solve(g, x, h, 0, tol=1e-9, check=False)
    assert st == B.NP_ENAN
