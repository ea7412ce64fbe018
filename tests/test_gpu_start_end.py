"""The start and the end of a Poisson solve: the FP64 cycles do not read a zero iterate
that x does not hold (same bits from an x of NaNs as from zeros), the right-hand side
is only read, a periodic solution has no mean, and a refinement returns its last
iterate whichever of its two buffers holds it."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2402_17913_amd import binding
    yield binding
    binding.np_release_all()


def rhs(d, n, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*([n] * d), dtype=torch.float64, device="cuda", generator=g)


def residual(f, x, h, bc):
    """|f - mean - A x| / |f - mean| with A = -Laplacian, cell-centred ghosts (minus the cell, or periodic)."""
    import torch
    r = f.clone()
    if bc:
        r -= f.mean()
    norm = r.norm()
    for a in range(f.dim()):
        for s in (1, -1):
            nb = torch.roll(x, s, a)
            if not bc:
                edge = [slice(None)] * f.dim()
                edge[a] = slice(0, 1) if s == 1 else slice(-1, None)
                nb[tuple(edge)] = -x[tuple(edge)]
            r -= (x - nb) / h ** 2
    return float(r.norm() / norm)


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("d,n", [(2, 4), (2, 128), (2, 1024), (3, 32), (3, 128)])
def test_zero_iterate_is_not_read(B, d, n, bc):
    import torch
    f, h = rhs(d, n, n + d), 1.0 / n
    keep = f.clone()
    print("cold start", d, n, bc, flush=True)
    for kw in (dict(), dict(nu1=1, nu2=1), dict(nu1=0, nu2=2), dict(nu1=3, nu2=1), dict(tol=2.0),
               dict(max_cycles=0), dict(fixed_cycles=2)):
        got = []
        for fill in (0.0, float("nan")):
            x = torch.full_like(f, fill)
            st, s = B.mg_poisson_solve(f, x, h, bc, check=False, **{"tol": 1e-8, "max_cycles": 40, **kw})
            got.append((x, st, s["hist"]))
        assert got[0][1:] == got[1][1:] and torch.equal(got[0][0], got[1][0]), kw
        if bc:  # the sum of m terms of size |x| rounds to at most m eps |x| each way
            assert abs(float(got[0][0].mean())) <= 1e-12 * max(float(got[0][0].abs().max()), 1e-300), kw
    assert torch.equal(f, keep)


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("d,n", [(2, 128), (3, 64), (3, 128)])
def test_refinement_returns_its_last_iterate(B, d, n, bc):
    """The residual of x after k refinement steps is the one the solve reports for step k
    (FP64 on both sides: 1e-6 relative of a residual above 1e-9)."""
    import torch
    f, h = rhs(d, n, n + d + 1), 1.0 / n
    keep = f.clone()
    print("refinement", d, n, bc, flush=True)
    for prec in (B.FP32, B.BF16):
        for k in (1, 2, 3):
            x = torch.full_like(f, 7.0)
            _, s = B.mg_poisson_solve(f, x, h, bc, check=False, smooth_prec=prec, fixed_cycles=k)
            want = s["hist"][k]
            assert want > 1e-9
            assert abs(residual(f, x, h, bc) - want) <= 1e-6 * want, (prec, k)
    assert torch.equal(f, keep)
