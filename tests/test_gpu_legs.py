"""One-pass legs: the 2D row-marching wavefronts (k_wave2) against the block and per-cell kernels
they replace, and the 2D and 3D legs with the advection-diffusion operator against its separate
kernels."""
import pytest

pytestmark = pytest.mark.gpu

DIR, PER = 0, 1


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2402_17913_amd import binding
    yield binding
    binding.np_set_tuning("w2min", 10)
    binding.np_release_all()


def _rhs(n, seed, offset=0):
    """A rough right-hand side; offset: that many values into its allocation."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(n * n + offset, dtype=torch.float64, device="cuda", generator=g)
    return a[offset:].view(n, n)


def _with(B, w2min, solve):
    B.np_set_tuning("w2min", w2min)
    try:
        return solve()
    finally:
        B.np_set_tuning("w2min", 10)


# 128: one strip with idle lanes; 256, 1024: strips of 120, 124 and 248 columns end inside a wave;
# 2048: the per-cell kernels on the other side
@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("bc", [DIR, PER])
@pytest.mark.parametrize("n", [128, 256, 1024, 2048])
def test_wavefront_legs_poisson(B, n, bc, prec):
    """Fixed cycles (outer steps): the same sums in the same order, so bit for bit."""
    import torch
    f = _rhs(n, n + bc)
    print("legs2 poisson", n, bc, prec, flush=True)

    def solve():
        x = torch.zeros_like(f)
        _, st = B.mg_poisson_solve(f, x, 1.0 / n, bc, smooth_prec=prec, fixed_cycles=3)
        return x, st["hist"]

    a, b = _with(B, 14, solve), _with(B, 7, solve)
    assert torch.isfinite(a[0]).all() and a[0].abs().max() > 0
    assert torch.equal(a[0], b[0])
    # the check sums its partials over other tiles: agreement to the rounding of n^2 terms
    assert all(abs(u - v) <= 1e-12 * max(u, 1e-300) for u, v in zip(a[1], b[1]))


@pytest.mark.parametrize("scheme,vel", [(0, [1.0, 1.0]), (0, [-1.0, 0.5]), (1, [0.2, -0.1])])
@pytest.mark.parametrize("bc", [DIR, PER])
@pytest.mark.parametrize("n", [128, 1024, 2048])
def test_wavefront_legs_advection_diffusion(B, n, bc, scheme, vel):
    """Against the block kernels bit for bit (up to 1024), against the separate sweep, restriction
    and prolongation kernels to rounding (2048: 1e-13 per cycle of values of order one)."""
    import torch
    f = _rhs(n, n + bc)
    op = B.ad_op(20.0, 2.0, vel, scheme)
    print("legs2 ad", n, bc, scheme, vel, flush=True)

    def solve():
        x = torch.zeros_like(f)
        B.np_ad_implicit_solve(f, x, 1.0, bc, op, fixed_cycles=3)
        return x

    a, b = _with(B, 14, solve), _with(B, 7, solve)
    assert torch.isfinite(a).all() and a.abs().max() > 0
    if n <= 1024:
        assert torch.equal(a, b)
    else:
        assert (a - b).abs().max() <= 3e-13 * a.abs().max()


@pytest.mark.parametrize("n", [1024, 2048])
def test_legs_unaligned_fields(B, n):
    """Fields that are not 16-byte aligned take the other kernels on the finest level."""
    import torch
    f = _rhs(n, n, offset=1)
    assert f.data_ptr() % 16 == 8
    g = f.clone()
    x, y = torch.zeros(n * n + 1, dtype=torch.float64, device="cuda")[1:].view(n, n), torch.zeros_like(g)
    B.mg_poisson_solve(f, x, 1.0 / n, DIR, fixed_cycles=2)
    B.mg_poisson_solve(g, y, 1.0 / n, DIR, fixed_cycles=2)
    assert torch.equal(x, y)
    op = B.ad_op(20.0, 2.0, [1.0, 1.0], 0)
    B.np_ad_implicit_solve(f, x, 1.0, DIR, op, fixed_cycles=2)
    B.np_ad_implicit_solve(g, y, 1.0, DIR, op, fixed_cycles=2)
    assert (x - y).abs().max() <= 2e-13 * y.abs().max()


@pytest.mark.parametrize("scheme,vel", [(0, [1.0, 1.0, 1.0]), (0, [-1.0, 0.5, -0.3]), (1, [0.2, -0.1, 0.15])])
@pytest.mark.parametrize("bc", [DIR, PER])
@pytest.mark.parametrize("n", [32, 64, 128, 256])
def test_legs3_advection_diffusion(B, n, bc, scheme, vel):
    """The 3D legs (z-marching tiles from 128^3, blocks below) against the separate sweep,
    restriction and prolongation kernels: 1e-13 per cycle of values of order one."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n + bc)
    f = torch.randn(n, n, n, dtype=torch.float64, device="cuda", generator=g)
    op = B.ad_op(20.0, 2.0, vel, scheme)
    print("legs3 ad", n, bc, scheme, vel, flush=True)
    out = []
    try:
        for on in (0, 1):
            B.np_set_tuning("sweep2z", on)
            B.np_set_tuning("fuseb", on)
            x = torch.zeros_like(f)
            _, st = B.np_ad_implicit_solve(f, x, 1.0, bc, op, fixed_cycles=3)
            out.append((x, st["hist"]))
    finally:
        B.np_set_tuning("sweep2z", 1)
        B.np_set_tuning("fuseb", 1)
    assert torch.isfinite(out[0][0]).all() and out[0][0].abs().max() > 0
    assert (out[0][0] - out[1][0]).abs().max() <= 3e-13 * out[0][0].abs().max()
    assert all(abs(u - v) <= 1e-12 * max(u, 1e-300) for u, v in zip(out[0][1], out[1][1]))


@pytest.mark.parametrize("prec", [0, 1])
def test_batched_legs(B, prec):
    """The batched V(2,2) legs against the per-stage tiles (one cell pair per thread), problems of
    one and of several strips and of every start (zero and not), bit for bit."""
    import torch
    sizes = [128, 1024, 64, 256, 512, 128, 16]
    fs = [torch.randn(n, n, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n + i))
          for i, n in enumerate(sizes)]
    out = []
    try:
        for rm in (0, 1):
            B.np_set_tuning("batched_rm", rm)
            xs = [torch.zeros_like(f) for f in fs]
            B.mg_poisson_solve_batched(fs, xs, [1.0 / n for n in sizes], smooth_prec=prec, inner_cycles=3, fixed_cycles=2)
            out.append(xs)
    finally:
        B.np_set_tuning("batched_rm", 1)
    for n, a, b in zip(sizes, *out):
        assert a.abs().max() > 0
        assert torch.equal(a, b), n


# every grid the one-workgroup solve takes, and the options it accepts
ONE = [dict(), dict(fixed_cycles=3), dict(nu1=1, nu2=2), dict(nu1=3, nu2=1, fixed_cycles=4), dict(warm_start=2),
       dict(smooth_prec=1), dict(smooth_prec=1, fixed_cycles=2), dict(smooth_prec=1, warm_start=2, inner_cycles=2),
       dict(max_cycles=2)]


@pytest.mark.parametrize("bc", [DIR, PER])
@pytest.mark.parametrize("d,n", [(2, 8), (2, 16), (2, 32), (2, 64), (3, 8), (3, 16)])
def test_one_workgroup_solves(B, d, n, bc):
    """A whole solve in one launch against the level kernels: the same cycles, status and history, the
    iterate to the rounding of the mean and of the coarsest product (1e-12 of its largest value)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n + bc)
    f = torch.randn((n,) * d, dtype=torch.float64, device="cuda", generator=g)
    op = B.ad_op(20.0, 2.0, [1.0, -0.5, 0.3][:d], 0)
    print("one workgroup", d, n, bc, flush=True)

    def pair(solve):
        out = []
        try:
            for one in (0, 1):
                B.np_set_tuning("one", one)
                x = 0.3 * f
                out.append((x,) + solve(x))
        finally:
            B.np_set_tuning("one", 1)
        (x, st, s), (y, tt, t) = out
        assert st == tt and s["cycles"] == t["cycles"] and s["outer_iters"] == t["outer_iters"]
        assert x.abs().max() > 0 and (x - y).abs().max() <= 1e-12 * x.abs().max()
        assert len(s["hist"]) == len(t["hist"])
        assert all(abs(u - v) <= 1e-10 * max(1.0, u) for u, v in zip(s["hist"], t["hist"]))

    for kw in ONE:
        pair(lambda x: B.mg_poisson_solve(f, x, 1.0 / n, bc, check=False, **kw))
    for kw in (dict(), dict(warm_start=2), dict(fixed_cycles=2)):
        pair(lambda x: B.np_ad_implicit_solve(f, x, 1.0, bc, op, check=False, **kw))


@pytest.mark.parametrize("prec", [0, 1])
def test_one_workgroup_right_hand_sides(B, prec):
    """A zero right-hand side gives zero in no cycles; a non-finite one leaves x alone."""
    import torch
    f = torch.zeros((32, 32), dtype=torch.float64, device="cuda")
    x = torch.full_like(f, 3.0)
    _, st = B.mg_poisson_solve(f, x, 1.0 / 32, DIR, smooth_prec=prec)
    assert st["cycles"] == 0 and bool((x == 0).all())
    for bad in (float("nan"), float("inf")):
        f[3, 4] = bad
        x.fill_(3.0)
        st, _ = B.mg_poisson_solve(f, x, 1.0 / 32, DIR, smooth_prec=prec, check=False)
        assert st == B.NP_ENAN and bool((x == 3.0).all())
