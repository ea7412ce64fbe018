"""The explicit step in one pass (2D row-marching wavefronts, 3D z-marching tiles) against its two
launches of one cell per thread: the same neighbourhoods and arithmetic, so bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2402_17913_amd import binding
    return binding


def _fields(d, n, offset=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    m = n ** d
    out = []
    for _ in range(d + 1):
        a = torch.randn(m + offset, dtype=torch.float64, device="cuda", generator=g)[offset:].view((n,) * d)
        out.append(a)
    return out[0], out[1:]


def _step(B, T, a, bc, scheme, on):
    t = T
    B.np_set_tuning("zmarch_explicit", on)
    try:
        B.np_ad_explicit_step(t, 1.0, 0.05, 0.3, bc, a=a, scheme=scheme)
    finally:
        B.np_set_tuning("zmarch_explicit", 1)
    return t


# 1281: odd rows, cells loaded one by one, a pair across the right wall; 1300: a last strip of 60
# columns and chunks that do not divide the rows; 1488 = 12 strips of 124; in 3D partial tiles along
# every axis and a last chunk of few planes
CASES = [(2, 1280, 0), (2, 1281, 0), (2, 1300, 0), (2, 1488, 1), (2, 2047, 0), (3, 97, 0), (3, 128, 0), (3, 131, 0),
         (3, 160, 1)]


@pytest.mark.parametrize("d,n,offset", CASES)
def test_one_pass_step(B, d, n, offset):
    import torch
    T, a = _fields(d, n, offset)
    print("explicit one pass", d, n, offset, flush=True)
    for scheme in (0, 1, 2):
        for bc in (0, 1, 2):
            for vel in (a, None):
                ref = _step(B, T.clone(), vel, bc, scheme, 0)
                x = torch.empty(n ** d + offset, dtype=torch.float64, device="cuda")[offset:].view((n,) * d)
                x.copy_(T)
                _step(B, x, vel, bc, scheme, 1)
                assert torch.isfinite(x).all()
                assert torch.equal(x, ref), (scheme, bc, vel is not None)
