"""The 3D finite-element step on z-marching tiles at its smallest grids (one 64-cell tile and one of a few columns
along x, chunks of four planes) against its two launches of one cell per thread: the same neighbourhoods and
arithmetic, so bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 65, 66, 72, 78, 95, 96])
def test_small_tiles(n):
    import torch
    from paper_2402_17913_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)
    T, *a = [torch.randn(n, n, n, dtype=torch.float64, device="cuda", generator=g) for _ in range(4)]
    print("explicit small tiles", n, flush=True)
    for bc in (0, 1, 2):
        for vel in (a, None):
            out = []
            for on in (0, 1):
                x = T.clone()
                B.np_set_tuning("zmarch_explicit", on)
                try:
                    B.np_ad_explicit_step(x, 1.0, 0.05, 0.3, bc, a=vel, scheme=2)
                finally:
                    B.np_set_tuning("zmarch_explicit", 1)
                out.append(x)
            assert torch.isfinite(out[0]).all() and torch.equal(*out), (bc, vel is not None)
