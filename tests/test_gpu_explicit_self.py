"""The explicit step of a field that is one of its own velocity components (u advecting itself) against
the same step with that component given as a copy: the same values everywhere, so bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


# 2D: two launches (301) and one pass at its smallest sizes, with rows that are loaded cell by cell (1281); 3D: two
# launches of one cell per thread (64) and on z-marching tiles, with partial tiles and a last chunk of few planes (131)
@pytest.mark.parametrize("d,n", [(2, 301), (2, 1280), (2, 1281), (2, 1488), (3, 64), (3, 96), (3, 128), (3, 131)])
def test_own_velocity(d, n):
    import torch
    from paper_2402_17913_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)
    T = torch.randn((n,) * d, dtype=torch.float64, device="cuda", generator=g)
    b = [torch.randn((n,) * d, dtype=torch.float64, device="cuda", generator=g) for _ in range(d)]
    print("explicit own velocity", d, n, flush=True)
    for scheme in (0, 1, 2):
        for bc in (0, 1, 2):
            for own in ((0,), (d - 1,), tuple(range(d))):
                ref, x = T.clone(), T.clone()
                B.np_ad_explicit_step(ref, 1.0, 0.05, 0.3, bc, a=[T if e in own else b[e] for e in range(d)],
                                      scheme=scheme)
                B.np_ad_explicit_step(x, 1.0, 0.05, 0.3, bc, a=[x if e in own else b[e] for e in range(d)],
                                      scheme=scheme)
                assert torch.equal(x, ref), (scheme, bc, own)
