"""The 3D explicit step on each side of its rule (two launches of one cell per thread, two launches on z-marching
tiles, one pass) against the two launches of one cell per thread: the same neighbourhoods and arithmetic, so bit for
bit, also of a field that is its own velocity component."""
import pytest

pytestmark = pytest.mark.gpu


# tiles: finite elements from 65^3, all families from 128^3 (partial tiles along every axis, a last chunk of few
# planes); one pass: from 192^3 with a velocity, finite elements without one from 288^3 (a last tile of a few columns
# or rows, uneven chunks); an offset of one value: fields that are not 16-byte aligned
@pytest.mark.parametrize("n,schemes,offset", [(64, (2,), 0), (65, (2,), 0), (78, (2,), 1), (127, (0, 1, 2), 0),
                                              (128, (0, 1), 0), (133, (0, 1, 2), 1), (191, (0, 2), 0), (192, (0, 1, 2), 0),
                                              (195, (0, 2), 1), (203, (1, 2), 0), (287, (2,), 0), (289, (2,), 0)])
def test_routes(n, schemes, offset):
    import torch
    from paper_2402_17913_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)

    def field():
        return torch.empty(n ** 3 + offset, dtype=torch.float64, device="cuda")[offset:].view(n, n, n)

    T, *a = [field().normal_(generator=g) for _ in range(4)]
    print("explicit routes", n, schemes, offset, flush=True)
    for scheme in schemes:
        for bc in (0, 1, 2):
            for vel in ("given", "own", None):
                out = []
                for on in (0, 1):
                    x = field().copy_(T)
                    v = None if vel is None else ([x] + a[1:] if vel == "own" else a)
                    B.np_set_tuning("zmarch_explicit", on)
                    try:
                        B.np_ad_explicit_step(x, 1.0, 0.05, 0.3, bc, a=v, scheme=scheme)
                    finally:
                        B.np_set_tuning("zmarch_explicit", 1)
                    out.append(x)
                assert torch.isfinite(out[0]).all() and torch.equal(*out), (scheme, bc, vel)


@pytest.mark.parametrize("n,scheme", [(131, 2), (195, 0), (195, 2)])
def test_own_velocity_equals_a_copy(n, scheme):
    import torch
    from paper_2402_17913_amd import binding as B
    T, b = [torch.randn(n, n, n, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(k))
            for k in (1, 2)]
    for bc in (0, 1, 2):
        ref, x = T.clone(), T.clone()
        B.np_ad_explicit_step(ref, 1.0, 0.05, 0.3, bc, a=[b, T, b], scheme=scheme)
        B.np_ad_explicit_step(x, 1.0, 0.05, 0.3, bc, a=[b, x, b], scheme=scheme)
        assert torch.equal(x, ref), bc
