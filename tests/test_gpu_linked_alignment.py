"""Linked cycles take fields in pairs of 16 bytes, so a solve of fields that are not so aligned runs unlinked.  Seen
from the workspace: only linked FP64 cycles allocate a second partner of the iterate (n^2 doubles), on first use, so
that the first solve of aligned fields takes that much memory after one of unaligned fields, and none later.  The two
results differ by rounding: at most the machine epsilon times the condition number, about n^2, of the solution."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["poisson", "ad"])
@pytest.mark.parametrize("shift", ["x", "f"])
def test_unaligned_fields_run_unlinked(what, shift):
    import torch
    from paper_2402_17913_amd import binding as B
    n = 2048
    g = torch.Generator(device="cuda").manual_seed(n)
    base = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g)
    print("linked alignment", what, shift, flush=True)

    def field(off):
        t = torch.empty(n * n + 1, dtype=torch.float64, device="cuda")[off:off + n * n].view(n, n)
        assert (t.data_ptr() % 16 == 0) == (off == 0)
        return t

    # every field of the test beforehand, so that torch allocates nothing between two looks at the free memory
    off = dict(x=int(shift == "x"), f=int(shift == "f"))
    pairs = [(field(0), field(0)), (field(off["f"]), field(off["x"]))]

    def solve(unaligned):
        f, x = pairs[unaligned]
        f.copy_(base)
        if what == "poisson":
            B.mg_poisson_solve(f, x, 1.0 / n, 0, fixed_cycles=3)
        else:
            B.np_ad_implicit_solve(f, x, 1.0, 0, B.ad_op(50.0, 2.0, [1.0, 1.0], 0), fixed_cycles=3)

    def taken(unaligned):
        """Device memory that a solve takes and keeps."""
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        solve(unaligned)
        torch.cuda.synchronize()
        return before - torch.cuda.mem_get_info()[0]

    need = 8 * n * n
    B.np_release_all()
    solve(1)  # the plan
    assert taken(1) < need // 2
    assert taken(0) >= need
    assert taken(0) < need // 2
    x0, x1 = pairs[0][1], pairs[1][1]
    assert (x1 - x0).abs().max() <= 2.3e-16 * n * n * x0.abs().max()
    B.np_release_all()
