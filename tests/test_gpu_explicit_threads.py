"""Explicit steps of equally large fields from several host threads, each on a stream of its own: they share
one scratch per size, so each result has to equal the one computed alone, bit for bit."""
import threading

import pytest

pytestmark = pytest.mark.gpu


# the step in two launches, its one-pass kernels in 2D and 3D, and the scalar step
@pytest.mark.parametrize("d,n,scheme", [(2, 512, 0), (2, 2048, 0), (3, 128, 2), (3, 64, None), (2, 1024, None)])
def test_threads(d, n, scheme):
    import torch
    from paper_2402_17913_amd import binding as B
    nthreads, steps = 4, 20
    print("explicit threads", d, n, scheme, flush=True)

    def step(T, a):
        if scheme is None:
            B.np_ad_scalar_step(T, 1.0, 0.01, 0.3, 1, a=a)
        else:
            B.np_ad_explicit_step(T, 1.0, 0.01, 0.3, 1, a=a, scheme=scheme)

    T, a, ref = [], [], []
    for k in range(nthreads):
        g = torch.Generator(device="cuda").manual_seed(10 * n + k)
        T.append(torch.randn((n,) * d, dtype=torch.float64, device="cuda", generator=g))
        a.append([torch.randn((n,) * d, dtype=torch.float64, device="cuda", generator=g) for _ in range(d)])
        ref.append(T[k].clone())
        for _ in range(steps):
            step(ref[k], a[k])
    torch.cuda.synchronize()
    gate, failed = threading.Barrier(nthreads), []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                gate.wait(30)
                for _ in range(steps):
                    step(T[k], a[k])
        except Exception as e:  # reported by the main thread
            failed.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(nthreads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(90)
    torch.cuda.synchronize()
    assert not failed and not any(t.is_alive() for t in ts)
    for k in range(nthreads):
        assert torch.isfinite(ref[k]).all() and torch.equal(T[k], ref[k]), k
