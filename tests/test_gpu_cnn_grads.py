"""Gradients of the learned network where the backward pass's fused kernels change
form: one level (no transfer, no skip), two and three levels, and activations that
are zero everywhere.  The FP64 reference runs on BF16-rounded weights and inputs;
the GPU rounds every activation and every masked gradient to BF16 (2^-9 relative,
independent errors over at most a few tens of roundings in sequence), hence the
relative L2 bound 2e-2 and the cosine bound 0.999 of the whole gradient."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def params_for(levels, seed):
    from oracle import cnn
    rng = np.random.default_rng(seed + 100)
    out = []
    ps = cnn.init_params(levels, seed=seed)
    for k, (W, b) in enumerate(ps):
        b = rng.standard_normal(16) * 0.05
        if k == len(ps) - 1:
            b[1:] = 0.0
        out.append((cnn.bf16_round(W), cnn.bf16_round(b).astype(np.float64)))
    return out


def gradients(n, levels, flat, f, t):
    import torch
    from paper_2402_17913_amd import binding as B
    net = B.Cnn(n, levels)
    net.set_params(flat.astype(np.float32))
    x = torch.from_numpy(f.astype(np.float32)).cuda()
    tt = torch.from_numpy(t.astype(np.float32)).cuda()
    loss = net.gradients([x, x], [tt, tt])  # a second sample reuses every buffer
    g = net.get_grads().astype(np.float64)
    net.close()
    return loss, g


@pytest.mark.parametrize("n,levels", [(16, 1), (32, 2), (64, 3)])
def test_gradients_of_two_samples(n, levels):
    from oracle import cnn
    print("cnn grads", n, levels, flush=True)
    ps = params_for(levels, seed=n + 5)
    rng = np.random.default_rng(n)
    f = cnn.bf16_round(rng.standard_normal((n, n, n)))
    t = rng.standard_normal((n, n, n)).astype(np.float32).astype(np.float64)
    loss_ref, grads = cnn.loss_and_grads(ps, f, t, levels)
    gref = cnn.flatten(grads)
    loss, g = gradients(n, levels, cnn.flatten(ps), f, t)
    # the mean over two equal samples, or their sum: take the scale from the loss
    k = round(loss / loss_ref)
    assert k in (1, 2) and abs(loss - k * loss_ref) / (k * loss_ref) <= 2e-2
    g = g / k
    rel = np.linalg.norm(g - gref) / np.linalg.norm(gref)
    cos = float(g @ gref / (np.linalg.norm(g) * np.linalg.norm(gref)))
    print("  rel L2 %.3e cos %.6f" % (rel, cos), flush=True)
    assert rel <= 2e-2 and cos >= 0.999


def test_zero_activations_stop_gradients():
    """Biases of -1 and zero weights leave every activation at zero: only the last
    convolution's bias has a gradient (its inputs are zero, and so is every mask)."""
    n, levels = 16, 1
    per = 27 * 16 * 16 + 16
    flat = np.zeros(3 * per)
    for k in range(2):
        flat[(k + 1) * per - 16:(k + 1) * per] = -1.0
    rng = np.random.default_rng(3)
    f, t = rng.standard_normal((2, n, n, n))
    _, g = gradients(n, levels, flat, f, t)
    assert g[-16] != 0.0
    g[-16] = 0.0
    assert not g.any()


def test_two_tiles_along_x():
    """128^3 has two tiles along x: the plane-marching convolution gives the bits of
    the one-plane form for every plane count, and the weight gradients agree with the
    FP32 vector path to FP32 rounding (sums in another order; 1e-5 relative)."""
    import torch
    from paper_2402_17913_amd import binding as B
    n, per = 128, 27 * 16 * 16 + 16
    rng = np.random.default_rng(4)
    net = B.Cnn(n, 1)
    net.set_params((rng.standard_normal(3 * per) * 0.05).astype(np.float32))
    f, t = (torch.from_numpy(a.astype(np.float32)).cuda() for a in rng.standard_normal((2, n, n, n)))
    got = {}
    try:
        for z, w in ((0, 1), (1, 1), (4, 1), (32, 1), (1, 0)):
            B.np_set_tuning("conv3z", z)
            B.np_set_tuning("wgrad_mfma", w)
            y = torch.empty_like(f)
            net.forward(f, y)
            loss = net.gradients([f], [t])
            got[z, w] = y.cpu().numpy(), loss, net.get_grads().astype(np.float64)
    finally:
        B.np_set_tuning("conv3z", 1)
        B.np_set_tuning("wgrad_mfma", 1)
        net.close()
    y0, l0, g0 = got[0, 1]
    for k in ((1, 1), (4, 1), (32, 1)):
        y, l, g = got[k]
        assert np.array_equal(y, y0) and l == l0 and np.array_equal(g, g0), k
    gv = got[1, 0][2]
    for k in range(3):
        a, b = g0[k * per:(k + 1) * per], gv[k * per:(k + 1) * per]
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), k
