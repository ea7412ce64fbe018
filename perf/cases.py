"""Performance cases of the library: the solves and steps a user's program runs.

Every case goes through the public binding (paper_2402_17913_amd.binding).
`listed()` names the standing cases, `draw(rng)` gives one more of the same
ranges, `prepare` makes a case's inputs on the GPU from a seed, `run` is one
pass, `work` counts what a pass cannot do without, and `exact` computes the
same outputs in 64 bits with plain torch.

Families (`path`):
  poisson   one multigrid Poisson solve from a zero guess (2D and 3D, both
            boundary rules, FP64 cycles or FP32/BF16 inner cycles with FP64
            refinement)
  batch     many 2D Poisson solves of uneven sizes in one call
  ad        one implicit (backward Euler) advection-diffusion step by multigrid
  explicit  one explicit advection-diffusion step with a filter family
  ns        one staggered incompressible projection step
  nsc       one collocated projection step
  net       the learned warm start's network: prediction, or loss and gradients
"""
import math

import numpy as np
import torch
import torch.utils.checkpoint

from paper_2402_17913_amd import binding as B

DEV = "cuda:0"
F64 = torch.float64
BC = {"dirichlet": B.BC_DIRICHLET0, "periodic": B.BC_PERIODIC, "neumann": B.BC_NEUMANN}
PREC = {"fp64": B.FP64, "fp32": B.FP32, "bf16": B.BF16}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: a solve that fits one workgroup, so launches and the host dominate
        dict(name="poisson2d_64_fp64", path="poisson", d=2, n=64, bc="dirichlet", prec="fp64", modes=8, tol=1e-10),
        # a large plane problem in plain FP64; 1e-9 is what FP64 resolves on fine 2D grids
        dict(name="poisson2d_2048_fp64", path="poisson", d=2, n=2048, bc="dirichlet", prec="fp64", modes=8, tol=1e-9),
        # the benchmark's headline: mixed-precision solve of 256^3
        dict(name="poisson3d_256_fp32", path="poisson", d=3, n=256, bc="dirichlet", prec="fp32", modes=8, tol=1e-10),
        # the largest call: 1.3e8 unknowns in plain FP64
        dict(name="poisson3d_512_fp64", path="poisson", d=3, n=512, bc="dirichlet", prec="fp64", modes=8, tol=1e-10),
        # many uneven solves in one call, with settings a program has tuned once
        dict(name="batch_64", path="batch", count=64, lo=64, hi=1024, pick=1, inner=4, prec="fp32", tol=1e-10),
        # time stepping in the plane, as a flow program calls it; the viscosity is visc * h (1e-3 here),
        # the same cell Reynolds number on every grid
        dict(name="ns2d_1024", path="ns", d=2, n=1024, prec="fp64", visc=0.163, tol=1e-10),
        # time stepping in the box, BF16 inner cycles, periodic solve
        dict(name="ns3d_256_bf16", path="ns", d=3, n=256, prec="bf16", visc=0.163, tol=1e-10),
        # implicit advection-diffusion at the paper's Courant number, large plane
        dict(name="ad2d_4096", path="ad", d=2, n=4096, bc="dirichlet", scheme=0, dt=50.0, tol=1e-10),
        # the same in the box
        dict(name="ad3d_256", path="ad", d=3, n=256, bc="dirichlet", scheme=0, dt=50.0, tol=1e-10),
        # the paper's 301^2 explicit grid: odd size, small call
        dict(name="explicit2d_301_central", path="explicit", d=2, n=301, bc="dirichlet", scheme=0),
        # the 27-point finite-element step on a large box
        dict(name="explicit3d_256_fe", path="explicit", d=3, n=256, bc="dirichlet", scheme=2),
        # training the warm-start network: forward and backward over a minibatch
        dict(name="net_grad_128_b2", path="net", n=128, levels=4, batch=2, grad=True),
    ]


def _pow2(rng, lo, hi):
    return 1 << rng.randint(lo, hi)


def draw(rng):
    path = rng.choice(["poisson", "poisson", "batch", "ad", "explicit", "ns", "nsc", "net"])
    if path == "poisson":
        d = rng.choice([2, 3])
        n = _pow2(rng, 4, 12) if d == 2 else _pow2(rng, 3, 8)
        prec = rng.choice(["fp64", "fp64", "fp32", "bf16"])
        if n > 1024:
            prec = rng.choice(["fp64", "fp32"])  # BF16 storage is too coarse on the finest planes
        return dict(path=path, d=d, n=n, bc=rng.choice(["dirichlet", "periodic"]), prec=prec,
                    modes=rng.randint(4, 12), tol=1e-9 if n > 1024 else 1e-10)
    if path == "batch":
        hi = rng.choice([128, 256, 512, 1024])
        return dict(path=path, count=int(round(math.exp(rng.uniform(math.log(3), math.log(64))))),
                    lo=rng.choice([16, 32, 64]), hi=hi, pick=rng.randint(0, 999), inner=rng.choice([2, 3, 4]),
                    prec=rng.choice(["fp32", "fp32", "fp64"]), tol=1e-10)
    if path == "ad":
        d = rng.choice([2, 3])
        n = _pow2(rng, 5, 12) if d == 2 else _pow2(rng, 4, 8)
        return dict(path=path, d=d, n=n, bc=rng.choice(["dirichlet", "periodic"]), scheme=rng.choice([0, 0, 1]),
                    dt=round(rng.uniform(10.0, 60.0), 1), tol=1e-10)
    if path == "explicit":
        d = rng.choice([2, 3])
        lo, hi = (33, 4096) if d == 2 else (20, 256)
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        if rng.random() < 0.4:  # as many users take round sizes as odd ones
            n = max(32, n // 32 * 32)
        return dict(path=path, d=d, n=n, bc=rng.choice(["dirichlet", "periodic", "neumann"]),
                    scheme=rng.choice([0, 1, 2]))
    if path == "ns":
        d = rng.choice([2, 3])
        n = _pow2(rng, 7, 10) if d == 2 else _pow2(rng, 5, 8)
        return dict(path=path, d=d, n=n, prec=rng.choice(["fp64", "fp32", "bf16"]), visc=round(rng.uniform(0.12, 0.5), 3),
                    tol=1e-10)
    if path == "nsc":
        d = rng.choice([2, 3])
        n = _pow2(rng, 7, 10) if d == 2 else _pow2(rng, 5, 8)
        return dict(path=path, d=d, n=n, scheme=rng.choice([0, 1, 2]), visc=round(rng.uniform(0.12, 0.5), 3), tol=1e-10)
    n, levels = rng.choice([(32, 2), (64, 2), (64, 3), (128, 2), (128, 3), (128, 4)])
    grad = rng.random() < 0.6
    return dict(path=path, n=n, levels=levels, batch=rng.randint(1, 4) if grad else 1, grad=grad)


# --------------------------------------------------------------------- inputs
def _centres(n, length=1.0):
    return (torch.arange(n, dtype=F64, device=DEV) + 0.5) * (length / n)


def _outer(cols):
    """sum_m of the products of per-axis profiles: cols[a] is (modes, n), x first; the
    result has x as its last (fastest) axis."""
    n = cols[0].shape[1]
    f = cols[0]
    for c in cols[1:-1]:
        f = (c[:, :, None] * f[:, None, :]).reshape(f.shape[0], -1)
    return (cols[-1].T @ f).reshape((n,) * len(cols)).contiguous()


def _sine_field(d, n, seed, modes=8, kmax=8):
    """Smooth source on the unit square or cube: sine modes up to kmax, coefficients in [-1, 1]."""
    rng = np.random.default_rng(seed)
    ks = torch.from_numpy(rng.integers(1, min(kmax, max(1, n // 4)) + 1, size=(modes, d)).astype(np.float64)).to(DEV)
    c = torch.from_numpy(rng.uniform(-1.0, 1.0, size=modes)).to(DEV)
    x = _centres(n)
    cols = [torch.sin(math.pi * ks[:, a:a + 1] * x) for a in range(d)]
    cols[0] = c[:, None] * cols[0]
    return _outer(cols)


def _wave_field(d, n, rng, power, half=(), kmax=16):
    """Real random field on the periodic grid of [0, 2 pi)^d, amplitudes |k|^-power up to
    |k| = kmax, sampled half a cell further along the axes (0 = x) in `half`."""
    kmax = min(kmax, n // 4)
    k1 = np.arange(-kmax, kmax + 1)
    K = np.meshgrid(*([k1] * d), indexing="ij")  # array axes z, y, x
    kk = np.sqrt(sum(k.astype(np.float64) ** 2 for k in K))
    amp = np.where((kk >= 1) & (kk <= kmax), np.maximum(kk, 1.0) ** -power, 0.0)
    z = (rng.standard_normal(kk.shape) + 1j * rng.standard_normal(kk.shape)) * amp
    for a in half:
        z = z * np.exp(1j * K[d - 1 - a] * math.pi / n)
    spec = torch.zeros((n,) * d, dtype=torch.complex128, device=DEV)
    at = torch.from_numpy(k1 % n).to(DEV)
    spec[torch.meshgrid(*([at] * d), indexing="ij")] = torch.from_numpy(z).to(DEV)
    return torch.fft.ifftn(spec).real.contiguous() * float(n ** d)


def _divfree(d, n, seed):
    """Divergence-free velocity on the staggered periodic grid (the discrete curl of a random
    potential), scaled to a largest component of 1, with h and a step of Courant number 1/2."""
    rng = np.random.default_rng(seed)
    h = 2 * math.pi / n
    if d == 2:
        psi = _wave_field(2, n, rng, 3.0, (0, 1))
        q = [_back(psi, 1) / h, -_back(psi, 0) / h]
    else:
        ax, ay, az = (_wave_field(3, n, rng, 3.5, e) for e in ((1, 2), (0, 2), (0, 1)))
        q = [(_back(az, 1) - _back(ay, 2)) / h, (_back(ax, 2) - _back(az, 0)) / h, (_back(ay, 0) - _back(ax, 1)) / h]
    top = max(float(c.abs().max()) for c in q)
    q = [(c / top).contiguous() for c in q]
    return q, h, 0.5 * h / sum(float(c.abs().max()) for c in q)


def _blob(d, n, seed, width):
    """A Gaussian of the given width, its centre drawn from the middle of n^d unit cells."""
    rng = np.random.default_rng(seed)
    x = torch.arange(n, dtype=F64, device=DEV)
    c = rng.uniform(0.35, 0.65, size=d) * n
    return _outer([torch.exp(-((x - c[a]) ** 2) / (2 * width ** 2))[None, :] for a in range(d)])


def _batch_sizes(case):
    rng = np.random.default_rng(case["pick"])
    choices = [s for s in (16, 32, 64, 128, 256, 512, 1024) if case["lo"] <= s <= case["hi"]]
    return [int(choices[i]) for i in rng.integers(0, len(choices), size=case["count"])]


def _rotation(d, n, seed):
    """Velocity of the explicit step: a solid-body rotation about a drawn centre (2D), or a
    divergence-free trigonometric field with drawn phases (3D); largest component about 1."""
    rng = np.random.default_rng(seed)
    x = torch.arange(n, dtype=F64, device=DEV)
    if d == 2:
        c = rng.uniform(0.45, 0.55, size=2) * n
        one = torch.ones(n, n, dtype=F64, device=DEV)
        return [((c[1] - x)[:, None] * one * (2 / n)).contiguous(), ((x - c[0])[None, :] * one * (2 / n)).contiguous()]
    s = [2 * math.pi * x / n + p for p in rng.uniform(0, 2 * math.pi, size=3)]
    sx, sy, sz = s[0][None, None, :], s[1][None, :, None], s[2][:, None, None]
    one = torch.ones(n, n, n, dtype=F64, device=DEV)
    return [(torch.sin(sy) * torch.cos(sz) * one).contiguous(), (torch.sin(sz) * torch.cos(sx) * one).contiguous(),
            (torch.sin(sx) * torch.cos(sy) * one).contiguous()]


def _net_pairs(case, seed):
    """Pairs as the solver gives them: a right-hand side of unit rms, its smooth solution."""
    xs, ts = [], []
    for k in range(case["batch"]):
        rng = np.random.default_rng([seed, k])
        f = _wave_field(3, case["n"], rng, 1.5)
        f = f / f.square().mean().sqrt()
        xs.append(f.float().contiguous())
        ts.append(_poisson_exact(f, 2 * math.pi / case["n"], "periodic").float().contiguous())
    return xs, ts


def prepare(case, seed):
    d, n = case.get("d"), case.get("n")
    path = case["path"]
    if path == "poisson":
        if case["bc"] == "dirichlet":
            f, h = _sine_field(d, n, seed, case["modes"]), 1.0 / n
        else:
            f, h = _wave_field(d, n, np.random.default_rng(seed), 1.5, kmax=2 * case["modes"]), 2 * math.pi / n
        return dict(case=case, f=f, x=torch.zeros_like(f), h=h)
    if path == "batch":
        sizes = _batch_sizes(case)
        fs = [_sine_field(2, s, seed * 1000 + i) for i, s in enumerate(sizes)]
        return dict(case=case, f=fs, x=[torch.zeros_like(f) for f in fs], h=[1.0 / s for s in sizes])
    if path == "ad":
        f = _blob(d, n, seed, n * 10.0 / 128.0)
        return dict(case=case, f=f, x=torch.zeros_like(f), op=B.ad_op(case["dt"], 2.0, [1.0] * d, case["scheme"]))
    if path == "explicit":
        return dict(case=case, T=_blob(d, n, seed, n / 10.0), a=_rotation(d, n, seed))
    if path in ("ns", "nsc"):
        q, h, dt = _divfree(d, n, seed)
        return dict(case=case, q=q, p=torch.zeros_like(q[0]), h=h, dt=dt, nu=case["visc"] * h)
    net = B.Cnn(case["n"], case["levels"])
    net.init(seed)
    xs, ts = _net_pairs(case, seed)
    return dict(case=case, net=_Net(net), x=xs, t=ts, y=torch.empty_like(xs[0]))


class _Net:
    """Closes the network with the state that holds it."""

    def __init__(self, net):
        self.net = net

    def __del__(self):
        self.net.close()


# ------------------------------------------------------------------- one pass
def run(state):
    c = state["case"]
    path = c["path"]
    if path == "poisson":
        B.mg_poisson_solve(state["f"], state["x"], state["h"], BC[c["bc"]], tol=c["tol"], smooth_prec=PREC[c["prec"]])
        return state["x"]
    if path == "batch":
        B.mg_poisson_solve_batched(state["f"], state["x"], state["h"], tol=c["tol"], smooth_prec=PREC[c["prec"]],
                                   inner_cycles=c["inner"])
        return state["x"]
    if path == "ad":
        B.np_ad_implicit_solve(state["f"], state["x"], 1.0, BC[c["bc"]], state["op"], tol=c["tol"])
        return state["x"]
    if path == "explicit":
        B.np_ad_explicit_step(state["T"], 1.0, 0.1, 0.5, BC[c["bc"]], a=state["a"], scheme=c["scheme"])
        return state["T"]
    if path in ("ns", "nsc"):
        q = state["q"]
        w = q[2] if c["d"] == 3 else None
        if path == "ns":
            B.ns_projection_step(q[0], q[1], w, state["p"], state["h"], state["dt"], state["nu"], tol=c["tol"],
                                 smooth_prec=PREC[c["prec"]])
        else:
            B.ns_collocated_step(q[0], q[1], w, state["p"], state["h"], state["dt"], state["nu"], scheme=c["scheme"],
                                 tol=c["tol"])
        return q + [state["p"]]
    net = state["net"].net
    if c["grad"]:
        loss = net.gradients(state["x"], state["t"])
        return dict(loss=loss, grads=net.get_grads())
    net.forward(state["x"][0], state["y"])
    return state["y"]


# ----------------------------------------------------------------------- work
def work(case):
    """Each input read once, each output written once; one evaluation of the operator (or of
    the stages, or of the network) in operations."""
    path = case["path"]
    if path == "batch":
        m = sum(s * s for s in _batch_sizes(case))
        return {"bytes": 16.0 * m, "flops": 11.0 * m}
    m = float(case["n"]) ** case.get("d", 3)
    d = case.get("d", 3)
    if path == "poisson":
        return {"bytes": 16.0 * m, "flops": (4 * d + 3) * m}
    if path == "ad":
        return {"bytes": 16.0 * m, "flops": (4 * d + 3) * m}
    if path == "explicit":
        taps = 3 ** d if case["scheme"] == 2 else 2 * d + 1
        return {"bytes": (16.0 + 8 * d) * m, "flops": 4.0 * taps * (d + 1) * m}
    if path in ("ns", "nsc"):
        return {"bytes": 16.0 * (d + 1) * m, "flops": 2.0 * d * (8 * d + 8) * m}
    flops = params = 0
    for level in range(case["levels"]):
        convs = (2 if level == case["levels"] - 1 else 4) + (1 if level == 0 else 0)
        flops += convs * 2 * 27 * 256 * m / 8 ** level
        params += convs * (27 * 256 + 16)
    b = case["batch"]
    if case["grad"]:
        return {"bytes": 8.0 * m * b + 8.0 * params, "flops": 3.0 * flops * b}
    return {"bytes": 8.0 * m + 4.0 * params, "flops": flops}


# ---------------------------------------------------------------------- exact
def _fwd(f, a):  # the value at index + 1 along axis a (0 = x), periodic, minus the value here
    return torch.roll(f, -1, f.dim() - 1 - a) - f


def _back(f, a):
    return f - torch.roll(f, 1, f.dim() - 1 - a)


def _shift(f, a, s, bc):
    """The neighbour's value at index + s (s = -1, 1) along axis a, ghosts by the boundary rule."""
    ax = f.dim() - 1 - a
    g = torch.roll(f, -s, ax)
    if bc != "periodic":
        edge = f.shape[ax] - 1 if s > 0 else 0
        g.select(ax, edge).copy_(f.select(ax, edge) * (-1.0 if bc == "dirichlet" else 1.0))
    return g


def _poisson_exact(f, h, bc):
    n, d = f.shape[0], f.dim()
    if bc == "periodic":
        lam1 = (2 - 2 * torch.cos(2 * math.pi * torch.arange(n, dtype=F64, device=DEV) / n)) / (h * h)
        s = torch.fft.fftn(f)
    else:
        k = torch.arange(1, n + 1, dtype=F64, device=DEV)
        q = torch.sin(math.pi * k[:, None] * _centres(n)[None, :]) * math.sqrt(2.0 / n)
        q[-1] /= math.sqrt(2.0)
        lam1 = (2 - 2 * torch.cos(math.pi * k / n)) / (h * h)
        s = f
        for a in range(d):
            s = torch.movedim(torch.tensordot(q, s, dims=([1], [a])), 0, a)
    lam = sum(lam1.reshape([-1 if b == a else 1 for b in range(d)]) for a in range(d))
    if bc == "periodic":
        lam.view(-1)[0] = 1.0
        s = s / lam
        s.view(-1)[0] = 0.0
        return torch.fft.ifftn(s).real.contiguous()
    s = s / lam
    for a in range(d):
        s = torch.movedim(torch.tensordot(q, s, dims=([0], [a])), 0, a)
    return s.contiguous()


def _ad_weights(d, h, dt, nu, a, scheme):
    """Centre, lower and upper weights of backward Euler advection-diffusion at spacing h."""
    dif = nu * dt / (h * h)
    c0, lo, up = 1 + 2 * d * dif, [-dif] * d, [-dif] * d
    for e in range(d):
        c = a[e] * dt / h
        if scheme == 1:
            lo[e], up[e] = lo[e] - c / 2, up[e] + c / 2
        elif c >= 0:
            c0, lo[e] = c0 + c, lo[e] - c
        else:
            c0, up[e] = c0 - c, up[e] + c
    return c0, lo, up


def _ad_exact(f, bc, scheme, dt):
    """Multigrid V(2,2) cycles in plain torch, until the residual no longer falls."""
    d, n0 = f.dim(), f.shape[0]

    def apply(x, w):
        y = w[0] * x
        for e in range(d):
            y += w[1][e] * _shift(x, e, -1, bc) + w[2][e] * _shift(x, e, 1, bc)
        return y

    def cycle(x, f, w):
        n = f.shape[0]
        if n <= 4:
            eye = torch.eye(n ** d, dtype=F64, device=DEV)
            dense = torch.stack([apply(r.reshape((n,) * d), w[0]).reshape(-1) for r in eye], 1)
            return torch.linalg.solve(dense, f.reshape(-1)).reshape(f.shape)
        jac = (2.0 / 3.0) / w[0][0]
        for _ in range(2):
            x = x + jac * (f - apply(x, w[0]))
        r = f - apply(x, w[0])
        for a in range(d):
            r = 0.5 * r.unflatten(a, (n // 2, 2)).sum(a + 1)
        e = cycle(torch.zeros_like(r), r, w[1:])
        for a in range(d):
            lo, up = _shift(e, d - 1 - a, -1, bc), _shift(e, d - 1 - a, 1, bc)
            e = torch.stack([0.75 * e + 0.25 * lo, 0.75 * e + 0.25 * up], a + 1).flatten(a, a + 1)
        x = x + e
        for _ in range(2):
            x = x + jac * (f - apply(x, w[0]))
        return x

    w, h = [], 1.0
    while n0 * 1.0 / h >= 4:
        w.append(_ad_weights(d, h, dt, 2.0, [1.0] * d, scheme))
        h *= 2
    x, best, norm = torch.zeros_like(f), math.inf, float(f.norm())
    for _ in range(80):
        new = cycle(x, f, w)
        res = float((f - apply(new, w[0])).norm()) / norm
        if not res < 0.9 * best:
            break
        x, best = new, res
    return x if best < 1e-12 else None


def _family(T, a, h, nu, bc, scheme):
    """sum_e a_e D_e T - nu Lap T with the filter family's stencils, and the family's D_e."""
    d = T.dim()

    def smooth(f, axes, w):  # (w, 4 - .., w)-type average over axes: weights w[0], w[1], w[0]
        for b in axes:
            f = w[1] * f + w[0] * (_shift(f, b, -1, bc) + _shift(f, b, 1, bc))
        return f

    out = torch.zeros_like(T)
    for e in range(d):
        if scheme == 1:
            lo, up = (T - _shift(T, e, -1, bc)) / h, (_shift(T, e, 1, bc) - T) / h
            out += a[e] * torch.where(a[e] >= 0, lo, up)
        else:
            out += a[e] * _first(T, e, h, bc, scheme)
    if scheme != 2:
        lap = sum(_shift(T, e, -1, bc) + _shift(T, e, 1, bc) for e in range(d)) - 2 * d * T
        return out - nu * lap / (h * h)
    if d == 2:
        return out + nu * (16 * T - smooth(T, (0, 1), (1.0, 2.0))) / (4 * h * h)
    # 88, -6, -3, -2 on the centre, faces, edges and corners, over 26
    box = smooth(T, (0, 1, 2), (1.0, 1.0))
    ax = [_shift(T, e, -1, bc) + _shift(T, e, 1, bc) for e in range(3)]
    face = ax[0] + ax[1] + ax[2]
    edge = sum(_shift(ax[b], c, -1, bc) + _shift(ax[b], c, 1, bc) for b, c in ((0, 1), (0, 2), (1, 2)))
    corner = box - T - face - edge
    return out + nu * (88 * T - 6 * face - 3 * edge - 2 * corner) / (26 * h * h)


def _first(T, e, h, bc, scheme):
    """The family's first derivative along e: central, averaged (1, 4, 1)/6 across for scheme 2."""
    g = (_shift(T, e, 1, bc) - _shift(T, e, -1, bc)) / (2 * h)
    if scheme == 2:  # the ghost of a padded field is padded, so averaging comes first
        t = T
        for b in range(T.dim()):
            if b != e:
                t = (4 * t + _shift(t, b, -1, bc) + _shift(t, b, 1, bc)) / 6
        g = (_shift(t, e, 1, bc) - _shift(t, e, -1, bc)) / (2 * h)
    return g


def _ns_exact(s):
    q, p, h, dt, nu = s["q"], s["p"], s["h"], s["dt"], s["nu"]
    d = len(q)

    def rhs(v, c):  # (a . grad) v - nu lap v + G p on the faces of component c
        out = _fwd(p, c) / h
        for e in range(d):
            a = q[e]
            if e != c:
                a = q[e] + torch.roll(q[e], 1, d - 1 - e)
                a = 0.25 * (a + torch.roll(a, -1, d - 1 - c))
            out = out + a * (_fwd(v, e) + _back(v, e)) / (2 * h) - nu * (_fwd(v, e) - _back(v, e)) / (h * h)
        return out

    half = [q[c] - dt * rhs(q[c], c) for c in range(d)]
    star = [q[c] - dt * rhs(0.5 * (half[c] + q[c]), c) for c in range(d)]
    f = -sum(_back(star[c], c) for c in range(d)) / (h * dt)
    dp = _poisson_exact(f, h, "periodic")
    return [star[c] - dt * _fwd(dp, c) / h for c in range(d)] + [p + dp]


def _nsc_exact(s, scheme):
    q, p, h, dt, nu = s["q"], s["p"], s["h"], s["dt"], s["nu"]
    d = len(q)
    grad = [_first(p, c, h, "periodic", scheme) for c in range(d)]
    step = lambda v, c: _family(v, q, h, nu, "periodic", scheme) + grad[c]  # noqa: E731
    half = [q[c] - dt * step(q[c], c) for c in range(d)]
    star = [q[c] - dt * step(0.5 * (half[c] + q[c]), c) for c in range(d)]
    dp = _poisson_exact(-sum(_first(star[c], c, h, "periodic", scheme) for c in range(d)) / dt, h, "periodic")
    return [star[c] - dt * _first(dp, c, h, "periodic", scheme) for c in range(d)] + [p + dp]


def _net_exact(s):
    c = s["case"]
    levels, n = c["levels"], c["n"]
    vec = torch.from_numpy(s["net"].net.get_params()).to(DEV, F64).requires_grad_(c["grad"])
    per = 27 * 256 + 16
    weights = [(vec[k * per:k * per + 6912].view(27, 16, 16), vec[k * per + 6912:(k + 1) * per])
               for k in range(vec.numel() // per)]
    taps = [(z, y, x) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1)]

    def conv(v, w, b):
        out = b[:, None].expand(16, v[0].numel())
        for t, (z, y, x) in enumerate(taps):
            out = out + w[t] @ torch.roll(v, (-z, -y, -x), (1, 2, 3)).reshape(16, -1)
        return out.reshape(v.shape)

    def layer(v, k, relu=True):
        y = torch.utils.checkpoint.checkpoint(conv, v, *weights[k], use_reentrant=False) if c["grad"] else conv(v, *weights[k])
        return torch.relu(y) if relu else y

    def up(v):
        for a in (1, 2, 3):
            lo, hi = 0.75 * v + 0.25 * torch.roll(v, 1, a), 0.75 * v + 0.25 * torch.roll(v, -1, a)
            v = torch.stack([lo, hi], a + 1).flatten(a, a + 1)
        return v

    def forward(x):
        v = torch.cat([x[None], torch.zeros((15,) + x.shape, dtype=F64, device=DEV)])
        k, enc = 0, []
        for level in range(levels):
            if level:
                m = v.shape[1] // 2
                v = v.reshape(16, m, 2, m, 2, m, 2).mean((2, 4, 6))
            v = layer(layer(v, k), k + 1)
            enc.append(v)
            k += 2
        for level in range(levels - 2, -1, -1):
            v = layer(layer(up(v) + enc[level], k), k + 1)
            k += 2
        return layer(v, k, False)[0]

    if not c["grad"]:
        return forward(s["x"][0].to(F64))
    total = 0.0
    for x, t in zip(s["x"], s["t"]):
        loss = (forward(x.to(F64)) - t.to(F64)).square().mean()
        loss.backward()
        total += float(loss.detach())
    return dict(loss=total, grads=vec.grad)


def exact(case, seed):
    s = prepare(case, seed)
    path = case["path"]
    if path == "poisson":
        f = s["f"]
        return _poisson_exact(f - f.mean() if case["bc"] == "periodic" else f, s["h"], case["bc"])
    if path == "batch":
        return [_poisson_exact(f, h, "dirichlet") for f, h in zip(s["f"], s["h"])]
    if path == "ad":
        return _ad_exact(s["f"], case["bc"], case["scheme"], case["dt"])
    if path == "explicit":
        T, a = s["T"], s["a"]
        rate = lambda v: _family(v, a, 1.0, 0.5, case["bc"], case["scheme"])  # noqa: E731
        half = T - 0.1 * rate(T)
        return T - 0.1 * rate(0.5 * (half + T))
    if path == "ns":
        return _ns_exact(s)
    if path == "nsc":
        return _nsc_exact(s, case["scheme"])
    return _net_exact(s)
