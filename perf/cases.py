"""The work measured when this framework's speed is compared between two builds.

Kinds of case:

  solve   one rks_solve on a context that is kept (matrix resident in HBM, a
          start vector of the seed on the device), a fixed number of restart
          cycles, then rks_eigpairs: Ritz values, Ritz vectors on the device
          and the verified FP64 residuals.  A bounded number of cycles is a
          solve as it runs in earnest (first extension, contractions,
          rotations, extensions, residual check), cut off before the
          operator's own conditioning separates two correct runs.
  sketch  rks_sketch_noalloc: z = Omega x in a caller's loop, nothing kept.
  start   the learned start: features of the velocity field on the host to
          an FP64 start vector on the N x N grid on the device.
  train   one training step of the start network: forward, loss, backward,
          Adam; returns losses, gradients and updated weights.
  layer   forward and backward of one 3x3 convolution layer.
"""
import math

import numpy as np
import torch

import paper_2508_05400_amd as P
from paper_2508_05400_amd.learned_start import LAYERS, StartNet

DEV = "cuda"


def _solve(name, op, size, k, m, d, which, restarts, sketch="sparse", precision="fp64", method="rks", keep=-1):
    return dict(name=name, kind="solve", op=op, size=size, k=k, m=m, d=d, which=which, restarts=restarts,
                sketch=sketch, precision=precision, method=method, keep=keep)


def listed():
    return [
        # a start vector for one new operator of the 512^2 family: six small
        # convolutions and an upsampling, latency counts
        dict(name="start-512", kind="start", N=512),
        # one step of the network's training at its batch size
        dict(name="train-32", kind="train", B=32),
        # the embedding alone in a serving loop, at the size of a 1000^2 grid
        dict(name="sketch-1m", kind="sketch", n=1_000_000, d=240, sketch="sparse"),
        # the smallest solver workload: 100^2 grid, Gaussian embedding
        _solve("cd2d-100-gauss", "cd2d", 100, 10, 40, 80, "LR", 4, sketch="gauss"),
        # one operator of the 512^2 variable-velocity family (8-byte values)
        _solve("field-512", "field", 512, 16, 48, 192, "SR", 6),
        # the 2D workload of middle size
        _solve("cd2d-1000", "cd2d", 1000, 20, 60, 240, "SR", 4),
        # the headline workload
        _solve("cd3d-160", "cd3d", 160, 30, 90, 360, "LR", 3),
        # the pair basis on an odd grid
        _solve("cd3d-101-pair", "cd3d", 101, 30, 90, 360, "LR", 2, precision="fp32+fx16"),
        # a low-precision phase with its FP64 refinement, odd grid
        _solve("cd2d-777-fp32", "cd2d", 777, 20, 60, 240, "LR", 4, precision="fp32"),
        # irregular rows, x gathered from everywhere, column-blocked layout
        _solve("powerlaw-2m", "powerlaw", 2_000_000, 50, 120, 480, "LM", 1),
        # irregular rows on a matrix of ordinary size: row tiles
        _solve("powerlaw-150k", "powerlaw", 150_001, 20, 60, 240, "LM", 4),
        # the comparison method on the tridiagonal family
        _solve("tridiag-1m-ks", "tridiag", 1_000_000, 40, 80, 160, "LM", 2, method="ks_cgs2"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["sketch", "start", "train", "layer"])
    if kind == "sketch":
        sk = rng.choice(["sparse", "gauss"])
        return dict(kind=kind, n=_log_int(rng, 5_000, 4_000_000 if sk == "sparse" else 200_000),
                    d=_log_int(rng, 50, 512), sketch=sk)
    if kind == "start":
        return dict(kind=kind, N=_log_int(rng, 100, 1000))
    if kind == "train":
        return dict(kind=kind, B=_log_int(rng, 1, 64))
    if kind == "layer":
        return dict(kind=kind, B=_log_int(rng, 1, 48), C=rng.choice([2, 5, 16]), O=rng.choice([1, 3, 16]),
                    H=rng.randint(9, 96), W=rng.randint(9, 96), dil=rng.choice([1, 2, 3, 4, 8, 16]),
                    relu=rng.random() < 0.7)
    op = rng.choice(["cd2d", "cd2d", "cd3d", "field", "powerlaw", "tridiag"])
    k = rng.randint(6, 30)
    m = 2 * k + rng.randint(8, 30)
    d = rng.choice([2, 3, 4]) * m + rng.randint(0, 5)
    sketch, precision, method = "sparse", rng.choice(["fp64", "fp64", "fp32+fx16", "fp32", "bf16"]), "rks"
    if op in ("cd2d", "field"):
        size = _log_int(rng, 60, 1000)
        which = rng.choice(["LR", "SR"])
        if size <= 200 and rng.random() < 0.5:
            sketch = "gauss"
    elif op == "cd3d":
        size, which = _log_int(rng, 20, 128), "LR"
    elif op == "powerlaw":
        size, which = _log_int(rng, 20_000, 1_500_000), "LM"
    else:
        size, which = _log_int(rng, 50_000, 2_000_000), "LM"
        if rng.random() < 0.4:
            method, precision = "ks_cgs2", "fp64"
    return dict(kind="solve", op=op, size=size, k=k, m=m, d=d, which=which, restarts=rng.randint(1, 3),
                sketch=sketch, precision=precision, method=method, keep=-1)


# ---- operators as CSR arrays on the device -----------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _stencil(N, dim, gammas):
    """-Laplace(u) + beta . grad(u), central differences on N^dim interior
    points, unknowns x-fastest; gammas: beta h / 2 per axis (numbers or node values)."""
    n = N ** dim
    ih2 = float((N + 1) ** 2)
    idx = torch.arange(n, device=DEV)
    co = [(idx // N ** c) % N for c in range(dim)]
    col = torch.empty((n, 2 * dim + 1), dtype=torch.int64, device=DEV)
    val = torch.empty((n, 2 * dim + 1), dtype=torch.float64, device=DEV)
    ok = torch.ones((n, 2 * dim + 1), dtype=torch.bool, device=DEV)
    for c in range(dim):
        lo, hi = dim - 1 - c, dim + 1 + c
        col[:, lo], col[:, hi] = idx - N ** c, idx + N ** c
        val[:, lo], val[:, hi] = (-1.0 - gammas[c]) * ih2, (-1.0 + gammas[c]) * ih2
        ok[:, lo], ok[:, hi] = co[c] > 0, co[c] < N - 1
    col[:, dim], val[:, dim] = idx, 2.0 * dim * ih2
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = ok.sum(1).cumsum(0)
    return rp.int(), col[ok].int(), val[ok]


def _field(N, seed, modes=8, amp=40.0, kmax=3):
    """Velocity components at the nodes: random Fourier modes."""
    rng = np.random.default_rng(seed)
    t = torch.arange(1, N + 1, dtype=torch.float64, device=DEV) / (N + 1)
    out = []
    for _ in range(2):
        f = torch.zeros((N, N), dtype=torch.float64, device=DEV)
        for _ in range(modes):
            p, r = int(rng.integers(-kmax, kmax + 1)), int(rng.integers(1, kmax + 1))
            a, phi = float(rng.uniform(0.0, amp)), float(rng.uniform(0.0, 2 * math.pi))
            f += a * torch.cos(2 * math.pi * (p * t[None, :] + r * t[:, None]) + phi)
        out.append(f.reshape(-1))
    return out


def _powerlaw(n, seed, lmin=4, lmax=512, alpha=2.0675):
    """Row lengths P(l) ~ l^-alpha, uniform columns, N(0,1)/sqrt(l), and a diagonal N(0, 0.1^2)."""
    g = _gen(seed)
    ell = torch.arange(lmin, min(lmax, n - 1) + 1, dtype=torch.float64, device=DEV)
    cdf = torch.cumsum(ell ** -alpha, 0)
    L = torch.searchsorted(cdf / cdf[-1], torch.rand(n, generator=g, device=DEV, dtype=torch.float64)) + lmin
    L = L.clamp(max=int(ell[-1]))
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), L)
    cols = torch.randint(0, n, (rows.numel(),), generator=g, device=DEV)
    diag = torch.arange(n, device=DEV) * (n + 1)
    key = torch.unique(torch.cat([rows * n + cols, diag]))
    rows, cols = key // n, key % n
    val = torch.randn(key.numel(), generator=g, device=DEV, dtype=torch.float64)
    val *= torch.where(rows == cols, 0.1, 1.0 / L.double()[rows].sqrt())
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.bincount(rows, minlength=n).cumsum(0)
    return rp.int(), cols.int(), val


def _tridiag(n, seed):
    """Diagonal exp(t / 10) on n points of [2, 10], off-diagonals N(0,1)/100."""
    g = _gen(seed)
    idx = torch.arange(n, device=DEV)
    col = torch.stack([idx - 1, idx, idx + 1], 1)
    val = torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64) / 100.0
    val[:, 1] = torch.exp(torch.linspace(2.0, 10.0, n, dtype=torch.float64, device=DEV) / 10.0)
    ok = (col >= 0) & (col < n)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = ok.sum(1).cumsum(0)
    return rp.int(), col[ok].int(), val[ok]


def _operator(op, size, seed):
    h2 = 0.5 / (size + 1)
    if op == "cd2d":
        return _stencil(size, 2, [20.0 * h2, 10.0 * h2])
    if op == "cd3d":
        return _stencil(size, 3, [40.0 * h2, 20.0 * h2, 10.0 * h2])
    if op == "field":
        return _stencil(size, 2, [b * h2 for b in _field(size, seed)])
    return _powerlaw(size, seed) if op == "powerlaw" else _tridiag(size, seed)


def _order(case):
    return case["size"] ** {"cd2d": 2, "field": 2, "cd3d": 3}.get(case["op"], 1)


class _Context:
    """A solver context that frees itself with the state."""

    def __init__(self, *a):
        self.ctx = P.rks_create(*a)

    def __del__(self):
        P.rks_destroy(self.ctx)


# ---- states ------------------------------------------------------------------

def _net(seed):
    return StartNet(seed=seed % (1 << 31))


def _batch(B, seed):
    """Velocity features (2 x 64 x 64 per sample) and orthonormal targets (4096 x 17)."""
    g = _gen(seed)
    x = torch.nn.functional.interpolate(torch.randn((B, 2, 8, 8), generator=g, device=DEV), size=(64, 64),
                                        mode="bilinear")
    V = torch.linalg.qr(torch.randn((B, 4096, 17), generator=g, device=DEV))[0].contiguous()
    return x.contiguous(), V


def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind == "solve":
        n = _order(case)
        rp, col, val = _operator(case["op"], case["size"], seed)
        opts = P.rks_opts_default(sketch_kind=case["sketch"], sketch_seed=5, precision=case["precision"],
                                  method=case["method"], max_restarts=case["restarts"], keep=case["keep"],
                                  stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        ctx = _Context(rp, col, val, n, case["k"], case["m"], case["d"], case["which"], 1e-10, opts)
        return dict(case=case, ctx=ctx, u0=torch.randn(n, generator=g, device=DEV, dtype=torch.float64),
                    X=torch.empty((case["k"] + 1, n), dtype=torch.float64, device=DEV))
    if kind == "sketch":
        return dict(case=case, seed=seed, x=torch.randn(case["n"], generator=g, device=DEV, dtype=torch.float64),
                    z=torch.empty(case["d"], dtype=torch.float64, device=DEV))
    if kind == "start":
        feats = np.random.default_rng(seed).standard_normal((2, 64, 64)).astype(np.float32)
        return dict(case=case, net=_net(seed), feats=feats)
    if kind == "train":
        x, V = _batch(case["B"], seed)
        return dict(case=case, net=_net(seed), x=x, V=V)
    B, C, O, H, W = (case[q] for q in "BCOHW")
    r = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    return dict(case=case, x=r(B, C, H, W), w=r(O, C, 3, 3) * math.sqrt(2.0 / (9 * C)), b=0.1 * r(O),
                dy=r(B, O, H, W), y=torch.empty((B, O, H, W), device=DEV), dx=torch.empty((B, C, H, W), device=DEV),
                dw=torch.empty((O, C, 3, 3), device=DEV), db=torch.empty(O, device=DEV))


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "solve":
        ctx = s["ctx"].ctx
        P.rks_solve(ctx, s["u0"])
        ke = P.rks_num_pairs(ctx)
        re, im, res = np.empty(ke), np.empty(ke), np.empty(ke)
        P.rks_eigpairs(ctx, re, im, s["X"], res)
        # (an extra member of a conjugate pair at the boundary is left out)
        X, step = s["X"][:c["k"]], max(1, s["u0"].numel() // 16384)
        # a Ritz vector is defined up to its sign: the one with a positive product with the start
        X.mul_((X[:, ::step] * s["u0"][::step]).sum(1, keepdim=True).sign())
        return dict(re=re[:c["k"]], im=im[:c["k"]], X=X, resid=res[:c["k"]])
    if kind == "sketch":
        P.rks_sketch_noalloc(c["n"], c["d"], c["sketch"], 8, s["seed"], s["x"], s["z"], torch.cuda.current_stream())
        return s["z"]
    if kind == "start":
        return s["net"].start_vector(s["feats"], c["N"])
    if kind == "train":
        net = s["net"]
        acts = net.forward(s["x"])
        loss, du = net.loss_and_grad(acts[-1], s["V"])
        gw, gb = net.backward(acts, du)
        net.adam(gw, gb, 2e-3)
        return dict(out=acts[-1], loss=loss, gw=gw, gb=gb, w=list(net.w), b=list(net.b))
    dims = tuple(c[q] for q in "BCOHW") + (c["dil"],)
    P.rks_net_conv3x3_forward(s["x"], s["w"], s["b"], s["y"], *dims, c["relu"])
    P.rks_net_conv3x3_backward(s["x"], s["w"], s["y"] if c["relu"] else None, s["dy"], s["dx"], s["dw"], s["db"],
                               *dims, c["relu"])
    return dict(y=s["y"], dx=s["dx"], dw=s["dw"], db=s["db"])


# ---- what a pass cannot do without ---------------------------------------------

def _conv_work(B, C, O, H, W, backward, dx):
    """Each tensor once; two operations per product and tap."""
    px, taps = B * H * W, 18.0 * B * H * W * C * O
    b, f = 4.0 * px * (C + O), taps
    if backward:
        b += 4.0 * px * (C + 2 * O + (C if dx else 0))
        f += taps * (2 if dx else 1)
    return b, f


def _nnz(case):
    n = _order(case)
    return {"cd2d": 5.0, "field": 5.0, "cd3d": 7.0, "powerlaw": 17.0, "tridiag": 3.0}[case["op"]] * n


def work(case):
    kind = case["kind"]
    if kind == "sketch":
        n, d = case["n"], case["d"]
        return dict(bytes=8.0 * (n + d), flops=2.0 * n * (8 if case["sketch"] == "sparse" else d))
    if kind in ("start", "train"):
        B, train = case.get("B", 1), kind == "train"
        b = f = 0.0
        for li, (cin, cout, _) in enumerate(LAYERS):
            x, y = _conv_work(B, cin, cout, 64, 64, train, li > 0)
            b, f = b + x, f + y
        if train:
            return dict(bytes=b + 4.0 * B * 4096 * (17 + 2), flops=f + 4.0 * B * 4096 * 17)
        return dict(bytes=b + 8.0 * case["N"] ** 2, flops=f)
    if kind == "layer":
        b, f = _conv_work(case["B"], case["C"], case["O"], case["H"], case["W"], True, True)
        return dict(bytes=b, flops=f)
    # a step reads A's pattern and values, x and w once, and the basis once per
    # projection (twice two for classical Gram-Schmidt); a restart reads m
    # columns and writes the kept ones
    n, m, k = _order(case), case["m"], case["k"]
    kept = k + (m - k) // 4 if case["keep"] < 0 else max(k, case["keep"])
    eb = {"fp64": 8, "fp32+fx16": 6, "fp32": 4, "bf16": 2}[case["precision"]]
    aval = 1 if case["op"] in ("cd2d", "cd3d") else 8
    passes = 3 if case["method"] == "ks_cgs2" else 1
    a_b = _nnz(case) * (4 + aval) + 16.0 * n
    two = case["precision"] in ("fp32", "bf16")
    phases = [(eb, max(1, case["restarts"] // 2) if two else case["restarts"])]
    if two:
        phases.append((8, max(1, case["restarts"] - phases[0][1])))
    b = f = 0.0
    for e, r in phases:
        for t0, t1, cycles in ((0, m, 1), (kept, m, r)):
            for t in range(t0, t1):
                b += cycles * (a_b + e * n * (passes * (t + 1) + 1.0))
                f += cycles * (2 * _nnz(case) + 4.0 * n * (t + 1))
        b += (r + 1) * e * n * float(m + kept)
        f += (r + 1) * 2.0 * n * m * kept
    # Ritz vectors: k columns read, k written; their residuals need A once
    b += eb * n * k + 8.0 * n * k + _nnz(case) * (4 + aval)
    f += 2.0 * n * k * k + 2.0 * k * _nnz(case)
    return dict(bytes=b, flops=f)


# ---- the same in 64 bits -------------------------------------------------------

def _taps(x, dil, sign):
    """x shifted by the nine taps, zero outside: list of (di, dj, shifted)."""
    H, W = x.shape[-2:]
    p = torch.nn.functional.pad(x, (dil,) * 4)
    return [(i, j, p[..., dil + sign * dil * (i - 1): dil + sign * dil * (i - 1) + H,
                     dil + sign * dil * (j - 1): dil + sign * dil * (j - 1) + W])
            for i in range(3) for j in range(3)]


def _conv(x, w, b, dil, relu):
    B, C, H, W = x.shape
    y = b.view(1, -1, 1).expand(B, -1, H * W).clone()
    for i, j, xs in _taps(x, dil, 1):
        y += torch.matmul(w[:, :, i, j].contiguous(), xs.reshape(B, C, -1))
    y = y.reshape(B, -1, H, W)
    return y.clamp_min(0.0) if relu else y


def _conv_back(x, w, y, dy, dil, relu):
    g = torch.where(y > 0, dy, torch.zeros_like(dy)) if relu else dy
    B, O, H, W = g.shape
    C = x.shape[1]
    dw, gf = torch.empty_like(w), g.reshape(B, O, -1).transpose(0, 1).reshape(O, -1)
    for i, j, xs in _taps(x, dil, 1):
        dw[:, :, i, j] = gf @ xs.reshape(B, C, -1).transpose(0, 1).reshape(C, -1).t()
    dx = torch.zeros((B, C, H * W), dtype=x.dtype, device=x.device)
    for i, j, gs in _taps(g, dil, -1):
        dx += torch.matmul(w[:, :, i, j].t().contiguous(), gs.reshape(B, O, -1))
    return dx.reshape(x.shape), dw, gf.sum(1)


def _upsample(u, N):
    h = u.shape[0]
    t = ((torch.arange(N, dtype=torch.float64, device=DEV) + 0.5) * h / N - 0.5).clamp(0.0, h - 1.0)
    i0 = t.floor().long()
    i1, f = (i0 + 1).clamp(max=h - 1), t - t.floor()
    rows = (1 - f)[:, None] * u[i0] + f[:, None] * u[i1]
    return ((1 - f)[None, :] * rows[:, i0] + f[None, :] * rows[:, i1]).reshape(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "sketch"):  # Ritz pairs of a bounded run, and a drawn embedding: no plain counterpart
        return None
    s = prepare(case, seed)
    if kind == "layer":
        x, w, b, dy = (s[q].double() for q in ("x", "w", "b", "dy"))
        y = _conv(x, w, b, case["dil"], case["relu"])
        dx, dw, db = _conv_back(x, w, y, dy, case["dil"], case["relu"])
        return dict(y=y, dx=dx, dw=dw, db=db)
    net = s["net"]
    w, b = [p.double() for p in net.w], [p.double() for p in net.b]
    x = torch.tensor(s["feats"][None], device=DEV).double() if kind == "start" else s["x"].double()
    acts, last = [x], len(LAYERS) - 1
    for li, (_, _, dil) in enumerate(LAYERS):
        acts.append(_conv(acts[-1], w[li], b[li], dil, li < last))
    if kind == "start":
        return _upsample(acts[-1][0, 0], case["N"])
    B = case["B"]
    u, V = acts[-1].reshape(B, -1), s["V"].double()
    pk = (V * u[:, :, None]).sum(1)
    uu = (u * u).sum(1)
    rho = (pk * pk).sum(1) / uu
    du = -2.0 / (uu * B)[:, None] * ((V * pk[:, None, :]).sum(2) - rho[:, None] * u)
    gw, gb, g = [None] * (last + 1), [None] * (last + 1), du.reshape(acts[-1].shape)
    for li in range(last, -1, -1):
        g, gw[li], gb[li] = _conv_back(acts[li], w[li], acts[li + 1], g, LAYERS[li][2], li < last)
    # Adam's first step: m / c1 = g, v / c2 = g^2
    step = lambda p, q: p - 2e-3 * q / (q.abs() + 1e-8)  # noqa: E731
    return dict(out=acts[-1], loss=1.0 - rho, gw=gw, gb=gb, w=[step(p, q) for p, q in zip(w, gw)],
                b=[step(p, q) for p, q in zip(b, gb)])
