"""Shapes of the convolution kernels at which the split of the work changes:
output channels that do not fill the channels per lane, images smaller than
one step of the filter gradient's chains, dilations beyond the image, tensors
beyond 32-bit offsets, and infinite or NaN operands next to the border.

The reference sums the taps inside the image in FP64.  Bars: a chain of n FP32
fused multiply-adds is within n u of the sum of its terms' magnitudes
(u = 2^-24; one more for the stored operand), n = 9 C + 1 forward, 9 O for the
input gradient, pixels / 256 + 9 (chain and tree) for the filter gradient."""
import pytest

import paper_2508_05400_amd as P

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _windows(H, W, dil, t):
    """Row and column ranges of the pixels whose tap t lies inside the image."""
    di, dj = dil * (t // 3 - 1), dil * (t % 3 - 1)
    return slice(max(0, -di), min(H, H - di)), slice(max(0, -dj), min(W, W - dj)), di, dj


def _shift(s, d):
    return slice(s.start + d, s.stop + d)


def _reference(torch, x, w, b, dy, dil, relu, yk=None):
    """y, dx, dw, db and the sums of the terms' magnitudes, taps outside left
    out; the ReLU's mask of the gradient from yk, the layer output it is given."""
    x, w, b, dy = (v.double() for v in (x, w, b, dy))
    B, C, H, W = x.shape
    O = w.shape[0]
    y, ya = b.view(1, -1, 1, 1).repeat(B, 1, H, W), b.abs().view(1, -1, 1, 1).repeat(B, 1, H, W)
    taps = [(t, *_windows(H, W, dil, t)) for t in range(9)]
    taps = [q for q in taps if q[1].stop > q[1].start and q[2].stop > q[2].start]
    for t, r, c, di, dj in taps:
        xs = x[:, :, _shift(r, di), _shift(c, dj)]
        for ch in range(C):
            term = w[:, ch, t // 3, t % 3].view(1, -1, 1, 1) * xs[:, ch:ch + 1]
            y[:, :, r, c] += term
            ya[:, :, r, c] += term.abs()
    g = torch.where(yk > 0, dy, torch.zeros_like(dy)) if relu else dy
    dx, dxa = torch.zeros_like(x), torch.zeros_like(x)
    dw, dwa = torch.zeros_like(w), torch.zeros_like(w)
    for t, r, c, di, dj in taps:
        for o in range(O):
            term = w[o, :, t // 3, t % 3].view(1, -1, 1, 1) * g[:, o:o + 1, r, c]
            dx[:, :, _shift(r, di), _shift(c, dj)] += term
            dxa[:, :, _shift(r, di), _shift(c, dj)] += term.abs()
            prod = x[:, :, _shift(r, di), _shift(c, dj)] * g[:, o:o + 1, r, c]
            prod = torch.where(g[:, o:o + 1, r, c] == 0, torch.zeros_like(prod), prod)
            dw[o, :, t // 3, t % 3] = prod.sum((0, 2, 3))
            dwa[o, :, t // 3, t % 3] = prod.abs().sum((0, 2, 3))
    if relu:
        y = torch.where(y < 0, torch.zeros_like(y), y)
    return (y, ya), (dx, dxa), (dw, dwa), (g.sum((0, 2, 3)), g.abs().sum((0, 2, 3)))


def _run(torch, x, w, b, dy, dil, relu):
    B, C, H, W = x.shape
    O = w.shape[0]
    y, dx, dw, db = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w), torch.empty_like(b)
    P.rks_net_conv3x3_forward(x, w, b, y, B, C, O, H, W, dil, relu)
    P.rks_net_conv3x3_backward(x, w, y if relu else None, dy, dx, dw, db, B, C, O, H, W, dil, relu)
    return y, dx, dw, db


def _near(torch, got, ref, n):
    want, mag = ref
    fin = torch.isfinite(want)
    assert torch.equal(fin, torch.isfinite(got)) and torch.equal(torch.isnan(want), torch.isnan(got))
    assert torch.equal(want[~fin & ~want.isnan()], got.double()[~fin & ~want.isnan()])
    err = (got.double() - want).abs()[fin]
    assert bool((err <= (n + 1) * U * mag[fin] + 1e-37).all()), float((err / (n * U * mag[fin] + 1e-37)).max())


def _bars(B, C, O, H, W):
    chain = B * H * W / 256 + 9
    return 9 * C + 1, 9 * O, chain, chain


SHAPES = [
    (6, 3, 9, 64, 64, 1, 1),    # eight channels per lane, one left over
    (4, 2, 13, 64, 64, 5, 0),   # four per lane, three left over
    (2, 4, 13, 64, 64, 2, 1),   # two per lane, one left over
    (1, 16, 8, 15, 17, 3, 1),   # 255 pixels: less than one step of a chain; 128 channel pairs
    (5, 16, 7, 16, 16, 2, 0),   # 256 pixels; 112 pairs
    (3, 2, 2, 1, 257, 1, 1),    # one row
    (2, 1, 1, 9, 13, 40, 1),    # dilation beyond the image: the centre tap alone
    (2, 3, 2, 40, 3, 7, 0),     # beyond its width
]


@pytest.mark.parametrize("B,C,O,H,W,dil,relu", SHAPES)
def test_conv_shapes(lib, cuda, B, C, O, H, W, dil, relu):
    torch = cuda
    g = torch.Generator().manual_seed(B + 10 * C + 100 * O + W)
    r = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    x, w, b, dy = r(B, C, H, W), 0.3 * r(O, C, 3, 3), r(O), r(B, O, H, W)
    got = _run(torch, *(v.cuda() for v in (x, w, b, dy)), dil, relu)
    ref = _reference(torch, x, w, b, dy, dil, relu, got[0].cpu())
    for v, q, n in zip(got, ref, _bars(B, C, O, H, W)):
        _near(torch, v.cpu(), q, n)


def test_conv_infinite_and_nan_operands(lib, cuda):
    """Taps outside the image and masked gradients add nothing, whatever the other factor is."""
    torch = cuda
    B, C, O, H, W, dil = 1, 2, 3, 12, 20, 2
    g = torch.Generator().manual_seed(4)
    r = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    inf, nan = float("inf"), float("nan")
    x, w, b, dy = r(B, C, H, W), r(O, C, 3, 3), r(O), r(B, O, H, W)
    for kind in ("weight", "input", "gradient"):
        xs, ws, ds = x.clone(), w.clone(), dy.clone()
        if kind == "weight":
            ws[1, 0, 0, 0], ws[2, 1, 2, 1] = inf, nan
        elif kind == "input":
            xs[0, 0, 0, 0], xs[0, 1, 5, 7] = inf, nan
        else:
            ds[0, 2, 0, 3], ds[0, 0, 11, 19] = -inf, nan
        ref = _reference(torch, xs, ws, b, ds, dil, 0)
        got = _run(torch, *(v.cuda() for v in (xs, ws, b, ds)), dil, 0)
        for v, q, n in zip(got, ref, _bars(B, C, O, H, W)):
            _near(torch, v.cpu(), q, n)
    # an infinite input under a gradient that the ReLU masks everywhere
    xs, bs = x.clone(), torch.full((O,), -1e4)
    xs[0, 0, 6, 6] = -inf
    ws = w.abs() + 0.1
    got = _run(torch, *(v.cuda() for v in (xs, ws, bs, dy)), dil, 1)
    ref = _reference(torch, xs, ws, bs, dy, dil, 1, got[0].cpu())
    assert not bool(got[0].any())
    for v, q in zip(got[1:], ref[1:]):
        assert torch.equal(v.cpu().double(), q[0]) and not bool(q[0].any())


def test_conv_beyond_32_bit_offsets(lib, cuda):
    """One channel of 2^28 pixels: rows at both ends and the whole filter gradient."""
    torch = cuda
    n = 1 << 14
    g = torch.Generator(device="cuda").manual_seed(7)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    x, w, b, dy = r(1, 1, n, n), r(1, 1, 3, 3), r(1), r(1, 1, n, n)
    y, dx, dw, db = _run(torch, x, w, b, dy, 3, 0)
    for r0 in (0, n - 8):  # 8 rows and their neighbours
        lo, hi = max(0, r0 - 3), min(n, r0 + 11)
        ref = _reference(torch, *(v.cpu() for v in (x[:, :, lo:hi], w, b, dy[:, :, lo:hi])), 3, 0)
        rows = slice(0, 8) if r0 == 0 else slice(hi - lo - 8, hi - lo)
        for v, q, m in ((y, ref[0], 10), (dx, ref[1], 9)):
            _near(torch, v[:, :, r0:r0 + 8].cpu(), tuple(e[:, :, rows] for e in q), m)
    for t in range(9):
        rs, cs, di, dj = _windows(n, n, 3, t)
        s = a = 0.0
        for k in range(rs.start, rs.stop, 1024):
            q = slice(k, min(rs.stop, k + 1024))
            prod = x[0, 0, _shift(q, di), _shift(cs, dj)].double() * dy[0, 0, q, cs].double()
            s, a = s + float(prod.sum()), a + float(prod.abs().sum())
        assert abs(float(dw[0, 0, t // 3, t % 3]) - s) <= (n * n / 256 + 10) * U * a
