"""GPU tests of the general kernels (any map, rectangular windows, cached
matrices, float32 as bf16 parts) against plain float64 torch, at the edges of
their stages, tiles and row loads."""
import pytest
import torch

from helpers import TORCH_DTYPE
from paper_2607_02097_amd import binding as W

pytestmark = pytest.mark.gpu

# One rounding of the result (half an ulp: 2^-9, 2^-12) plus the float32 sums
# of at most 256 products: |error| <= half ulp |y| + 256 2^-24 sum |x m|, taken
# relative to sum |x m| per output, with a factor of two in hand.  float32:
# what the six partial products leave out is below 2^-24 of each product.
REL = {"f32": 2.0 ** -16, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}
# and half the spacing of the smallest values (float16's subnormals, 2^-24)
ABS = {"f32": 0.0, "bf16": 0.0, "f16": 2.0 ** -25}


def windows(v, wh, ww):
    B, C, H, Wd = v.shape
    v = torch.nn.functional.pad(v, (0, -Wd % ww, 0, -H % wh))
    nh, nw = v.shape[2] // wh, v.shape[3] // ww
    return v.reshape(B, C, nh, wh, nw, ww).permute(1, 0, 2, 4, 3, 5).reshape(C, B * nh * nw, wh * ww)


def unwindows(v, shape, wh, ww):
    B, C, H, Wd = shape
    nh, nw = -(-H // wh), -(-Wd // ww)
    v = v.reshape(C, B, nh, nw, wh, ww).permute(1, 0, 2, 4, 3, 5)
    return v.reshape(B, C, nh * wh, nw * ww)[:, :, :H, :Wd]


def index(wh, ww):
    p = torch.arange(wh * ww)
    h, x = p // ww, p % ww
    return (h[:, None] - h[None] + wh - 1) * (2 * ww - 1) + x[:, None] - x[None] + ww - 1


def data(B, C, H, Wd, wh, ww, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    td = TORCH_DTYPE[dtype]
    x = torch.randn((B, C, H, Wd), generator=g).to(td)
    t = (0.02 * torch.randn((C, (2 * wh - 1) * (2 * ww - 1)), generator=g)).to(td)
    return x, t


def check(got, x, m, wh, ww, dtype, label):
    """got against x m per window, each output relative to its sum |x m|."""
    xw = windows(x.double(), wh, ww)
    want = unwindows(xw @ m, x.shape, wh, ww)
    scale = unwindows(xw.abs() @ m.abs(), x.shape, wh, ww)
    err = (got.double().cpu() - want).abs()
    worst = float(((err - ABS[dtype]) / (scale + 1e-30)).max())
    print(label, "worst %.2e" % worst, flush=True)
    assert worst <= REL[dtype], label


# K steps 1..8 of both row pitches, their remainders, one stage and several
WINDOWS = [(1, 1), (1, 16), (2, 9), (3, 8), (4, 7), (5, 16), (7, 14), (8, 8), (9, 3), (10, 9), (12, 12), (13, 8),
           (14, 7), (14, 14), (15, 15), (16, 16)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("win", WINDOWS, ids=lambda w: "%dx%d" % w)
def test_matrix_and_table_products(win, dtype):
    """Dense forward and transposed product with an arbitrary matrix, and the
    rectangular-window forms with the matrix built from a table: maps smaller
    than a window, cut windows, odd widths, several stages."""
    wh, ww = win
    for B, C, H, Wd in ((1, 2, max(wh - 1, 4), ww + 1), (3, 3, 2 * wh + 1, 3 * ww - 1), (2, 1, 6 * wh, 11 * ww)):
        x, t = data(B, C, H, Wd, wh, ww, dtype, seed=wh * 31 + ww)
        g = torch.Generator().manual_seed(5)
        m = (0.1 * torch.randn((C, wh * ww, wh * ww), generator=g)).to(TORCH_DTYPE[dtype])
        xd, md, td = x.cuda(), m.cuda(), t.cuda()
        label = "%s %s %s" % (dtype, win, (B, C, H, Wd))
        check(W.wbmm_dense_forward(xd, md, wh, ww), x, m.double(), wh, ww, dtype, "dense " + label)
        check(W.wbmm_dense_backward_input(xd, md, wh, ww), x, m.double().transpose(1, 2), wh, ww, dtype,
              "dense^T " + label)
        mt = t.double()[:, index(wh, ww)]
        check(W.wbmm_rect_forward(xd, td, wh, ww), x, mt, wh, ww, dtype, "rect " + label)
        check(W.wbmm_rect_backward_input(xd, td, wh, ww), x, mt.transpose(1, 2), wh, ww, dtype, "rect^T " + label)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 3, 1, 5), (1, 1, 3, 5), (2, 2, 2, 2), (1, 1, 4, 4)],
                         ids=lambda s: "B%dC%dH%dW%d" % s)
def test_tensors_shorter_than_a_row_load(shape, dtype):
    """Fewer than, and exactly, the sixteen elements that a row load takes, in
    the map and (windows of one to three positions) in the matrix."""
    B, C, H, Wd = shape
    for w in (2, 7, 14):
        x, t = data(B, C, H, Wd, w, w, dtype, seed=w)
        m = t.double()[:, index(w, w)]
        check(W.wbmm_forward(x.cuda(), t.cuda(), w), x, m, w, w, dtype, "fwd %s %s w%d" % (dtype, shape, w))
        check(W.wbmm_rect_forward(x.cuda(), t.cuda(), w, w), x, m, w, w, dtype, "rect %s %s w%d" % (dtype, shape, w))
    for C in (1, 3, 15, 16):
        for wh, ww in ((1, 1), (1, 3), (2, 1)):
            x, t = data(2, C, 9, 20, wh, ww, dtype, seed=C)
            m = t.double()[:, index(wh, ww)]
            check(W.wbmm_rect_forward(x.cuda(), t.cuda(), wh, ww), x, m, wh, ww, dtype, "small matrix %d %dx%d" % (C, wh, ww))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("w", [7, 8, 9, 13, 14, 16])
def test_cut_maps_equal_padded_maps(w, dtype):
    """A map cut inside its last windows takes the general kernel, the same
    map padded with zeros to whole windows the fixed-layout kernels: the same
    products in the same order, so the same bits."""
    B, C, nh, nw = 2, 3, 4, 4
    H, Wd = nh * w - 1, nw * w - 3
    x, t = data(B, C, H, Wd, w, w, dtype, seed=w)
    xd, td = x.cuda(), t.cuda()
    xp = torch.nn.functional.pad(xd, (0, nw * w - Wd, 0, nh * w - H)).contiguous()
    for f in (W.wbmm_forward, W.wbmm_backward_input):
        assert torch.equal(f(xd, td, w), f(xp, td, w)[:, :, :H, :Wd])


# few channels: the staged kernel (rows of eight: the direct one); many: enough
# 16-window units for the direct one
@pytest.mark.parametrize("w,C", [(9, 2), (14, 2), (16, 2), (5, 2), (7, 3), (9, 1024), (12, 700), (14, 1024), (16, 600)])
def test_float32_range(w, C):
    """float32 rows and tables outside the range of the bf16 parts take
    float32 products: infinities and NaN reach exactly the outputs of their
    window, huge, tiny and denormal values keep float32's precision, and a
    zero table or zero rows give zeros."""
    B, H, Wd = 3, 2 * w, 3 * w
    fwd = W.wbmm_forward if w > 8 else (lambda x, t, w: W.wbmm_rect_forward(x, t, w, w))
    x, t = data(B, C, H, Wd, w, w, "f32", seed=w)
    m = t.double()[:, index(w, w)]
    check(fwd(x.cuda(), t.cuda(), w), x, m, w, w, "f32", "plain")
    for s in (2.0 ** 70, 2.0 ** -100, 2.0 ** -120):
        xs = x * s
        check(fwd(xs.cuda(), t.cuda(), w) / s, xs / s, m, w, w, "f32", "x scaled by %g" % s)
    for s in (2.0 ** 66, 2.0 ** -70):
        check(fwd(x.cuda(), (t * s).cuda(), w) / s, x, m, w, w, "f32", "table scaled by %g" % s)
    # a few rows far out of range beside ordinary ones
    xm = x.clone()
    xm[1, 0, 3] *= 2.0 ** 80
    xm[2, 1, w + 1] *= 2.0 ** -110
    check(fwd(xm.cuda(), t.cuda(), w), xm, m, w, w, "f32", "mixed rows")
    for bad in (float("inf"), float("-inf"), float("nan")):
        xb = x.clone()
        xb[1, 1, w + 2, 3] = bad
        y = fwd(xb.cuda(), t.cuda(), w).cpu()
        hit = torch.zeros_like(xb, dtype=torch.bool)
        hit[1, 1, w:2 * w, 0:w] = True
        assert not torch.isfinite(y[hit]).any() and torch.isfinite(y[~hit]).all()
        if bad != bad:
            assert torch.isnan(y[hit]).all()
        else:
            assert torch.isinf(y[hit]).all()
    assert not fwd(torch.zeros_like(x).cuda(), t.cuda(), w).any()
    assert not fwd(x.cuda(), torch.zeros_like(t).cuda(), w).any()


# rows without fixed offsets at the sizes the general gradients take, windows
# of every K-step count: cut maps, odd windows, window counts that are no
# power of two, one and several slabs, more channels than compute units
GRAD = [(24, 96, 31, 31, 3), (40, 64, 29, 31, 4), (9, 300, 28, 28, 7), (64, 40, 29, 31, 7), (16, 96, 42, 42, 8),
        (30, 200, 27, 27, 9), (6, 64, 113, 99, 10), (2, 600, 61, 61, 12), (8, 96, 100, 61, 14), (11, 96, 84, 84, 14),
        (3, 17, 301, 299, 15), (9, 40, 111, 109, 16)]


def exact_gradients(x, dy, t, w):
    idx = index(w, w).to(x.device)
    xw, gw = windows(x.double(), w, w), windows(dy.double(), w, w)
    m = t.double()[:, idx]
    g = torch.bmm(xw.transpose(1, 2).contiguous(), gw.contiguous())
    dt = torch.zeros(t.shape, dtype=torch.float64, device=x.device).index_add_(1, idx.flatten(), g.flatten(1))
    dx = unwindows(torch.bmm(gw.contiguous(), m.transpose(1, 2).contiguous()), x.shape, w, w)
    return dx, dt


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", GRAD, ids=lambda s: "B%dC%dH%dW%dw%d" % s)
def test_general_gradients(shape, dtype):
    """The fused backward equals the separate calls bit for bit and the exact
    gradients within tolerance (dT: float32 sums of exact products, held to
    1e-5 of the largest entry as in the parity tests)."""
    B, C, H, Wd, w = shape
    x, t = (v.cuda() for v in data(B, C, H, Wd, w, w, dtype, seed=w))
    dy, _ = (v.cuda() for v in data(B, C, H, Wd, w, w, dtype, seed=w + 100))
    dx, dt = W.wbmm_backward(x, dy, t, w)
    assert torch.equal(dt, W.wbmm_backward_table(x, dy, w))
    assert torch.equal(dx, W.wbmm_backward_input(dy, t, w))
    wdx, wdt = exact_gradients(x, dy, t, w)
    e_t = float((dt.double() - wdt).abs().max() / wdt.abs().max())
    e_x = float((dx.double() - wdx).abs().max() / wdx.abs().max())
    print(shape, dtype, "dt %.1e dx %.1e" % (e_t, e_x), flush=True)
    assert e_t <= 1e-5 and e_x <= 2e-2


@pytest.mark.parametrize("shape", [(20, 200, 27, 27, 13), (14, 192, 28, 28, 14), (10, 300, 30, 31, 15),
                                   (3, 40, 160, 150, 16), (64, 192, 14, 14, 7), (8, 96, 61, 50, 7), (5, 60, 96, 96, 8),
                                   (9, 96, 56, 56, 5), (30, 90, 28, 28, 9)], ids=lambda s: "B%dC%dH%dW%dw%d" % s)
def test_general_gradients_float32(shape):
    """As above in float32 (and the forward), then with rows of x or dy out of the range of the
    bf16 parts (their stages take float32 products)."""
    B, C, H, Wd, w = shape
    x, t = (v.cuda() for v in data(B, C, H, Wd, w, w, "f32", seed=w))
    dy, _ = (v.cuda() for v in data(B, C, H, Wd, w, w, "f32", seed=w + 100))
    for case in ("plain", "huge", "tiny"):
        if case == "huge":
            x[1, 3, 5] *= 2.0 ** 70
        if case == "tiny":
            x[1, 3, 5] *= 2.0 ** -70
            dy[0, :, :w] *= 2.0 ** -110
        dx, dt = W.wbmm_backward(x, dy, t, w)
        assert torch.equal(dt, W.wbmm_backward_table(x, dy, w))
        assert torch.equal(dx, W.wbmm_backward_input(dy, t, w))
        assert torch.equal(W.wbmm_forward(x, t, w), W.wbmm_rect_forward(x, t, w, w))
        wdx, wdt = exact_gradients(x, dy, t, w)
        err = (dt.double() - wdt).abs().amax(1) / wdt.abs().amax(1)  # per channel: each has its own scale
        e_x = float((dx.double() - wdx).abs().max() / wdx.abs().max())
        print(shape, case, "dt %.1e dx %.1e" % (float(err.max()), e_x), flush=True)
        assert float(err.max()) <= 1e-5 and e_x <= 1e-5
    x[0, 2, 7, 9] = float("nan")
    _, dt = W.wbmm_backward(x, dy, t, w)
    assert torch.isnan(dt[2]).any() and not torch.isnan(dt[:2]).any() and not torch.isnan(dt[3:]).any()


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("win", WINDOWS, ids=lambda w: "%dx%d" % w)
def test_rectangular_table_gradient(win, dtype):
    """From the table, against float64 and against the matrix gradient folded
    by wbmm_bin_matrix; tiny maps, cut windows, several slabs."""
    wh, ww = win
    for B, C, H, Wd in ((1, 1, 2, 3), (1, 2, max(wh - 1, 4), ww + 5), (3, 3, 2 * wh + 1, 3 * ww - 1),
                        (7, 5, 6 * wh, 11 * ww)):
        x, _ = data(B, C, H, Wd, wh, ww, dtype, seed=wh + ww)
        dy, _ = data(B, C, H, Wd, wh, ww, dtype, seed=wh * ww)
        xw, gw = windows(x.double(), wh, ww), windows(dy.double(), wh, ww)
        idx = index(wh, ww).flatten()
        want = torch.zeros((C, (2 * wh - 1) * (2 * ww - 1)), dtype=torch.float64)
        want.index_add_(1, idx, (xw.transpose(1, 2) @ gw).flatten(1))
        scale = torch.zeros_like(want).index_add_(1, idx, (xw.abs().transpose(1, 2) @ gw.abs()).flatten(1))
        got = W.wbmm_rect_backward_table(x.cuda(), dy.cuda(), wh, ww)
        fold = W.wbmm_bin_matrix(W.wbmm_dense_backward_matrix(x.cuda(), dy.cuda(), wh, ww), wh, ww)
        # float32 sums of exact products (f32: of parts that leave out 2^-24)
        for r in (got, fold):
            worst = float(((r.double().cpu() - want).abs() / (scale + 1e-30)).max())
            assert worst <= 2.0 ** -18, (win, dtype, (B, C, H, Wd), worst)


def test_rectangular_errors_and_streams():
    x, t = (v.cuda() for v in data(2, 3, 20, 30, 4, 9, "bf16", seed=1))
    with pytest.raises(ValueError):
        W.wbmm_rect_forward(x, t[:2].contiguous(), 4, 9)
    with pytest.raises(ValueError):
        W.wbmm_rect_forward(x, t.float(), 4, 9)
    with pytest.raises(ValueError):
        W.wbmm_rect_backward_table(x, x[:1].contiguous(), 4, 9)
    with pytest.raises(W.WbmmError):
        W.wbmm_rect_backward_table(x, x, 17, 9)
    want = W.wbmm_rect_backward_table(x, x, 4, 9)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    got = W.wbmm_rect_backward_table(x, x, 4, 9, stream=s)
    s.synchronize()
    assert torch.equal(got, want)


# one unit of 16 windows per wave (1024 units and more) against the staged
# kernel, which the matrix form takes: the same products in the same order.
# K steps 1..8, rows that fill the last K step and rows that do not, one round
# of units per wave and several, cut maps that end inside a row load.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B", [2, 13])
@pytest.mark.parametrize("win", [(1, 1), (4, 8), (7, 7), (9, 5), (16, 3), (13, 8), (2, 16), (3, 9), (5, 11), (7, 14),
                                 (9, 9), (12, 12), (13, 13), (14, 14), (15, 15), (16, 16)], ids=lambda w: "%dx%d" % w)
def test_units_equal_stages(win, B, dtype):
    wh, ww = win
    C, H, Wd = 1030, 2 * wh - wh // 2, 2 * ww + 1
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn((B, C, H, Wd), generator=g, device="cuda").to(TORCH_DTYPE[dtype])
    t = (0.02 * torch.randn((C, (2 * wh - 1) * (2 * ww - 1)), generator=g, device="cuda")).to(TORCH_DTYPE[dtype])
    # infinities stay where they belong
    x[0, 3, 0, 0] = x[-1, 5, -1, -1] = float("inf")
    t[7, 0] = t[9, -1] = float("inf")
    m = W.wbmm_build_matrix(t, wh, ww)
    for got, want in ((W.wbmm_rect_forward(x, t, wh, ww), W.wbmm_dense_forward(x, m, wh, ww)),
                      (W.wbmm_rect_backward_input(x, t, wh, ww), W.wbmm_dense_backward_input(x, m, wh, ww))):
        assert torch.equal(got.isnan(), want.isnan()), "NaN"
        assert torch.equal(got.nan_to_num(1.0, 2.0, -2.0), want.nan_to_num(1.0, 2.0, -2.0))


# three windows a map row (rows without fixed offsets), 135 windows a channel,
# channels on either side of the line for rows of eight: the windows one by one
# as images of their own, at most 100 a call (from 128 on odd windows would take
# the general kernels again), take the fixed-layout kernels, with the same sums
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("w,C", [(4, 120), (5, 120), (6, 113), (7, 120), (8, 114), (8, 3), (9, 3), (11, 5), (14, 120), (16, 3)])
def test_rows_without_fixed_offsets(w, C, dtype):
    td = TORCH_DTYPE[dtype]
    g = torch.Generator(device="cuda").manual_seed(w)
    x = torch.randn((15, C, 3 * w, 3 * w), generator=g, device="cuda").to(td)
    dy = torch.randn(x.shape, generator=g, device="cuda").to(td)
    t = (0.02 * torch.randn((C, (2 * w - 1) ** 2), generator=g, device="cuda")).to(td)

    def apart(v):
        return v.reshape(15, C, 3, w, 3, w).permute(0, 2, 4, 1, 3, 5).reshape(135, C, w, w).contiguous()

    def alone(f, v):
        return torch.cat([f(part.contiguous(), t, w) for part in apart(v).split(100)])
    assert torch.equal(apart(W.wbmm_forward(x, t, w)), alone(W.wbmm_forward, x))
    dx = W.wbmm_backward_input(dy, t, w)
    assert torch.equal(apart(dx), alone(W.wbmm_backward_input, dy))
    assert torch.equal(W.wbmm_backward(x, dy, t, w)[0], dx)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_more_channels_than_one_grid_dimension(dtype):
    """2^23 + 5 channels of one 1 x 2 window: at 512 threads a channel more
    than the 2^32 threads of a grid dimension.  y0 = x0 T1 + x1 T2, y1 = x0 T0
    + x1 T1; dT = (x0 dy1, x0 dy0 + x1 dy1, x1 dy0).  Small whole numbers:
    every result is exact."""
    C, td = 2 ** 23 + 5, TORCH_DTYPE[dtype]
    g = torch.Generator(device="cuda").manual_seed(5)
    x, dy, t = (torch.randint(-3, 4, s, generator=g, device="cuda").to(td) for s in ((1, C, 1, 2), (1, C, 1, 2), (C, 3)))
    x0, x1, d0, d1 = x[0, :, 0, 0], x[0, :, 0, 1], dy[0, :, 0, 0], dy[0, :, 0, 1]
    t0, t1, t2 = t.unbind(1)
    y = W.wbmm_rect_forward(x, t, 1, 2)
    assert torch.equal(y[0, :, 0], torch.stack([x0 * t1 + x1 * t2, x0 * t0 + x1 * t1], 1))
    dx = W.wbmm_rect_backward_input(dy, t, 1, 2)
    assert torch.equal(dx[0, :, 0], torch.stack([d0 * t1 + d1 * t0, d0 * t2 + d1 * t1], 1))
    dt = W.wbmm_rect_backward_table(x, dy, 1, 2)
    assert torch.equal(dt, torch.stack([x0 * d1, x0 * d0 + x1 * d1, x1 * d0], 1).float())


def pattern(v):
    """0: finite, 1 and 2: the infinities, 3: NaN."""
    v = v.float().cpu()
    return torch.where(v.isnan(), 3, 0) + torch.where(v == float("inf"), 1, 0) + torch.where(v == -float("inf"), 2, 0)


# rows of eight and of sixteen that the window fills and does not, odd and even
# heights; square windows at sizes where both gradients take the general kernel
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 3, 2 * h + 1, 2 * w + 1, h, w) for h, w in (
    (1, 3), (2, 8), (5, 5), (7, 7), (8, 6), (9, 3), (11, 8), (13, 7), (15, 4), (16, 8), (1, 16), (3, 9), (6, 14),
    (9, 12), (11, 16), (13, 13), (14, 14), (15, 10), (16, 16))]
    + [(64, 40, 29, 31, 7, 7), (5, 60, 96, 96, 8, 8), (20, 200, 27, 27, 13, 13), (8, 96, 100, 61, 14, 14)],
    ids=lambda s: "B%dC%dH%dW%dw%dx%d" % s)
def test_gradient_infinities_stay_in_their_pairs(shape, dtype):
    """Infinities and NaN at the corners of windows reach the table entries
    of the pairs they are in and no others: entry by entry what the matrix
    gradient, which has no pad positions, folds to."""
    B, C, H, Wd, wh, ww = shape
    x, _ = (v.cuda() for v in data(B, C, H, Wd, wh, ww, dtype, seed=1))
    dy, t = (v.cuda() for v in data(B, C, H, Wd, wh, ww, dtype, seed=2))
    inf, nan = float("inf"), float("nan")
    x[1, 0, wh - 1, ww - 1] = inf
    x[0, 1, 0, 0] = -inf
    dy[1, 1, wh - 1, 0] = inf
    dy[0, 2, 0, ww - 1] = nan
    x[-1, 2, -1, -1] = inf
    want = pattern(W.wbmm_bin_matrix(W.wbmm_dense_backward_matrix(x, dy, wh, ww), wh, ww))
    assert want.any() and (wh * ww < 4 or not want[:, (2 * wh - 1) * (2 * ww - 1) // 2 - 1].all())
    assert torch.equal(pattern(W.wbmm_rect_backward_table(x, dy, wh, ww)), want)
    if B * C * H * Wd >= 2 ** 21:
        assert torch.equal(pattern(W.wbmm_backward_table(x, dy, wh)), want)
        assert torch.equal(pattern(W.wbmm_backward(x, dy, t, wh)[1]), want)


def rounding(adds):
    """The relative 2-norm error of a float32 sum of random terms added one by
    one: an addition rounds by at most 2^-23 / sqrt(12) = 2^-24.8 of the partial
    sum (rms), which after k of n has sqrt(k / n) of the result's size; half as
    much again for the sums that do not grow so evenly.  (Leaving out any of the
    six partial products would show as 2^-18 / 3 = 1.3e-6.)"""
    return 1.5 * 2.0 ** -24.8 * (adds / 2) ** 0.5


# table gradients with one and several stages per partial sum, up to six K
# steps and more, many channels and one; products in units, in stages and from
# a matrix
@pytest.mark.parametrize("shape", [(28, 36, 98, 98, 14, 14), (1, 1, 1500, 1500, 13, 13), (1, 2, 1100, 1100, 16, 16),
                                   (8, 195, 53, 71, 15, 15), (64, 192, 28, 28, 14, 14), (4, 31, 72, 60, 12, 12),
                                   (64, 96, 56, 56, 7, 7), (9, 16, 65, 80, 16, 8), (1, 3, 40, 50, 9, 14),
                                   (2, 8, 33, 40, 5, 5)], ids=lambda s: "B%dC%dH%dW%dw%dx%d" % s)
def test_float32_precision(shape):
    """float32 results are as good as sums of float32 products rounded once
    per addition."""
    B, C, H, Wd, wh, ww = shape
    x, t = (v.cuda() for v in data(B, C, H, Wd, wh, ww, "f32", seed=wh))
    dy, _ = (v.cuda() for v in data(B, C, H, Wd, wh, ww, "f32", seed=wh + 100))
    xw, gw = windows(x.double(), wh, ww).contiguous(), windows(dy.double(), wh, ww).contiguous()
    idx = index(wh, ww).cuda()
    m = t.double()[:, idx]
    ksteps = -(-wh // (4 if ww <= 8 else 2))  # of 32 positions; then the smaller parts' sum
    windows_, rows = xw.shape[1], 16 + wh
    want = {"y": unwindows(torch.bmm(xw, m), x.shape, wh, ww),
            "dx": unwindows(torch.bmm(gw, m.transpose(1, 2).contiguous()), x.shape, wh, ww),
            "dt": torch.zeros(t.shape, dtype=torch.float64, device="cuda").index_add_(
                1, idx.flatten(), torch.bmm(xw.transpose(1, 2).contiguous(), gw).flatten(1))}
    got = {"y": W.wbmm_rect_forward(x, t, wh, ww), "dx": W.wbmm_rect_backward_input(dy, t, wh, ww),
           "dt": W.wbmm_rect_backward_table(x, dy, wh, ww)}
    got["y matrix"] = W.wbmm_dense_forward(x, W.wbmm_build_matrix(t, wh, ww), wh, ww)
    if wh == ww and B * C * H * Wd >= 2 ** 21:
        got["dt square"] = W.wbmm_backward_table(x, dy, wh)
    for k, v in got.items():
        w = want[k.split()[0]]
        err = float((v.double() - w).norm() / w.norm())
        bound = rounding(-(-windows_ // 32) + rows if k[:2] == "dt" else ksteps + 2)
        print(shape, k, "%.1e of %.1e" % (err, bound), flush=True)
        assert err <= bound, k


# the direct kernels (many channels; rows of eight: always), the staged kernel,
# the matrix form and the table gradient
@pytest.mark.parametrize("shape", [(3, 2, 28, 42, 14, 14), (3, 1024, 28, 42, 14, 14), (7, 3, 21, 30, 7, 7),
                                   (2, 5, 40, 50, 16, 9), (9, 4, 70, 65, 11, 8)], ids=lambda s: "B%dC%dH%dW%dw%dx%d" % s)
def test_float32_tiny_beside_ordinary(shape):
    """A value far below the others of its row or table keeps float32's
    precision where it decides an output alone: coefficients that are zero for
    every other position of its row, inputs that are zero wherever the other
    coefficients apply."""
    B, C, H, Wd, wh, ww = shape
    x, t = (v.cuda() for v in data(B, C, H, Wd, wh, ww, "f32", seed=3))
    k = (2 * wh - 1) * (2 * ww - 1)
    mid = k // 2
    x = x + torch.where(x < 0, -0.5, 0.5)  # (no result becomes denormal)
    eps = 2.0 ** -21  # one product: three roundings and what the parts leave out, 2^-24 each
    for e in (-100, -110, -118):
        # every second column tiny, the table's centre alone: y = x T_0
        xs = x.clone()
        xs[..., ::2] *= 2.0 ** e
        only = torch.zeros_like(t)
        only[:, mid] = 1.0 + t[:, mid]
        want = xs.double() * only[:, mid].double()[None, :, None, None]
        m = W.wbmm_build_matrix(only, wh, ww)
        for name, y in (("forward", W.wbmm_rect_forward(xs, only, wh, ww)),
                        ("input gradient", W.wbmm_rect_backward_input(xs, only, wh, ww)),
                        ("matrix", W.wbmm_dense_forward(xs, m, wh, ww)),
                        ("matrix^T", W.wbmm_dense_backward_input(xs, m, wh, ww))):
            worst = float(((y.double() - want).abs() / want.abs()).max())
            print(shape, e, name, "%.1e" % worst, flush=True)
            assert worst <= eps, name
        # a tiny centre beside ordinary entries, inputs in one position a window
        ts = t.clone()
        ts[:, mid] = (1.0 + t[:, mid]) * 2.0 ** e
        xo = torch.zeros_like(x)
        xo[:, :, ::wh, ::ww] = x[:, :, ::wh, ::ww]
        want = xo[:, :, ::wh, ::ww].double() * ts[:, mid].double()[None, :, None, None]
        m = W.wbmm_build_matrix(ts, wh, ww)
        for name, y in (("table", W.wbmm_rect_forward(xo, ts, wh, ww)),
                        ("table reversed", W.wbmm_rect_backward_input(xo, ts, wh, ww)),
                        ("table's matrix", W.wbmm_dense_forward(xo, m, wh, ww)),
                        ("table's matrix^T", W.wbmm_dense_backward_input(xo, m, wh, ww))):
            y = y[:, :, ::wh, ::ww].double()
            worst = float(((y - want).abs() / want.abs()).max())
            print(shape, e, name, "%.1e" % worst, flush=True)
            assert worst <= eps, name
        # small inputs and a small centre: their product is still a float32
        if e == -110:
            ts[:, mid] = (1.0 + t[:, mid]) * 2.0 ** -62
            y = W.wbmm_rect_forward(xo * 2.0 ** -62, ts, wh, ww)[:, :, ::wh, ::ww].double()
            want = (xo * 2.0 ** -62)[:, :, ::wh, ::ww].double() * ts[:, mid].double()[None, :, None, None]
            worst = float(((y - want).abs() / want.abs()).max())
            print(shape, "both small %.1e" % worst, flush=True)
            assert worst <= eps, "both small"
        # dT of a tiny column and one dY beside it: the centre is one product
        # (the other columns of x are ordinary and meet zeros there)
        xg, dy = torch.zeros_like(x), torch.zeros_like(x)
        xg[0, :, 0] = x[0, :, 0]
        xg[0, :, 0, 0] *= 2.0 ** e
        dy[0, :, 0, 0] = x[0, :, 1, 1]
        want = xg[0, :, 0, 0].double() * dy[0, :, 0, 0].double()
        dt = W.wbmm_rect_backward_table(xg, dy, wh, ww)[:, mid].double()
        assert float(((dt - want).abs() / want.abs()).max()) <= eps, "table gradient"
        dt = W.wbmm_rect_backward_table(dy, xg, wh, ww)[:, mid].double()
        assert float(((dt - want).abs() / want.abs()).max()) <= eps, "table gradient, dY"


@pytest.mark.parametrize("odd", ["x", "dy", "dx"])
@pytest.mark.parametrize("shape", [(32, 96, 56, 56, 14), (16, 192, 28, 28, 14), (64, 96, 32, 32, 8)],
                         ids=lambda s: "B%dC%dH%dW%dw%d" % s)
def test_gradients_at_odd_addresses(shape, odd):
    """16-bit tensors at addresses that are no multiple of four, on maps with
    fixed-offset rows: one call for both gradients equals the separate ones."""
    B, C, H, Wd, w = shape
    x, t = (v.cuda() for v in data(B, C, H, Wd, w, w, "bf16", seed=1))
    dy, _ = (v.cuda() for v in data(B, C, H, Wd, w, w, "bf16", seed=2))
    base = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
    moved = base[1:].view(x.shape)
    dx = None
    if odd == "dx":
        dx = moved
    else:
        x, dy = (moved.copy_(x), dy) if odd == "x" else (x, moved.copy_(dy))
    dx, dt = W.wbmm_backward(x, dy, t, w, dx=dx)
    assert torch.equal(dt, W.wbmm_backward_table(x, dy, w))
    assert torch.equal(dx, W.wbmm_backward_input(dy, t, w))

# channels and windows on either side of the lines between the row kernel and
# the general ones, on cut maps and on maps as wide as a window
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(4, 256, 8, 14, 14), (4, 257, 8, 14, 14), (5, 257, 8, 14, 14), (1, 700, 20, 30, 15),
                                   (8, 512, 5, 9, 9), (8, 513, 5, 9, 9), (9, 513, 5, 9, 9), (16, 1030, 5, 3, 7),
                                   (17, 1030, 5, 3, 7), (33, 600, 7, 8, 13), (33, 683, 7, 8, 13), (15, 114, 79, 14, 14),
                                   (10, 200, 44, 11, 11), (60, 300, 9, 9, 9), (16, 200, 63, 8, 8)],
                         ids=lambda s: "B%dC%dH%dW%dw%d" % s)
def test_channel_counts_change_no_bit(shape, dtype):
    B, C, H, Wd, w = shape
    x, t = (v.cuda() for v in data(B, C, H, Wd, w, w, dtype, seed=w))
    for f in (W.wbmm_forward, W.wbmm_backward_input):
        y = f(x, t, w)
        for lo in (0, C - 20):
            part = slice(lo, lo + 20)
            assert torch.equal(y[:, part], f(x[:, part].contiguous(), t[part].contiguous(), w))


# on either side of the lines between the general gradient kernel and the
# four-wave ones, on tiled maps without fixed-offset rows
@pytest.mark.parametrize("shape", [(36, 108, 30, 60, 10), (78, 17, 100, 60, 10), (12, 612, 18, 36, 9), (20, 257, 33, 33, 11),
                                   (20, 256, 33, 33, 11), (8, 600, 30, 30, 15), (9, 600, 30, 30, 15), (14, 260, 28, 42, 14),
                                   (10, 420, 28, 42, 14)], ids=lambda s: "B%dC%dH%dW%dw%d" % s)
def test_gradients_on_tiled_maps(shape):
    test_general_gradients(shape, "bf16")


@pytest.mark.parametrize("kind", ["forward", "forward w7", "backward", "matrix", "rectangular gradient"])
def test_time_of_values_out_of_range(kind):
    """Values that take float32 products cost what those cost (the bf16 rate
    is 16 times theirs and each product takes six bf16 ones, so 2.7 times where
    the matrix cores are the bound), not much more: at most five times."""
    B, C, H, Wd, wh, ww = {"forward": (32, 256, 56, 56, 14, 14), "forward w7": (128, 192, 56, 56, 7, 7),
                           "backward": (128, 192, 28, 28, 14, 14), "matrix": (64, 192, 28, 28, 14, 14),
                           "rectangular gradient": (64, 192, 56, 56, 7, 14)}[kind]
    x, t = (v.cuda() for v in data(B, C, H, Wd, wh, ww, "f32", seed=1))
    m = W.wbmm_build_matrix(t, wh, ww) if kind == "matrix" else None

    def once(x):
        if kind == "backward":
            return W.wbmm_backward(x, x.flip(0), t, wh)
        if kind == "matrix":
            return W.wbmm_dense_forward(x, m, wh, ww)
        if kind == "rectangular gradient":
            return W.wbmm_rect_backward_table(x, x, wh, ww)
        return W.wbmm_forward(x, t, wh)

    def time(x):
        once(x)
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            once(x)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    plain, far = time(x), time(x * 2.0 ** -100)
    print(kind, "%.0f us, out of range %.0f us" % (1e3 * plain, 1e3 * far), flush=True)
    assert far <= 5 * plain
