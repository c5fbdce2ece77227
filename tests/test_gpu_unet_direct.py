"""Convolutions at the sizes where their kernels' tiles, slices and fallbacks
meet: remainders of 32- and 64-pixel tiles, of 32- and 64-channel tiles and of
the four-wave blocks, one-row and one-column images, channel slices on both
sides, more tiles than blocks, and outputs that take the general kernel (channels
or offsets that are not whole vectors of eight).
Bound: BF16 products are exact and summed in FP32 (1e-5 of the sum of |terms|,
fewer than 2^12 terms), then rounded to BF16 once (2^-8 of the value)."""
import numpy as np
import pytest

import oracle.unet_oracle as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_08666_amd import surrogate
    surrogate.lib()
    return surrogate


def _round(S, a):
    return S.bf16_to_float(S.bf16_bits(a)).astype(np.float64)


def _dev(S, a):
    import torch
    return torch.from_numpy(S.bf16_bits(a).view(np.int16)).cuda()


def _filled(*shape):
    import torch
    return torch.full(shape, 0x4321, dtype=torch.int16, device="cuda")


def _check(S, y, co, cout, ref, terms):
    import torch
    torch.cuda.synchronize()
    raw = y.cpu().numpy()
    outside = np.ones(raw.shape[-1], bool)
    outside[co:co + cout] = False
    assert np.all(raw[..., outside] == 0x4321)  # the channels beside the slice
    got = S.bf16_to_float(raw[..., co:co + cout].view(np.uint16)).astype(np.float64)
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * terms)


@pytest.mark.parametrize("n,h,w,cin,cout,xc,xo,yc,yo", [
    # tap outermost (any width)
    (1, 1, 1, 16, 8, 16, 0, 8, 0), (1, 1, 33, 16, 40, 16, 0, 40, 0), (1, 33, 1, 32, 72, 40, 8, 88, 16),
    (3, 7, 11, 48, 64, 48, 0, 64, 0), (2, 3, 300, 16, 24, 24, 8, 24, 0),
    (1, 257, 259, 16, 40, 16, 0, 40, 0),   # 64 x 32 tiles, four waves a block
    (1, 257, 259, 16, 72, 16, 0, 72, 0),   # 64 x 64 tiles
    (1, 181, 183, 16, 24, 16, 0, 24, 0), (1, 61, 67, 32, 104, 32, 0, 104, 0),
    # 16-channel groups outermost (whole rows per 256 or 512 pixels)
    (1, 16, 16, 16, 8, 16, 0, 8, 0), (1, 16, 16, 48, 96, 56, 8, 104, 8), (1, 8, 32, 64, 40, 64, 0, 40, 0),
    (3, 4, 128, 32, 24, 32, 0, 32, 8), (2, 256, 128, 16, 24, 16, 0, 24, 0),
    (2, 32, 32, 48, 256, 48, 0, 256, 0), (3, 32, 32, 64, 248, 64, 0, 248, 0),
    # the same through LDS, in tiles of 512 pixels: last tiles that are not whole, one and an odd
    # number of groups, more tiles than blocks, 64-channel tiles with 32 or fewer in the last
    (33, 24, 32, 48, 8, 48, 0, 8, 0), (8, 12, 64, 64, 104, 72, 8, 120, 8), (33, 2, 128, 48, 40, 48, 0, 40, 0),
    (17, 63, 256, 16, 24, 24, 8, 32, 8), (4, 65, 256, 32, 72, 32, 0, 72, 0), (9, 65, 256, 48, 40, 48, 0, 40, 0),
    # sixteen columns, staged 256 pixels at a time
    (70, 16, 16, 16, 40, 16, 0, 40, 0),
    # input layer
    (1, 1, 1, 8, 8, 8, 0, 8, 0), (2, 9, 13, 8, 40, 24, 8, 48, 8), (1, 257, 259, 8, 72, 8, 0, 72, 0),
    # general kernel: partial groups, outputs that are not whole vectors
    (2, 9, 13, 24, 40, 24, 0, 40, 0), (2, 9, 13, 32, 12, 32, 0, 12, 0), (2, 9, 13, 32, 16, 32, 0, 20, 4),
    (1, 16, 16, 16, 12, 16, 0, 12, 0), (2, 9, 13, 8, 12, 8, 0, 12, 0),
])
def test_conv3x3(S, n, h, w, cin, cout, xc, xo, yc, yo):
    import torch
    r = np.random.default_rng(1000 * h + w + cin)
    x = _round(S, r.normal(size=(n, h, w, xc)))
    wt = _round(S, r.normal(0, 0.2, size=(cout, 3, 3, cin)))
    b = r.normal(0, 0.1, size=cout).astype(np.float32)
    xs = x[..., xo:xo + cin]
    ref = U.conv3x3(xs, wt, b.astype(np.float64))
    terms = U.conv3x3(np.abs(xs), np.abs(wt), np.abs(b).astype(np.float64))
    xd, wd, bd = _dev(S, x), _dev(S, wt), torch.from_numpy(b).cuda()
    for relu in (0, 1):
        y = _filled(n, h, w, yc)
        S.call("unet_conv3x3_fwd", S.ptr(xd), n, h, w, cin, xc, xo, S.ptr(wd), S.ptr(bd), cout, S.ptr(y), yc, yo, relu,
               None)
        _check(S, y, yo, cout, np.maximum(ref, 0) if relu else ref, terms)


@pytest.mark.parametrize("n,h,w,cin,cout,yc,yo", [
    (1, 1, 1, 16, 16, 16, 0), (1, 1, 35, 32, 48, 64, 16), (3, 7, 5, 64, 32, 64, 32), (1, 129, 257, 16, 32, 32, 0),
    (1, 129, 257, 80, 16, 16, 0), (1, 129, 257, 144, 32, 40, 8),
    (2, 5, 7, 24, 24, 24, 0),  # general kernel, both ways
    (2, 5, 7, 16, 16, 20, 4),  # general kernel forward
])
def test_upconv(S, n, h, w, cin, cout, yc, yo):
    """Forward into a slice and the data gradient back out of it."""
    import torch
    r = np.random.default_rng(h + w)
    x = _round(S, r.normal(size=(n, h, w, cin)))
    wt = _round(S, r.normal(0, 0.2, size=(cout, 2, 2, cin)))
    b = r.normal(0, 0.1, size=cout).astype(np.float32)
    xd, wd, bd = _dev(S, x), _dev(S, wt), torch.from_numpy(b).cuda()
    y = _filled(n, 2 * h, 2 * w, yc)
    S.call("unet_upconv_fwd", S.ptr(xd), n, h, w, cin, cin, 0, S.ptr(wd), S.ptr(bd), cout, S.ptr(y), yc, yo, None)
    b64 = b.astype(np.float64)
    _check(S, y, yo, cout, U.upconv2(x, wt, b64), U.upconv2(np.abs(x), np.abs(wt), np.abs(b64)))

    if yo % 8:  # gradients are read as vectors
        return
    dy = _round(S, r.normal(size=(n, 2 * h, 2 * w, yc)))
    sl = dy[..., yo:yo + cout]
    for dc, do in ((cin, 0), (cin + 12, 4)):  # vector and general stores
        dx, scratch, dyd = _filled(n, h, w, dc), _filled(4 * cin * cout), _dev(S, dy)
        S.call("unet_upconv_bwd_data", S.ptr(dyd), n, h, w, cout, yc, yo, S.ptr(wd), cin, S.ptr(scratch), S.ptr(dx), dc, do,
               None)
        ref, _, _ = U.upconv2_grad(x, wt, sl)
        terms, _, _ = U.upconv2_grad(np.abs(x), np.abs(wt), np.abs(sl))
        _check(S, dx, do, cin, ref, terms)
