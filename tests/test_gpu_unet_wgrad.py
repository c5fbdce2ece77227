"""Weight gradients with all taps in one wave, at the sizes where their march
over 16-column segments, images and rows can go wrong: one-pixel images, widths
around whole segments, more shares of the work than steps, shares that end
inside an image or a segment, channel counts that do not fill a 32 x 32 tile,
and infinite inputs beside the zero padding.  Bound as for every FP32 gradient: 1e-5 of the sum of
|terms| (FP32 accumulation of exact BF16 products, fewer than 2^15 per sum)."""
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


def _zeros(*s):
    import torch
    return torch.zeros(s, dtype=torch.float32, device="cuda")


def _conv_wgrad(S, x, dy):
    import torch
    n, h, w, cin = x.shape
    cout = dy.shape[3]
    part = _zeros(S.lib().unet_wgrad_scratch_floats(n, h, w, cin, cout, 9))
    part.fill_(float("nan"))  # every partial sum has to be written
    dw, db = _zeros(cout, 3, 3, cin), _zeros(cout)
    xd, dyd = _dev(S, x), _dev(S, dy)
    S.call("unet_conv3x3_wgrad", S.ptr(xd), n, h, w, cin, cin, 0, S.ptr(dyd), cout, cout, 0, S.ptr(dw), S.ptr(db),
           S.ptr(part), 0, None)
    torch.cuda.synchronize()
    return dw.cpu().numpy(), db.cpu().numpy()


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 1, 1, 8, 8), (3, 1, 1, 40, 8), (5, 3, 2, 8, 40), (2, 17, 16, 32, 32), (40, 4, 4, 16, 72),
    (2, 9, 15, 8, 16), (2, 9, 31, 8, 16), (1, 7, 129, 8, 8), (1, 5, 1000, 8, 8), (1, 700, 3, 16, 8),
    (2, 9, 48, 40, 24), (1, 3, 144, 8, 8), (1, 2, 256, 8, 40), (3, 65, 128, 8, 8), (1, 33, 272, 8, 8),
    (8, 33, 32, 64, 96),  # 8448 pixels: three chunks, each ends inside an image
    (32, 32, 32, 8, 32),  # eight chunks
    (2, 260, 256, 8, 16), (3, 211, 212, 8, 40),  # 33 chunks: eight threads to a sum
])
def test_conv_weight_gradient(S, n, h, w, cin, cout):
    r = np.random.default_rng(h * w + cin)
    x, dy = _round(S, r.normal(size=(n, h, w, cin))), _round(S, r.normal(size=(n, h, w, cout)))
    dw, db = _conv_wgrad(S, x, dy)
    wt = np.zeros((cout, 3, 3, cin))
    _, rdw, rdb = U.conv3x3_grad(x, wt, dy)
    _, tdw, _ = U.conv3x3_grad(np.abs(x), wt, np.abs(dy))
    assert np.all(np.abs(dw - rdw) <= 1e-5 * tdw)
    assert np.all(np.abs(db - rdb) <= 1e-5 * np.abs(dy).sum(axis=(0, 1, 2)))


@pytest.mark.parametrize("w", [5, 16, 200])
def test_infinite_input_beside_the_padding(S, w):
    """An infinite pixel in column 0 (row 0) enters only the taps that reach
    it from a pixel of the image: not the tap that would come from column -1
    (row -1)."""
    n, h, c = 2, 6, 8
    r = np.random.default_rng(w)
    dy = _round(S, r.normal(size=(n, h, w, c)))
    x = _round(S, r.normal(size=(n, h, w, c)))
    x[1, 3, 0, 2] = np.inf
    x[1, 0, 2, 5] = -np.inf
    dw, db = _conv_wgrad(S, x, dy)
    want = np.ones((c, 3, 3, c), bool)
    want[:, :, :2, 2] = False   # x[p + (kx - 1)] with p = column 1 or 0
    want[:, :2, :, 5] = False   # x[p + (ky - 1)] with p = row 1 or 0
    assert np.array_equal(np.isfinite(dw), want)
    assert np.all(np.isfinite(db))


@pytest.mark.parametrize("n,h,w,cin,cout", [(1, 1, 1, 8, 8), (3, 5, 7, 40, 24), (9, 31, 33, 32, 64), (2, 3, 16, 8, 40), (5, 33, 32, 32, 64),
                                            (1, 9, 112, 8, 8), (3, 31, 128, 16, 32), (1, 3, 144, 8, 8)])
def test_upconv_weight_gradient(S, n, h, w, cin, cout):
    import torch
    r = np.random.default_rng(h + w)
    x, dy = _round(S, r.normal(size=(n, h, w, cin))), _round(S, r.normal(size=(n, 2 * h, 2 * w, cout)))
    part = _zeros(S.lib().unet_wgrad_scratch_floats(n, h, w, cin, cout, 4))
    part.fill_(float("nan"))
    dw, db = _zeros(cout, 2, 2, cin), _zeros(cout)
    xd, dyd = _dev(S, x), _dev(S, dy)
    S.call("unet_upconv_wgrad", S.ptr(xd), n, h, w, cin, cin, 0, S.ptr(dyd), cout, cout, 0, S.ptr(dw), S.ptr(db),
           S.ptr(part), None)
    torch.cuda.synchronize()
    wt = np.zeros((cout, 2, 2, cin))
    _, rdw, rdb = U.upconv2_grad(x, wt, dy)
    _, tdw, _ = U.upconv2_grad(np.abs(x), wt, np.abs(dy))
    assert np.all(np.abs(dw.cpu().numpy() - rdw) <= 1e-5 * tdw)
    assert np.all(np.abs(db.cpu().numpy() - rdb) <= 1e-5 * np.abs(dy).sum(axis=(0, 1, 2)))
