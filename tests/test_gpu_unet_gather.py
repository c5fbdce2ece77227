"""Weight gradients on the grids that take the gathering kernel, and on the other side
of each of its limits: one to four columns, 128 and 256 pixels, many blocks of a
transposed convolution.  Every partial sum starts as NaN.  Bound as for every FP32
gradient: 1e-5 of the sum of |terms|."""
import numpy as np
import pytest

import oracle.unet_oracle as U
from test_gpu_unet_wgrad import S, _conv_wgrad, _dev, _round, _zeros  # noqa: F401

pytestmark = pytest.mark.gpu

NARROW = [(1, 1, 1, 8, 8), (2, 700, 1, 8, 40), (3, 300, 2, 24, 16), (1, 4111, 3, 8, 40), (1, 4111, 3, 8, 32),
          (2, 100, 4, 40, 72), (5, 210, 4, 16, 8), (1, 300, 5, 8, 8)]
FEW = [(1, 8, 16, 40, 24), (1, 16, 16, 8, 40), (1, 8, 17, 8, 40), (2, 11, 12, 16, 32), (4, 8, 8, 32, 8), (1, 257, 6, 8, 40)]


@pytest.mark.parametrize("n,h,w,cin,cout", NARROW + FEW)
def test_conv_weight_gradient(S, n, h, w, cin, cout):  # noqa: F811
    r = np.random.default_rng(h + cin)
    x, dy = _round(S, r.normal(size=(n, h, w, cin))), _round(S, r.normal(size=(n, h, w, cout)))
    dw, db = _conv_wgrad(S, x, dy)
    wt = np.zeros((cout, 3, 3, cin))
    _, rdw, rdb = U.conv3x3_grad(x, wt, dy)
    _, tdw, tdb = U.conv3x3_grad(np.abs(x), wt, np.abs(dy))
    assert np.all(np.abs(dw - rdw) <= 1e-5 * tdw)
    assert np.all(np.abs(db - rdb) <= 1e-5 * tdb)


@pytest.mark.parametrize("n,h,w,cin,cout", NARROW + FEW + [
    (3, 33, 96, 512, 512), (1, 43, 96, 512, 512),  # three and two shares, three quarters of a stage
    (1, 300, 6, 256, 512), (1, 900, 12, 512, 512), (1, 9, 33, 1024, 1024), (2, 40, 60, 64, 512)])
def test_upconv_weight_gradient(S, n, h, w, cin, cout):  # noqa: F811
    import torch
    r = np.random.default_rng(h + cin)
    x, dy = _round(S, r.normal(size=(n, h, w, cin))), _round(S, r.normal(size=(n, 2 * h, 2 * w, cout)))
    part = _zeros(S.lib().unet_wgrad_scratch_floats(n, h, w, cin, cout, 4))
    part.fill_(float("nan"))
    dw, db = _zeros(cout, 2, 2, cin), _zeros(cout)
    xd, dyd = _dev(S, x), _dev(S, dy)
    S.call("unet_upconv_wgrad", S.ptr(xd), n, h, w, cin, cin, 0, S.ptr(dyd), cout, cout, 0, S.ptr(dw), S.ptr(db),
           S.ptr(part), None)
    torch.cuda.synchronize()
    # the oracle on some of the output channels where there are many
    k = np.arange(cout) if cout <= 128 else np.array([0, 31, 32, cout - 1])
    dy, wt = dy[..., k], np.zeros((len(k), 2, 2, cin))
    _, rdw, rdb = U.upconv2_grad(x, wt, dy)
    _, tdw, tdb = U.upconv2_grad(np.abs(x), wt, np.abs(dy))
    assert np.all(np.abs(dw.cpu().numpy()[k] - rdw) <= 1e-5 * tdw)
    assert np.all(np.abs(db.cpu().numpy()[k] - rdb) <= 1e-5 * tdb)


def test_infinite_input_in_a_narrow_image(S):  # noqa: F811
    """As beside the padding of wider ones: only the taps that reach it from a pixel."""
    n, h, w, c = 2, 90, 2, 8
    r = np.random.default_rng(2)
    dy, x = _round(S, r.normal(size=(n, h, w, c))), _round(S, r.normal(size=(n, h, w, c)))
    x[1, 3, 0, 2] = np.inf
    dw, db = _conv_wgrad(S, x, dy)
    want = np.ones((c, 3, 3, c), bool)
    want[:, :, :2, 2] = False
    assert np.array_equal(np.isfinite(dw), want) and np.all(np.isfinite(db))
