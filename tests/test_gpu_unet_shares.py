"""Weight gradients over many shares of the pixels: eight, nine and more than
thirty-two of them with one and several channel tiles, so that the ranges of blocks
the XCDs take end inside a share and in a last block that has none.  Every partial
sum starts as NaN.  Bound as for every FP32 gradient: 1e-5 of the sum of |terms|."""
import numpy as np
import pytest

import oracle.unet_oracle as U
from test_gpu_unet_wgrad import S, _conv_wgrad, _dev, _round, _zeros  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(2, 128, 128, 40, 24), (3, 96, 128, 8, 72),   # eight and nine shares, whole rows
          (3, 101, 109, 24, 40), (1, 180, 200, 72, 8),  # nine, rows of no whole 16-pixel segments
          (2, 260, 256, 8, 8), (2, 258, 254, 8, 40)]    # 33, both ways


@pytest.mark.parametrize("n,h,w,cin,cout", SHAPES)
def test_conv_weight_gradient(S, n, h, w, cin, cout):  # noqa: F811
    r = np.random.default_rng(h + cin)
    x, dy = _round(S, r.normal(size=(n, h, w, cin))), _round(S, r.normal(size=(n, h, w, cout)))
    dw, db = _conv_wgrad(S, x, dy)
    wt = np.zeros((cout, 3, 3, cin))
    _, rdw, rdb = U.conv3x3_grad(x, wt, dy)
    _, tdw, tdb = U.conv3x3_grad(np.abs(x), wt, np.abs(dy))
    assert np.all(np.abs(dw - rdw) <= 1e-5 * tdw)
    assert np.all(np.abs(db - rdb) <= 1e-5 * tdb)


@pytest.mark.parametrize("n,h,w,cin,cout", SHAPES)
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
    wt = np.zeros((cout, 2, 2, cin))
    _, rdw, rdb = U.upconv2_grad(x, wt, dy)
    _, tdw, tdb = U.upconv2_grad(np.abs(x), wt, np.abs(dy))
    assert np.all(np.abs(dw.cpu().numpy() - rdw) <= 1e-5 * tdw)
    assert np.all(np.abs(db.cpu().numpy() - rdb) <= 1e-5 * tdb)
