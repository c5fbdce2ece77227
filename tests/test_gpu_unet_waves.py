"""The direct convolution kernels with four waves to a block: more than 4096 waves,
not a multiple of four, in every order and tile that can have so many, and the
transposed convolution's data gradient in tiles of 64 pixels by 32 channels.  The
launch's rule is repeated here, so that a moved threshold shows.  Bound as for every
convolution: 1e-5 of the sum of |terms|, rounded once (2^-8)."""
import numpy as np
import pytest

import oracle.unet_oracle as U
from test_gpu_unet_direct import S, _check, _dev, _filled, _round  # noqa: F401

pytestmark = pytest.mark.gpu

H, W = 513, 517  # 265 221 pixels: 4145 tiles of 64


def _four_waves(pix, nout, tn):
    """Waves of 64 pixels by 32 tn channels: four to a block, the last one not full."""
    waves = -(-pix // 64) * -(-nout // (32 * tn))
    return waves > 4096 and waves % 4 != 0


@pytest.mark.parametrize("cin,cout,tn", [(8, 24, 1),     # two taps a step
                                         (16, 24, 1), (16, 40, 2)])  # tap by tap
def test_conv3x3(S, cin, cout, tn):  # noqa: F811
    import torch
    assert _four_waves(H * W, cout, tn)
    r = np.random.default_rng(cin + cout)
    x, wt = _round(S, r.normal(size=(1, H, W, cin))), _round(S, r.normal(0, 0.2, size=(cout, 3, 3, cin)))
    b = r.normal(0, 0.1, size=cout).astype(np.float32)
    xd, wd, bd, y = _dev(S, x), _dev(S, wt), torch.from_numpy(b).cuda(), _filled(1, H, W, cout)
    S.call("unet_conv3x3_fwd", S.ptr(xd), 1, H, W, cin, cin, 0, S.ptr(wd), S.ptr(bd), cout, S.ptr(y), cout, 0, 0, None)
    _check(S, y, 0, cout, U.conv3x3(x, wt, b.astype(np.float64)),
           U.conv3x3(np.abs(x), np.abs(wt), np.abs(b).astype(np.float64)))


def test_upconv(S):  # noqa: F811
    import torch
    cin, cout = 16, 8
    assert _four_waves(H * W, cout, 1)
    r = np.random.default_rng(7)
    x, wt = _round(S, r.normal(size=(1, H, W, cin))), _round(S, r.normal(0, 0.2, size=(cout, 2, 2, cin)))
    b = r.normal(0, 0.1, size=cout).astype(np.float32)
    xd, wd, bd, y = _dev(S, x), _dev(S, wt), torch.from_numpy(b).cuda(), _filled(1, 2 * H, 2 * W, cout)
    S.call("unet_upconv_fwd", S.ptr(xd), 1, H, W, cin, cin, 0, S.ptr(wd), S.ptr(bd), cout, S.ptr(y), cout, 0, None)
    b64 = b.astype(np.float64)
    _check(S, y, 0, cout, U.upconv2(x, wt, b64), U.upconv2(np.abs(x), np.abs(wt), np.abs(b64)))


@pytest.mark.parametrize("h,w,cin,tn", [(H, W, 72, 4), (H, W, 40, 2), (H, W, 24, 1), (257, 259, 24, 1)])
def test_upconv_data_gradient(S, h, w, cin, tn):  # noqa: F811
    cout = 16
    tiles = -(-h * w // 32) * -(-cin // 32)  # of 32 x 32
    assert tiles >= {4: 4096, 2: 1024, 1: 2048}[tn] and (h != H or _four_waves(h * w, cin, tn))
    r = np.random.default_rng(cin + h)
    wt, dy = _round(S, r.normal(0, 0.2, size=(cout, 2, 2, cin))), _round(S, r.normal(size=(1, 2 * h, 2 * w, cout)))
    dx, scratch, dyd, wd = _filled(1, h, w, cin), _filled(4 * cin * cout), _dev(S, dy), _dev(S, wt)
    S.call("unet_upconv_bwd_data", S.ptr(dyd), 1, h, w, cout, cout, 0, S.ptr(wd), cin, S.ptr(scratch), S.ptr(dx), cin, 0,
           None)
    x = np.zeros((1, h, w, cin))
    _check(S, dx, 0, cin, U.upconv2_grad(x, wt, dy)[0], U.upconv2_grad(x, np.abs(wt), np.abs(dy))[0])
