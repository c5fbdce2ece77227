"""The staged 3x3 convolution in blocks of 512 pixels by 32 channels, and of 256 by
64 beside the limits: fewer than 256 blocks, more than 32 output channels, images
that are not whole blocks of 512.  Bound as for every convolution: BF16 products
summed in FP32 (1e-5 of the sum of |terms|), rounded once (2^-8)."""
import numpy as np
import pytest

import oracle.unet_oracle as U
from test_gpu_unet_direct import S, _check, _dev, _filled, _round  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,cin,cout,yc,yo", [
    (256, 32, 16, 16, 24, 24, 0), (257, 32, 16, 32, 32, 40, 8),   # sixteen columns: 512 pixels
    (255, 32, 16, 16, 24, 24, 0), (512, 16, 16, 16, 8, 8, 0),     # too few blocks; 256 pixels an image
    (2, 256, 256, 16, 12, 12, 0), (4, 256, 128, 48, 20, 23, 3),   # outputs that are not whole vectors
    (2, 256, 256, 16, 36, 36, 0), (1, 256, 256, 16, 12, 12, 0),
])
def test_conv3x3(S, n, h, w, cin, cout, yc, yo):  # noqa: F811
    import torch
    r = np.random.default_rng(n + w + cin + cout)
    x, wt = _round(S, r.normal(size=(n, h, w, cin))), _round(S, r.normal(0, 0.2, size=(cout, 3, 3, cin)))
    b = r.normal(0, 0.1, size=cout).astype(np.float32)
    xd, wd, bd, y = _dev(S, x), _dev(S, wt), torch.from_numpy(b).cuda(), _filled(n, h, w, yc)
    S.call("unet_conv3x3_fwd", S.ptr(xd), n, h, w, cin, cin, 0, S.ptr(wd), S.ptr(bd), cout, S.ptr(y), yc, yo, 0, None)
    # the oracle on one image at a time, the first, the last and one between
    for i in sorted({0, n // 2, n - 1}):
        ref = U.conv3x3(x[i:i + 1], wt, b.astype(np.float64))
        _check(S, y[i:i + 1], yo, cout, ref, U.conv3x3(np.abs(x[i:i + 1]), np.abs(wt), np.abs(b).astype(np.float64)))
