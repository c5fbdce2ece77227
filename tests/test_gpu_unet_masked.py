"""Data gradients masked by the activation they go to, with finite gradients and
weights: bit for bit the plain call followed by unet_relu_bwd on every kernel that
writes them, among them both tiles of the staged convolution with a mask, which a
training step of large images runs; and that most of what is compared is a number."""
import numpy as np
import pytest

from test_gpu_unet_direct import S  # noqa: F401

pytestmark = pytest.mark.gpu


def _gradient(S, r, *shape):  # noqa: F811
    import torch
    return torch.from_numpy(S.bf16_bits(r.normal(size=shape)).view(np.int16)).cuda()


def _activation(S, r, *shape):  # noqa: F811
    """Positive and negative values, zeros of both signs, infinities and NaN."""
    import torch
    v = r.normal(size=shape)
    v.flat[::7], v.flat[1::29] = 0.0, -0.0
    v.flat[3::31], v.flat[5::37], v.flat[6::41] = np.inf, -np.inf, np.nan
    return torch.from_numpy(S.bf16_bits(v).view(np.int16)).cuda()


def _same(plain, masked, act):
    """Equal bits, and where act > 0 finite and nearly all non-zero."""
    import torch
    torch.cuda.synchronize()
    assert torch.equal(plain, masked)
    kept = masked[act.view(torch.bfloat16) > 0].view(torch.bfloat16)
    assert kept.numel() > 0.3 * act.numel() and bool(torch.isfinite(kept).all())
    assert int((kept != 0).sum()) > 0.95 * kept.numel()
    assert not bool(masked[~(act.view(torch.bfloat16) > 0)].any())


@pytest.mark.parametrize("n,h,w,cout,cin,cs,co", [
    (1, 9, 13, 16, 40, 40, 0), (2, 16, 16, 32, 24, 40, 8), (1, 9, 13, 8, 40, 40, 0),   # direct: three orders
    (1, 64, 64, 64, 64, 64, 0),
    (33, 24, 32, 48, 8, 16, 8), (20, 20, 256, 16, 32, 32, 0),                          # staged, 32 channels a tile
    (8, 128, 128, 16, 64, 72, 8), (9, 65, 256, 48, 40, 48, 8),                         # 64 channels a tile
    (70, 16, 16, 16, 40, 40, 0),                                                       # sixteen columns
    (2, 9, 13, 24, 40, 40, 0), (2, 9, 13, 32, 12, 12, 0), (1, 9, 13, 16, 16, 20, 4),   # general
])
def test_conv3x3(S, n, h, w, cout, cin, cs, co):  # noqa: F811
    r = np.random.default_rng(h + w + cin)
    dy, wt, act = _gradient(S, r, n, h, w, cout), _gradient(S, r, cin, 3, 3, cout), _activation(S, r, n, h, w, cs)
    before = _gradient(S, r, n, h, w, cs)
    a, b = before.clone(), before.clone()
    S.call("unet_conv3x3_fwd", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), None, cin, S.ptr(a), cs, co, 0, None)
    S.call("unet_relu_bwd", S.ptr(act), n * h * w, cin, cs, co, S.ptr(a), cs, co, None)
    S.call("unet_conv3x3_relu_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), cin, S.ptr(b), cs, co, S.ptr(act),
           cs, co, None)
    sl = slice(co, co + cin)
    _same(a[..., sl], b[..., sl], act[..., sl])
    for k in (slice(0, co), slice(co + cin, cs)):  # beside the slice: untouched
        assert bool((b[..., k] == before[..., k]).all())


@pytest.mark.parametrize("n,h,w,cout,cin", [(1, 5, 7, 16, 40), (1, 129, 257, 16, 32), (1, 129, 257, 16, 72),
                                            (2, 5, 7, 24, 16), (2, 5, 7, 16, 12)])
def test_upconv(S, n, h, w, cout, cin):  # noqa: F811
    import torch
    r = np.random.default_rng(h + cin)
    dy, wt, act = _gradient(S, r, n, 2 * h, 2 * w, cout), _gradient(S, r, cout, 2, 2, cin), _activation(S, r, n, h, w, cin)
    a, b, sc = (torch.zeros(s, dtype=torch.int16, device="cuda") for s in ((n, h, w, cin), (n, h, w, cin), 4 * cin * cout))
    S.call("unet_upconv_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), cin, S.ptr(sc), S.ptr(a), cin, 0, None)
    S.call("unet_relu_bwd", S.ptr(act), n * h * w, cin, cin, 0, S.ptr(a), cin, 0, None)
    S.call("unet_upconv_relu_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), cin, S.ptr(sc), S.ptr(b), cin, 0,
           S.ptr(act), cin, 0, None)
    _same(a, b, act)


def test_one_infinite_gradient(S):  # noqa: F811
    """Reaches its nine pixels' kept gradients, and no other."""
    import torch
    n, h, w, c = 8, 128, 128, 64
    r = np.random.default_rng(5)
    dy, wt, act = _gradient(S, r, n, h, w, 16), _gradient(S, r, c, 3, 3, 16), _activation(S, r, n, h, w, c)
    dy.view(torch.bfloat16)[3, 77, 127, 5] = float("inf")
    dx = torch.zeros((n, h, w, c), dtype=torch.int16, device="cuda")
    S.call("unet_conv3x3_relu_bwd_data", S.ptr(dy), n, h, w, 16, 16, 0, S.ptr(wt), c, S.ptr(dx), c, 0, S.ptr(act), c, 0, None)
    torch.cuda.synchronize()
    bad = ~torch.isfinite(dx.view(torch.bfloat16))
    want = torch.zeros_like(bad)
    want[3, 76:79, 126:128] = act.view(torch.bfloat16)[3, 76:79, 126:128] > 0
    assert torch.equal(bad, want)
