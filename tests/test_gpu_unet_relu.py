"""Data gradients whose ReLU backward is done as they are written: bit for bit
the result of the plain call followed by unet_relu_bwd, on every kernel that
writes them (direct, staged in tiles, sixteen columns, general) and on the
shapes where vectors do not fit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_08666_amd import surrogate
    surrogate.lib()
    return surrogate


def _bits(S, r, *shape):
    import torch
    v = r.normal(size=shape)
    v.flat[::7] = 0.0
    v.flat[3::11] = np.inf
    return torch.from_numpy(S.bf16_bits(v).view(np.int16)).cuda()


def _same(a, b):
    import torch
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("n,h,w,cout,cin,cs,co", [
    (1, 9, 13, 16, 40, 40, 0), (2, 16, 16, 32, 24, 40, 8), (1, 9, 13, 8, 40, 40, 0),   # direct
    (33, 24, 32, 48, 8, 16, 8), (8, 12, 64, 64, 104, 104, 0), (9, 65, 256, 48, 40, 48, 8),  # tiles
    (70, 16, 16, 16, 40, 40, 0),                                                       # sixteen columns
    (2, 9, 13, 24, 40, 40, 0), (2, 9, 13, 32, 12, 12, 0), (1, 9, 13, 16, 16, 20, 4),   # general
])
def test_conv3x3(S, n, h, w, cout, cin, cs, co):
    import torch
    r = np.random.default_rng(h + w + cin)
    dy, wt, act = _bits(S, r, n, h, w, cout), _bits(S, r, cin, 3, 3, cout), _bits(S, r, n, h, w, cs)
    a, b = (torch.full((n, h, w, cs), 77, dtype=torch.int16, device="cuda") for _ in range(2))
    S.call("unet_conv3x3_fwd", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), None, cin, S.ptr(a), cs, co, 0, None)
    S.call("unet_relu_bwd", S.ptr(act), n * h * w, cin, cs, co, S.ptr(a), cs, co, None)
    S.call("unet_conv3x3_relu_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), cin, S.ptr(b), cs, co, S.ptr(act),
           cs, co, None)
    _same(a, b)


@pytest.mark.parametrize("n,h,w,cout,cin", [(1, 5, 7, 16, 40), (1, 129, 257, 16, 32), (2, 5, 7, 24, 16), (2, 5, 7, 16, 12)])
def test_upconv(S, n, h, w, cout, cin):
    import torch
    r = np.random.default_rng(h + cin)
    dy, wt, act = _bits(S, r, n, 2 * h, 2 * w, cout), _bits(S, r, cout, 2, 2, cin), _bits(S, r, n, h, w, cin)
    a, b, sc = (torch.zeros(s, dtype=torch.int16, device="cuda") for s in ((n, h, w, cin), (n, h, w, cin), 4 * cin * cout))
    S.call("unet_upconv_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), cin, S.ptr(sc), S.ptr(a), cin, 0, None)
    S.call("unet_relu_bwd", S.ptr(act), n * h * w, cin, cin, 0, S.ptr(a), cin, 0, None)
    S.call("unet_upconv_relu_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt), cin, S.ptr(sc), S.ptr(b), cin, 0,
           S.ptr(act), cin, 0, None)
    _same(a, b)


@pytest.mark.parametrize("c,cs,co", [(16, 24, 8), (12, 12, 0)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_maxpool(S, c, cs, co, accumulate):
    r = np.random.default_rng(c)
    n, h, w = 2, 6, 10
    x, dy, a = _bits(S, r, n, h, w, cs), _bits(S, r, n, h // 2, w // 2, c), _bits(S, r, n, h, w, cs)
    b = a.clone()
    args = (n, h, w, c, cs, co, S.ptr(dy), c, 0)
    S.call("unet_maxpool_bwd", S.ptr(x), *args, S.ptr(a), cs, co, accumulate, None)
    S.call("unet_relu_bwd", S.ptr(x), n * h * w, c, cs, co, S.ptr(a), cs, co, None)
    S.call("unet_maxpool_relu_bwd", S.ptr(x), *args, S.ptr(b), cs, co, accumulate, None)
    _same(a, b)


@pytest.mark.parametrize("c", [8, 64, 128, 4])
def test_head(S, c):
    import torch
    r = np.random.default_rng(c)
    n = 300
    x = torch.from_numpy(S.bf16_bits(r.normal(size=(n, c))).view(np.int16)).cuda()
    w, b, t = (torch.from_numpy(r.normal(size=k).astype(np.float32)).cuda() for k in (c, 1, n))
    m = torch.ones(n, dtype=torch.uint8, device="cuda")
    out = []
    for name in ("unet_head_loss_bwd", "unet_head_loss_relu_bwd"):
        f = [torch.zeros(k, dtype=torch.float32, device="cuda") for k in (1, c, 1, S.lib().unet_head_scratch_floats(n, c))]
        dx = torch.zeros((n, c), dtype=torch.int16, device="cuda")
        S.call(name, S.ptr(x), n, c, c, S.ptr(w), S.ptr(b), S.ptr(t), S.ptr(m), 1.0, S.ptr(f[0]), S.ptr(dx), S.ptr(f[1]),
               S.ptr(f[2]), S.ptr(f[3]), None)
        out.append((dx, f))
    S.call("unet_relu_bwd", S.ptr(x), n, c, c, 0, S.ptr(out[0][0]), c, 0, None)
    _same(out[0][0], out[1][0])
    for k in range(3):
        _same(out[0][1][k], out[1][1][k])
