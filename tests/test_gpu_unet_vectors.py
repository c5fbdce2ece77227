"""Pooling and head kernels by vectors of eight channels, at the sizes where their
thread blocks and chunks end, beside the element-wise forms of the same calls:
pooling is exact; head sums are FP32 (1e-5 of the sum of |terms|, at most 2^13
terms in eight or more partial sums, with the fast exponential's 1e-6)."""
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


def _host(S, t):
    return S.bf16_to_float(t.cpu().numpy().view(np.uint16)).astype(np.float64)


@pytest.mark.parametrize("n,h,w,c,cs,co", [
    (1, 2, 2, 8, 8, 0), (2, 6, 2, 24, 40, 16), (3, 4, 34, 16, 24, 8), (2, 32, 64, 64, 64, 0),
    (2, 6, 10, 12, 12, 0), (2, 6, 10, 8, 12, 4),  # element-wise
])
def test_maxpool(S, n, h, w, c, cs, co):
    import torch
    r = np.random.default_rng(h * w + c)
    x = _round(S, r.normal(size=(n, h, w, cs)))
    x[0, 0, 0] = x[0, 0, 1]          # a tie
    x[-1, :2, :2] = -np.inf          # no maximum: zero forward, the first pixel backward
    dy, base = _round(S, r.normal(size=(n, h // 2, w // 2, c))), _round(S, r.normal(size=(n, h, w, cs)))
    xs = x[..., co:co + c]
    xd, dyd = _dev(S, x), _dev(S, dy)
    y = torch.zeros((n, h // 2, w // 2, c), dtype=torch.int16, device="cuda")
    dx0, dx1 = _dev(S, base), _dev(S, base)
    S.call("unet_maxpool_fwd", S.ptr(xd), n, h, w, c, cs, co, S.ptr(y), c, 0, None)
    for dx, acc in ((dx0, 0), (dx1, 1)):
        S.call("unet_maxpool_bwd", S.ptr(xd), n, h, w, c, cs, co, S.ptr(dyd), c, 0, S.ptr(dx), cs, co, acc, None)
    torch.cuda.synchronize()
    ref = U.maxpool2(xs)
    assert np.array_equal(_host(S, y), np.where(np.isinf(ref), 0.0, ref))
    route = U.maxpool2_grad(xs, dy)
    want0, want1 = base.copy(), base.copy()
    want0[..., co:co + c] = route
    want1[..., co:co + c] = _round(S, base[..., co:co + c] + route)
    assert np.array_equal(_host(S, dx0), want0)
    assert np.array_equal(_host(S, dx1), want1)


@pytest.mark.parametrize("n_pix,c,cs", [(1, 8, 8), (255, 16, 24), (257, 64, 64), (4097, 32, 32), (8192, 8, 8), (700, 128, 128)])
def test_head_loss(S, n_pix, c, cs):
    import torch
    r = np.random.default_rng(n_pix + c)
    x = _round(S, np.abs(r.normal(size=(n_pix, cs))))
    xs = x[:, :c]
    w = r.normal(0, 0.3, size=c).astype(np.float32)
    b = np.array([0.1], np.float32)
    t = r.uniform(size=n_pix).astype(np.float32)
    mask = (r.uniform(size=n_pix) > 0.3).astype(np.uint8)
    mask[0] = 1
    scale = np.float32(1.0 / mask.sum())

    def f32(*s):
        return torch.zeros(s, dtype=torch.float32, device="cuda")

    dx = torch.zeros((n_pix, c), dtype=torch.int16, device="cuda")
    loss, dw, db, part = f32(1), f32(c), f32(1), f32(S.lib().unet_head_scratch_floats(n_pix, c))
    xd, wd, bd, td, md = _dev(S, x), *(torch.from_numpy(a).cuda() for a in (w, b, t, mask))
    S.call("unet_head_loss_bwd", S.ptr(xd), n_pix, c, cs, S.ptr(wd), S.ptr(bd), S.ptr(td), S.ptr(md), float(scale),
           S.ptr(loss), S.ptr(dx), S.ptr(dw), S.ptr(db), S.ptr(part), None)
    torch.cuda.synchronize()
    z = xs @ w.astype(np.float64) + float(b[0])
    g = np.where(mask, U.sigmoid(z) - t, 0.0) * float(scale)
    terms = np.where(mask, np.logaddexp(0, z) + np.abs(t * z), 0.0) * float(scale)
    lz = np.where(mask, np.logaddexp(0, z) - t * z, 0.0) * float(scale)
    # the logit's own rounding: 1e-6 of the sum of its |terms|
    ez = 1e-6 * (np.abs(xs) @ np.abs(w.astype(np.float64)) + 1.0) * float(scale)
    assert abs(loss.item() - lz.sum()) <= 1e-5 * terms.sum() + 2 * ez.sum()
    assert abs(db.item() - g.sum()) <= 1e-5 * np.abs(g).sum() + ez.sum()
    assert np.all(np.abs(dw.cpu().numpy() - g @ xs) <= 1e-5 * (np.abs(g) @ xs) + ez @ xs)
    ref = g[:, None] * w[None, :].astype(np.float64)
    assert np.all(np.abs(_host(S, dx) - ref) <= 2.0 ** -8 * np.abs(ref) + 1.01 * ez[:, None] * np.abs(w)[None, :])
