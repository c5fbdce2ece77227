"""Tensors that start one element past a multiple of 16 bytes: the results of the
same tensors copied to aligned memory, bit for bit."""
import numpy as np
import pytest

from test_gpu_unet_direct import S  # noqa: F401

pytestmark = pytest.mark.gpu


def _bf16(S, r, *shape):  # noqa: F811
    import torch
    return torch.from_numpy(S.bf16_bits(r.normal(size=shape)).view(np.int16)).cuda()


def _shifted(t):
    """A copy of t one element off."""
    import torch
    base = torch.zeros(t.numel() + 8, dtype=t.dtype, device=t.device)
    v = base[1:1 + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == 2
    return v


def _both(tensors, run):
    """run on aligned copies and on shifted ones; it returns what it wrote."""
    import torch
    a, b = run(*[t.clone() for t in tensors]), run(*[_shifted(t) for t in tensors])
    torch.cuda.synchronize()
    for u, v in zip(a, b):
        assert torch.equal(u, v)


def test_relu_bwd(S):  # noqa: F811
    r = np.random.default_rng(1)

    def run(y, dy):
        S.call("unet_relu_bwd", S.ptr(y), 99, 16, 24, 8, S.ptr(dy), 24, 8, None)
        return [dy]
    _both([_bf16(S, r, 99, 24), _bf16(S, r, 99, 24)], run)


@pytest.mark.parametrize("c", [8, 64, 128])
def test_head(S, c):  # noqa: F811
    import torch
    r = np.random.default_rng(c)
    n = 5000
    w, b, t = (torch.from_numpy(r.normal(size=k).astype(np.float32)).cuda() for k in (c, 1, n))
    m = torch.ones(n, dtype=torch.uint8, device="cuda")
    for name in ("unet_head_loss_bwd", "unet_head_loss_relu_bwd"):
        def run(x, dx):
            f = [torch.zeros(k, device="cuda") for k in (1, c, 1, S.lib().unet_head_scratch_floats(n, c), n)]
            S.call(name, S.ptr(x), n, c, c, S.ptr(w), S.ptr(b), S.ptr(t), S.ptr(m), 1.0, S.ptr(f[0]), S.ptr(dx),
                   S.ptr(f[1]), S.ptr(f[2]), S.ptr(f[3]), None)
            S.call("unet_head_fwd", S.ptr(x), n, c, c, S.ptr(w), S.ptr(b), S.ptr(f[4]), None)
            return [dx, f[0], f[1], f[2], f[4]]
        _both([_bf16(S, r, n, c), _bf16(S, r, n, c)], run)


@pytest.mark.parametrize("accumulate", [0, 1])
def test_maxpool(S, accumulate):  # noqa: F811
    r = np.random.default_rng(3)

    def run(x, dy, dx, y):
        S.call("unet_maxpool_fwd", S.ptr(x), 2, 6, 10, 16, 24, 8, S.ptr(y), 16, 0, None)
        S.call("unet_maxpool_relu_bwd", S.ptr(x), 2, 6, 10, 16, 24, 8, S.ptr(dy), 16, 0, S.ptr(dx), 24, 8, accumulate, None)
        return [y, dx]
    _both([_bf16(S, r, 2, 6, 10, 24), _bf16(S, r, 2, 3, 5, 16), _bf16(S, r, 2, 6, 10, 24), _bf16(S, r, 2, 3, 5, 16)], run)


@pytest.mark.parametrize("n,h,w,cin,cout", [(2, 9, 13, 16, 40), (1, 32, 32, 48, 24), (8, 32, 64, 32, 64), (2, 9, 13, 8, 16)])
def test_convolutions(S, n, h, w, cin, cout):  # noqa: F811
    import torch
    r = np.random.default_rng(h + cin)
    part = torch.zeros(S.lib().unet_wgrad_scratch_floats(n, h, w, cin, cout, 9), device="cuda")

    def run(x, dy, act, wt, wt2, y, dx):
        dw, db = torch.zeros((cout, 9, cin), device="cuda"), torch.zeros(cout, device="cuda")
        S.call("unet_conv3x3_fwd", S.ptr(x), n, h, w, cin, cin, 0, S.ptr(wt), None, cout, S.ptr(y), cout, 0, 1, None)
        S.call("unet_conv3x3_flip", S.ptr(wt), cout, cin, S.ptr(wt2), None)
        S.call("unet_conv3x3_relu_bwd_data", S.ptr(dy), n, h, w, cout, cout, 0, S.ptr(wt2), cin, S.ptr(dx), cin, 0,
               S.ptr(act), cin, 0, None)
        S.call("unet_conv3x3_wgrad", S.ptr(x), n, h, w, cin, cin, 0, S.ptr(dy), cout, cout, 0, S.ptr(dw), S.ptr(db),
               S.ptr(part), 0, None)
        return y, dx, dw, db
    ts = [_bf16(S, r, *s) for s in ((n, h, w, cin), (n, h, w, cout), (n, h, w, cin), (cout, 9, cin), (cin, 9, cout),
                                    (n, h, w, cout), (n, h, w, cin))]
    a, b = run(*[t.clone() for t in ts]), run(*[_shifted(t) for t in ts])
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    # another kernel, another order of the weight gradients' sums
    for u, v in zip(a[2:], b[2:]):
        assert (u - v).abs().max() <= 2 ** -14 * u.abs().max()
