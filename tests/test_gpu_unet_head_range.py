"""The head's loss at the end of its range of pixels (2^31 - 1), where the number of
blocks does not come out of 32 bits: three masked pixels, against the closed form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_head_loss_of_all_pixels():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 80 * 2 ** 30:
        pytest.skip("needs 80 GB")
    from paper_2111_08666_amd import surrogate as S
    n, c = 2 ** 31 - 1, 8
    r = np.random.default_rng(3)
    at = [0, 2 ** 30 + 12345, n - 1]
    x = torch.zeros((n, c), dtype=torch.int16, device="cuda")
    t, m = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")
    xs = S.bf16_to_float(S.bf16_bits(r.normal(size=(3, c)))).astype(np.float64)
    ts = r.uniform(size=3).astype(np.float32)
    for k, p in enumerate(at):
        x[p] = torch.from_numpy(S.bf16_bits(xs[k]).view(np.int16)).cuda()
        t[p], m[p] = float(ts[k]), 1
    w, b = r.normal(size=c).astype(np.float32), r.normal(size=1).astype(np.float32)
    wd, bd = torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda()
    loss, dw, db = (torch.full((k,), float("nan"), device="cuda") for k in (1, c, 1))
    part = torch.empty(S.lib().unet_head_scratch_floats(n, c), dtype=torch.float32, device="cuda")
    S.call("unet_head_loss_bwd", S.ptr(x), n, c, c, S.ptr(wd), S.ptr(bd), S.ptr(t), S.ptr(m), 0.5, S.ptr(loss), None,
           S.ptr(dw), S.ptr(db), S.ptr(part), None)
    torch.cuda.synchronize()
    z = xs @ w.astype(np.float64) + b
    g = 0.5 * (1 / (1 + np.exp(-z)) - ts)
    # FP32 logits and exponentials of magnitude below 10: 1e-5
    assert abs(float(loss) - 0.5 * (np.logaddexp(0, z) - ts * z).sum()) <= 1e-5
    assert abs(float(db) - g.sum()) <= 1e-5
    assert np.all(np.abs(dw.cpu().numpy() - g @ xs) <= 1e-5 * (np.abs(g) @ np.abs(xs)) + 1e-6)
