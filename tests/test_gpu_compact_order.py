"""The compacted D3Q19 collision walks its nodes backwards where the population
buffers are large (608 MB here, against 34 MB): the dense split step's node
arithmetic, bit for bit."""
import numpy as np
import pytest

from paper_2111_08666_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [48, 126])
def test_compact_equals_split(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_08666_amd import lbm
    lbm.lib()
    m = np.zeros((n, n, n), np.uint8)
    m[10:14, 8:20, 5:17] = 1
    r0 = I.tanh_droplet(m.shape, (n / 2, n / 2, n / 2), n / 4, (1.0, 0.027), (0.027, 1.0), mask=m)
    p = I.Problem(q=19, mask=m, rho0=r0, periodic=7, open_x=0, tau=I.TAU_M10, G=3.5, xi=-0.3, collision=2)
    a, b = lbm.Solver(p, strategy=lbm.SPLIT), lbm.Solver(p, strategy=lbm.COMPACT)
    a.step(5)
    b.step(5)
    np.testing.assert_array_equal(a.density(), b.density())
    a.step(6)
    b.step_graph(2, 3)
    np.testing.assert_array_equal(a.density(), b.density())
