"""Waves and rows of the fused D2Q9 tile on both sides of the tile counts at which
they change: the densities are those of the 16-row tile, bit for bit."""
import numpy as np
import pytest

from paper_2111_08666_amd import inputs as I

pytestmark = pytest.mark.gpu


def _problem(ny, collision):
    """Two tiles of 60 x 8 nodes per eight rows."""
    m = np.zeros((ny, 61), np.uint8)
    m[ny // 2, 20:30] = 1
    return I.Problem(q=9, mask=m, rho0=I.tanh_droplet(m.shape, (30, ny / 2), 9, (1.0, 0.027), (0.027, 1.0), mask=m),
                     periodic=3, open_x=0, tau=I.TAU_M10, G=3.5, xi=-0.3, collision=collision)


@pytest.mark.parametrize("compact,storage,math,collision,ny,tile_rows,rows,threads", [
    (False, 0, 0, 2, 24000, 0, 8, 512), (False, 0, 0, 2, 24001, 0, 8, 256),   # dense FP32: 6000 tiles
    (False, 0, 1, 2, 4096, 0, 8, 512), (False, 0, 1, 0, 4097, 0, 8, 256),     # dense FP64: 1024
    (False, 1, 0, 1, 5120, 8, 8, 512), (False, 1, 0, 1, 5121, 8, 8, 256),     # dense BF16: 1280
    (False, 1, 1, 1, 5121, 8, 8, 512), (False, 1, 1, 2, 5121, 8, 8, 256),     # the same in FP64: MRT keeps eight
    (True, 0, 1, 0, 12000, 0, 8, 512), (True, 0, 1, 0, 12001, 0, 12, 256),    # compacted FP64: 3000
    (True, 0, 1, 2, 12001, 8, 8, 256),
])
def test_waves_by_tile_count(compact, storage, math, collision, ny, tile_rows, rows, threads):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_08666_amd import lbm
    p = _problem(ny, collision)
    kw = dict(strategy=lbm.COMPACT_FUSED if compact else lbm.FUSED, storage=storage, math=math)
    a, b = lbm.Solver(p, tile_rows=tile_rows, **kw), lbm.Solver(p, tile_rows=16, **kw)
    name, _, block = a.kernel_info()
    assert (",%d>" % rows in name or ",%d,compact>" % rows in name) and block == threads
    a.step(5)
    b.step(5)
    np.testing.assert_array_equal(a.density(), b.density())
    a.step_graph(2, 2)
    b.step(4)
    np.testing.assert_array_equal(a.density(), b.density())
