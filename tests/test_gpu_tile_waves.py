"""Waves and rows of the fused D2Q9 tile on both sides of the tile counts at which
they change: the densities are those of the 16-row tile, bit for bit."""
import numpy as np
import pytest

from paper_2111_08666_amd import inputs as I

pytestmark = pytest.mark.gpu


def _problem(nx, ny, collision):
    m = np.zeros((ny, nx), np.uint8)
    m[ny // 2, 20:30] = 1
    return I.Problem(q=9, mask=m, rho0=I.tanh_droplet(m.shape, (30, ny / 2), 9, (1.0, 0.027), (0.027, 1.0), mask=m),
                     periodic=3, open_x=0, tau=I.TAU_M10, G=3.5, xi=-0.3, collision=collision)


# (61 columns: two tiles of 60 x 8 nodes per eight rows; 640: eleven)
@pytest.mark.parametrize("compact,storage,math,collision,nx,ny,tile_rows,rows,threads", [
    (False, 0, 0, 2, 61, 24000, 0, 8, 512), (False, 0, 0, 2, 61, 24001, 0, 8, 256),   # dense FP32: 6000 tiles
    (False, 0, 1, 2, 61, 1600, 0, 8, 512), (False, 0, 1, 0, 61, 1601, 0, 8, 256),     # dense FP64: 400
    (False, 0, 1, 0, 61, 3600, 0, 8, 256), (False, 0, 1, 0, 61, 3601, 0, 12, 256),    # and 900
    (False, 1, 0, 1, 61, 1600, 0, 8, 512), (False, 1, 0, 1, 61, 1601, 0, 8, 256),     # dense BF16: 400
    (False, 1, 0, 2, 640, 500, 0, 8, 256), (False, 1, 0, 2, 640, 501, 0, 12, 256),    # 320 000 nodes
    (False, 1, 1, 2, 640, 501, 0, 12, 256), (False, 1, 1, 1, 640, 501, 0, 8, 512),    # (MRT in FP64: eight waves on)
    (False, 1, 1, 1, 61, 5121, 8, 8, 512), (False, 1, 1, 2, 61, 5121, 8, 8, 256),
    (True, 0, 1, 0, 61, 1600, 0, 8, 512), (True, 0, 1, 0, 61, 1601, 0, 8, 256),       # compacted FP64: 400 tiles
    (True, 0, 1, 2, 61, 3200, 0, 8, 256), (True, 0, 1, 2, 61, 3201, 0, 12, 256),      # and 800
])
def test_waves_by_tile_count(compact, storage, math, collision, nx, ny, tile_rows, rows, threads):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_08666_amd import lbm
    p = _problem(nx, ny, collision)
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
