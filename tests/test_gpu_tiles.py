"""The default tile of the fused D2Q9 step (8 rows, one wave per interior row
where the block has eight) against the 16-row tile with four waves: the same
node arithmetic, so the densities are equal bit for bit, at heights around
the tile's edges and on every storage, node arithmetic and layout."""
import numpy as np
import pytest

from paper_2111_08666_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_08666_amd import lbm as L
    L.lib()
    return L


def _problem(ny, periodic):
    if periodic:
        m = np.zeros((ny, 61), np.uint8)
        m[ny // 2, 20:30] = 1
        return I.Problem(q=9, mask=m, rho0=I.tanh_droplet(m.shape, (30, ny / 2), 3, (1.0, 0.027), (0.027, 1.0), mask=m),
                         periodic=3, open_x=0, tau=I.TAU_M10, G=3.5, xi=-0.3, collision=1)
    return I.drainage_2d(nx=121, ny=ny, r=(2.0, 4.0), porosity=0.75, seed=ny, G=3.5, theta=60, tau=I.TAU_M10,
                         rho_in1=1.01, minor=0.027, collision=1)


@pytest.mark.parametrize("ny,periodic", [(7, True), (8, True), (9, True), (17, True), (15, False), (33, False)])
@pytest.mark.parametrize("compact", [False, True])
@pytest.mark.parametrize("storage,math", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_default_tile_matches_the_four_wave_tile(lbm, ny, periodic, compact, storage, math):
    p = _problem(ny, periodic)
    kw = dict(strategy=lbm.COMPACT_FUSED if compact else lbm.FUSED, storage=storage, math=math)
    a, b = lbm.Solver(p, **kw), lbm.Solver(p, tile_rows=16, **kw)
    eight = not compact or (math == lbm.MATH_F64 and storage == lbm.STORE_F32)
    assert a.kernel_info()[2] == (512 if eight else 256) and b.kernel_info()[2] == 256
    for _ in range(3):
        a.step(7)
        b.step(7)
        np.testing.assert_array_equal(a.density(), b.density())
    a.step_graph(4, 3)  # replays, with the eager work above in between
    b.step(12)
    np.testing.assert_array_equal(a.density(), b.density())


@pytest.mark.parametrize("ny,rows", [(5120, 8), (5121, 12)])
def test_default_tile_of_many_tiles_with_bf16_storage(lbm, ny, rows):
    """1280 tiles of 60 x 8 nodes take 8 rows, more take 12: the same densities."""
    m = np.zeros((ny, 61), np.uint8)
    m[ny // 2, 20:30] = 1
    p = I.Problem(q=9, mask=m, rho0=I.tanh_droplet(m.shape, (30, ny / 2), 9, (1.0, 0.027), (0.027, 1.0), mask=m),
                  periodic=3, open_x=0, tau=I.TAU_M10, G=3.5, xi=-0.3, collision=1)
    kw = dict(strategy=lbm.FUSED, storage=1)
    a, b = lbm.Solver(p, **kw), lbm.Solver(p, tile_rows=16, **kw)
    assert a.kernel_info()[0].endswith(",%d>" % rows)
    a.step(6)
    b.step(6)
    np.testing.assert_array_equal(a.density(), b.density())
