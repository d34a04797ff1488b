"""An FP64 field of few potentials is the direct sum, whatever the grid's size: a
large grid's nodes equal those of small windows of it bit for bit (x0 and h are
dyadic, so that the windows' nodes are the same numbers)."""
import numpy as np
import pytest

import synthlens as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lens():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1902_03252_amd as lens
    lens.context()
    return lens


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("p,nx,ny", [(4, 2300, 2300), (5, 4100, 1025), (8, 1601, 1700), (11, 1300, 1290)])
def test_large_grid_equals_windows(lens, p, nx, ny):
    h = 2.0 ** -4
    grid = S.Grid(-64.0, -48.0, h, nx, ny)
    prm = S.draw_galaxies(np.random.default_rng(p), p, 40.0)
    prm[:, 0] = (10.25, 20.5, 0.05, 0.3, 5.0, 1000.0, 1000.0)
    prm[4, 1], prm[5, 2] = 0.0, np.inf
    ax, ay = lens.lens_deflect(dev(prm), grid, "fp64")
    for i, j in ((0, 0), (nx // 2, ny // 3), (127, 129), (nx - 65, ny - 33)):
        bx, by = lens.lens_deflect(dev(prm), S.Grid(grid.x0 + i * h, grid.y0 + j * h, h, 65, 33), "fp64")
        assert torch.equal(ax[j:j + 33, i:i + 65], bx) and torch.equal(ay[j:j + 33, i:i + 65], by), (i, j)
