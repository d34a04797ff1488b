"""A wide grid of few rows is the direct sum: its tiles would hold fewer nodes than
their Chebyshev points are worth.  Its nodes equal those of small windows of it
bit for bit (x0 and h are dyadic, so that the windows' nodes are the same numbers)."""
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


def check(call, nx, ny, h):
    x0, y0 = -0.5 * nx * h, -0.25
    ax, ay = call(S.Grid(x0, y0, h, nx, ny))
    for i in (0, nx // 3, nx // 2 - 31, nx - 65):
        bx, by = call(S.Grid(x0 + i * h, y0, h, 65, ny))
        assert torch.equal(ax[:, i:i + 65], bx) and torch.equal(ay[:, i:i + 65], by), i


@pytest.mark.parametrize("prec,nx,ny,p", [("fp64", 120000, 2, 100), ("fp64", 90000, 8, 60), ("fp32", 120000, 2, 100),
                                          ("fp32", 100000, 4, 100)])
def test_thin_field(lens, prec, nx, ny, p):
    h = 2.0 ** -9
    prm = S.draw_galaxies(np.random.default_rng(p), p, 60.0)
    prm[:, 0] = (1.25, 3.5, 0.05, 0.3, 5.0, 1000.0, 1000.0)
    prm = dev(prm)
    check(lambda g: lens.lens_deflect(prm, g, prec), nx, ny, h)


@pytest.mark.parametrize("nx,ny,p", [(120000, 2, 100), (90000, 6, 60)])
def test_thin_nfw_field(lens, nx, ny, p):
    h = dev(S.nfw_cluster(S.Grid(-50.0, -50.0, 0.1, 1001, 1001), n_galaxies=p - 2, seed=3))
    check(lambda g: lens.lens_deflect_nfw(h, g, "fp64"), nx, ny, 2.0 ** -9)
