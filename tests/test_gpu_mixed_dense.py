"""GPU parity of the mixed-precision SIE gradient where the halos' FP64 blocks overlap
(a dense image, blocks that cover it, halos on one node, blocks clipped by the edges,
more halos than one list of 256) and with more halos than a tile's lists hold: the
bars of test_gpu_mixed, and the counts of the mask."""
import numpy as np
import pytest

import oracle
import synthlens as S
from test_gpu_mixed import check_rows, criterion_margin, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lens():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1902_03252_amd as lens
    lens.context()
    return lens


@pytest.mark.parametrize("nx,ny,p,n_cluster,pc,pg", [
    (100, 64, 702, 2, 30, 20), (130, 97, 300, 3, 40, 9), (70, 65, 40, 2, 400, 400), (300, 211, 60, 0, 50, 60),
    (140, 90, 258, 258, 12, 0), (90, 80, 2049, 2, 16, 3), (60, 50, 2300, 2, 0, 0), (1025, 700, 11, 2, 0, 0),
    (1025, 700, 12, 2, 7, 3)])
def test_overlapping_blocks(lens, nx, ny, p, n_cluster, pc, pg):
    grid = S.paper_grid(nx, ny=ny)
    prm = S.paper_sie_cluster(grid, n_galaxies=p - 2, seed=p)
    prm[:2, p // 2:p // 2 + 3] = prm[:2, 2:3]           # four halos on one node
    prm[0, -1], prm[1, -1] = grid.x0 - 5 * grid.h, grid.y0 + 2 * grid.h  # a block reaching in from outside
    res = lens.lens_deflect_mixed(dev(prm), grid, n_cluster=n_cluster, patch_cluster=pc, patch_galaxy=pg)
    torch.cuda.synchronize()
    ax, ay = oracle.alpha_grid(prm, grid)
    patch = oracle.dp_patches(prm, grid, n_cluster, pc, pg)
    crit = oracle.criteria(ax, ay, grid.h)
    mask = res.mask.cpu().numpy()
    n_dp = check_rows(res.ax.cpu().numpy(), res.ay.cpu().numpy(), mask, ax, ay, patch, crit,
                      criterion_margin(ax, ay, grid.h), f"{nx}x{ny} P={p} {n_cluster} {pc}/{pg}")
    st = res.stats.cpu().numpy()
    assert st[3] == 0 and st[0] == (mask == 1).sum() and st[1] == (mask == 2).sum() and st[2] == n_dp


@pytest.mark.parametrize("nx,ny,p,t12,t34", [(1025, 700, 60, 1e-5, 0.5), (1025, 700, 60, 1e-3, 0.1), (513, 1300, 30, 5e-3, 0.02),
                                             (700, 650, 62, 0.0, 1e9), (1600, 1500, 24, 9.2e-3, 1.04e-2)])
def test_criteria_pixels_few_and_many(lens, nx, ny, p, t12, t34):
    """From no criteria pixels to nearly all: FP64 pixels within 1e-10 arcsec, the others within the FP32 bound, the
    criteria set within rounding of the thresholds."""
    grid = S.paper_grid(nx, ny=ny)
    prm = S.paper_sie_cluster(grid, n_galaxies=p - 2, seed=p)
    res = lens.lens_deflect_mixed(dev(prm), grid, n_cluster=2, patch_cluster=16, patch_galaxy=4, t12=t12, t34=t34)
    torch.cuda.synchronize()
    ax, ay = oracle.alpha_grid(prm, grid)
    patch = oracle.dp_patches(prm, grid, 2, 16, 4).astype(bool)
    want = oracle.criteria(ax, ay, grid.h, t12, t34).astype(bool) & ~patch
    mask = res.mask.cpu().numpy()
    np.testing.assert_array_equal(mask == 1, patch)
    err = np.maximum(np.abs(res.ax.cpu().numpy() - ax), np.abs(res.ay.cpu().numpy() - ay))
    assert err[mask >= 1].max() <= 1e-10
    e32 = err[mask == 0].max() if (mask == 0).any() else 0.0
    assert e32 <= 2.3e-3
    diff = (mask == 2) != want
    print(f"  {nx}x{ny} P={p}: criteria {int((mask == 2).sum())} of {nx * ny}, differ {int(diff.sum())}, FP32 {e32:.2e}",
          flush=True)
    dist = np.full(ax.shape, np.inf)
    for axis in (0, 1):
        s, b = ([slice(1, None), slice(None)], [slice(None, -1), slice(None)]) if axis == 0 else \
            ([slice(None), slice(1, None)], [slice(None), slice(None, -1)])
        s, b = tuple(s), tuple(b)
        d, o = (ay[s] - ay[b], ax[s] - ax[b]) if axis == 0 else (ax[s] - ax[b], ay[s] - ay[b])
        dist[s] = np.minimum(dist[s], np.minimum(np.abs(np.abs(grid.h - d) - t12), np.abs(np.abs(o) - t34)))
    assert (dist[diff] <= 2 * e32 + 1e-12).all()
    assert int(res.stats.cpu()[1]) == (mask == 2).sum()
