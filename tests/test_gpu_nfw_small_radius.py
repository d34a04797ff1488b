"""GPU parity of the NFW deflection where x^2 = (R / r_s)^2 is at the small end of
its type: a scale radius so large that every node has x^2 near or below the
smallest normal number, and a centre 1e-20 arcsec off a node.

Reference: 4 kappa_s m (ln(2/x) - 1/2)/2, the profile's limit for x -> 0 (the next
term is smaller by x^2).  Bars, relative to the halo's largest deflection on the
grid: FP32 64 u (one halo's evaluation, as test_gpu_tiled) plus 4e-5, the rounding
of a denormal x^2 of at least 2^-138 and of its reciprocal r_s^2, divided by
ln(2/x) > 40 (its halves: 2^-12 / 2 / 40 each); FP64 64 u the same way, x^2 normal."""
import numpy as np
import pytest

import oracle
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


def small_x(halos, grid):
    x, y = np.meshgrid(grid.x0 + np.arange(grid.nx) * grid.h, grid.y0 + np.arange(grid.ny) * grid.h)
    ax, ay = np.zeros(x.shape), np.zeros(x.shape)
    for xc, yc, eps, phi, rs, ks in halos.T:
        a, b, c = 1 - eps * np.cos(2 * phi), -eps * np.sin(2 * phi), 1 + eps * np.cos(2 * phi)
        dx, dy = x - xc, y - yc
        m1, m2 = a * dx + b * dy, b * dx + c * dy
        r = np.sqrt(dx * m1 + dy * m2)
        f = 4 * ks * 0.5 * (np.log(2.0 * rs / r) - 0.5)
        ax += f * m1
        ay += f * m2
    return ax, ay


# direct and tiled sums (P = 1 and 4)
@pytest.mark.parametrize("nx,ny,p", [(65, 50, 1), (65, 50, 4), (2100, 1050, 4)])
@pytest.mark.parametrize("prec,rs", [("fp32", 3e19), ("fp32", 1e20), ("fp32", 1e21), ("fp64", 1e20), ("fp64", 3e151),
                                     ("fp64", 9e151)])
def test_large_scale_radius(lens, nx, ny, p, prec, rs):
    grid = S.Grid(-30.013, -27.9, 60.0 / nx, nx, ny)
    g = np.random.default_rng(p)
    h = np.stack([g.uniform(-20, 20, p), g.uniform(-20, 20, p), g.uniform(0, 0.4, p), g.uniform(0, 3, p),
                  rs * g.uniform(1.0, 1.2, p), g.uniform(0.1, 0.3, p)])
    # sizes of order 10 from every centre: x^2 of 1e-40 and up (FP32), 1e-303 (FP64)
    ax, ay = lens.lens_deflect_nfw(dev(h), grid, prec)
    want = small_x(h, grid)
    scale = np.abs(want[0]).max() + np.abs(want[1]).max()
    far = np.ones((ny, nx), bool)
    if prec == "fp32":  # nodes so near a centre that x^2 has no digits left
        for xc, yc in h[:2].T:
            x, y = np.meshgrid(grid.x0 + np.arange(nx) * grid.h - xc, grid.y0 + np.arange(ny) * grid.h - yc)
            far &= (x * x + y * y) * 0.6 / (1.2 * rs) ** 2 >= 2.0 ** -138
        assert far.any() or rs == 1e21
    tol = 64 * 2.0 ** -53 if prec == "fp64" else 64 * 2.0 ** -24 + 4e-5
    for got, w in ((ax, want[0]), (ay, want[1])):
        got = got.double().cpu().numpy()
        assert np.isfinite(got).all()
        err = np.abs(got - w)[far].max() / scale if far.any() else 0.0
        print(f"  {prec} {nx}x{ny} P={p} r_s={rs:.0e}: {err:.2e} (bar {tol:.2e})", flush=True)
        assert err <= tol


@pytest.mark.parametrize("nx,ny,p", [(80, 70, 5), (2100, 1050, 5)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("off", [1e-17, 1e-20, 1e-23])
def test_centre_next_to_a_node(lens, nx, ny, p, prec, off):
    """The halo contributes next to nothing at its own node: there the field is the other halos'."""
    grid = S.Grid(0.0, 0.0, 0.05, nx, ny)
    h = S.nfw_cluster(S.Grid(0.0, 0.0, 0.05, 80, 70), n_galaxies=p - 2, seed=3)
    h[0, p - 1] = h[1, p - 1] = off
    got = lens.lens_deflect_nfw(dev(h), grid, prec)
    want = oracle.nfw_alpha_grid(h[:, : p - 1], S.Grid(0.0, 0.0, 0.05, 2, 2))
    w = (1.3 * h[5] * h[4] * (1 + h[2]) / np.sqrt(1 - h[2])).sum()
    tol = 2.0 ** -24 * (64 + p) * w if prec == "fp32" else 1e-10
    for a, b in zip(got, want):
        assert torch.isfinite(a).all()
        assert abs(float(a[0, 0]) - b[0, 0]) <= tol
