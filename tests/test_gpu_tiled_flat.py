"""GPU parity of the tiled deflection field with potentials of ellipticity close to
1, far away along their long axis: R^2 = d . M d is then a small difference of
large terms, and the singular line of the nearly flat potential passes close to
the tiles although its centre is far off.

Reference: the profile in long double.  Bar (FP64): the direct sum's own error,
8 roundings of the terms A dx^2, 2 B dx dy, C dy^2 (together at most 4 d^2) in
R^2, relative to the R^2 of the long axis, (1 - eps) d^2, for deflections of at
most K sqrt(1 + eps) (|M d| <= sqrt(1 + eps) R); and 1e-10 arcsec for everything
else.  FP32: the library's bound u (64 + P) sum_p w_p with these potentials in it."""
import numpy as np
import pytest

import synthlens as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LD = np.longdouble


@pytest.fixture(scope="module")
def lens():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1902_03252_amd as lens
    lens.context()
    return lens


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def alpha(t, x, y):
    pi = LD("3.14159265358979323846264338327950288")
    sx, sy = np.zeros(x.shape, LD), np.zeros(x.shape, LD)
    for q in t.T:
        xc, yc, e, ph, a, s, sg = [LD(v) for v in q]
        c, sn = np.cos(ph), np.sin(ph)
        k = 4 * pi * (sg / LD("299792.458")) ** 2 * (LD(180) * 3600 / pi)
        u, v = (x - xc) * c + (y - yc) * sn, (y - yc) * c - (x - xc) * sn
        r2 = (1 - e) * u * u + (1 + e) * v * v
        f = k / (np.sqrt(a * a + r2) + a)
        if np.isfinite(s):
            f = s / (s - a) * (f - k / (np.sqrt(s * s + r2) + s))
        sx += f * ((1 - e) * u * c - (1 + e) * v * sn)
        sy += f * ((1 - e) * u * sn + (1 + e) * v * c)
    return sx, sy


# directions in which FP32 takes the quadratic for larger than it is
PHI = (0.751002, 0.839762, 0.887604, 2.389629, 2.431259, 2.395361)


@pytest.mark.parametrize("flat,nodes", [(1e-6, 1e4), (1e-9, 1e6), (1e-10, 1e6), (1e-11, 1e6), (1e-11, 3e6)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_flat_potentials_far_along_their_axes(lens, flat, nodes, prec):
    grid = S.Grid(-30.0, -29.0, 0.1, 601, 585)
    g = np.random.default_rng(5)
    prm = S.draw_galaxies(g, 60, 20.0)
    n = len(PHI)
    for k, ph in enumerate(PHI):
        prm[:, k] = (grid.x0 + (300 + np.rint(-nodes * np.cos(ph))) * grid.h,
                     grid.y0 + (290 + np.rint(-nodes * np.sin(ph))) * grid.h, 1.0 - flat, ph, 0.0, np.inf, 100.0)
    kk = 4 * np.pi * (prm[6] / 299792.458) ** 2 * 206264.806
    if prec == "fp64":
        tol = 1e-10 + 8 * 2.0 ** -53 * 4 / flat * 1.42 * kk[:n].sum()
    else:
        w = kk * (1 + prm[2]) / np.sqrt(1 - prm[2])
        fin = np.isfinite(prm[5])
        w[fin] *= prm[5, fin] / (prm[5, fin] - prm[4, fin])
        tol = 2.0 ** -24 * (64 + 60) * w.sum()
    # along the axes, where the singular lines pass, and anywhere
    i, j = g.integers(0, grid.nx, 6000), g.integers(0, grid.ny, 6000)
    r, k = g.uniform(-280, 280, 6000), g.integers(0, n, 6000)
    ph = np.array(PHI)[k]
    i = np.concatenate([i, np.rint(300 + r * np.cos(ph)).astype(int)])
    j = np.concatenate([j, np.rint(290 + r * np.sin(ph) + g.uniform(-12, 12, 6000)).astype(int)])
    want = alpha(prm, (grid.x0 + i * grid.h).astype(LD), (grid.y0 + j * grid.h).astype(LD))
    got = lens.lens_deflect(dev(prm), grid, prec)
    err = max(float(np.abs(a.double().cpu().numpy()[j, i] - b).max()) for a, b in zip(got, want))
    print(f"  1 - eps = {flat:.0e}, {nodes:.0e} nodes, {prec}: max err {err:.2e} (bar {tol:.2e})", flush=True)
    assert err <= tol


@pytest.mark.parametrize("core,cut", [(1e19, np.inf), (3e19, np.inf), (1e20, 1e21), (1e25, np.inf)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_core_whose_square_leaves_fp32(lens, core, cut, prec):
    """A core radius beyond the square root of FP32's largest number: far from every tile, its deflection in FP64."""
    grid = S.Grid(-30.0, -29.0, 0.1, 601, 585)
    g = np.random.default_rng(5)
    prm = S.draw_galaxies(g, 60, 20.0)
    prm[:, 3] = (5.0, -3.0, 0.3, 0.4, core, cut, 1000.0)
    i, j = g.integers(0, grid.nx, 3000), g.integers(0, grid.ny, 3000)
    want = alpha(prm, (grid.x0 + i * grid.h).astype(LD), (grid.y0 + j * grid.h).astype(LD))
    got = lens.lens_deflect(dev(prm), grid, prec)
    assert all(torch.isfinite(a).all() for a in got)
    err = max(float(np.abs(a.double().cpu().numpy()[j, i] - b).max()) for a, b in zip(got, want))
    kk = 4 * np.pi * (prm[6] / 299792.458) ** 2 * 206264.806 * (1 + prm[2]) / np.sqrt(1 - prm[2]) * 1.2
    assert err <= (1e-10 if prec == "fp64" else 2.0 ** -24 * (64 + 60) * kk.sum())
