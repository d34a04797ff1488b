"""GPU accuracy of the tiled fields for every tile side, on ragged grids: against the
profiles in long double at random nodes and at those around tile edges, the grid's
last tiles among them.

Bars, relative to the root mean square of the deflection over the nodes (u = 2^-53 or
2^-24).  FP64: 8 u (rms) and 40 u (largest): a node is the sum of a few dozen rounded
terms and of an interpolation of values with the same rounding, each about 1 ulp of a
part of the field; a truncation that is not negligible (1e-12 w_p, as with c = 3
instead of 4.5) is 10 to 100 times the bars.  FP32: 4 u and 16 u the same way, the
near terms with 2 ulp roots, where the truncation of the far ones (c = 3: 5e-7 w_p of
one galaxy, a hundredth of the field) belongs to it.  NFW: 8 times that, the
profile's functions amplifying the rounding of x near 1 and the sum of its terms."""
import numpy as np
import pytest

import oracle
import synthlens as S
from test_tile_rule import LD, SIDES
from test_gpu_tiled_flat import alpha

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(t, *s) for t, v in SIDES.items() for s in v]


@pytest.fixture(scope="module")
def lens():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1902_03252_amd as lens
    lens.context()
    return lens


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def nodes(g, n, nx, ny, t):
    """n random nodes, and as many next to tile edges or the grid's."""
    i, j = g.integers(0, nx, 2 * n), g.integers(0, ny, 2 * n)
    edge = lambda m: np.clip(np.where(g.uniform(size=n) < 0.5, t * g.integers(0, m // t + 1, n), m - 1) +
                             g.integers(-1, 2, n), 0, m - 1)
    i[n:] = np.where(g.uniform(size=n) < 0.5, edge(nx), i[n:])
    j[n:] = np.where(g.uniform(size=n) < 0.5, edge(ny), j[n:])
    return i, j


def check(got, want, u, rms_bar, max_bar, what):
    scale = np.sqrt(float((want[0] ** 2 + want[1] ** 2).mean()))
    d = [g.double().cpu().numpy().astype(LD) - w for g, w in zip(got, want)]
    rms = np.sqrt(float((d[0] ** 2 + d[1] ** 2).mean())) / scale
    top = max(float(np.abs(v).max()) for v in d) / scale
    print(f"  {what}: rms {rms:.2e} (bar {rms_bar * u:.1e}), max {top:.2e} (bar {max_bar * u:.1e})", flush=True)
    assert rms <= rms_bar * u and top <= max_bar * u


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("t,nx,ny,p", SHAPES)
def test_side(lens, t, nx, ny, p, prec):
    h = 160.0 / max(nx, ny)
    grid = S.Grid(-0.5 * h * nx + 0.3 * h, -0.5 * h * ny - 0.2 * h, h, nx, ny)
    g = np.random.default_rng(nx + p)
    prm = S.draw_galaxies(g, p, 60.0)
    prm[:, 0] = (0.3, -0.2, 0.05, 0.3, 5.0, 1000.0, 1000.0)
    prm[4, 1::5] = 0.0
    prm[5, 2::5] = np.inf
    i, j = nodes(g, 1500, nx, ny, t)
    want = alpha(prm, (grid.x0 + i * h).astype(LD), (grid.y0 + j * h).astype(LD))
    ax, ay = lens.lens_deflect(dev(prm), grid, prec)
    ij = torch.as_tensor(j, device="cuda"), torch.as_tensor(i, device="cuda")
    u, bars = (2.0 ** -53, (8, 40)) if prec == "fp64" else (2.0 ** -24, (4, 16))
    check((ax[ij], ay[ij]), want, u, *bars, f"{prec} {nx}x{ny} P={p} side {t}")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,p", [(700, 701, 60), (2501, 2495, 12), (4097, 4095, 20), (4097, 4127, 200)])
def test_nfw_side(lens, nx, ny, p, prec):
    grid = S.Grid(-30.1, -29.7, 60.0 / max(nx, ny), nx, ny)
    h = S.nfw_cluster(grid, n_galaxies=p - 2, seed=p)
    g = np.random.default_rng(p)
    rows = sorted({1, 63, 64, 127, 128, ny - 2} | set(int(v) for v in g.integers(0, ny - 1, 4)))
    got, want = [[], []], [[], []]
    ax, ay = lens.lens_deflect_nfw(dev(h), grid, prec)
    for r in rows:
        o = oracle.nfw_alpha_grid(h, S.Grid(grid.x0, grid.y0 + r * grid.h, grid.h, nx, 2))
        for c, a in enumerate((ax, ay)):
            got[c].append(a[r])
            want[c].append(o[c][0])
    u, bars = (2.0 ** -53, (64, 320)) if prec == "fp64" else (2.0 ** -24, (32, 128))
    check([torch.cat(v) for v in got], [np.concatenate(v).astype(LD) for v in want], u, *bars, f"nfw {prec} {nx}x{ny} P={p}")


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,tile", [(4097, 4095, 1), (4127, 4033, 2), (4225, 4001, 3), (4095, 4102, 4)])
def test_chi2_on_ragged_128_tiles(lens, nx, ny, tile, prec):
    """Range records of clipped 128-node tiles: the hits are the oracle's, taken from the FP64 field's own rule."""
    from conftest import load_inputs
    prm, _, obs_np = load_inputs(2)
    prm = prm[:, :20]
    h = 120.0 / max(nx, ny)
    grid = S.Grid(-0.5 * h * nx, -0.5 * h * ny, h, nx, ny)
    want = oracle.image_chi2(prm, grid, obs_np)
    got = lens.lens_image_chi2(dev(prm), grid, lens.Obs.from_numpy(obs_np), prec=prec, tile=tile).host()
    assert got["status"] == 0 and len(got["hit_tid"]) > 0
    np.testing.assert_array_equal(got["hit_sys"], want["hit_sys"])
    np.testing.assert_array_equal(got["hit_tid"], want["hit_tid"])
    np.testing.assert_array_equal(got["n_pred"], want["n_pred"])


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batch_beyond_a_million_arcsec(lens, prec):
    """Grids of 3e6 arcsec, where the coordinates' rounding exceeds 1e-10 arcsec: batched hits are the single calls'
    and the oracle's; sources within a few ulps of nodes, so that they lie at the corners of their cells."""
    g = np.random.default_rng(2)
    grids = [S.Grid(-1.4e6 + 1e3 * k, 1.1e6, 1.0e4, 300 - k, 280 + k) for k in range(3)]
    prm = S.draw_galaxies(g, 20, 30.0)
    prm[0] += grids[0].x0 + 1.5e6
    prm[1] += grids[0].y0 + 1.4e6
    n = 60
    i, j = g.integers(1, 290, n), g.integers(1, 270, n)
    x, y = grids[0].x0 + i * grids[0].h, grids[0].y0 + j * grids[0].h
    for v in (x, y):
        for _ in range(3):
            v[:] = np.nextafter(v, np.where(g.uniform(size=n) < 0.5, -np.inf, np.inf))
    obs_np = dict(sys_off=np.arange(n + 1, dtype=np.int32), x=x, y=y, sigma=np.full(n, 1.0), dls=g.uniform(0.4, 0.9, n))
    obs = lens.Obs.from_numpy(obs_np)
    layout = lens.BatchLayout(np.arange(4, dtype=np.int32) * 20, grids)
    out = lens.batch_buffers(3, obs, "cuda", hits=True)
    got = lens.lens_image_chi2_batched(dev(np.concatenate([prm] * 3, axis=1)), layout, obs, prec=prec, out=out)
    torch.cuda.synchronize()
    for s, grid in enumerate(grids):
        one = lens.lens_image_chi2(dev(prm), grid, obs, prec=prec).host()
        want = oracle.image_chi2(prm, grid, obs_np)
        h = got.sample_hits(s)
        assert len(h["hit_tid"]) > 0
        for r in (one, h):
            np.testing.assert_array_equal(r["hit_sys"], want["hit_sys"])
            np.testing.assert_array_equal(r["hit_tid"], want["hit_tid"])
