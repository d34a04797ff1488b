"""GPU parity of the tiled deflection field (near potentials per node, the far
ones through one Chebyshev polynomial per tile) against the FP64 CPU oracle, at
the edges of its tiles and of the rule that selects it: grids a node short of,
on and past multiples of the tile sides, thin grids, few and many potentials,
every profile kind, centres on nodes and outside the grid.

Bars: FP64 within 1e-10 arcsec, FP32 within the library's stated FP32
deflection bound (test_gpu_parity).  The oracle evaluates sampled rows: the first and last two, and the rows around
every kind of tile boundary."""
import numpy as np
import pytest

import oracle
import synthlens as S
from test_gpu_parity import fp32_alpha_bound

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


def potentials(grid, p, seed, overflow):
    """Galaxies of every profile kind over a field a little wider than the grid, one halo, one centre exactly on a
    node, one 1e-9 nodes off a node, and (FP32 only) one with a cut radius whose square overflows."""
    g = np.random.default_rng(seed)
    lx, ly = 0.5 * (grid.nx - 1) * grid.h, 0.5 * (grid.ny - 1) * grid.h
    prm = S.draw_galaxies(g, p, 1.0)
    prm[0] = grid.x0 + lx + 1.2 * lx * prm[0]
    prm[1] = grid.y0 + ly + 1.2 * ly * prm[1]
    kind = g.integers(0, 4, p)
    prm[4, kind % 2 == 1] = 0.0
    prm[5, kind // 2 == 1] = np.inf
    prm[:, 0] = (grid.x0 + lx, grid.y0 + ly, 0.05, 0.3, 5.0, 1000.0, 1000.0)
    prm[0, 1], prm[1, 1] = grid.x0 + (grid.nx // 3) * grid.h, grid.y0 + (grid.ny // 2) * grid.h
    prm[0, 2], prm[1, 2] = prm[0, 1] + 1e-9 * grid.h, prm[1, 1] - grid.h
    if overflow:
        prm[5, 3] = 1e160
    prm[2, p // 2] = 0.95
    return prm


def sampled_rows(ny, g):
    rows = {0, 1, ny - 2, ny - 1} | {r + d for r in (32, 64, 128, 256) for d in (-1, 0, 1)}
    rows |= set(int(v) for v in g.integers(0, ny, 4))
    return sorted(r for r in rows if 0 <= r < ny - 1)


def check_rows(ax, ay, prm, grid, tol, what):
    worst = 0.0
    for j in sampled_rows(grid.ny, np.random.default_rng(1)):
        sub = S.Grid(grid.x0, grid.y0 + j * grid.h, grid.h, grid.nx, 2)
        ox, oy = oracle.alpha_grid(prm, sub)
        for got, want in ((ax, ox), (ay, oy)):
            worst = max(worst, np.abs(got[j:j + 2].double().cpu().numpy() - want).max())
    print(f"  {what}: max err {worst:.2e} (bar {tol:.2e})", flush=True)
    assert worst <= tol


# (nx, ny, P): the rule's sides 32, 64 and 128 and both of its limits in P
SHAPES = [(512, 512, 64), (513, 511, 70), (545, 481, 80), (1025, 1023, 40), (2049, 1500, 120), (1999, 2113, 700),
          (40007, 9, 60), (9, 40007, 60), (2300, 2300, 4), (2300, 2300, 3), (300, 280, 2048), (300, 280, 2049)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,p", SHAPES)
def test_tiled_field(lens, nx, ny, p, prec):
    grid = S.Grid(-61.3, -47.9, 120.0 / max(nx, ny), nx, ny)
    prm = potentials(grid, max(p, 4), nx + p, prec == "fp32")[:, :p]
    ax, ay = lens.lens_deflect(dev(prm), grid, prec)
    prm = prm.copy()
    prm[5, prm[5] > 1e100] = np.inf  # the oracle squares the cut radius
    tol = 1e-10 if prec == "fp64" else fp32_alpha_bound(prm, grid)
    check_rows(ax, ay, prm, grid, tol, f"{prec} {nx}x{ny} P={p}")


# NFW halos: (nx, ny, P) around the tile sides and the rule's limits
NFW_SHAPES = [(512, 500, 40), (545, 481, 80), (1025, 1023, 60), (2049, 1500, 302), (40007, 9, 60), (300, 280, 2048),
              (300, 280, 2049), (2300, 2300, 3)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,p", NFW_SHAPES)
def test_tiled_nfw_field(lens, nx, ny, p, prec):
    """FP64 within 1e-10 arcsec; FP32 within u (64 + P) sum_p w_p, w_p = 1.3 kappa_s r_s (1 + eps)/sqrt(1 - eps)
    the largest deflection of a halo (4 g(x)/x is at most 1.3), 64 u w_p for one halo's evaluation (about 30
    operations, five of them 1-2 ulp functions, doubled) and (P - 1) u sum w for the sum."""
    grid = S.Grid(-31.3, -27.9, 60.0 / max(nx, ny), nx, ny)
    h = S.nfw_cluster(grid, n_galaxies=p - 2, seed=p)
    h[0, p - 1], h[1, p - 1] = grid.x0 + (nx // 3) * grid.h, grid.y0 + (ny // 2) * grid.h  # a centre on a node
    w = (1.3 * h[5] * h[4] * (1 + h[2]) / np.sqrt(1 - h[2])).sum()
    tol = 1e-10 if prec == "fp64" else 2.0 ** -24 * (64 + p) * w
    ax, ay = lens.lens_deflect_nfw(dev(h), grid, prec)
    worst = 0.0
    for j in sampled_rows(ny, np.random.default_rng(1)):
        sub = S.Grid(grid.x0, grid.y0 + j * grid.h, grid.h, nx, 2)
        want = oracle.nfw_alpha_grid(h, sub)
        for got, o in ((ax, want[0]), (ay, want[1])):
            worst = max(worst, np.abs(got[j:j + 2].double().cpu().numpy() - o).max())
    print(f"  nfw {prec} {nx}x{ny} P={p}: max err {worst:.2e} (bar {tol:.2e})", flush=True)
    assert worst <= tol
