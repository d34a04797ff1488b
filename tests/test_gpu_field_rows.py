"""Rows of a tiled field that do not start at multiples of 16 bytes: the nodes are the
same bits as in a grid, and a buffer, of aligned rows; nothing around the planes is
written; and the rows cost what aligned ones do (a plane is written with the same
instructions: at 4 potentials, where the writes are most of the time, a width one
less took 1.9 times as long when its lanes stored single nodes; bar 1.4)."""
import ctypes as C

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


def guarded(lens, prm, grid, prec, shift):
    """Both planes in one buffer, `shift` elements from an aligned address, guards between."""
    n, dt = grid.nx * grid.ny, torch.float64 if prec == "fp64" else torch.float32
    buf = torch.full((2 * n + 64 + 2 * shift,), -7.0, dtype=dt, device="cuda")
    ax, ay = buf[shift:shift + n], buf[2 * shift + n + 32:2 * shift + 2 * n + 32]
    L, ctx = lens._lib, lens.context()
    p, status = lens._pots(prm), torch.zeros(1, dtype=torch.int32, device="cuda")
    L.check(ctx._lib.lens_deflect(ctx.handle, C.byref(p), C.byref(lens._grid(grid)), lens._PREC[prec], L.ptr(ax),
                                  L.ptr(ay), L.ptr(status), ctx.stream()), "lens_deflect")
    assert int(status) == 0
    rest = torch.ones_like(buf, dtype=torch.bool)
    rest[shift:shift + n] = False
    rest[2 * shift + n + 32:2 * shift + 2 * n + 32] = False
    assert bool((buf[rest] == -7.0).all())
    return ax.view(grid.ny, grid.nx), ay.view(grid.ny, grid.nx)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,p", [(1056, 1000, 20), (2304, 2303, 24), (4224, 4097, 24)])  # FP64 sides 32, 64, 128
def test_rows_at_any_address(lens, nx, ny, p, prec):
    h = 2.0 ** -5
    prm = dev(S.draw_galaxies(np.random.default_rng(p), p, 60.0))
    grid = lambda nx: S.Grid(-40.0, -40.0, h, nx, ny)
    want = lens.lens_deflect(prm, grid(nx), prec)
    for less in (0, 1, 2, 3, 31):
        for shift in (0, 1, 2, 3):
            got = guarded(lens, prm, grid(nx - less), prec, shift)
            assert all(torch.equal(a, b[:, :nx - less]) for a, b in zip(got, want)), (less, shift)


@pytest.mark.parametrize("prec,p", [("fp32", 4), ("fp64", 12)])
def test_odd_width_costs_what_an_even_one_does(lens, prec, p):
    prm = dev(S.draw_galaxies(np.random.default_rng(p), p, 60.0))

    def best(nx):
        grid, t = S.Grid(-40.0, -40.0, 80.0 / nx, nx, 4096), []
        for _ in range(60):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            lens.lens_deflect(prm, grid, prec, check=False)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    even, odd = best(4096), best(4095)
    print(f"  {prec} P={p}: 4096 columns {1e3 * even:.1f} us, 4095 {1e3 * odd:.1f}", flush=True)
    assert odd <= 1.4 * even
