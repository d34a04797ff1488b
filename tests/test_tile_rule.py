"""Host-side checks of the tiled fields: the worst truncation of the far terms over
the profile family at the criterion's constants, and the rule that picks a tile side
or the direct sum (through the library's host functions; no GPU)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from conftest import ROOT

LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")
CSRC = os.path.join(ROOT, "paper_1902_03252_amd", "csrc")


# ---------------------------------------------------------------- truncation

def alpha(e, ph, a, s, dx, dy):
    """grad Psi / K0 of one potential, K0 the uncut strength."""
    c, sn = np.cos(LD(ph)), np.sin(LD(ph))
    u, v = dx * c + dy * sn, dy * c - dx * sn
    r2 = (1 - e) * u * u + (1 + e) * v * v
    f = 1 / (np.sqrt(a * a + r2) + a)
    if np.isfinite(s):
        f = s / (s - a) * (f - 1 / (np.sqrt(s * s + r2) + s))
    return f * ((1 - e) * u * c - (1 + e) * v * sn), f * ((1 - e) * u * sn + (1 + e) * v * c)


def distance(e, ph, a, dx, dy):
    """The criterion's c^2 for a tile of half width 1 centred at (dx, dy) from the potential."""
    c, sn = np.cos(ph), np.sin(ph)
    A, B, D = (1 - e) * c * c + (1 + e) * sn * sn, -2 * e * c * sn, (1 - e) * sn * sn + (1 + e) * c * c
    t, u = min(max(-B * dx / D, dy - 1), dy + 1), min(max(-B * dy / A, dx - 1), dx + 1)
    return min((A * dx * dx + 2 * B * dx * t + D * t * t + a * a) / A, (A * u * u + 2 * B * dy * u + D * dy * dy + a * a) / D)


def truncation(n, c, e, ph, a, s, th):
    """Largest error of the n x n Chebyshev interpolant over the tile, the potential exactly at the criterion in the
    direction th, in units of w_p."""
    hi = 1.0
    at = lambda r: distance(e, ph, a, r * np.cos(th), r * np.sin(th)) >= c * c
    while not at(hi):
        hi *= 2
    lo = 0.0
    for _ in range(60):
        m = 0.5 * (lo + hi)
        lo, hi = (lo, m) if at(m) else (m, hi)
    x, y = LD(hi * np.cos(th)), LD(hi * np.sin(th))
    k = np.arange(n)
    xi = np.cos(PI * (2 * k + 1) / (2 * n))
    v = np.cos(np.outer(k.astype(LD), np.arccos(xi)))
    d = v * (LD(2) / n)
    d[0] /= 2
    t = np.linspace(-1, 1, 17).astype(LD)
    w = np.cos(np.outer(np.arccos(t), k.astype(LD))) @ d
    gx, gy = np.meshgrid(xi, xi)
    tx, ty = np.meshgrid(t, t)
    f, g = alpha(LD(e), ph, LD(a), LD(s), x + gx, y + gy), alpha(LD(e), ph, LD(a), LD(s), x + tx, y + ty)
    wp = (1 + e) / np.sqrt(1 - e) * (s / (s - a) if np.isfinite(s) else 1)
    return max(float(np.abs(w @ f[q] @ w.T - g[q]).max()) for q in (0, 1)) / wp


@pytest.mark.parametrize("n,name,bar", [(8, "kFarC32", 5.2e-7), (16, "kFarC64", 3e-16)])
def test_truncation_at_the_criterion(n, name, bar):
    """The bars are the ones stated beside the constants."""
    src = open(os.path.join(CSRC, "lens_tiles.hpp")).read()
    c = float(re.search(rf"constexpr float {name} = ([0-9.]+)f;", src).group(1))
    worst = 0.0
    for e in (0.0, 0.3, 0.6, 0.95, 0.999):
        for ph in np.linspace(0, np.pi, 7)[:-1]:
            for th in np.linspace(0, 2 * np.pi, 25)[:-1]:
                for a, s in ((0.0, np.inf), (0.0, 3.0), (1.0, np.inf), (2.5, 4.0)):
                    worst = max(worst, truncation(n, c, e, ph, a, s, th))
    print(f"  N = {n}, c = {c}: {worst:.2e} w_p (bar {bar:.1e})")
    assert worst <= bar


# ---------------------------------------------------------------- side

class Grid(C.Structure):
    _fields_ = [("x0", C.c_double), ("y0", C.c_double), ("h", C.c_double), ("nx", C.c_int), ("ny", C.c_int)]


@pytest.fixture(scope="module")
def side():
    lib = os.path.join(ROOT, "paper_1902_03252_amd", "liblens.so")
    if not os.path.exists(lib):
        pytest.skip("the library is not built")
    f = C.CDLL(lib)._ZN4lens10tiled_sideERKNS_8GridDescEib  # lens::tiled_side(const GridDesc&, int, bool)
    f.restype = C.c_int
    return lambda nx, ny, p, fp32: f(C.byref(Grid(0.0, 0.0, 1.0, nx, ny)), p, C.c_bool(fp32))


# ragged shapes for each side, in both precisions (test_gpu_tiled_sides runs them)
SIDES = {32: [(601, 599, 50), (545, 481, 80), (801, 777, 75)], 64: [(2501, 2495, 12), (2049, 1500, 120), (1025, 8200, 12)],
         128: [(4097, 4095, 20), (4097, 4127, 200), (5001, 4999, 700)]}


def test_sides(side):
    for want, shapes in SIDES.items():
        for s in shapes:
            assert side(*s, True) == want and side(*s, False) == want, s


def test_direct(side):
    for fp32 in (True, False):
        assert side(400, 400, 100, fp32) == 0 and side(420, 420, 100, fp32) != 0    # 2^24 terms
        assert side(4000, 4000, 2048, fp32) != 0 and side(4000, 4000, 2049, fp32) == 0
        assert side(200000, 2, 60, fp32) == 0 and side(2, 65535, 200, fp32) != 0     # thin, narrow
    assert side(4000, 4000, 4, True) != 0 and side(4000, 4000, 3, True) == 0
    assert side(4000, 4000, 12, False) != 0 and side(4000, 4000, 11, False) == 0
