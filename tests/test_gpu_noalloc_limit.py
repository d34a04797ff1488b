"""The no-allocation entry point near its fixed scratch: a field that is the direct sum
elsewhere (few potentials in FP64) goes by tiles where only their smaller records fit.
Same hits as the context's call, chi^2 within the FP64 path's bar (1e-9 relative)."""
import numpy as np
import pytest

import synthlens as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,p", [(5500, 5500, 8), (5441, 5555, 11), (5500, 5500, 4)])
def test_few_potentials_near_the_limit(nx, ny, p):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1902_03252_amd as lens
    g = np.random.default_rng(p)
    prm = torch.as_tensor(S.draw_galaxies(g, p, 30.0), dtype=torch.float64, device="cuda")
    grid = S.Grid(-40.0, -40.0, 80.0 / nx, nx, ny)
    n = 6
    obs = lens.Obs.from_numpy(dict(sys_off=np.array([0, 3, 6], dtype=np.int32), x=g.uniform(-30, 30, n),
                                   y=g.uniform(-30, 30, n), sigma=np.full(n, 0.5), dls=np.array([0.6, 0.8])))
    want = lens.lens_image_chi2(prm, grid, obs, prec="fp64").host()
    got = lens.lens_image_chi2_noalloc(prm, grid, obs, prec="fp64").host()
    assert got["status"] == 0 and len(want["hit_tid"]) > 0
    np.testing.assert_array_equal(got["hit_sys"], want["hit_sys"])
    np.testing.assert_array_equal(got["hit_tid"], want["hit_tid"])
    np.testing.assert_array_equal(got["n_pred"], want["n_pred"])
    np.testing.assert_allclose(got["chi2"], want["chi2"], rtol=1e-9)
    with pytest.raises(RuntimeError, match="fixed no-allocation buffer"):
        lens.lens_image_chi2_noalloc(prm, S.Grid(-40.0, -40.0, 80.0 / nx, 6000, 6000), obs, prec="fp64")
