"""GPU parity of the batched triangle stage with single evaluations at the edges
of its work items: 32 tiles of a row and one more, a single column of cells, more
systems than one chunk of 64, each tile shape.  The two forms cull and test
independently, so hits, predicted images, (tile, system) pairs and bounding-box
passes have to agree exactly (the latter two in FP64: the FP32 fields of the two
forms may differ by rounding, which moves a box by less than the hit's bound but
may move a count).  chi^2 within 1e-13, the bar of the same hits in another order."""
import numpy as np
import pytest

import synthlens as S
from conftest import load_inputs

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


def systems(n, seed):
    """n systems: the cluster workload's, in turn, each moved by up to half an arcsecond."""
    _, _, base = load_inputs(2)
    g = np.random.default_rng(seed)
    off, x, y, sg, dls = [0], [], [], [], []
    for s in range(n):
        q = s % (len(base["sys_off"]) - 1)
        sl = slice(base["sys_off"][q], base["sys_off"][q + 1])
        dx, dy = g.uniform(-0.5, 0.5, 2)
        x.append(base["x"][sl] + dx)
        y.append(base["y"][sl] + dy)
        sg.append(base["sigma"][sl])
        dls.append(base["dls"][q])
        off.append(off[-1] + len(x[-1]))
    return dict(sys_off=np.asarray(off, np.int32), x=np.concatenate(x), y=np.concatenate(y), sigma=np.concatenate(sg),
                dls=np.asarray(dls))


SHAPES = [(1025, 66), (1026, 67), (2, 300), (300, 2), (33, 258), (258, 257), (2050, 41)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n_sys,tile", [(1, 1), (63, 2), (64, 3), (65, 4), (130, 1)])
def test_batched_triangles_match_single(lens, prec, n_sys, tile):
    prm, grid, _ = load_inputs(2)
    obs = lens.Obs.from_numpy(systems(n_sys, 7 + n_sys))
    h = 120.0 / 1024
    grids = [S.Grid(-0.5 * h * (nx - 1) + 0.37 * h, -0.5 * h * (ny - 1) - 0.21 * h, h, nx, ny) for nx, ny in SHAPES]
    layout = lens.BatchLayout(np.arange(len(grids) + 1, dtype=np.int32) * prm.shape[1], grids)
    out = lens.batch_buffers(layout.n, obs, "cuda", hits=True)
    got = lens.lens_image_chi2_batched(dev(np.concatenate([prm] * len(grids), axis=1)), layout, obs, prec=prec,
                                       out=out, tile=tile)
    torch.cuda.synchronize()
    pairs = boxes = 0
    for s, g in enumerate(grids):
        print(f"  {g.nx}x{g.ny} {prec} systems {n_sys} tile {tile}", flush=True)
        one = lens.lens_image_chi2(dev(prm), g, obs, prec=prec, tile=tile).host()
        h = got.sample_hits(s)
        np.testing.assert_array_equal(h["hit_sys"], one["hit_sys"])
        np.testing.assert_array_equal(h["hit_tid"], one["hit_tid"])
        np.testing.assert_array_equal(got.n_pred[s].cpu().numpy(), one["n_pred"])
        np.testing.assert_allclose(got.chi2_sys[s].cpu().numpy(), one["chi2_sys"], rtol=1e-13, atol=0)
        pairs += int(one["stats"][2])
        boxes += int(one["stats"][3])
    if prec == "fp64":
        assert (int(got.stats[2]), int(got.stats[3])) == (pairs, boxes)
