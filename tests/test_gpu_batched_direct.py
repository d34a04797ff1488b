"""GPU parity of the batched samples whose field is the direct sum (fewer than 4
potentials, in FP64 fewer than 12, more than the tiles' lists hold, a few rows)
with single evaluations, next to tiled samples in one call: at the edges of the
direct sum's units (64 columns, 8 rows, 64 potentials' row parts at a time) and of
the rule.  The two forms cull and test independently, so hits and predicted images
have to agree exactly, and in FP64 the (tile, system) pairs and bounding-box passes;
chi^2 within 1e-13, the bar of the same hits in another order."""
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


def model(p):
    """The cluster's first p potentials, or all of them and faint galaxies."""
    prm, _, _ = load_inputs(2)
    if p > prm.shape[1]:
        more = S.draw_galaxies(np.random.default_rng(p), p - prm.shape[1], 60.0)
        more[6] *= 0.1
        more[4, ::3] = 0.0
        more[5, ::5] = np.inf
        prm = np.concatenate([prm, more], axis=1)
    return prm[:, :p]


# (nx, ny, P)
MIXES = [
    [(65, 50, 0), (64, 64, 1), (129, 127, 2), (512, 500, 3), (63, 9, 4), (300, 301, 11), (300, 301, 12)],
    [(120, 121, 2048), (120, 121, 2049), (66, 33, 2100), (257, 256, 50), (2, 64, 2049)],
    [(4097, 2, 50), (2000, 3, 50), (30000, 8, 12), (30001, 9, 50), (3, 4096, 50), (700, 16, 50)],
]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("mix", range(3))
def test_direct_samples_match_single(lens, prec, mix):
    _, _, obs_np = load_inputs(2)
    obs = lens.Obs.from_numpy(obs_np)
    rng = np.random.default_rng(mix)
    grids, blocks = [], []
    for nx, ny, p in MIXES[mix]:
        h = 120.0 / max(nx, ny)
        grids.append(S.Grid(-0.5 * h * (nx - 1) + h * rng.uniform(), -0.5 * h * (ny - 1) + h * rng.uniform(), h, nx, ny))
        blocks.append(model(p))
    layout = lens.BatchLayout(np.concatenate([[0], np.cumsum([b.shape[1] for b in blocks])]).astype(np.int32), grids)
    out = lens.batch_buffers(layout.n, obs, "cuda", hits=True)
    got = lens.lens_image_chi2_batched(dev(np.concatenate(blocks, axis=1)), layout, obs, prec=prec, out=out)
    torch.cuda.synchronize()
    pairs = boxes = hits = 0
    for s, (g, b) in enumerate(zip(grids, blocks)):
        print(f"  {g.nx}x{g.ny} P={b.shape[1]} {prec}", flush=True)
        one = lens.lens_image_chi2(dev(b), g, obs, prec=prec).host()
        h = got.sample_hits(s)
        np.testing.assert_array_equal(h["hit_sys"], one["hit_sys"])
        np.testing.assert_array_equal(h["hit_tid"], one["hit_tid"])
        np.testing.assert_array_equal(got.n_pred[s].cpu().numpy(), one["n_pred"])
        np.testing.assert_allclose(got.chi2_sys[s].cpu().numpy(), one["chi2_sys"], rtol=1e-13, atol=0)
        pairs += int(one["stats"][2])
        boxes += int(one["stats"][3])
        hits += len(h["hit_tid"])
    assert hits > 0
    if prec == "fp64":
        assert (int(got.stats[2]), int(got.stats[3])) == (pairs, boxes)
