"""The autotuner where the call's field has no nodes per thread (tiled single calls,
batches): it times the tile shapes only, so that the entry's nodes per thread is the
one that the bucket had, or the default, and never the winner among equal kernels."""
import json

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


def entry(path, batched, npl):
    path.write_text(json.dumps({"arch": "gfx950", "entries": [
        {"prec": 2, "batched": batched, "n_log2": 10, "p_log2": 6, "tile": 1, "field_npl": npl, "ms": 1.0}]}))
    return str(path)


@pytest.mark.parametrize("batched", [False, True])
def test_layout_is_left_alone(lens, batched, tmp_path):
    prm, _, obs_np = load_inputs(2)
    obs = lens.Obs.from_numpy(obs_np)
    grid = S.Grid(-60.0, -60.0, 120.0 / 599, 600, 600)  # 360000 x 50 terms: tiled
    if batched:
        layout = lens.BatchLayout(np.arange(3, dtype=np.int32) * 50, [grid] * 2)
        p = dev(np.concatenate([prm[:, :50]] * 2, axis=1))
        tune = lambda ctx: lens.autotune_chi2_batched(p, layout, obs, prec="mixed", ctx=ctx, reps=1)
    else:
        p = dev(prm[:, :50])
        tune = lambda ctx: lens.autotune_chi2(p, grid, obs, prec="mixed", ctx=ctx, reps=1)
    default = 0x41 if batched else 1
    for _ in range(6):
        ctx = lens.Context()
        _, npl, _ = tune(ctx)
        assert npl == default and lens.autotune_lookup("mixed", batched, 600, 50, ctx=ctx)[1] == default
    ctx = lens.Context()
    lens.autotune_load(entry(tmp_path / "t.json", int(batched), 4), ctx=ctx)
    _, npl, _ = tune(ctx)
    assert npl == 4 and lens.autotune_lookup("mixed", batched, 600, 50, ctx=ctx)[1] == 4
