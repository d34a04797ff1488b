"""GPU parity of the HMC step at the limits of its one-workgroup form (n_img n
<= 6144 terms and 64 KB of LDS) against the oracle's plain FP64 step on the same
draws: one potential, potential counts around the 16 and 64 lane groups, every
profile kind, uneven systems (an empty one and single images among them), and
models just inside and outside the limits.

Bars as in test_gpu_sampler: the end state within 1e-7 of a step, chi^2 within
1e-9 relative, decisions identical (the draw is kept off the threshold)."""
import math

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


def model(n, n_img, seed):
    g = np.random.default_rng(seed)
    prm = S.draw_galaxies(g, n)
    kind = np.arange(n) % 4
    prm[4, kind % 2 == 1] = 0.0
    prm[5, kind // 2 == 1] = np.inf
    prm[:, 0] = S.CLUSTER_HALO
    counts = []
    while sum(counts) < n_img:
        counts.append(int(min(g.integers(0, 6), n_img - sum(counts))))
    obs = dict(sys_off=np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), x=g.uniform(-40, 40, n_img),
               y=g.uniform(-40, 40, n_img), sigma=g.uniform(5.0, 9.0, n_img), dls=g.uniform(0.4, 0.9, len(counts)))
    st = np.zeros_like(prm)
    st[0, 0] = st[1, 0] = 2e-3
    st[2, 0], st[3, 0], st[4, 0], st[6, 0] = 2e-4, 2e-3, 2e-3, 0.05
    st[6, 1:] = 0.05
    st[3, 1::3] = 1e-3   # some galaxies turn, some do not
    return prm, obs, st, g.normal(size=prm.shape), g


@pytest.mark.parametrize("n,n_img,leap", [(1, 1, 1), (1, 40, 3), (15, 63, 4), (17, 65, 2), (64, 96, 3), (65, 94, 3),
                                          (96, 64, 2), (128, 48, 2), (128, 49, 2), (12, 512, 2), (3, 1100, 2)])
def test_hmc_step_sizes(lens, n, n_img, leap):
    prm, obs_np, st, mom, g = model(n, n_img, 100 * n + n_img)
    obs = lens.Obs.from_numpy(obs_np)
    for u in (1e-9, 1.0 - 1e-9):  # one that accepts any finite energy change of a few, one that takes energy losses only
        want_q, want_c, want_acc = oracle.hmc_step(prm, obs_np, st, leap, mom, u)
        state = dev(prm)
        chi2, acc = lens.hmc_step(state, obs, dev(st), leap, dev(mom), dev([u]))
        got_q, got_c, got_acc = state.cpu().numpy(), float(chi2.cpu()[0]), bool(acc.cpu()[0])
        print(f"  n={n} n_img={n_img} u={u:.1e}: accepted {got_acc} (oracle {want_acc}), chi2 {got_c:.8e}", flush=True)
        assert got_acc == want_acc
        assert got_c == pytest.approx(want_c, rel=1e-9)
        same = np.isinf(prm) & (got_q == want_q)
        assert (same | (np.abs(got_q - want_q) <= 1e-7 * st + 1e-13 * np.abs(np.where(same, 0.0, want_q)))).all()


def test_hmc_small_invalid_offsets(lens):
    """Offsets that do not cover the images: no step is taken, chi^2 is NaN."""
    prm, obs_np, st, mom, _ = model(10, 30, 5)
    obs_np["sys_off"][-1] = 29
    obs = lens.Obs.from_numpy(obs_np)
    state = dev(prm)
    chi2, acc = lens.hmc_step(state, obs, dev(st), 3, dev(mom), dev([0.5]))
    assert math.isnan(float(chi2.cpu()[0])) and not bool(acc.cpu()[0])
    assert torch.equal(state, dev(prm))
