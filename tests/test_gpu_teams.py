"""Small launches and drains of the lane kernels, where a team of lanes holds
each run: every per-run outcome equals the node-by-node execution's bit for
bit, over team sizes from 64 lanes to one, ragged last chunks, short and odd
step caps, clipped units and a wide flag distance (runs that come near the
threshold and go on)."""
import numpy as np
import pytest

from paper_2110_15425_amd import cm, workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 5), (3, 67), (37, 27), (5, 1021), (64, 1024), (7, 18725), (1, 262_145)]
PREC = {"fp64": W.FP64, "fp32": W.FP32_STEP}


def _same(h, w):
    ds = cm.DeviceSweep(h, w, dumps=True)
    ds.launch()
    got = ds.results()
    ds.launch_unfused()
    want = ds.results()
    for k in ("run_choice", "run_step", "run_flag", "run_state", "hist", "stats"):
        assert np.array_equal(got[k], want[k]), k


def _grid(s):
    return np.stack([np.linspace(0.0, 5.0, s), np.linspace(1.0, 0.5, s)], 1)


@pytest.mark.parametrize("prec", sorted(PREC))
@pytest.mark.parametrize("settings,trials", SIZES)
def test_lca_teams(settings, trials, prec):
    print(f"lca {settings} x {trials} {prec}", flush=True)
    _same(cm.Handle(0), W.conflict(trials=trials, seed=5, grid=_grid(settings), precision=PREC[prec]))


@pytest.mark.parametrize("prec", sorted(PREC))
@pytest.mark.parametrize("settings,trials", SIZES)
def test_ddm_teams(settings, trials, prec):
    print(f"ddm {settings} x {trials} {prec}", flush=True)
    h = cm.Handle(0)
    h.set_tuning(W.DDM, PREC[prec], lanes_per_run=1)
    _same(h, W.ddm(trials=trials, seed=6, drifts=np.linspace(-0.4, 0.9, settings), precision=PREC[prec]))


@pytest.mark.parametrize("prec", sorted(PREC))
@pytest.mark.parametrize("steps", [1, 2, 7, 64, 65, 201])
def test_team_caps_and_near_misses(steps, prec):
    h = cm.Handle(0)
    h.set_tuning(W.DDM, PREC[prec], lanes_per_run=1)
    kw = dict(seed=9, max_steps=steps, n_bins=min(steps, 10), precision=PREC[prec])
    for eps in (1e-10, 0.05):
        print(f"steps {steps} {prec} eps {eps}", flush=True)
        _same(h, W.ddm(trials=301, drifts=[0.0, 0.5], flag_eps=eps, **kw))
        for nonneg in (0.0, 1.0):
            _same(h, W.conflict(trials=301, grid=_grid(2), nonneg=nonneg, flag_eps=eps, **kw))
