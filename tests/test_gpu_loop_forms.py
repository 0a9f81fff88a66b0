"""The closed loop's team forms and run counting at the edges of their rules,
FP64 per run against the oracle, FP32 steps against the same sweep with the
window out of the way: allocations at each team size and either side of a
wavefront's lanes, sample counts that are and are not powers of two, exact ties
of every score, a wide flag distance, runs of many settings in one workgroup
and histograms too large for the window."""
import numpy as np
import pytest

import oracle
from paper_2110_15425_amd import cm, workloads as W

pytestmark = pytest.mark.gpu


def _check(w):
    print({k: w[k] for k in ("n_settings", "trials", "n_bins")}, w["params"][10:13], flush=True)
    g, o = cm.run(w, dumps=True), oracle.run(w, dumps=True)
    ok = (g["run_flag"] == 0) & (o["run_flag"] == 0)
    assert np.array_equal(g["run_choice"][ok], o["run_choice"][ok])
    assert np.array_equal(g["run_step"][ok], o["run_step"][ok])
    assert ok.all() or w["flag_eps"] > 1e-6
    if ok.all():
        assert np.array_equal(g["hist"], o["hist"]) and np.array_equal(g["stats"], o["stats"])
    else:
        assert np.array_equal(g["run_flag"], o["run_flag"])


@pytest.mark.parametrize("levels,trials", [(1, 9), (2, 70), (3, 33), (4, 33), (5, 33), (8, 33), (9, 20), (15, 9),
                                           (16, 9), (17, 9), (31, 5), (33, 4)])
@pytest.mark.parametrize("samples", [1, 3])
def test_team_sizes(levels, trials, samples):
    _check(W.control_loop(trials=trials, levels=levels, samples=samples, costs=[0.0, 0.01], seed=levels,
                          max_steps=150))


@pytest.mark.parametrize("levels", [4, 8, 9, 17])
def test_exact_ties_and_near_picks(levels):
    # no noise and no control: every allocation scores the same
    _check(W.control_loop(trials=20, levels=levels, samples=2, amax=0.0, noise=0.0, seed=2, max_steps=60,
                          n_bins=20))
    # scores within the flag distance of each other
    _check(W.control_loop(trials=20, levels=levels, samples=2, seed=3, max_steps=60, n_bins=20,
                          flag_eps=1e-3))


@pytest.mark.parametrize("settings,trials,bins", [(300, 1, 100), (41, 3, 100), (1, 700, 150), (200, 2, 4000)])
def test_windows(settings, trials, bins):
    kw = dict(trials=trials, levels=5, samples=2, costs=np.linspace(0.0, 0.03, settings), seed=6,
              max_steps=max(150, bins))
    _check(W.control_loop(n_bins=bins, **kw))
    a = cm.run(W.control_loop(n_bins=bins, precision=W.FP32_STEP, **kw), dumps=True)
    recount = np.zeros_like(a["hist"])
    s = np.repeat(np.arange(settings), trials)
    for c in (0, 1):
        at = a["run_choice"] == c
        np.add.at(recount, (s[at], c, (a["run_step"][at].astype(np.int64) - 1) * bins // kw["max_steps"]), 1)
    assert np.array_equal(a["hist"], recount)
    assert np.array_equal(a["stats"][:, cm.ST["undec"]], np.bincount(s[a["run_choice"] < 0], minlength=settings))
