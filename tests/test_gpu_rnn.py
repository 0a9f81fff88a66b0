"""GPU parity for the recurrent rate network (matrix-core kernels).

FP64: per-run integers bit-exact on unflagged runs, final readout and unit
states within 1e-9 relative.  BF16 projection: paired with the FP64 oracle
(same random words), compared by decision agreement and histogram L1."""
import numpy as np
import pytest

import oracle
from paper_2110_15425_amd import cm, workloads as W
from parity import assert_parity, hist_l1

pytestmark = pytest.mark.gpu


def _case(n_units, trials, seed=1, **kw):
    return W.rnn(trials=trials, seed=seed, n_units=n_units,
                 weights=W.rnn_weights(n_units, 7), **kw)


def _both(w):
    print(f"case rnn prec={w['precision']} n={w['n_units']} S={w['n_settings']} "
          f"T={w['trials']} N={w['max_steps']} seed={w['seed']}", flush=True)
    return cm.run(w, dumps=True), oracle.run(w, dumps=True, n_threads=0)


@pytest.mark.parametrize("n_units,trials", [(64, 600), (128, 300), (192, 200), (256, 250)])
def test_rnn_fp64_parity(n_units, trials):
    w = _case(n_units, trials)
    g, o = _both(w)
    assert_parity(w, g, o, [-1])
    # both choices occur and some runs hit the cap at the reference shape
    if n_units == 256:
        st = g["stats"][0]
        assert st[0] > 0 and st[1] > 0


def test_rnn_fp64_gain_grid_and_ragged():
    w = _case(128, 37, seed=3, gains=np.linspace(0.5, 1.5, 7))
    g, o = _both(w)
    assert_parity(w, g, o, [-1])


def test_rnn_fp64_short_cap_and_bins():
    w = _case(64, 500, seed=4, max_steps=17, n_bins=17)
    g, o = _both(w)
    assert_parity(w, g, o, [-1])


def test_rnn_uncoupled_noise_free():
    nu = 64
    wts = np.concatenate([np.zeros(nu * nu), W.rnn_weights(nu, 3)[nu * nu:] * 4.0])
    w = W.rnn(trials=100, seed=2, n_units=nu, noise=0.0, weights=wts, max_steps=120)
    g, o = _both(w)
    assert_parity(w, g, o, [-1])


@pytest.mark.parametrize("n_units,trials", [(64, 2000), (256, 400)])
def test_rnn_bf16_against_fp64(n_units, trials):
    w = _case(n_units, trials, seed=5)
    wb = W.with_(w, precision=W.BF16_PROJ)
    g = cm.run(wb, dumps=True)
    o64 = oracle.run(w, dumps=True)
    ob = oracle.run(wb, dumps=True)
    agree = (g["run_choice"] == o64["run_choice"]).mean()
    agree_b = (g["run_choice"] == ob["run_choice"]).mean()
    print(f"bf16 n={n_units}: choice agreement with fp64 oracle {agree:.4f}, "
          f"with bf16 oracle {agree_b:.4f}, L1 {hist_l1(g, o64, trials)[0]:.4f}")
    assert agree > 0.9 and agree_b > 0.9
    # aggregate outcome probabilities close to the fp64 oracle
    T = trials
    pg = np.array([g["stats"][0, k] for k in (0, 1, 2)]) / T
    po = np.array([o64["stats"][0, k] for k in (0, 1, 2)]) / T
    assert np.abs(pg - po).max() < 0.05


def test_rnn_full_size_sampled():
    """65,536 runs of the 256-unit network as the benchmark launches it; a
    sample of runs recomputed one by one by the oracle."""
    w = W.rnn()
    g = cm.run(w, dumps=True)
    st = g["stats"][0]
    assert st[0] + st[1] + st[2] == 65536
    rng = np.random.default_rng(0)
    for t in rng.choice(65536, 6, replace=False):
        traj, ch, fl = oracle.trajectory(w, 0, int(t))
        if fl or g["run_flag"][t]:
            continue
        assert g["run_choice"][t] == ch and g["run_step"][t] == traj.shape[0], t
        np.testing.assert_allclose(g["run_state"][t], traj[-1], rtol=1e-9, atol=1e-12)
    # the reduction agrees with the per-run dumps
    from parity import reduce_dumps
    h, s = reduce_dumps(w, g, [-1])
    assert np.array_equal(h, g["hist"]) and np.array_equal(s, g["stats"])


def test_rnn_invariant_to_dumps():
    w = _case(256, 3000, seed=9, precision=W.BF16_PROJ)
    a, b = cm.run(w), cm.run(w, dumps=True)
    assert np.array_equal(a["hist"], b["hist"]) and np.array_equal(a["stats"], b["stats"])


@pytest.mark.parametrize("prec", [W.FP64, W.BF16_PROJ])
def test_rnn_coupled_fixed_point(prec):
    """Two groups of 32 units, coupled within and across groups with
    different strengths each way, no noise, no input: every run settles at
    the fixed point of the continuous dynamics, found by root finding
    (bf16 weights move it by their rounding)."""
    from scipy.optimize import fsolve
    a, b, c_ab, c_ba = 1.0, -0.5, 0.8, -0.6
    nu, h = 64, 32
    Wm = np.zeros((nu, nu))
    Wm[:h, :h] = a / (h - 1)
    Wm[:h, h:] = c_ab / h
    Wm[h:, :h] = c_ba / h
    Wm[h:, h:] = b / (h - 1)
    np.fill_diagonal(Wm, 0.0)
    wts = np.concatenate([Wm.ravel(), np.zeros(2 * nu)])
    w = W.rnn(trials=40, seed=5, n_units=nu, dt=0.05, noise=0.0, thresh=1e300, input_gain=0.0,
              max_steps=1500, n_bins=10, weights=wts, precision=prec)
    g = cm.run(w, dumps=True)

    def s(x):
        return 1.0 / (1.0 + np.exp(-x))

    xa, xb = fsolve(lambda v: [v[0] - a * s(v[0]) - c_ab * s(v[1]),
                               v[1] - c_ba * s(v[0]) - b * s(v[1])], [0.5, -0.5], xtol=1e-14)
    tol = 1e-9 if prec == W.FP64 else 2e-2
    x = g["run_state"][:, 2:]
    assert np.abs(x[:, :h] - xa).max() < tol and np.abs(x[:, h:] - xb).max() < tol
    assert int(g["stats"][0, 2]) == 40  # undecided at the cap


@pytest.mark.parametrize("n_units,gain,trials", [(64, 3e3, 40), (192, 3e4, 40), (256, 1e6, 40), (128, 1e4, 1100)])
def test_rnn_fp64_large_states(n_units, gain, trials):
    """Drives that carry some states past |x| = 80, where the logistic leaves
    its table form, and past 700, in the same wavefronts as small ones."""
    w = _case(n_units, trials, seed=11, gains=np.array([1.0, gain]), max_steps=40, n_bins=10, thresh=1e300)
    g, o = _both(w)
    assert_parity(w, g, o, [-1])
    x = np.abs(g["run_state"][:, 2:])
    assert (x > 700).any() and (x < 1).any()


@pytest.mark.parametrize("n_units,settings,trials,max_steps", [
    (256, 1, 1, 40), (256, 1, 5, 60), (192, 3, 2, 60), (128, 1, 4, 60),  # one group and less
    (256, 1, 1025, 30), (192, 1, 1100, 30), (128, 7, 293, 30),  # a second group in some workgroups, in all
    (64, 1, 1024, 60), (64, 1, 1025, 60), (128, 1, 2048, 30), (128, 1, 2049, 30),  # on both sides of
    (192, 1, 2049, 20), (256, 1, 2048, 20), (256, 1, 2049, 20),  # the rule
])
def test_rnn_fp64_few_runs(n_units, settings, trials, max_steps):
    """Launches of few runs, whose groups of four slots are freed as runs end."""
    w = _case(n_units, trials, seed=21, max_steps=max_steps, n_bins=max_steps // 2, thresh=0.1,
              gains=None if settings == 1 else np.linspace(0.5, 2.0, settings))
    g, o = _both(w)
    assert_parity(w, g, o, [-1])
    b = cm.run(w)  # without dumps
    assert np.array_equal(b["hist"], g["hist"]) and np.array_equal(b["stats"], g["stats"])


@pytest.mark.parametrize("n_units,settings,trials,n_bins", [
    (64, 3, 500, 1200), (256, 5, 3, 1200),  # window too large: counted in global memory
    (64, 700, 2, 40), (128, 30, 41, 40),    # many settings in a window, few
    (256, 1, 8300, 60), (256, 1, 8192, 60), (128, 7, 2400, 60),  # workgroups of 16 and 17 runs
])
@pytest.mark.parametrize("prec", [W.FP64, W.BF16_PROJ])
def test_rnn_counting(n_units, settings, trials, n_bins, prec):
    """Histograms and statistics equal the reduction of the per-run outputs."""
    from parity import reduce_dumps
    w = _case(n_units, trials, seed=31, max_steps=max(n_bins, 60), n_bins=n_bins, thresh=0.2,
              gains=np.linspace(0.5, 2.0, settings), precision=prec)
    g = cm.run(w, dumps=True)
    h, s = reduce_dumps(w, g, [-1] * settings)
    assert np.array_equal(h, g["hist"]) and np.array_equal(s, g["stats"])
    assert int(g["stats"][:, :3].sum()) == settings * trials


@pytest.mark.parametrize("n_units,settings", [(64, 100), (128, 100), (192, 100), (256, 100),  # launches of few runs
                                              (64, 600), (128, 600), (192, 600), (256, 600)])
def test_rnn_fp64_companions(n_units, settings):
    """A run's bits do not depend on the runs beside it: the even settings' states with
    and without odd settings whose units leave the logistic's table form."""
    kw = dict(n_units=n_units, trials=4, seed=41, max_steps=30, n_bins=10, thresh=1e300)
    print(f"rnn companions {n_units} units {settings} settings", flush=True)
    tame = np.linspace(0.5, 1.5, settings)
    wild = tame.copy()
    wild[1::2] = 3e4
    a, b = (cm.run(W.rnn(gains=g, **kw), dumps=True)["run_state"].reshape(settings, 4, -1) for g in (tame, wild))
    assert np.abs(b[1::2, :, 2:]).max() > 700 and np.abs(b[::2, :, 2:]).max() < 80
    assert np.array_equal(a[::2], b[::2])


@pytest.mark.parametrize("n_units,settings,trials,n_bins", [
    (192, 3, 10_923, 60), (256, 17, 2000, 100), (256, 19, 1800, 100),  # 64 runs each and more; the widest window
    (256, 20, 1700, 100), (192, 1000, 33, 40), (256, 33_000, 1, 60),  # in global memory
    (256, 2, 16_400, 60), (192, 3, 10_922, 60), (256, 3, 1, 40),  # consecutive
])
def test_rnn_bf16_dealt_runs(n_units, settings, trials, n_bins):
    """Runs dealt out to the workgroups in turn: every run is there once, counted as its
    own outputs say, and the same whatever other settings it is dealt out with."""
    from parity import reduce_dumps
    gains = np.geomspace(0.02, 30.0, settings)
    kw = dict(n_units=n_units, trials=trials, seed=51, max_steps=max(n_bins, 60), n_bins=n_bins, thresh=0.2,
              precision=W.BF16_PROJ)
    print(f"rnn dealt {n_units} units {settings} x {trials}", flush=True)
    w = W.rnn(gains=gains, **kw)
    g = cm.run(w, dumps=True)
    h, s = reduce_dumps(w, g, [-1] * settings)
    assert np.array_equal(h, g["hist"]) and np.array_equal(s, g["stats"])
    assert int(g["stats"][:, :3].sum()) == settings * trials
    part = cm.run(W.rnn(gains=gains[:2], **kw), dumps=True)
    n = min(settings, 2) * trials
    for k in ("run_choice", "run_step", "run_flag", "run_state"):
        assert np.array_equal(part[k], g[k][:n]), k
