"""The drift-diffusion form with one wavefront per run, 128 steps at a time: per-run
outcomes equal the node-by-node execution's, over step caps at the edges of its
blocks, starts off the centre and flag distances from the default to wider than
the threshold (where no block can be skipped).  States are sums of at most 400
increments below 1 in another order: 400 x 2^-53 x 4 apart at most."""
import numpy as np
import pytest

from paper_2110_15425_amd import cm, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_STEP])
@pytest.mark.parametrize("max_steps", [1, 2, 127, 128, 129, 256, 257, 400])
@pytest.mark.parametrize("flag_eps", [0.0, 1e-10, 0.3, 1.5])
def test_ddm_scan(prec, max_steps, flag_eps):
    h = cm.Handle(0)
    for settings, trials, start in ((1, 1, 0.0), (3, 41, -0.4), (1, 4001, 0.2)):
        print(f"scan {prec} {settings} x {trials} cap {max_steps} eps {flag_eps}", flush=True)
        w = W.ddm(trials=trials, seed=9, drifts=np.linspace(-0.5, 0.5, settings), start=start,
                  max_steps=max_steps, n_bins=min(100, max_steps), precision=prec, flag_eps=flag_eps)
        ds = cm.DeviceSweep(h, w, dumps=True)
        ds.launch()
        got = ds.results()
        ds.launch_unfused()
        want = ds.results()
        for k in ("run_choice", "run_step", "run_flag", "hist", "stats"):
            assert np.array_equal(got[k], want[k]), k
        np.testing.assert_allclose(got["run_state"], want["run_state"], rtol=0, atol=400 * 4 * 2.0 ** -53)


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_STEP])
def test_ddm_scan_with_four_wavefronts(prec):
    """Launches of more than 2^17 runs, whose workgroups have four wavefronts."""
    h = cm.Handle(0)
    runs = (1 << 17) + 1
    print(f"scan {prec} 1 x {runs}", flush=True)
    w = W.ddm(trials=runs, seed=10, max_steps=400, precision=prec)
    ds = cm.DeviceSweep(h, w, dumps=True)
    ds.launch()
    got = ds.results()
    ds.launch_unfused()
    want = ds.results()
    for k in ("run_choice", "run_step", "run_flag", "hist", "stats"):
        assert np.array_equal(got[k], want[k]), k
    np.testing.assert_allclose(got["run_state"], want["run_state"], rtol=0, atol=400 * 4 * 2.0 ** -53)


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_STEP])
def test_form_either_side_of_its_limit(prec):
    """At 2^18 runs a sweep takes the scan's form, one run more takes lanes, alone and in a
    batch beside each other: bit for bit what the form gives when it is named."""
    kw = dict(max_steps=150, n_bins=10, precision=prec)
    small, big = W.ddm(trials=1 << 18, seed=3, **kw), W.ddm(trials=(1 << 18) + 1, seed=4, **kw)
    keys = ("run_state", "run_choice", "run_step", "run_flag", "hist", "stats")
    h = cm.Handle(0)
    print(f"limit {prec}", flush=True)
    ds = [cm.DeviceSweep(h, w, dumps=True) for w in (small, big)]
    cm.launch_batch(h, ds)
    for w, d, lanes in ((small, ds[0], 64), (big, ds[1], 1)):
        named = cm.Handle(0)
        named.set_tuning(W.DDM, prec, lanes_per_run=lanes)
        want, other = cm.run(w, dumps=True, handle=named), cm.run(w, dumps=True, handle=h)
        got = d.results()
        for k in keys:
            assert np.array_equal(got[k], want[k]) and np.array_equal(other[k], want[k]), (lanes, k)
