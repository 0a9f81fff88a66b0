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
