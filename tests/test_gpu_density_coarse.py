"""The coarse form of the density propagation (samples of the survivor mass
and powers of their step matrix) against the oracle's cell-by-cell one, at the
edges of its rules: cell counts either side of each, step counts around the
16-step passes, the outputs' buffer and the least number of steps it takes,
early stops on the full grid and inside a pass, and drifts that leave some
settings of a grid to the full-grid form."""
import math

import numpy as np
import pytest

import oracle
from paper_2110_15425_amd import cm, workloads as W

pytestmark = pytest.mark.gpu

# absolute: the propagation's acceptance; relative, where a probability is above
# 10^-9: the samples' absolute rounding, 2^-52, over 10^-9, over the few hundred
# entries of a sum
ATOL, RTOL, FLOOR = 1e-12, 1e-5, 1e-9


def _check(cells, steps, drifts, start=0.0, noise=1.0, dt=0.01, tol=1e-15):
    print(f"{cells} cells, {steps} steps, drifts {drifts}, start {start}, noise {noise}, tol {tol}", flush=True)
    w = W.ddm(drifts=drifts, start=start, noise=noise, dt=dt, max_steps=steps, n_bins=min(steps, 10))
    out = cm.ddm_density(w, cells=cells, tol=tol)
    for s, d in enumerate(drifts):
        lo, up = oracle.ddm_density(d * dt, noise * math.sqrt(dt), 1.0, start=start, cells=cells,
                                    max_steps=steps, tol=tol)
        for got, want in ((out[s, 0], lo), (out[s, 1], up)):
            np.testing.assert_allclose(got, want, rtol=0, atol=ATOL)
            big = want > FLOOR
            np.testing.assert_allclose(got[big], want[big], rtol=RTOL, atol=0)


@pytest.mark.parametrize("cells", [79, 80, 97, 127, 128, 129, 171, 255, 256, 257, 400, 512, 769, 1025, 1300])
def test_cell_counts(cells):
    _check(cells, 320, [0.3, -0.1])


@pytest.mark.parametrize("steps", [191, 192, 199, 200, 201, 215, 216, 217, 4103, 4104, 4105, 4200])
def test_step_counts(steps):
    _check(96, steps, [0.05], tol=0.0)


@pytest.mark.parametrize("tol", [0.9999, 0.97, 0.5, 1e-3])
def test_early_stops(tol):
    _check(160, 400, [0.3, 0.0], tol=tol)


@pytest.mark.parametrize("start", [-0.6, 0.25, 0.93])
def test_starts(start):
    _check(333, 250, [0.2], start=start)


def test_drifts_either_side_of_the_rule():
    # 2 drift theta / noise^2 = 4 at drift 2
    _check(200, 260, [0.0, 1.99, 2.01, -1.99, -2.5, 6.0])


@pytest.mark.parametrize("noise,dt", [(0.4, 0.02), (2.0, 0.01), (2.6, 0.01), (1.0, 0.001)])
def test_kernel_widths(noise, dt):
    _check(500, 300, [0.1], noise=noise, dt=dt)
