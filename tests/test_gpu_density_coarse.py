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


def _exact(cells, steps, a, b, th, start):
    """The cell-by-cell propagation in 80 bits: (probabilities [2, steps], mass before each
    step).  Gaussian cell masses by 12-point Gauss quadrature, the absorption as the sum of
    the masses of the cells beyond a bound."""
    f80 = np.longdouble
    x, g = (v.astype(f80) for v in np.polynomial.legendre.leggauss(12))
    for _ in range(3):  # nodes and weights to 80 bits
        p0, p1 = np.ones_like(x), x
        for k in range(2, 13):
            p0, p1 = p1, ((2 * k - 1) * x * p1 - (k - 1) * p0) / k
        d = 12 * (x * p1 - p0) / (x * x - 1)
        x, g = x - p1 / d, 2 / ((1 - x * x) * d * d)
    a, b, h = f80(a), f80(b), 2 * f80(th) / cells
    pi = 4 * np.arctan(f80(1))

    def mass(edge):  # of [edge, edge + h] under the step's normal density
        z = (edge[:, None] + (x[None] + 1) * (h / 2) - a) / b
        return (np.exp(-z * z / 2) * g).sum(1) * (h / 2) / (b * np.sqrt(2 * pi))

    D = cells + int(np.ceil(float(12 * b / h)))
    row = mass((np.arange(-D, D + 1) - f80(0.5)) * h)  # by displacement
    above, below = np.cumsum(row[::-1])[::-1], np.cumsum(row)  # displacements >= d, <= d
    at = np.arange(cells)
    up, lo = above[cells - at + D], below[-1 - at + D]
    band = row[D - cells + 1:D + cells]
    ext = mass((np.arange(-D, cells + D) * h - f80(th)) - f80(start))
    m = ext[D:D + cells]
    out, left = np.zeros((2, steps), f80), np.ones(steps, f80)
    out[0, 0], out[1, 0] = ext[:D].sum(), ext[D + cells:].sum()
    for n in range(1, steps):
        left[n] = m.sum()
        out[0, n], out[1, n] = (m * lo).sum(), (m * up).sum()
        m = np.convolve(m, band)[cells - 1:2 * cells - 1]
    return out, left


# The samples' rounding is relative to the mass that is left: an entry is off by at most
# 16 x 2^-52 of the survivor mass (a sum of 128 terms whose weights add up to a few), and by
# what the mass itself has gathered, below 10^-13 of the entry.  The error's norm: twice
# what either form is from an 80-bit propagation (3.5e-15), and its own rounding again.
def _check_close(cells, steps, drifts, start=0.0, noise=1.0, dt=0.01, tol=1e-15):
    print(f"close: {cells} cells, {steps} steps, drifts {drifts}, start {start}, noise {noise}, tol {tol}", flush=True)
    w = W.ddm(drifts=drifts, start=start, noise=noise, dt=dt, max_steps=steps, n_bins=min(steps, 10))
    out = cm.ddm_density(w, cells=cells, tol=tol)
    assert (out >= 0.0).all()
    for s, d in enumerate(drifts):
        want, left = _exact(cells, steps, d * dt, noise * math.sqrt(dt), 1.0, start)
        if tol > 0.0:  # both forms end once the survivor mass is below tol
            end = int(np.flatnonzero(out[s].sum(0) > 0.0).max()) + 1
            assert end == steps or left[end] < tol * (1.0 + 1e-9), (end, left[end])
            assert end < 3 or left[end - 1] >= tol * (1.0 - 1e-9), (end, left[end - 1])
            assert not out[s][:, end:].any()
            want[:, end:] = 0.0
        err = np.abs(out[s] - want)
        worst = float((err / (16 * 2.0 ** -52 * left + 1e-13 * want + 1e-300)).max())
        norm = float(np.sqrt((err * err).sum() / (want * want).sum()))
        print(f"  drift {d}: worst {worst:.3f} of its bound, norm {norm:.1e}", flush=True)
        assert worst <= 1.0 and norm <= 1e-14


@pytest.mark.parametrize("cells,noise", [(32, 2.5), (33, 2.45), (48, 1.7), (48, 2.5), (64, 1.3), (64, 2.4), (79, 1.1),
                                         (80, 1.0), (127, 2.5), (128, 0.7)])
def test_wide_steps_on_few_cells(cells, noise):
    """Where the step reaches beyond the whole grid: 32 to 128 cells."""
    _check_close(cells, 260, [0.0, 0.3, -1.0], noise=noise)


@pytest.mark.parametrize("cells,steps,noise,start", [(96, 900, 1.0, 0.0), (171, 900, 1.0, 0.4), (333, 400, 2.0, -0.7),
                                                     (512, 400, 1.0, 0.9), (1000, 300, 1.0, 0.0), (1300, 250, 1.0, 0.2)])
def test_error_against_the_mass_left(cells, steps, noise, start):
    edge = 1.99 * noise * noise  # the rule's largest drift
    _check_close(cells, steps, [0.1, edge, -edge], noise=noise, start=start)


@pytest.mark.parametrize("cells", [96, 171])
@pytest.mark.parametrize("tol", [0.2, 0.05, 1e-2, 1e-3, 1e-6])
def test_stops_inside_a_pass(cells, tol):
    _check_close(cells, 1600, [0.0, 0.37, -0.9], tol=tol)


@pytest.mark.parametrize("cells", [171, 333, 1000])
def test_no_entry_is_negative(cells):
    """Down to masses that are denormal and beyond."""
    print(f"{cells} cells, 30000 steps, tol 0", flush=True)
    out = cm.ddm_density(W.ddm(drifts=[1.99, -1.99], max_steps=30_000, n_bins=10), cells=cells, tol=0.0)
    assert (out >= 0.0).all() and out[:, :, 23_000].any() and not out[:, :, 29_000].any()
