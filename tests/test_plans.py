"""Launch plans of the lane kernels, on the host: what the rules send a sweep to."""
import os
import shutil
import subprocess

import pytest

from paper_2110_15425_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LIB = os.path.join(ROOT, "paper_2110_15425_amd", "libcm.so")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-ffp-contract=off", "-w",
                    "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "helpers", "plan_check.hip"),
                    "-L", os.path.dirname(LIB), "-lcm", "-Wl,-rpath," + os.path.dirname(LIB), "-o", exe],
                   check=True, capture_output=True)

    def run(where, kind, prec, settings, trials, max_steps=1000, n_bins=100, every=0):
        r = subprocess.run([exe, where] + [str(v) for v in (kind, prec, settings, trials, max_steps, n_bins, every)],
                           capture_output=True, text=True, check=True)
        return dict(zip(("chunk", "groups", "team", "direct", "scan"), map(int, r.stdout.split())))

    return run


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_STEP])
@pytest.mark.parametrize("settings,trials", [(1, 1), (37, 27), (32, 500), (64, 1000), (1, 50_000), (2000, 100),
                                             (64, 10_000), (64, 200_000)])
def test_queue_chunks(plan, settings, trials, prec):
    """A request of the device queue: few chunks, since each costs a claim, a descriptor
    copy and a write-back of the L2, and none beyond what a large launch takes."""
    runs = settings * trials
    p = plan("queue", W.LCA, prec, settings, trials)
    assert p["chunk"] * p["groups"] >= runs > p["chunk"] * (p["groups"] - 1)
    assert 4 <= p["chunk"] <= 8 * 256 and p["team"] == 256
    assert p["groups"] <= max(128, -(-runs // 512))


@pytest.mark.parametrize("kind,prec", [(W.DDM, W.FP64), (W.LCA, W.FP64), (W.LCA, W.FP32_STEP)])
@pytest.mark.parametrize("settings,trials,wide", [(1, 1000, False), (1, 65_536, False), (1, 65_537, True), (1, 400_000, True),
                                                  (4, 5000, False), (4, 5001, True), (47, 512, False), (47, 513, True),
                                                  (2000, 32, False), (2000, 200, True)])
def test_sampled_in_global_memory(plan, settings, trials, wide, kind, prec):
    """A time course whose window does not fit: two runs per lane where many runs share a
    setting's words, else the chunks of a launch."""
    p = plan("launch", kind, prec, settings, trials, every=1)
    assert p["direct"] == 1 and not p["scan"]
    assert (p["chunk"] >= 512) == wide, p


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_STEP])
@pytest.mark.parametrize("settings,trials,scan", [(1, 1, True), (1, 1 << 18, True), (1, (1 << 18) + 1, False),
                                                  (64, 4096, True), (64, 4097, False)])
def test_ddm_forms(plan, settings, trials, scan, prec):
    assert plan("launch", W.DDM, prec, settings, trials)["scan"] == scan


@pytest.mark.parametrize("every", [0, 10])
@pytest.mark.parametrize("kind,prec,runs,per_lane", [
    (W.LCA, W.FP64, 640_000, 2), (W.LCA, W.FP64, 655_361, 2), (W.LCA, W.FP64, 1_310_720, 2), (W.LCA, W.FP64, 1_310_721, 3),
    (W.LCA, W.FP32_STEP, 458_753, 2), (W.LCA, W.FP32_STEP, 1_000_000, 2), (W.LCA, W.FP32_STEP, 1_835_008, 2),
    (W.LCA, W.FP32_STEP, 1_835_009, 3), (W.DDM, W.FP64, 1_000_000, 3), (W.DDM, W.FP32_STEP, 1_000_000, 3)])
def test_runs_per_lane(plan, kind, prec, runs, per_lane, every):
    """Conflict networks stay at two runs per lane while the GPU would hold up to four."""
    p = plan("launch", kind, prec, 1, runs, every=every)
    assert not p["scan"] and not p["direct"] and p["chunk"] == 256 * per_lane


@pytest.mark.parametrize("prec", [W.FP64, W.FP32_STEP])
@pytest.mark.parametrize("settings,trials,chunk", [(1, 1000, 8), (1, 5000, 16), (1, 10_000, 24), (1, 20_000, 32),
                                                   (1, 30_000, 32), (1, 32_768, 32), (10, 1000, 16), (10, 2000, 24)])
def test_scan_chunks(plan, settings, trials, chunk, prec):
    """Runs of a scan workgroup of eight wavefronts: five to four times sqrt(runs / 600)."""
    p = plan("launch", W.DDM, prec, settings, trials)
    assert p["scan"] and p["chunk"] == chunk


@pytest.mark.parametrize("units,prec,settings,trials,dealt", [
    (256, W.BF16_PROJ, 16, 4096, True), (192, W.BF16_PROJ, 3, 10_923, True), (192, W.BF16_PROJ, 3, 10_922, False),
    (256, W.BF16_PROJ, 1, 65_536, False), (256, W.BF16_PROJ, 2, 32_768, False), (256, W.BF16_PROJ, 3, 1, False),
    (128, W.BF16_PROJ, 16, 4096, False), (64, W.BF16_PROJ, 16, 4096, False), (256, W.FP64, 16, 4096, False)])
def test_rate_networks_that_deal_runs_out(plan, units, prec, settings, trials, dealt):
    """Where all workgroups are resident at once, two on a CU, and settings may differ in length."""
    assert plan("rnn", units, prec, settings, trials)["scan"] == dealt
