"""The device queue hands a request's tables over between workgroups (and
XCDs): with every buffer filled with other values beforehand, no chunk may see
what was there before the preparation."""
import numpy as np
import pytest
import torch

from paper_2110_15425_amd import cm, workloads as W

pytestmark = pytest.mark.gpu


def test_tables_are_seen_by_every_chunk():
    h = cm.Handle(0)
    ws = [W.conflict(trials=300, seed=61, grid=W.control_grid(4), reward=1.0, cost=0.1, precision=W.FP32_STEP),
          W.conflict(trials=2000, seed=62, grid=W.control_grid(8)[::5], precision=W.FP32_STEP)]
    ref = [cm.run(w, handle=h) for w in ws]
    q = cm.DeviceQueue(h, W.LCA, W.FP32_STEP, slots=4, idle_us=20000)
    try:
        for i in range(300):
            ds = [cm.DeviceSweep(h, w) for w in (ws[0], ws[1])]
            for d in ds:
                d.workspace.fill_(0x7F)
                d.hist.fill_(5)
                d.stats.fill_(7)
            left = {q.submit(d) for d in ds}
            while left:
                left -= {t for t in left if q.poll(t)}
            torch.cuda.synchronize()
            for d, r in zip(ds, ref):
                assert np.array_equal(d.stats.cpu().numpy().view(np.uint64), r["stats"]), i
                assert np.array_equal(d.hist.cpu().numpy().view(np.uint64), r["hist"]), i
    finally:
        q.close()
