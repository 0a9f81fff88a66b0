"""The work a user of this library has it do, as timed cases.

Every case is one pass through a public entry point (``DeviceSweep.launch``,
``launch_timecourse``, ``launch_batch`` or ``ddm_density``) on buffers the
caller keeps between passes, as a parameter study or a server does: the sweep
is described and uploaded once and launched again and again.  ``prepare``
draws the noise seed (and, for the density, the drifts) from its seed.

The ranges are those of the library's own workloads: sweeps of 10^3 to 10^7
runs over 1 to 4,096 settings, rate networks of 64 to 256 units with up to
65,536 runs, closed loops of up to 100 control levels and densities of up to
64 settings.
"""
import math

import numpy as np
import torch

from paper_2110_15425_amd import cm, workloads as W

PRECISION = {"fp64": W.FP64, "fp32": W.FP32_STEP, "bf16": W.BF16_PROJ}


def listed():
    return [
        # one setting of the drift-diffusion model with per-run outcomes, as a
        # fit of response-time data reads them
        dict(name="ddm_10k_dumps_fp64", kind="ddm", precision="fp64", settings=1, trials=10_000,
             max_steps=3000, dumps=True),
        # a drift sweep at the top of the served range (10^6 runs), ragged sizes
        dict(name="ddm_61x16393_fp32", kind="ddm", precision="fp32", settings=61, trials=16_393,
             max_steps=3000, dumps=False),
        # a whole outcome distribution of one setting: 10^7 runs
        dict(name="ddm_10m_fp64", kind="ddm", precision="fp64", settings=1, trials=10_000_000,
             max_steps=3000, dumps=False),
        # the smallest request a server sees, about 10^3 runs: latency and launches
        dict(name="conflict_37x27_fp64", kind="conflict", precision="fp64", settings=37, trials=27,
             max_steps=1000, batch=1),
        # the conflict network's reference sweep in the default precision
        dict(name="conflict_64x10k_fp64", kind="conflict", precision="fp64", settings=64,
             trials=10_000, max_steps=1000, batch=1),
        # the benchmark's step: twelve replicate sweeps in one batched launch
        dict(name="conflict_12x64x10k_fp32", kind="conflict", precision="fp32", settings=64,
             trials=10_000, max_steps=1000, batch=12),
        # exhaustive grid search over the 64 x 64 control allocations
        dict(name="grid_4096x100_fp32", kind="conflict", precision="fp32", settings=4096,
             trials=100, max_steps=1000, batch=1),
        # dynamics over time beside the outcomes
        dict(name="timecourse_64x10k_fp32", kind="timecourse", precision="fp32", settings=64,
             trials=10_000, max_steps=1000, every=10),
        # the recurrent rate network on the matrix cores, reference size
        dict(name="rnn_256x65536_bf16", kind="rnn", precision="bf16", units=256, settings=1,
             trials=65_536, max_steps=200, dumps=False),
        # the same network in double precision, final states kept
        dict(name="rnn_256x8192_dumps_fp64", kind="rnn", precision="fp64", units=256, settings=1,
             trials=8192, max_steps=200, dumps=True),
        # closed-loop control: 64 allocations, 4 look-ahead samples each, four cost weights
        dict(name="loop_l8_m4_4x20k_fp32", kind="loop", precision="fp32", settings=4,
             trials=20_000, levels=8, samples=4, max_steps=1000),
        # exact first-passage distributions of a drift sweep
        dict(name="density_64x1000", kind="density", settings=64, cells=1000, max_steps=3000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ddm", "ddm", "conflict", "conflict", "conflict", "timecourse", "rnn", "loop",
                       "density"])
    prec = rng.choice(["fp64", "fp32"])
    if kind in ("ddm", "conflict", "timecourse"):
        settings = _log_int(rng, 1, 4096)
        if kind == "ddm":
            runs = _log_int(rng, 1_000, 8_000_000)
        else:
            runs = _log_int(rng, 1_000, 2_000_000)
        trials = max(1, runs // settings)
        if kind == "ddm":
            return dict(kind=kind, precision=prec, settings=settings, trials=trials,
                        max_steps=rng.choice([1000, 1501, 3000]),
                        dumps=runs <= 100_000 and rng.random() < 0.5)
        if kind == "conflict":
            return dict(kind=kind, precision=prec, settings=settings, trials=trials,
                        max_steps=rng.choice([400, 999, 1000]), batch=rng.choice([1, 1, 2, 3, 5]))
        settings = min(settings, 256)
        return dict(kind=kind, precision=prec, settings=settings,
                    trials=max(1, min(runs, 800_000) // settings), max_steps=1000,
                    every=rng.choice([5, 10, 25, 50]))
    if kind == "rnn":
        prec = rng.choice(["fp64", "bf16"])
        units = rng.choice([64, 128, 192, 256])
        settings = rng.choice([1, 1, 3, 16])
        runs = _log_int(rng, 500, 8192 if prec == "fp64" else 65_536)
        return dict(kind=kind, precision=prec, units=units, settings=settings,
                    trials=max(1, runs // settings), max_steps=rng.randint(60, 200),
                    dumps=rng.random() < 0.3)
    if kind == "loop":
        levels = _log_int(rng, 2, 100)
        samples = rng.choice([1, 2, 3, 4, 8])
        settings = rng.choice([1, 4])
        most = 20_000_000 // (levels * levels * samples)
        trials = max(16, min(_log_int(rng, 250, 80_000), most) // settings)
        return dict(kind=kind, precision=prec, settings=settings, trials=trials, levels=levels,
                    samples=samples, max_steps=1000)
    return dict(kind="density", settings=_log_int(rng, 1, 64), cells=rng.randint(120, 1000),
                max_steps=_log_int(rng, 300, 3000))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _conflict_grid(n):
    """n control settings: one level of c_B for up to 256 settings, else the
    first n rows of the smallest square grid that holds them."""
    if n == 1:
        return np.array([[2.5, 1.0]])
    if n <= 256:
        lv = W.control_levels(n)
        return np.stack([lv, np.ones_like(lv)], 1)
    return W.control_grid(math.isqrt(n - 1) + 1)[:n]


def _workload(case, seed, replicate=0):
    k = case["kind"]
    noise_seed = 1000 * seed + replicate + 1
    if k == "density":
        top = 0.25 + 0.1 * float(np.random.default_rng(seed).uniform())
        n = case["settings"]
        return W.ddm(drifts=[top * (i + 1) / n for i in range(n)], max_steps=case["max_steps"])
    common = dict(precision=PRECISION[case["precision"]], trials=case["trials"], seed=noise_seed,
                  max_steps=case["max_steps"])
    if k == "ddm":
        n = case["settings"]
        return W.ddm(drifts=None if n == 1 else np.linspace(0.0, 0.6, n), **common)
    if k == "conflict":
        return W.conflict(grid=_conflict_grid(case["settings"]), reward=1.0, cost=0.1, **common)
    if k == "timecourse":
        return W.conflict(grid=_conflict_grid(case["settings"]), **common)
    if k == "rnn":
        n = case["settings"]
        return W.rnn(n_units=case["units"], gains=None if n == 1 else np.linspace(0.5, 1.5, n),
                     n_bins=min(100, case["max_steps"]), **common)
    n = case["settings"]
    return W.control_loop(levels=case["levels"], samples=case["samples"],
                          costs=None if n == 1 else [0.0, 0.003, 0.01, 0.03][:n], **common)


def prepare(case, seed):
    n = case.get("batch", 1)
    ws = [_workload(case, seed, r) for r in range(n)]
    if case["kind"] == "density":
        return case, ws, None
    h = cm.default_handle()
    return case, ws, [cm.DeviceSweep(h, w, dumps=case.get("dumps", False)) for w in ws]


def _outputs(ds):
    out = dict(hist=ds.hist, stats=ds.stats)
    if ds.score is not None:
        out.update(score=ds.score, best=ds.best)
    if ds.dumps:
        out.update(run_choice=ds.run_choice, run_step=ds.run_step, run_flag=ds.run_flag,
                   run_state=ds.run_state)
    return out


def run(state):
    case, ws, sweeps = state
    if case["kind"] == "density":
        return cm.ddm_density(ws[0], cells=case["cells"])
    if case["kind"] == "timecourse":
        sweeps[0].launch_timecourse(case["every"])
        return dict(_outputs(sweeps[0]), timecourse=sweeps[0].timecourse)
    if len(sweeps) == 1:
        sweeps[0].launch()
    else:
        cm.launch_batch(sweeps[0].handle, sweeps)
    return [_outputs(d) for d in sweeps]


# ---------------------------------------------------------------------------
# Work: each input read once and each output written once, and the arithmetic
# of the executed steps (mean decision steps of these workloads).
# ---------------------------------------------------------------------------

PHILOX_OPS = 60   # ten rounds of two products and four exclusive ors
NORMAL_OPS = 20   # a Box-Muller pair


def _ddm_steps(case, drift):
    v = max(drift, 1e-6)
    return min(case["max_steps"], 1.12 * math.tanh(v) / v / 0.01)


def work(case):
    k = case["kind"]
    S = case["settings"]
    if k == "density":
        w = _workload(case, 1)
        cells, p = case["cells"], w["params"]
        h = 2.0 * p[3] / cells
        b = p[2] * math.sqrt(p[0])
        band = min(2 * cells - 1, 2 * 8.5 * b / h)  # displacements that carry mass
        per_step = 2.0 * cells * min(band, cells) + 6.0 * cells
        return dict(bytes=8.0 * S + 16.0 * S * case["max_steps"], flops=S * case["max_steps"] * per_step)
    T, B = case["trials"], min(100, case["max_steps"])
    n = case.get("batch", 1)
    runs = float(S) * T * n
    out = n * S * (2 * B + 9) * 8.0
    if k == "ddm":
        drifts = [0.3] if S == 1 else np.linspace(0.0, 0.6, min(S, 64))
        steps = float(np.mean([_ddm_steps(case, float(d)) for d in drifts]))
        byt = out + 8.0 * S + (runs * 14 if case["dumps"] else 0)
        return dict(bytes=byt, flops=runs * steps * ((PHILOX_OPS + NORMAL_OPS) / 2 + 6))
    if k in ("conflict", "timecourse"):
        byt = out + n * (S * 24.0 + 320)
        if k == "timecourse":
            byt += S * (case["max_steps"] // case["every"]) * 48.0
        return dict(bytes=byt, flops=runs * 52 * (PHILOX_OPS + NORMAL_OPS + 18))
    if k == "rnn":
        u = case["units"]
        byt = out + 8.0 * (u * u + 2 * u) + (runs * (6 + 8 * (u + 2)) if case["dumps"] else 0)
        per = 2.0 * u * u + u * ((PHILOX_OPS + NORMAL_OPS) / 2 + 14)
        return dict(bytes=byt, flops=runs * 0.9 * case["max_steps"] * per)
    looks = case["levels"] ** 2 * case["samples"]
    return dict(bytes=out + 8.0 * S + 320, flops=runs * 23 * looks * (PHILOX_OPS + NORMAL_OPS + 20))


# ---------------------------------------------------------------------------
# The same results in plain 64-bit torch.
# ---------------------------------------------------------------------------

MASK = 0xFFFFFFFF
M0, M1, KW0, KW1 = 0xD2511F53, 0xCD9E8D57, 0x9E3779B9, 0xBB67AE85


def _mul(c, x):
    """High and low words of a 32 x 32 bit product (int64 tensors)."""
    p1, p0 = c * (x >> 16), c * (x & 0xFFFF)
    low = p0 + ((p1 & 0xFFFF) << 16)
    return (p1 >> 16) + (low >> 32), low & MASK


def _philox(c, seed):
    """Philox4x32-10 (Salmon et al., SC'11) of four int64 counter tensors."""
    k0, k1 = seed & MASK, (seed >> 32) & MASK
    c0, c1, c2, c3 = c
    for _ in range(10):
        h0, l0 = _mul(M0, c0)
        h1, l1 = _mul(M1, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + KW0) & MASK, (k1 + KW1) & MASK
    return c0, c1, c2, c3


def _normals(c, seed, fp32=False):
    """Box-Muller pair in double; fp32: from the top 24 bits of two words, as
    the FP32-steps mode draws them."""
    w0, w1, w2, w3 = _philox(c, seed)
    if fp32:
        ua, ub = ((w1 >> 8) + 1).double() * 2.0 ** -24, ((w3 >> 8) + 1).double() * 2.0 ** -24
    else:
        ua = (((w1 << 21) | (w0 >> 11)) + 1).double() * 2.0 ** -53
        ub = (((w3 << 21) | (w2 >> 11)) + 1).double() * 2.0 ** -53
    rho = torch.sqrt(-2.0 * torch.log(ua))
    ang = 2.0 * math.pi * ub
    return rho * torch.cos(ang), rho * torch.sin(ang)


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _counters(w, dev):
    S, T = w["n_settings"], w["trials"]
    r = torch.arange(S * T, device=dev)
    return r // T, r % T


def _ddm_states(w):
    dev, p = _device(), w["params"]
    fp32 = w["precision"] == W.FP32_STEP
    s, t = _counters(w, dev)
    grid = np.full(w["n_settings"], p[1]) if w["grid"] is None else w["grid"][:, 0]
    a = torch.as_tensor(grid, device=dev)[s] * p[0]
    b, th = p[2] * math.sqrt(p[0]), p[3]
    x = torch.full(s.shape, float(p[4]), dtype=torch.float64, device=dev)
    live = torch.arange(s.numel(), device=dev)
    for n in range(w["max_steps"]):
        if n % 2 == 0:
            zero = torch.zeros_like(live)
            z = _normals((zero + n // 2, t[live], s[live], zero), w["seed"], fp32)
        x[live] = (x[live] + a[live]) + b * z[n % 2]
        if n % 2:
            live = live[x[live].abs() < th]
            if not live.numel():
                break
        else:  # a run that ended on the first step of a pair keeps its state
            on = x[live].abs() < th
            z = (z[0][on], z[1][on])
            live = live[on]
    return x.reshape(-1, 1)


def _conflict_score(w):
    dev, p = _device(), w["params"]
    fp32 = w["precision"] == W.FP32_STEP
    wt = w["weights"]
    WA, WB, OA, OB = wt[:12].reshape(4, 3), wt[12:24].reshape(4, 3), wt[24:32].reshape(2, 4), wt[32:].reshape(2, 4)
    gain, bias = p[6], p[7]
    logistic = lambda v: 1.0 / (1.0 + np.exp(-v))  # noqa: E731
    stim = np.arange(9)
    cA, cB = w["grid"][:, 0], w["grid"][:, 1]
    hA = logistic((cA[:, None, None] * gain) * (WA[None] + bias))
    hB = logistic((cB[:, None, None] * gain) * (WB[None] + bias))
    drive = (np.einsum("jk,skc->scj", OA, hA)[:, stim // 3] + np.einsum("jk,skc->scj", OB, hB)[:, stim % 3]) + p[5]
    unit = np.einsum("jk,kc->cj", OA, logistic(gain * (WA + bias)))[stim // 3]
    correct = torch.as_tensor((unit[:, 1] > unit[:, 0]).astype(np.int64), device=dev)
    s, t = _counters(w, dev)
    inp = torch.as_tensor(drive, device=dev)[s, t % 9]
    target = correct[t % 9]
    hits = torch.zeros(w["n_settings"], dtype=torch.float64, device=dev)
    dt, leak, comp, b, th = p[0], p[1], p[2], p[3] * math.sqrt(p[0]), p[4]
    x0 = torch.zeros(s.shape, dtype=torch.float64, device=dev)
    x1 = x0.clone()
    for n in range(w["max_steps"]):
        z0, z1 = _normals((torch.full_like(s, n), t, s, torch.zeros_like(s)), w["seed"], fp32)
        x0, x1 = (x0 + ((inp[:, 0] - leak * x0) - comp * x1) * dt + b * z0,
                  x1 + ((inp[:, 1] - leak * x1) - comp * x0) * dt + b * z1)
        done = torch.maximum(x0, x1) >= th
        if bool(done.any()):
            right = done & ((x1 > x0).long() == target)
            hits += torch.bincount(s[right], minlength=w["n_settings"]).double()
            on = ~done
            s, t, inp, target, x0, x1 = s[on], t[on], inp[on], target[on], x0[on], x1[on]
            if not s.numel():
                break
    pen = torch.as_tensor(cA * cA + cB * cB, device=dev)
    return w["reward"] * (hits / w["trials"]) - w["cost"] * pen


def _rnn_states(w):
    dev, p, n = _device(), w["params"], w["n_units"]
    Wm = torch.as_tensor(w["weights"][:n * n].reshape(n, n), device=dev)
    R = torch.as_tensor(w["weights"][n * n:].reshape(2, n), device=dev)
    dt, b, th = p[0], p[1] * math.sqrt(p[0]), p[2]
    s, t = _counters(w, dev)
    gain = np.full(w["n_settings"], p[3]) if w["grid"] is None else w["grid"][:, 0]
    pair = torch.arange(n // 2, device=dev)

    def draws(step, stream):
        shape = (s.numel(), n // 2)
        at = [t[:, None].expand(shape), s[:, None].expand(shape)]
        m = pair[None].expand(shape)
        c = (m, *at, torch.full(shape, stream, device=dev)) if stream else (torch.full(shape, step, device=dev), *at, m)
        return torch.stack(_normals(c, w["seed"]), 2).reshape(s.numel(), n)

    out = torch.zeros((s.numel(), 2 + n), dtype=torch.float64, device=dev)
    u = torch.as_tensor(gain, device=dev)[s][:, None] * draws(0, 0x40000000)
    run = torch.arange(s.numel(), device=dev)
    x = torch.zeros((s.numel(), n), dtype=torch.float64, device=dev)
    y = torch.zeros((s.numel(), 2), dtype=torch.float64, device=dev)
    for step in range(w["max_steps"]):
        r = torch.sigmoid(x)
        y = y + dt * ((r - 0.5) @ R.T.contiguous())
        x = (x + dt * ((r @ Wm.T.contiguous() - x) + u)) + b * draws(step, 0)
        done = y.max(1).values >= th
        if step == w["max_steps"] - 1:
            done = torch.ones_like(done)
        if bool(done.any()):
            out[run[done]] = torch.cat([y[done], x[done]], 1)
            on = ~done
            s, t, u, run, x, y = s[on], t[on], u[on], run[on], x[on], y[on]
    return out


def _density(w, cells):
    dev, p = _device(), w["params"]
    dt, b, th, start = p[0], p[2] * math.sqrt(p[0]), p[3], p[4]
    a = torch.as_tensor(w["grid"][:, 0] * dt, device=dev)[:, None]
    h = 2.0 * th / cells
    phi = lambda v: 0.5 * torch.special.erfc(-v / math.sqrt(2.0))  # noqa: E731
    j = torch.arange(cells, device=dev, dtype=torch.float64)[None]
    centre = -th + (j + 0.5) * h
    up, lo = phi(-((th - centre) - a) / b), phi(((-th - centre) - a) / b)
    d = torch.arange(-(cells - 1), cells, device=dev, dtype=torch.float64)[None]
    row = phi(((d + 0.5) * h - a) / b) - phi(((d - 0.5) * h - a) / b)
    at = torch.arange(cells, device=dev)
    T = row[:, (at[:, None] - at[None] + cells - 1)]  # [settings, to, from]
    out = torch.zeros((a.shape[0], 2, w["max_steps"]), dtype=torch.float64, device=dev)
    out[:, 1, 0] = phi(-((th - start) - a[:, 0]) / b)
    out[:, 0, 0] = phi(((-th - start) - a[:, 0]) / b)
    m = phi(((-th + (j + 1) * h - start) - a) / b) - phi(((-th + j * h - start) - a) / b)
    for n in range(1, w["max_steps"]):
        out[:, 1, n] = (m * up).sum(1)
        out[:, 0, n] = (m * lo).sum(1)
        m = torch.bmm(T, m[:, :, None])[:, :, 0]
        m = torch.where(m.sum(1, keepdim=True) < 1e-15, 0.0, m)
    return out.cpu().numpy()


def exact(case, seed):
    k = case["kind"]
    ws = [_workload(case, seed, r) for r in range(case.get("batch", 1))]
    if k == "density":
        return _density(ws[0], case["cells"])
    none = dict(hist=None, stats=None)
    dumps = dict(none, run_choice=None, run_step=None, run_flag=None)
    if k == "conflict":
        return [dict(none, score=_conflict_score(w), best=None) for w in ws]
    if k == "ddm" and case["dumps"]:
        return [dict(dumps, run_state=_ddm_states(ws[0]))]
    if k == "rnn" and case["dumps"] and case["precision"] == "fp64":
        return [dict(dumps, run_state=_rnn_states(ws[0]))]
    return None  # whole numbers only, or the rounding of bf16 products
