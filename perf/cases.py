"""The work a user of this framework has it do, as cases that can be timed one by one.

Each case goes through the package's public classes (``binding.Detector``, ``StreamSet``,
``Trainer``, ``ConfigScanner``) on synthetic monitoring series of the kinds and shapes that
``workloads`` defines: z-scored windows of W steps x M metrics of many LLM services, a detector of
H hidden and L latent units, reference prefix = first half of a stream.

``prepare`` draws the series on the GPU from the seed alone and builds the handles; ``run`` is one
call (or the one sequence of calls) a program makes; ``exact`` is the same result in 64 bits from
plain torch. All AR(1) series have coefficient 0.8 (``workloads.PHI``).
"""
import math

import numpy as np
import torch

from paper_2407_09486_amd import binding
from paper_2407_09486_amd import workloads as wl

DEV = "cuda"


# ----------------------------------------------------------------------------- the cases
def listed():
    f32 = dict(latent=16, dtype="f32", act="relu")
    return [
        # an operator looks at one service: a whole detection (statistics, scores, threshold, flags)
        # of 2048 steps x 8 metrics; all launches and round trips
        dict(name="detect_one_service", kind="detect", streams=1, t_min=2048, t_max=2048, metrics=8, window=32,
             stride=1, hidden=32, **f32),
        # the seven metrics of the paper's Table II, one-hour windows of one-minute steps, services
        # deployed at different times (ragged lengths): an odd metric count that no 16-byte row fits
        dict(name="score_seven_metrics", kind="score", streams=96, t_min=1441, t_max=20161, metrics=7, window=60,
             stride=1, hidden=64, latent=16, dtype="f32", act="tanh"),
        # an ordinary batch: 64 services of eleven days of minutes
        dict(name="score_services", kind="score", streams=64, t_min=16384, t_max=16384, metrics=8, window=64,
             stride=1, hidden=64, **f32),
        # a large fleet of ragged streams (an eighth of the benchmark's default workload)
        dict(name="score_ragged_fleet", kind="score", streams=512, t_min=512, t_max=65536, metrics=16, window=64,
             stride=1, hidden=128, **f32),
        # the bf16 detector: long strided windows of 32 metrics (a sixteenth of the bf16 workload)
        dict(name="score_bf16", kind="score", streams=1024, t_min=4096, t_max=4096, metrics=32, window=256,
             stride=8, hidden=256, latent=16, dtype="bf16", act="relu"),
        # the threshold refit over a batch's scores and the flags of every window
        dict(name="threshold", kind="threshold", streams=64, t_min=16384, t_max=16384, window=64),
        # one live step of 4096 streams: append, score, thresholds (the streaming benchmark)
        dict(name="stream_push", kind="stream", streams=4096, metrics=16, window=64, stride=1, hidden=128, **f32),
        # training: four minibatches of an epoch at the training benchmark's shape, then the weights
        dict(name="train_large_batches", kind="train", batch=8192, batches=4, metrics=16, window=64, hidden=128,
             latent=16, act="relu"),
        # training a per-service detector on its own few windows: small minibatches, launch-bound
        dict(name="train_small_batches", kind="train", batch=500, batches=8, metrics=7, window=60, hidden=64,
             latent=16, act="tanh"),
        # the configuration scan of a fleet (every window's fits and each service's recommendation)
        dict(name="config_scan", kind="config", streams=1024, t_len=16384, window=64, stride=1, dtype="f32"),
        # every output variant (per-metric direction, reconstruction error), per-window normalisation
        dict(name="variants_window_norm", kind="variants", streams=64, t_min=512, t_max=65536, metrics=16, window=64,
             stride=1, hidden=128, norm="window", **f32),
        # the same outputs for the seven Table II metrics, normalised against the reference prefix
        dict(name="variants_seven_metrics", kind="variants", streams=32, t_min=1441, t_max=20161, metrics=7,
             window=60, stride=1, hidden=64, latent=16, dtype="f32", act="tanh", norm="reference"),
    ]


# The largest listed pass, as the product of windows and first-layer multiply-adds (score_ragged_fleet).
_MOST_MACS = 512 * 33000 * 1024 * 128


def _log(rng, lo, hi):
    """A whole number of [lo, hi], even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: any of the calls above, over the range of sizes that its kind stands for."""
    kind = rng.choice(["detect", "score", "score", "score", "threshold", "stream", "train", "config", "variants",
                       "variants"])
    if kind == "threshold":
        t = _log(rng, 2000, 60000)
        return dict(kind=kind, streams=_log(rng, 4, max(4, min(1024, 8_000_000 // t))), t_min=t // 2, t_max=t,
                    window=rng.randint(16, 128))
    if kind == "config":
        t = _log(rng, 512, 16384)
        return dict(kind=kind, streams=_log(rng, 1, 1024), t_len=t, window=_log(rng, 16, 240),
                    stride=rng.choice([1, 1, 2, 5]), dtype=rng.choice(["f32", "f32", "bf16"]))
    metrics = rng.choice([4, 5, 7, 7, 8, 8, 12, 16, 16, 32])
    window = _log(rng, 16, 256 if metrics <= 16 else 128)
    hidden = rng.choice([24, 32, 64, 64, 100, 128, 128, 200, 256])
    latent = rng.choice([8, 16, 16])
    act = rng.choice(["relu", "relu", "tanh"])
    if kind == "train":
        batch = _log(rng, 128, 8192)
        return dict(kind=kind, batch=batch, batches=rng.randint(2, 8) if batch < 2048 else 2, metrics=metrics,
                    window=min(window, 1024 // metrics), hidden=min(hidden, 128), latent=latent, act=act)
    dtype = rng.choice(["f32", "f32", "bf16"])
    if kind == "stream":
        return dict(kind=kind, streams=_log(rng, 16, 6000), metrics=metrics, window=min(window, 128), stride=1,
                    hidden=hidden, latent=latent, dtype=dtype, act=act)
    stride = rng.choice([1, 1, 1, 2, 4, 8]) if window >= 32 else 1
    t_max = _log(rng, 1000, 40000)
    macs = (t_max * 0.75 / stride) * window * metrics * hidden * (2 if kind == "variants" else 1)
    most = max(1, min(2048, int(_MOST_MACS / (8 if kind == "variants" else 3) / macs),
                      int(2e8 / (t_max * 0.75 * metrics))))
    if kind == "detect":
        most = min(most, 64)
    c = dict(kind=kind, streams=_log(rng, 1, most), t_min=max(window + 1, t_max // 2), t_max=t_max, metrics=metrics,
             window=window, stride=stride, hidden=hidden, latent=latent, dtype=dtype, act=act)
    if kind == "variants":
        c["norm"] = rng.choice(["reference", "window"])
    return c


# ----------------------------------------------------------------------------- series on the GPU
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 12345)
    return g


def _ar1(e):
    """AR(1) of unit variance along dim 0 from white noise e (the first 32 terms of its moving-average
    form, by doubling; 0.8^32 < 1e-3)."""
    x = e
    for k in (1, 2, 4, 8, 16):
        y = x.clone()
        y[k:] += (wl.PHI ** k) * x[:-k]
        x = y
    return x.mul_(1.0 / wl.SIGMA_MARG)


def _lengths(case):
    """Steps of every stream: the same for every seed, so that every seed's windows are as many."""
    rng = np.random.default_rng(case["t_max"] * 4099 + case["streams"])
    return rng.integers(case["t_min"], case["t_max"] + 1, size=case["streams"]).astype(np.int64)


def _offsets(lengths):
    offs = np.zeros(len(lengths) + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    return offs


def _series(case, seed, rows):
    """Metrics of every service, one after another: per metric a level and a scale of its own (requests,
    seconds, shares), AR(1) around it, and 6-sigma spikes of all metrics at one step in 512."""
    g = _gen(seed)
    M = case["metrics"]
    x = _ar1(torch.randn(rows, M, device=DEV, generator=g))
    x += 6.0 * (torch.rand(rows, 1, device=DEV, generator=g) < 1.0 / 512)
    level = torch.rand(M, device=DEV, generator=g) * 8 - 4
    scale = torch.exp(torch.rand(M, device=DEV, generator=g) * 3 - 1.5)
    x = x.mul_(scale).add_(level * scale)
    return x.to(torch.bfloat16) if case["dtype"] == "bf16" else x


def _config(case):
    return wl.CONFIGS["c1"].replace(metrics=case["metrics"], window=case["window"], stride=case.get("stride", 1),
                                    hidden=case["hidden"], latent=case["latent"], dtype=case.get("dtype", "f32"),
                                    act=case["act"])


def _weights(case, seed):
    return wl.make_weights(_config(case), seed=int(seed) % (1 << 31), bias_scale=0.05)


def _detector(case, seed):
    return binding.Detector(case["metrics"], case["window"], case["stride"], case["hidden"],
                            binding.weights_for_library(_weights(case, seed), case["dtype"]), latent=case["latent"],
                            dtype=case["dtype"], act=case["act"])


def _train_data(case, seed):
    """A shuffled training set: unit-variance AR(1) windows, a tenth of them with a level shift of 3 to 6
    standard deviations of one metric from some step on (labels +1 normal, -1 anomalous), and the noise."""
    g = _gen(seed)
    n, W, M = case["batch"] * case["batches"], case["window"], case["metrics"]
    v = _ar1(torch.randn(W, n * M, device=DEV, generator=g)).view(W, n, M).permute(1, 0, 2).contiguous()
    bad = torch.rand(n, device=DEV, generator=g) < 0.1
    start = torch.randint(0, W, (n,), device=DEV, generator=g)
    metric = torch.randint(0, M, (n,), device=DEV, generator=g)
    size = (torch.rand(n, device=DEV, generator=g) * 3 + 3) * (torch.randint(0, 2, (n,), device=DEV, generator=g) * 2 - 1)
    late = torch.arange(W, device=DEV)[None, :] >= start[:, None]
    one = torch.arange(M, device=DEV)[None, :] == metric[:, None]
    v += (size * bad)[:, None, None] * late[:, :, None] * one[:, None, :]
    labels = torch.where(bad, -1.0, 1.0).float()
    eps = torch.randn(n, case["latent"], device=DEV, generator=g)
    return v.reshape(n, W * M), labels, eps


def _config_series(case, seed):
    """Serving metrics in Table II's order (the recipe of ``workloads.config_series``, drawn on the GPU)."""
    g = _gen(seed)
    n, T = case["streams"], case["t_len"]

    def u(lo, hi):
        return torch.rand(n, 1, device=DEV, generator=g) * (hi - lo) + lo

    def z(std):
        return torch.randn(n, T, device=DEV, generator=g) * std

    base, phase, t0 = u(20.0, 80.0), u(0.0, 1440.0), u(1.0, 4.0)
    even = (torch.arange(n, device=DEV) % 2 == 0)[:, None]
    cap = base * torch.where(even, 3.0, 0.8)
    t = torch.arange(T, device=DEV, dtype=torch.float32)[None, :]
    lam = base * (1.0 + 0.5 * torch.sin(2.0 * math.pi * (t + phase) / 1440.0))
    n_a = torch.poisson(lam, generator=g)
    t_r = t0 * (1.0 + 0.5 * torch.clamp(lam / cap, max=1.5)) * torch.exp(z(0.05))
    n_r = torch.poisson(torch.minimum(lam, cap) * t_r, generator=g)
    n_f = torch.where(lam >= cap, cap + z(0.05) * cap, n_r / t_r + z(0.02) * base)
    n_p = torch.poisson(5.0 * torch.clamp(lam - cap, min=0.0), generator=g)
    m_u = 0.05 + 0.9 * torch.clamp(n_r / (2.0 * cap * t0), max=1.0) + z(0.005)
    g_u = torch.clamp(torch.sigmoid(4.0 * (lam / cap - 0.7)) + z(0.02), 0.0, 1.0)
    x = torch.stack([n_f, n_r, n_a, n_p, t_r, m_u, g_u], dim=2).reshape(n * T, 7).contiguous()
    return x.to(torch.bfloat16) if case["dtype"] == "bf16" else x


def _score_series(seed, n):
    """KL scores: half a sum of squares of 16 latents, with a heavier tail in one window of 200."""
    g = _gen(seed)
    z = torch.randn(n, 16, device=DEV, generator=g)
    return 0.5 * (z * z).sum(1) * torch.where(torch.rand(n, device=DEV, generator=g) < 0.005, 4.0, 1.0)


# ----------------------------------------------------------------------------- one pass
def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        V, labels, eps = _train_data(case, seed)
        w = _weights(case, seed)
        B, D = case["batch"], case["window"] * case["metrics"]
        tr = binding.Trainer(D, case["hidden"], case["latent"], {k: getattr(w, k) for k in binding.TRAIN_PARAMS},
                             act=case["act"], margin=float(D))
        batches = [(V[i:i + B], labels[i:i + B], eps[i:i + B]) for i in range(0, B * case["batches"], B)]
        return dict(kind=kind, trainer=tr, batches=batches)
    if kind == "config":
        x = _config_series(case, seed)
        sc = binding.ConfigScanner(7, case["window"], case["stride"], col_finished=0, col_running=1, col_exec_time=4,
                                   col_mem_util=5, dtype=case["dtype"])
        so = np.arange(case["streams"] + 1, dtype=np.int64) * case["t_len"]
        wo = sc.window_offsets(so)
        return dict(kind=kind, scanner=sc, x=x, so=torch.from_numpy(so).to(DEV), wo=torch.from_numpy(wo).to(DEV),
                    n=int(wo[-1]))
    if kind == "stream":
        n, W, M = case["streams"], case["window"], case["metrics"]
        live, calib = 256, 1024
        g = _gen(seed + 1)
        x = _series(case, seed, 2048).float()                                  # reference steps of one service
        mean = x.mean(0).repeat(n, 1).contiguous()
        std = x.std(0, unbiased=False).repeat(n, 1).contiguous()
        steps = _ar1(torch.randn(W - 1 + live, n * M, device=DEV, generator=g)).view(W - 1 + live, n, M) * std + mean
        steps = steps.to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float32).contiguous()
        det = _detector(case, seed)
        # calibration scores: those of an earlier stretch of such a service, each stream at a place of its own
        T = calib * 8 + W - 1
        hist = (_ar1(torch.randn(T, M, device=DEV, generator=g)) * std[0] + mean[0]).to(steps.dtype)
        so = torch.tensor([0, T], device=DEV, dtype=torch.int64)
        wo = torch.tensor([0, calib * 8], device=DEV, dtype=torch.int64)
        past = det.score(hist, so, wo, calib * 8, mean[:1].contiguous(), std[:1].contiguous(), md=False)[0]
        at = torch.randint(0, calib * 7, (n, 1), device=DEV, generator=g) + torch.arange(calib, device=DEV)[None, :]
        cal = past[at].reshape(-1).contiguous()
        st = binding.StreamSet(det, mean, std, cal, np.arange(n + 1, dtype=np.int64) * calib)
        for k in range(W - 1):
            st.push(steps[k])
        out = [torch.zeros(n, device=DEV), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV, dtype=torch.uint8)]
        return dict(kind=kind, det=det, set=st, steps=steps, at=W - 1, first=W - 1, out=out, mean=mean, std=std)
    lengths = _lengths(case)
    so = _offsets(lengths)
    if kind == "threshold":
        det = binding.Detector(1, case["window"], 1, 1, _one_unit(case["window"]), latent=1)
        wo = det.window_offsets(so)
        return dict(kind=kind, det=det, scores=_score_series(seed, int(wo[-1])), so=torch.from_numpy(so).to(DEV),
                    wo=torch.from_numpy(wo).to(DEV))
    x = _series(case, seed, int(so[-1]))
    det = _detector(case, seed)
    wo = det.window_offsets(so)
    return dict(kind=kind, det=det, x=x, so=torch.from_numpy(so).to(DEV), wo=torch.from_numpy(wo).to(DEV),
                n=int(wo[-1]), norm=case.get("norm"))


def _one_unit(window):
    """Weights of the smallest detector (the threshold call uses only a detector's window geometry)."""
    shapes = dict(w1=(1, window), b1=(1,), wmu=(1, 1), bmu=(1,), wlv=(1, 1), blv=(1,), wd1=(1, 1), bd1=(1,),
                  wd2=(window, 1), bd2=(window,))
    return {k: np.full(s, 0.1, np.float32) for k, s in shapes.items()}


def run(state):
    kind = state["kind"]
    if kind == "score":
        scores, md, _ = state["det"].score(state["x"], state["so"], state["wo"], state["n"])
        return scores, md
    if kind == "detect":
        det = state["det"]
        scores, md, _ = det.score(state["x"], state["so"], state["wo"], state["n"])
        thr, _, flags = det.threshold(scores, state["so"], state["wo"], flags=True)
        return scores, md, thr, flags
    if kind == "threshold":
        thr, info, flags = state["det"].threshold(state["scores"], state["so"], state["wo"], flags=True)
        return thr, info["gamma"], info["sigma"], info["n_peaks"], flags
    if kind == "stream":
        if state["at"] >= state["steps"].shape[0]:
            state["at"] = state["first"]
        x = state["steps"][state["at"]]
        state["at"] += 1
        scores, md, flags = state["out"]
        state["set"].push(x, scores, md, flags)
        return scores, md, flags
    if kind == "train":
        tr = state["trainer"]
        for V, labels, eps in state["batches"]:
            tr.step(V, labels, eps)
        return tr.params()
    if kind == "config":
        sc = state["scanner"]
        fits = sc.scan(state["x"], state["so"], state["wo"], state["n"])
        return fits, sc.recommend(state["x"], state["so"])
    return state["det"].score_ext(state["x"], state["so"], state["wo"], state["n"], norm=state["norm"])


# ----------------------------------------------------------------------------- what a pass needs
def _windows(case):
    """Windows and steps of a pass."""
    lengths = np.full(case["streams"], case["t_len"]) if case["kind"] == "config" else _lengths(case)
    W, S = case["window"], case.get("stride", 1)
    return int(np.where(lengths >= W, (lengths - W) // S + 1, 0).sum()), int(lengths.sum())


def work(case):
    kind = case["kind"]
    W, M = case["window"], case.get("metrics", 1)
    H, L, D = case.get("hidden", 0), case.get("latent", 0), W * M
    size = 2 if case.get("dtype") == "bf16" else 4
    weights = 4.0 * (2 * H * D + 3 * H * L + 2 * H + 2 * L + D)
    if kind == "train":
        B, k = case["batch"], case["batches"]
        # forward and backward products; the windows, noise and labels once, weights and both moments
        # read and written in each step, the weights copied out at the end
        return dict(bytes=k * (4.0 * B * (D + L + 1) + 6 * weights) + weights, flops=k * 2.0 * B * (5 * H * D + 9 * H * L))
    if kind == "stream":
        n = case["streams"]
        # every stream's newest window is read, its new step read and kept, three outputs written
        return dict(bytes=n * (D * size + 2.0 * M * size + 9) + n * M * 8, flops=n * (2.0 * H * D + 6 * H * L + 2 * H))
    n, rows = _windows(case)
    if kind == "threshold":
        # every score read, every flag written
        return dict(bytes=5.0 * n, flops=0.0)
    if kind == "config":
        # the series once, 21 bytes a window; three means and four centred sums, each window's change by
        # one stride of samples at the least
        return dict(bytes=rows * 7.0 * size + 21.0 * n, flops=n * (14.0 * case["stride"] + 20))
    score = 2.0 * H * D + 4 * H * L + 2 * H * L + 2 * H
    if kind == "variants":
        return dict(bytes=rows * M * size + n * 4.0 * (3 + M) + weights, flops=n * (score + 2.0 * H * D))
    return dict(bytes=rows * M * size + n * (9.0 if kind == "detect" else 8.0) + weights, flops=n * score)


def tolerance(case):
    """About four times the largest error against ``exact`` over the listed and some drawn cases."""
    kind = case["kind"]
    if kind == "threshold":
        # an exact order statistic and a fit in 64 bits, the threshold rounded to 32
        return dict(rel=1e-6, differ=1e-6)
    if kind == "config":
        # 64-bit statistics written as 32-bit numbers (seen: 2.8e-8); the t-test's decision at |t| = critical
        return dict(rel=1.2e-7, max=1e-5, differ=1e-5)
    if kind == "train":
        # 32-bit sums of one order or another decide on which side of zero a ReLU's input falls, and Adam
        # turns the sign of a small first gradient into a whole step (seen: 3.5e-4 with ReLU, 1.6e-7 with tanh)
        return dict(rel=1.4e-3, max=0.3) if case["act"] == "relu" else dict(rel=1e-4, max=0.1)
    if case.get("dtype") == "bf16":
        # one bf16 rounding of each normalised input decides; 32-bit sums (seen: 9.4e-6 over long windows)
        return dict(rel=2e-4, max=2e-2, differ=3e-3)
    if kind == "variants":
        # the per-metric direction is a small difference of sums (seen: 8.2e-6)
        return dict(rel=4e-5)
    # 32-bit sums (seen: 1.7e-6); flags of a few thousand windows within that of the threshold
    return dict(rel=1e-5, differ=2e-3)


# ----------------------------------------------------------------------------- the same in 64 bits
def _act(a, act):
    return a.clamp(min=0.0) if act == "relu" else torch.tanh(a)


def _ref_len(T):
    return T // 2                      # the reference prefix: the first half of a stream


def _norm_rows(x, std_guard=True):
    mean = x.mean(0)
    std = x.std(0, unbiased=False)
    std = torch.where(std <= 1e-6 * torch.clamp(mean.abs(), min=1.0), torch.ones_like(std), std)
    return mean, std


def _encode(v, w, act):
    h = _act(v @ w["w1"].T + w["b1"], act)
    mu, lv = h @ w["wmu"].T + w["bmu"], h @ w["wlv"].T + w["blv"]
    return mu, 0.5 * (mu * mu + torch.expm1(lv) - lv).sum(1)


def _decode(mu, w, act):
    return _act(mu @ w["wd1"].T + w["bd1"], act) @ w["wd2"].T + w["bd2"]


def _w64(case, seed):
    return {k: torch.from_numpy(v).to(DEV) for k, v in _weights(case, seed).as_f64().items()}


def _exact_scores(case, seed):
    """Scores and md of every window (and md_m and the reconstruction error for the variants)."""
    W, S, M, act = case["window"], case["stride"], case["metrics"], case["act"]
    so = _offsets(_lengths(case))
    x = _series(case, seed, int(so[-1]))
    w = _w64(case, seed)
    u, b = w["wd2"].sum(0), w["bd2"].sum()
    D = W * M
    ext = case["kind"] == "variants"
    out = [[], [], [], []]
    for s in range(case["streams"]):
        xs = x[so[s]:so[s + 1]].double()
        if xs.shape[0] < W:
            continue
        if case.get("norm") != "window":
            mean, std = _norm_rows(xs[:_ref_len(xs.shape[0])])
            xs = (xs - mean) / std
            if case["dtype"] == "bf16":
                xs = xs.to(torch.bfloat16).double()
        win = xs.unfold(0, W, S).transpose(1, 2)                     # [windows, W, M], a view
        for a in range(0, win.shape[0], 1 << 15):
            v = win[a:a + (1 << 15)]
            if case.get("norm") == "window":
                m, sd = v.mean(1), v.std(1, unbiased=False)
                sd = torch.where(sd <= 1e-6 * torch.clamp(m.abs(), min=1.0), torch.ones_like(sd), sd)
                v = (v - m[:, None]) / sd[:, None]
                if case["dtype"] == "bf16":
                    v = v.to(torch.bfloat16).double()
            v = v.reshape(-1, D)
            mu, kl = _encode(v, w, act)
            out[0].append(kl)
            if not ext:
                hd = _act(mu @ w["wd1"].T + w["bd1"], act)
                out[1].append((v.sum(1) - hd @ u - b) / D)
                continue
            d = v - _decode(mu, w, act)
            out[1].append(d.mean(1))
            out[2].append(d.view(-1, W, M).mean(1))
            out[3].append((d * d).mean(1))
    return [torch.cat(o) for o in out if o]


def _fit_tail(y, t, n, q):
    """Grimshaw's maximum-likelihood fit of a generalised Pareto tail to the excesses y and the threshold
    at probability q (Siffer et al. 2017)."""
    N = y.numel()
    mean, mn, mx = float(y.mean()), float(y.min()), float(y.max())

    def sums(xs):
        a = torch.empty_like(xs)
        b = torch.empty_like(xs)
        for i in range(0, xs.numel(), 64):
            p = xs[i:i + 64, None] * y[None, :]
            a[i:i + 64] = (p / (1.0 + p)).mean(1)
            b[i:i + 64] = torch.log1p(p).mean(1)
        return a, b

    def w(xs):
        a, b = sums(xs)
        return b - a - a * b

    e = 1e-8 / mean
    grids = []
    f0 = e * mx
    if f0 < 0.5:
        z = torch.linspace(math.log(f0 / (1.0 - f0)), 30.0, 512, device=DEV, dtype=torch.float64)
        grids.append(-torch.sigmoid(z) / mx)
    top = 2.0 * (mean - mn) / mn ** 2
    if top > 2.0 * e:
        grids.append(torch.logspace(math.log10(e), math.log10(top), 512, device=DEV, dtype=torch.float64))
    best = (-N * math.log(mean) - N, 0.0, mean)
    for xs in grids:
        v = w(xs)
        at = torch.nonzero(v[:-1] * v[1:] < 0).flatten()
        if not at.numel():
            continue
        lo, hi, s = xs[at].clone(), xs[at + 1].clone(), torch.sign(v[at])
        for _ in range(100):
            mid = 0.5 * (lo + hi)
            same = torch.sign(w(mid)) == s
            lo, hi = torch.where(same, mid, lo), torch.where(same, hi, mid)
        for x in (0.5 * (lo + hi)).tolist():
            g = float(torch.log1p(x * y).mean())
            if g == 0.0 or g / x <= 0.0:
                continue
            ll = -N * math.log(g / x) - (1.0 + 1.0 / g) * N * g
            if ll > best[0]:
                best = (ll, g, g / x)
    _, g, s = best
    r = q * n / N
    z = t - s * math.log(r) if abs(g) < 1e-9 else t + s / g * (r ** -g - 1.0)
    return z, g, s


def _exact_threshold(scores, so, W, S, level=0.98, q=1e-3):
    cal, at = [], 0
    for T in np.diff(so):
        n = (T - W) // S + 1 if T >= W else 0
        R = _ref_len(int(T))
        cal.append(scores[at:at + ((R - W) // S + 1 if R >= W else 0)])
        at += n
    cal = torch.cat(cal)
    k = max(0, math.ceil(level * cal.numel()) - 1)
    t = float(torch.sort(cal).values[k])
    y = cal[cal > t].double() - t
    if y.numel() < 10:
        return None, t, None, int(y.numel())
    z, g, s = _fit_tail(y, t, cal.numel(), q)
    return z, g, s, int(y.numel())


def _exact_train(case, seed):
    V, labels, eps = _train_data(case, seed)
    p = _w64(case, seed)
    m, v = ({k: torch.zeros_like(t) for k, t in p.items()} for _ in range(2))
    B, act, integ = case["batch"], case["act"], 0.0
    lr, kl_set, kp, ki = 1e-3, 3.0, 0.01, 1e-4                       # the trainer's defaults
    margin = float(case["window"] * case["metrics"])

    def dact(a):
        return (a > 0).double() if act == "relu" else 1.0 - torch.tanh(a) ** 2

    for k in range(case["batches"]):
        x, l, e = (t[k * B:(k + 1) * B].double() for t in (V, labels, eps))
        a1 = x @ p["w1"].T + p["b1"]
        h = _act(a1, act)
        mu, lv = h @ p["wmu"].T + p["bmu"], h @ p["wlv"].T + p["blv"]
        sd = torch.exp(0.5 * lv)
        z = mu + sd * e
        a2 = z @ p["wd1"].T + p["bd1"]
        hd = _act(a2, act)
        d = hd @ p["wd2"].T + p["bd2"] - x
        kl = 0.5 * (mu * mu + torch.expm1(lv) - lv).sum(1)
        normal = l > 0
        err = kl_set - float(kl[normal].mean()) if bool(normal.any()) else kl_set
        integ -= ki * err
        beta = min(max(kp / (1.0 + math.exp(err)) + integ, 0.0), 1.0)
        live = normal | (0.5 * (d * d).sum(1) < margin)
        gd = d * (l * live / B)[:, None]
        ga2 = (gd @ p["wd2"]) * dact(a2)
        gz = ga2 @ p["wd1"]
        c = (0.5 * (1.0 + l) * beta / B)[:, None]
        gmu = gz + c * mu
        glv = gz * e * 0.5 * sd + c * 0.5 * torch.expm1(lv)
        ga1 = (gmu @ p["wmu"] + glv @ p["wlv"]) * dact(a1)
        grads = dict(w1=ga1.T @ x, b1=ga1.sum(0), wmu=gmu.T @ h, bmu=gmu.sum(0), wlv=glv.T @ h, blv=glv.sum(0),
                     wd1=ga2.T @ z, bd1=ga2.sum(0), wd2=gd.T @ hd, bd2=gd.sum(0))
        for name, g in grads.items():
            m[name] = 0.9 * m[name] + 0.1 * g
            v[name] = 0.999 * v[name] + 0.001 * g * g
            mh, vh = m[name] / (1.0 - 0.9 ** (k + 1)), v[name] / (1.0 - 0.999 ** (k + 1))
            p[name] = p[name] - lr * mh / (torch.sqrt(vh) + 1e-8)
    return {k: p[k] for k in binding.TRAIN_PARAMS}


def _kde_quantile(v, q):
    """Quantile q[s] of the Gaussian kernel density estimate of each row of v."""
    n = v.shape[1]
    srt = torch.sort(v, dim=1).values

    def at(p):
        h = (n - 1) * p
        lo = int(math.floor(h))
        return srt[:, lo] + (h - lo) * (srt[:, min(lo + 1, n - 1)] - srt[:, lo])

    sd, iqr = v.std(1), at(0.75) - at(0.25)
    h = 0.9 * torch.where(iqr > 0, torch.minimum(sd, iqr / 1.34), sd) * n ** -0.2
    lo, hi = srt[:, 0] - 10 * h, srt[:, -1] + 10 * h
    for _ in range(90):
        mid = 0.5 * (lo + hi)
        F = 0.5 * torch.erfc(-(mid[:, None] - v) / (h[:, None] * math.sqrt(2.0))).mean(1)
        lo, hi = torch.where(F < q, mid, lo), torch.where(F < q, hi, mid)
    return torch.where(h > 0, 0.5 * (lo + hi), v[:, 0])


def _exact_config(case, seed):
    W, S, n, T = case["window"], case["stride"], case["streams"], case["t_len"]
    x = _config_series(case, seed).view(n, T, 7)
    parts = [[] for _ in range(5)]

    def fit(f, r, m):
        rm, fm, mm = r.mean(-1, True), f.mean(-1, True), m.mean(-1, True)
        dr, df = r - rm, f - fm
        sxx, sxy, syy = (dr * dr).sum(-1), (dr * df).sum(-1), (df * df).sum(-1)
        flat = sxx == 0
        one = torch.where(flat, torch.ones_like(sxx), sxx)
        b = torch.where(flat, torch.zeros_like(sxx), sxy / one)
        g1 = torch.where(flat, torch.zeros_like(sxx), (dr * (m - mm)).sum(-1) / one)
        rss = torch.clamp(syy - b * sxy, min=0.0)
        t = torch.where(b == 0, torch.zeros_like(b), b * torch.sqrt((W - 2) * sxx / rss))
        return [fm[..., 0] - b * rm[..., 0], b, t, mm[..., 0] - g1 * rm[..., 0], g1]

    step = max(1, (1 << 21) // T)
    last = []
    for s in range(0, n, step):
        c = [x[s:s + step, :, k].double().contiguous().unfold(1, W, S) for k in (0, 1, 5)]
        got = fit(*c)
        for o, g in zip(parts, got):
            o.append(g.reshape(-1))
        last.append([got[2][:, -1], got[3][:, -1], got[4][:, -1]])
    t, g0, g1 = (torch.cat(k) for k in zip(*last))
    end = ((T - W) // S) * S
    tail = x[:, end:end + W].double()
    crit = binding.enova_config_t_critical(0.05, W - 2)
    q = torch.full_like(t, 0.5).masked_fill(t.abs() > crit, 0.99)
    nl, tl = _kde_quantile(tail[:, :, 0].contiguous(), q), _kde_quantile(tail[:, :, 4].contiguous(), q)
    a, b, tt, g0w, g1w = (torch.cat(o) for o in parts)
    return (a, b, tt, None, g0w, g1w), (None, nl, tl, nl * tl, g0 + g1 * nl * tl)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "config":
        return _exact_config(case, seed)
    if kind == "threshold":
        so = _offsets(_lengths(case))
        n = int(np.maximum(np.diff(so) - case["window"] + 1, 0).sum())
        z, g, s, _ = _exact_threshold(_score_series(seed, n), so, case["window"], 1)
        return z, g, s, None, None
    if kind == "stream":
        st = prepare(case, seed)
        W, M, act = case["window"], case["metrics"], case["act"]
        w = _w64(case, seed)
        v = (st["steps"][:W].double() - st["mean"].double()) / st["std"].double()
        if case["dtype"] == "bf16":
            v = v.to(torch.bfloat16).double()
        v = v.permute(1, 0, 2).reshape(-1, W * M)
        mu, kl = _encode(v, w, act)
        return kl, (v - _decode(mu, w, act)).mean(1), None
    got = _exact_scores(case, seed)
    if kind == "detect":
        z = _exact_threshold(got[0], _offsets(_lengths(case)), case["window"], case["stride"])[0]
        return got[0], got[1], z, None
    return got
