"""The output variants on the 16-bit matrix cores: padded metric counts, tile edges, output rows that end
inside a 32-row block, hidden layers of one to four blocks, and the windows outside the range of the 16-bit
parts (evaluated in fp32, up to 64 at a time), against the fp64 oracle. Every call asserts the evaluation it
takes: calls of few windows take the chunked one at some shapes, and the split pass with a long stream added. Sums of D products in fp32 differ by about
sqrt(D) 2^-24 of their scale; the tests allow 3e-6 in the 2-norm (D <= 1024)."""
import numpy as np
import pytest

from harness import detector, log, upload
from oracle import variants as ov
from paper_2407_09486_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _run(cfg, weights, w, norm, route="split", pairs=None):
    import torch
    det = detector(cfg, weights)
    x, so = upload(w)
    woff = det.window_offsets(w.stream_offsets)
    assert det.ext_route(len(w.stream_offsets) - 1, int(woff[-1]), norm) == route
    out = det.score_ext(x, so, torch.from_numpy(woff).cuda(), int(woff[-1]), norm=norm)
    torch.cuda.synchronize()
    res = [o.cpu().numpy().astype(np.float64) for o in out]
    det.close()
    ref = ov.score_ext(w.values_f64(), w.stream_offsets, window=cfg.window, stride=cfg.stride,
                       weights={k: np.asarray(getattr(weights, k), np.float64) for k in
                                ("w1", "b1", "wmu", "bmu", "wlv", "blv", "wd1", "bd1", "wd2", "bd2")},
                       act=cfg.act, norm=norm, ref_frac=cfg.ref_frac, pairs=pairs)
    if pairs is not None:
        res = [r[[woff[i] + k for i, k in pairs]] for r in res]
    return res, ref


def _with_long_stream(lengths, W, S, windows):
    """The lengths with a stream of so many windows behind the first two, and the windows to check: all of the
    other streams, and of the long one its first, last and every 97th."""
    if not windows:
        return lengths, None
    lengths = lengths[:2] + [W + (windows - 1) * S] + lengths[2:]
    n = [max(0, (T - W) // S + 1) if T >= W else 0 for T in lengths]
    pairs = [(i, k) for i in range(len(n)) for k in range(n[i]) if i != 2 or k % 97 == 0 or k == n[2] - 1]
    return lengths, pairs


def _check(res, ref, sel):
    scale = ref["scale"][sel]
    for name, g, o, s in (("score", res[0], ref["score"], None), ("md", res[1], ref["md"], scale),
                          ("md_m", res[2], ref["md_metric"], scale[:, None]),
                          ("recon", res[3], ref["recon"], None)):
        g, o = g[sel], o[sel]
        if s is None:
            assert np.linalg.norm(g - o) <= 3e-6 * np.linalg.norm(o), name
            assert np.all(np.abs(g - o) <= 1e-4 * np.abs(o) + 1e-6), name
        else:
            assert np.linalg.norm(g - o) <= 3e-6 * np.linalg.norm(s * np.ones_like(o)), name
            assert np.all(np.abs(g - o) <= 1e-4 * s), name


@pytest.mark.parametrize("norm", ["reference", "window"])
@pytest.mark.parametrize("M,W,S,H,act,more,route", [
    (7, 9, 1, 64, "tanh", 0, "split"), (5, 33, 8, 32, "relu", 0, "chunked"), (5, 32, 3, 32, "relu", 0, "split"),
    (12, 11, 1, 128, "tanh", 13000, "split"), (16, 14, 3, 100, "tanh", 0, "chunked"), (16, 14, 1, 100, "tanh", 13000, "split"),
    (1, 50, 1, 40, "relu", 0, "chunked"), (1, 50, 1, 40, "relu", 20000, "split"), (8, 6, 9, 128, "relu", 0, "chunked"),
    (8, 3, 5, 128, "relu", 0, "split"), (9, 7, 1, 20, "relu", 0, "split"), (16, 64, 1, 128, "relu", 0, "split"),
    (7, 60, 1, 64, "tanh", 0, "chunked"), (7, 60, 1, 64, "tanh", 9000, "split")])
def test_tile_and_block_edges(norm, M, W, S, H, act, more, route):
    counts = [1, 31, 64, 65, 255, 257, 513]
    lengths = [W + (k - 1) * S for k in counts] + [W - 1, 0, W + 100 * S + S - 1]
    lengths, pairs = _with_long_stream(lengths, W, S, more)
    cfg = wl.CONFIGS["c1"].replace(metrics=M, window=W, stride=S, hidden=H, act=act, n_streams=len(lengths))
    log(f"[ext split] {norm} M={M} W={W} S={S} H={H} {act}")
    rng = np.random.default_rng(M + W)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    w = wl.from_arrays(cfg, rng.standard_normal((int(offs[-1]), M)) * np.exp(rng.uniform(-2, 2, M)) + 3, offs)
    res, ref = _run(cfg, wl.make_weights(cfg, bias_scale=0.1), w, norm, route, pairs)
    _check(res, ref, np.arange(len(ref["score"])))


@pytest.mark.parametrize("norm", ["reference", "window"])
@pytest.mark.parametrize("M,H", [(7, 64), (16, 128)])
def test_windows_outside_the_range(norm, M, H):
    """Spikes, infinities, NaN and nearly constant stretches; every window that holds neither infinity nor
    NaN against the oracle, the others not finite."""
    cfg = wl.CONFIGS["c1"].replace(metrics=M, window=20, stride=1, hidden=H, n_streams=2)
    rng = np.random.default_rng(4)
    offs = np.array([0, 1500, 2300], np.int64)
    x = rng.standard_normal((2300, M)).astype(np.float32)
    x[900, 1] = 3e5
    x[1000:1060] = 0.25 * np.arange(M)                    # constant metrics
    x[1100:1160] = 2.0 + 2e-7 * rng.integers(0, 3, (60, M)).astype(np.float32)   # within a few last places
    x[1300, 0] = np.inf
    x[1400, M - 1] = np.nan
    x[2200, 2] = -7e7
    w = wl.from_arrays(cfg, x, offs)
    log(f"[ext split] range {norm} M={M} H={H}")
    res, ref = _run(cfg, wl.make_weights(cfg, bias_scale=0.1), w, norm)
    start = np.concatenate([np.arange(1500 - 19), 1500 + np.arange(800 - 19)])
    odd = np.zeros(len(start), bool)
    for row in (1300, 1400):
        odd |= (start <= row) & (start + 20 > row)
    big = np.zeros(len(start), bool)
    for row in (900, 2200):
        big |= (start <= row) & (start + 20 > row)
    _check(res, ref, np.flatnonzero(~odd & ~big))
    sel = np.flatnonzero(big)
    for g, o in ((res[0], ref["score"]), (res[3], ref["recon"])):
        with np.errstate(over="ignore"):            # e^lv overflows on both sides
            o = o.astype(np.float32).astype(np.float64)
        np.testing.assert_allclose(g[sel], o[sel], rtol=1e-4, atol=1e-6)
    nan = np.flatnonzero((start <= 1400) & (start + 20 > 1400))
    assert np.all(np.isnan(res[0][nan])) and np.all(np.isnan(res[3][nan]))
    assert not np.any(np.isfinite(res[3][odd]))


@pytest.mark.parametrize("norm", ["reference", "window"])
@pytest.mark.parametrize("where", ["rows", "units"])
def test_decoder_output_scales(norm, where):
    """Decoder output weights whose rows (here one metric's) or columns (hidden units, whose activations make
    up for it) lie far apart: the other metrics' md keep fp32's precision (|v| and |m'| of about 1, one
    rounding of 2^-24 each: 6e-8 rms; fp32 sums measure 5e-8)."""
    M, W, H = 8, 8, 64
    cfg = wl.CONFIGS["c1"].replace(metrics=M, window=W, stride=1, hidden=H, n_streams=2)
    rng = np.random.default_rng(8)
    offs = np.array([0, 1200, 2100], np.int64)
    w = wl.from_arrays(cfg, rng.standard_normal((2100, M)) * 2 + 1, offs)
    weights = wl.make_weights(cfg, bias_scale=0.1)
    if where == "rows":
        weights.wd2.reshape(W, M, H)[:, 0] *= 1e6
    else:
        weights.wd1[:H // 2] *= 1e-6
        weights.bd1[:H // 2] *= 1e-6
        weights.wd2[:, :H // 2] *= 1e6
    log(f"[ext split] decoder scales {norm} {where}, largest |Wd2| {np.abs(weights.wd2).max():.3g}")
    res, ref = _run(cfg, weights, w, norm, "fused")      # 8 metrics: the pass in fp32
    err = np.sqrt(np.mean((res[2] - ref["md_metric"])[:, 1:] ** 2))
    log(f"  rms error {err:.2e}")
    assert err <= 1e-7


@pytest.mark.parametrize("norm", ["reference", "window"])
@pytest.mark.parametrize("M,W,S,H,L,act,more,route", [
    (7, 60, 1, 64, 16, "tanh", 9000, "split"), (16, 64, 1, 128, 16, "relu", 0, "split"), (3, 9, 1, 96, 3, "relu", 0, "split"),
    (12, 11, 2, 30, 5, "tanh", 0, "chunked"), (12, 11, 1, 30, 5, "tanh", 400, "split"), (5, 40, 3, 128, 16, "relu", 6000, "split"),
    (1, 100, 1, 64, 2, "relu", 0, "chunked"), (1, 100, 1, 64, 2, "relu", 46000, "split"), (8, 32, 1, 33, 16, "relu", 0, "split"),
    # windows left to the fp32 pass of whole tiles (strides that divide the window, whole hidden blocks), or just not
    (4, 16, 1, 64, 3, "tanh", 0, "split"), (8, 12, 3, 32, 16, "relu", 0, "split"), (8, 12, 5, 64, 16, "relu", 0, "split"),
    (8, 16, 4, 128, 7, "tanh", 0, "split"), (16, 8, 2, 64, 16, "tanh", 0, "split"), (16, 6, 1, 32, 16, "relu", 0, "split")])
def test_stretches_outside_the_range(norm, M, W, S, H, L, act, more, route):
    """Windows left to the fp32 kernel in all numbers, from one of a tile's 64 to whole tiles, beside others: a
    metric that was constant over the reference prefix and moves by thousands later (reference normalisation),
    stretches constant but for their last places (window normalisation)."""
    counts = [700, 300, 64, 1]
    lengths, pairs = _with_long_stream([W + (k - 1) * S + W * S for k in counts], W, S, more)
    cfg = wl.CONFIGS["c1"].replace(metrics=M, window=W, stride=S, hidden=H, latent=L, act=act, n_streams=len(lengths))
    log(f"[ext split] stretches {norm} M={M} W={W} S={S} H={H} L={L} {act}")
    rng = np.random.default_rng(M + H)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    x = rng.standard_normal((int(offs[-1]), M)).astype(np.float32)
    small = rng.integers(-1, 2, x.shape).astype(np.float32) * np.float32(2.0 ** -20)
    for i, T in enumerate(lengths):
        y, z = x[offs[i]:offs[i + 1]], small[offs[i]:offs[i + 1]]
        if norm == "reference":
            y[:T // 2 + 1, 0] = 0.5
            y[T // 2 + 1:, 0] = rng.uniform(-1, 1, T - T // 2 - 1)
            y[5 * T // 8, 0] = 4500.0
            y[3 * T // 4:, 0] = rng.uniform(4100, 5000, T - 3 * T // 4)
            y[min(7 * T // 8 + 3, T - 1), 0] = -0.2
        else:
            for part in (slice(T // 8, T // 8 + W + 2 * S), slice(T // 2, 3 * T // 4)):
                y[part] = 2.0 + z[part]
    w = wl.from_arrays(cfg, x, offs)
    weights = wl.make_weights(cfg, bias_scale=0.1)
    if norm == "reference":
        weights.w1 *= 1e-3                               # e^lv stays finite
    res, ref = _run(cfg, weights, w, norm, route, pairs)
    keep = np.ones(len(ref["score"]), bool)
    if norm == "window":
        # a window that ends in the first step of a stretch may hold a metric that is next to constant: v is then
        # off by the rounding of its fp32 mean, 2^-24 mean / sd, 1.2e-4 at a deviation of 1e-3
        where = pairs or [(i, k) for i, T in enumerate(lengths) for k in range((T - W) // S + 1 if T >= W else 0)]
        sd = np.array([x[offs[i] + k * S:offs[i] + k * S + W].astype(np.float64).std(axis=0) for i, k in where])
        keep = ~np.any((sd > 1e-6) & (sd < 1e-3), axis=1)
        assert keep.mean() > 0.99
    _check(res, ref, np.flatnonzero(keep))
    import torch
    det = detector(cfg, weights)
    xd, so = upload(w)
    wo = det.window_offsets(offs)
    only = det.score_ext(xd, so, torch.from_numpy(wo).cuda(), int(wo[-1]), norm=norm, scores_only=True)[0]
    only = only.cpu().numpy().astype(np.float64)
    if pairs is not None:
        only = only[[wo[i] + k for i, k in pairs]]
    assert np.array_equal(only, res[0])
    det.close()


@pytest.mark.parametrize("M,W,S,H", [(6, 1, 1, 64), (7, 9, 1, 50), (8, 6, 5, 33)])
def test_infinite_reference_mean(M, W, S, H):
    """A metric whose reference mean is infinite makes v infinite at every step; tanh's hidden layer is then all ones
    in size and the scores are finite, as the chunked evaluation has them: the padding of the list's runs
    may not turn them into NaN."""
    import torch
    cfg = wl.CONFIGS["c1"].replace(metrics=M, window=W, stride=S, hidden=H, act="tanh", n_streams=2)
    rng = np.random.default_rng(M * W)
    offs = np.array([0, 400, 700], np.int64)
    w = wl.from_arrays(cfg, rng.standard_normal((700, M)), offs)
    # one sign for every step's weight, or infinities of both would meet
    weights = wl.make_weights(cfg, bias_scale=0.1)
    weights.w1.reshape(H, W, M)[:, :, 0] = np.sign(weights.w1.reshape(H, W, M)[:, :1, 0])
    log(f"[ext split] infinite mean M={M} W={W} S={S} H={H}")
    mean, std = np.zeros((2, M)), np.ones((2, M))
    mean[1, 0] = np.inf
    det = detector(cfg, weights)
    x, so = upload(w)
    wo = det.window_offsets(offs)
    assert det.ext_route(2, int(wo[-1])) == "split"
    out = det.score_ext(x, so, torch.from_numpy(wo).cuda(), int(wo[-1]), ref_mean=torch.from_numpy(mean).float().cuda(),
                        ref_std=torch.from_numpy(std).float().cuda())[0].cpu().numpy().astype(np.float64)
    det.close()
    ref = ov.score_ext(w.values_f64(), offs, window=W, stride=S, weights={k: np.asarray(getattr(weights, k), np.float64) for k in
                       ("w1", "b1", "wmu", "bmu", "wlv", "blv", "wd1", "bd1", "wd2", "bd2")},
                       act="tanh", ref_mean=mean, ref_std=std)["score"]
    out, ref = out[wo[1]:], ref[wo[1]:]                  # the second stream's: sums of H exact products, 16 squares
    assert np.all(np.isfinite(ref)) and np.all(np.abs(out - ref) <= 1e-5 * np.abs(ref))
