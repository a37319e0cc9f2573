"""The split-precision scoring kernel (fp32 detectors): tile edges, both tile sizes, odd geometries and
the range its 16-bit parts hold, against the fp64 oracle, and the windows outside that range against the
vector kernel. Two fp32 sums of D products in different order differ by about sqrt(D) 2^-24 of the
score's scale; the tests allow 2e-6 (D <= 1024)."""
import numpy as np
import pytest

import oracle
from harness import check_md, check_scores, detector, gpu_score, log, oracle_score
from paper_2407_09486_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _cfg(M, W, S, H, L=16, act="relu", n=1):
    return wl.CONFIGS["c1"].replace(metrics=M, window=W, stride=S, hidden=H, latent=L, act=act, n_streams=n)


def _check(cfg, w, weights, what):
    det = detector(cfg, weights)
    sc, md, _, _ = gpu_score(det, w, pad=32)
    o_sc, o_md, info = oracle_score(cfg, w, weights)
    scale = float(np.sqrt(np.mean(o_sc ** 2)))
    assert np.linalg.norm(sc - o_sc) <= 2e-6 * np.linalg.norm(o_sc), what
    assert np.max(np.abs(sc - o_sc)) <= 2e-5 * scale + 2e-5 * np.max(np.abs(o_sc)), what
    check_scores(sc, o_sc, "f32", what)
    check_md(md, o_md, info["md_scale"], "f32", what)
    det.close()


# chunk counts of a super-row of 1 (two rows a step), 2, 3 (odd), padded metrics, strides, S > W;
# windows around the tiles' 64, 128, 256 and 512; hidden layers of one to eight 32-row blocks
@pytest.mark.parametrize("M,W,S,H,act", [(8, 6, 1, 32, "relu"), (7, 9, 1, 64, "tanh"), (16, 5, 1, 100, "relu"),
                                         (3, 4, 8, 33, "relu"), (24, 3, 1, 200, "tanh"), (4, 11, 2, 256, "relu"),
                                         (5, 16, 3, 128, "tanh"), (32, 2, 5, 8, "relu")])
def test_tile_edges(M, W, S, H, act):
    counts = [1, 31, 33, 64, 65, 128, 129, 257, 512, 513]
    lengths = [W + (k - 1) * S for k in counts] + [W - 1, 0, W + 300 * S + S - 1]
    cfg = _cfg(M, W, S, H, act=act, n=len(lengths))
    log(f"[split] edges M={M} W={W} S={S} H={H} {act}")
    rng = np.random.default_rng(5)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    w = wl.from_arrays(cfg, rng.standard_normal((int(offs[-1]), M)) * 3 + 1, offs)
    _check(cfg, w, wl.make_weights(cfg, bias_scale=0.1), f"{M} {W} {S} {H}")


@pytest.mark.parametrize("H", [32, 64, 128, 256])
def test_large_tiles(H):
    """Enough windows for the large tile of each hidden width."""
    cfg = _cfg(2, 4, 1, H, n=2)
    n = {32: 262200, 64: 262200, 128: 131200, 256: 65700}[H]
    log(f"[split] large tiles H={H}, {n} windows")
    rng = np.random.default_rng(H)
    offs = np.array([0, n // 2 + 17, n + 40], np.int64)
    w = wl.from_arrays(cfg, rng.standard_normal((n + 40, 2)), offs)
    _check(cfg, w, wl.make_weights(cfg, bias_scale=0.1), f"large {H}")


@pytest.mark.parametrize("H", [32, 128, 256])
def test_windows_outside_the_range(H):
    """Spikes beyond the f16 range, infinities, NaN and nearly constant stretches: the windows that hold
    them agree with the vector kernel, and every window is bitwise what its stream gives alone."""
    cfg = _cfg(7, 20, 1, H, n=3)
    rng = np.random.default_rng(9)
    lengths = [900, 2500, 700]
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    x = rng.standard_normal((int(offs[-1]), 7)).astype(np.float32)
    x[offs[0] + 600, 2] = 1e6
    x[offs[0] + 800, 0] = -3e38
    x[offs[1] + 1400:offs[1] + 1460] = x[offs[1]:offs[1] + 1250].mean(0) + 1e-4     # nearly constant
    x[offs[1] + 1700, 3] = np.inf
    x[offs[1] + 1900, 6] = np.nan
    x[offs[1] + 2100, 1] = 4001.0                                                  # about the limit
    x[offs[2]:] = 5.0                                                              # constant: scores of v = 0
    w = wl.from_arrays(cfg, x, offs)
    weights = wl.make_weights(cfg, bias_scale=0.1)
    log(f"[split] range H={H}")
    det, ref = detector(cfg, weights), detector(cfg, weights, "valu")
    (sc, md, _, woff), (rsc, rmd, _, _) = gpu_score(det, w, pad=16), gpu_score(ref, w)
    fin = np.isfinite(rsc) & (np.abs(rsc) < 1e30)
    assert np.array_equal(np.isnan(sc), np.isnan(rsc)) and np.array_equal(np.isinf(sc), np.isinf(rsc))
    np.testing.assert_allclose(sc[fin], rsc[fin], rtol=1e-5, atol=1e-6)
    ok = np.isfinite(rmd) & (np.abs(rmd) < 1e30)
    np.testing.assert_allclose(md[ok], rmd[ok], rtol=1e-5, atol=2e-6)
    for i in range(3):
        one = wl.from_arrays(cfg, x[offs[i]:offs[i + 1]], np.array([0, lengths[i]]))
        a, b, _, _ = gpu_score(det, one)
        assert np.array_equal(a, sc[woff[i]:woff[i + 1]], equal_nan=True)
        assert np.array_equal(b, md[woff[i]:woff[i + 1]], equal_nan=True)
    det.close()
    ref.close()


def test_weight_scales():
    """Hidden rows of very different scale keep their precision (each row has its own power of two); rows
    of zeros; a weight outside the supported range falls back to the fp32 kernel."""
    cfg = _cfg(8, 16, 1, 64, n=1)
    rng = np.random.default_rng(2)
    w = wl.from_arrays(cfg, rng.standard_normal((1500, 8)), np.array([0, 1500]))
    weights = wl.make_weights(cfg, bias_scale=0.05)
    scale = np.exp2(rng.integers(-30, 6, 64)).astype(np.float32)
    scale[:3] = 0.0
    weights.w1[:] *= scale[:, None]
    weights.wmu[:] /= np.maximum(scale, 2.0 ** -10)[None, :]
    log("[split] weight scales")
    _check(cfg, w, weights, "row scales")
    weights.w1[5, 7] = 2e6
    det, ref = detector(cfg, weights), detector(cfg, weights, "valu")
    sc, rsc = gpu_score(det, w)[0], gpu_score(ref, w)[0]
    np.testing.assert_allclose(sc, rsc, rtol=1e-5)
    det.close()
    ref.close()


# Half the inputs small under large weights, the other half ordinary: by metric, by step (the first half
# of every stream, so windows at its end hold both) or with the large factor in the heads' weights.
@pytest.mark.parametrize("where", ["metrics", "steps", "heads"])
@pytest.mark.parametrize("small,big,other", [(1e-5, 1e5, 1.0), (1e-6, 9e5, 1.0), (1e-8, 1e6, 1e-2)])
def test_small_inputs_under_large_weights(small, big, other, where):
    """A 16-bit part holds nothing below 2^-24, so inputs far below the window's largest may lose digits that
    large weights would bring back: such detectors keep fp32's precision (relative 2-norm 4e-6; fp32 sums
    measure 6e-7 to 9e-7)."""
    M, W, H = 8, 32, 64
    cfg = _cfg(M, W, 1, H, n=2)
    rng = np.random.default_rng(11)
    offs = np.array([0, 700, 1500], np.int64)
    x = rng.standard_normal((1500, M)) * 2.0
    weights = wl.make_weights(cfg, bias_scale=0.1)
    w1 = weights.w1.reshape(H, W, M)
    if where == "metrics":
        x[:, :4] *= small
        w1[:, :, :4] *= big
        w1[:, :, 4:] *= other
    elif where == "steps":
        x[:350] *= small
        x[700:1100] *= small
        w1[:, :W // 2] *= big
        w1[:, W // 2:] *= other
    else:
        x[:, :4] *= small
        w1[:H // 2, :, 4:] = 0.0
        w1[H // 2:, :, :4] = 0.0
        weights.b1[:H // 2] *= small
        for a in (weights.wmu, weights.wlv):
            a[:, :H // 2] *= big
            a[:, H // 2:] *= other
    w = wl.from_arrays(cfg, x, offs)
    ref = (np.zeros((2, M)), np.ones((2, M)))
    log(f"[split] small inputs {where} {small} {big} {other}")
    det = detector(cfg, weights)
    sc, md, _, _ = gpu_score(det, w, ref=ref)
    o_sc, o_md, info = oracle_score(cfg, w, weights, ref=ref)
    # large windows and the others apart: e^lv spans many decades, and leaves fp32's where ordinary inputs
    # meet the large weights
    few = np.flatnonzero(o_sc < 1e4)
    assert len(few) > 200
    for sel in (few, few[o_sc[few] < 10 * np.median(o_sc[few])]):
        err = np.linalg.norm(sc[sel] - o_sc[sel]) / np.linalg.norm(o_sc[sel])
        log(f"  {len(sel)} windows, relative error {err:.2e}")
        assert err <= 4e-6
    check_scores(sc[few], o_sc[few], "f32", where)
    check_md(md[few], o_md[few], info["md_scale"][few], "f32", where)
    det.close()


@pytest.mark.parametrize("M,W,S,H", [(7, 5, 2, 64), (4, 4, 8, 32), (5, 9, 4, 128), (3, 10, 8, 256), (16, 7, 3, 100)])
def test_steps_beside_a_window_do_not_count(M, W, S, H):
    """With W no multiple of S (or below it), a window's last super-row holds steps behind the window. Large,
    infinite and NaN ones there leave it finite, as the vector kernel has it, and its bits those of the
    stream cut off at its end, also where the window itself is out of the range."""
    cfg = _cfg(M, W, S, H, n=1)
    rng = np.random.default_rng(M * W)
    K = 150
    T = W + (K - 1) * S + S
    x = rng.standard_normal((T, M)).astype(np.float32)
    tail = W - (W - 1) // S * S                          # steps of the last super-row inside the window
    behind = [(k * S + W + (S - tail) // 2, k) for k in range(10, K - 1, 10)]
    for i, (t, k) in enumerate(behind):
        x[t, i % M] = [1e6, np.inf, np.nan, -np.inf, 4500.0][i % 5]
        if i % 2:
            x[k * S, 0] = 2e5                             # window k is out of the range by itself
    w = wl.from_arrays(cfg, x, np.array([0, T]))
    weights = wl.make_weights(cfg, bias_scale=0.1)
    ref = (np.zeros((1, M)), np.ones((1, M)))
    log(f"[split] steps beside a window M={M} W={W} S={S} H={H}")
    det, valu = detector(cfg, weights), detector(cfg, weights, "valu")
    (sc, md, _, _), (rsc, rmd, _, _) = gpu_score(det, w, pad=16, ref=ref), gpu_score(valu, w, ref=ref)
    own = np.array([np.isfinite(x[k * S:k * S + W]).all() for k in range(len(sc))])
    assert own[[k for _, k in behind]].all() and np.array_equal(np.isfinite(rmd), own)
    assert np.array_equal(np.isnan(md) | np.isinf(md), ~own)
    fin = own & np.isfinite(rsc) & (np.abs(rsc) < 1e30)
    assert np.array_equal(np.isinf(sc[own]), np.isinf(rsc[own])) and not np.any(np.isnan(sc[own]))
    np.testing.assert_allclose(sc[fin], rsc[fin], rtol=1e-5, atol=1e-6)
    for t, k in behind:
        cut = wl.from_arrays(cfg, x[:k * S + W], np.array([0, k * S + W]))
        a, b, _, _ = gpu_score(det, cut, ref=ref)
        assert len(a) == k + 1 and a[k] == sc[k] and b[k] == md[k], (k, a[k], sc[k])
    det.close()
    valu.close()


@pytest.mark.parametrize("M,W,H", [(1, 1, 64), (3, 1, 200), (1, 3, 32), (2, 2, 128), (1, 5, 64)])
def test_windows_of_few_values(M, W, H):
    """Below four values a window the fp32 kernel scores; from four on the split kernel leaves the quiet windows to
    its list."""
    cfg = _cfg(M, W, 1, H, n=2)
    rng = np.random.default_rng(M + W)
    offs = np.array([0, 3000, 4100], np.int64)
    log(f"[split] few values M={M} W={W} H={H}")
    w = wl.from_arrays(cfg, rng.standard_normal((4100, M)), offs)
    _check(cfg, w, wl.make_weights(cfg, bias_scale=0.1), f"M={M} W={W} H={H}")


@pytest.mark.parametrize("H", [32, 64, 128, 256])
def test_marked_parts_of_large_tiles(H):
    """Large tiles whose windows leave the range at the edges of their parts and waves, for one window, for a
    wave's, for a whole tile and more, against the vector kernel."""
    cfg = _cfg(2, 4, 1, H, n=2)
    n = {32: 262200, 64: 262200, 128: 131200, 256: 65700}[H]
    rng = np.random.default_rng(H)
    x = rng.standard_normal((n + 40, 2)).astype(np.float32)
    offs = np.array([0, n // 2 + 17, n + 40], np.int64)
    for at in (0, 31, 127, 131, 255, 512 + 64, 1024 + 383, 2048 + 511, offs[1] - 1, offs[1] + 3, offs[2] - 4):
        x[at, 1] = 1e5
    for a, b in ((5000, 5200), (7168, 8192), (9000, 11000), (int(offs[1]) + 4096 - 3, int(offs[1]) + 4608)):
        x[a:b, 0] = -7e4
    x[12000:60000:300, 1] = np.nan
    x[12100:60000:700, 0] = np.inf
    w = wl.from_arrays(cfg, x, offs)
    weights = wl.make_weights(cfg, bias_scale=0.1)
    ref = (np.zeros((2, 2)), np.ones((2, 2)))
    log(f"[split] marked parts H={H}, {n} windows")
    det, valu = detector(cfg, weights), detector(cfg, weights, "valu")
    (sc, md, _, _), (rsc, rmd, _, _) = gpu_score(det, w, pad=32, ref=ref), gpu_score(valu, w, ref=ref)
    assert np.array_equal(np.isfinite(md), np.isfinite(rmd)) and np.array_equal(np.isnan(sc), np.isnan(rsc))
    fin = np.isfinite(rsc) & (np.abs(rsc) < 1e30)
    np.testing.assert_allclose(sc[fin], rsc[fin], rtol=2e-5, atol=1e-6)
    ok = np.isfinite(rmd)
    np.testing.assert_allclose(md[ok], rmd[ok], rtol=2e-5, atol=1e-5)
    det.close()
    valu.close()
