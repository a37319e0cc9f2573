"""The threshold call over the sizes at which its launches change: more streams than its offsets table
in LDS holds, both block sizes (beyond 4 M windows), several runs a block (beyond 33 M), calibration
sets that end inside a block, none, one and nine peaks, and heavy and light tails, against the oracle's
order statistic and fit on the same scores. Both sides fit in fp64; the roots agree to rounding, gamma
and sigma to 1e-7."""
import numpy as np
import pytest

import oracle
from harness import log
from paper_2407_09486_amd import binding

pytestmark = pytest.mark.gpu


def _det(W, S):
    D = W
    shapes = dict(w1=(1, D), b1=(1,), wmu=(1, 1), bmu=(1,), wlv=(1, 1), blv=(1,), wd1=(1, 1), bd1=(1,), wd2=(D, 1),
                  bd2=(D,))
    return binding.Detector(1, W, S, 1, {k: np.full(s, 0.1, np.float32) for k, s in shapes.items()}, latent=1)


@pytest.mark.parametrize("what,lengths,W,S,level,tail", [
    ("one block", [2048 + 8], 9, 1, 0.98, 0.3),
    ("ragged streams", [5000, 3, 0, 9, 777, 20000], 7, 2, 0.9, -0.2),
    ("2047 streams", [40] * 2047, 4, 1, 0.98, 0.1),
    ("2048 streams", [40] * 2047 + [900], 4, 1, 0.98, 0.1),
    ("3000 streams", list(range(3, 3003)), 4, 3, 0.95, 0.5),
    ("over 4 M windows", [4_300_000, 200_001], 2, 1, 0.98, 0.2),
    ("over 33 M windows", [33_600_000, 3, 500_001], 2, 1, 0.999, 0.2),
    ("nine peaks", [920], 2, 1, 0.98, 0.2),
    ("ten peaks", [1002], 2, 1, 0.98, 0.2),
    ("one peak", [60], 2, 1, 0.98, 0.2),
    ("no peak", [6], 2, 1, 0.98, 0.2),
    ("low level", [9000, 100], 5, 1, 0.05, 0.0),
])
def test_threshold_over_sizes(what, lengths, W, S, level, tail):
    import torch
    log(f"[threshold] {what}")
    det = _det(W, S)
    so_h = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    wo_h = det.window_offsets(so_h)
    n = int(wo_h[-1])
    rng = np.random.default_rng(len(lengths))
    u = rng.random(n)
    scores = ((u ** -tail - 1) / tail if tail else -np.log(u)).astype(np.float32)
    so, wo, sc = torch.from_numpy(so_h).cuda(), torch.from_numpy(wo_h).cuda(), torch.from_numpy(scores).cuda()
    cal = oracle.calibration_scores(scores.astype(np.float64), so_h, window=W, stride=S)
    want, info_o = oracle.pot_threshold(cal, level=level, q=1e-3)
    for _ in range(2):                                  # the second call finds the first one's state
        thr, info, flags = det.threshold(sc, so, wo, level=level, q=1e-3, flags=True)
        assert info["t"] == info_o["t"] and info["n"] == len(cal) and info["n_peaks"] == info_o["n_peaks"]
        assert info["method"] == info_o["method"]
        assert abs(thr - want) <= 2e-7 * abs(want), (thr, want)
        for k in ("gamma", "sigma"):
            a, b = info[k], info_o[k]
            assert (np.isnan(a) and (b is None or np.isnan(b))) or abs(a - b) <= 1e-7 * max(abs(b), 1e-3), (k, a, b)
        assert np.array_equal(flags.cpu().numpy(), (scores > np.float32(thr)).astype(np.uint8))
    det.close()


def test_threshold_errors_write_no_flags():
    import torch
    det = _det(4, 1)
    so_h = np.array([0, 300], np.int64)
    wo_h = det.window_offsets(so_h)
    so, wo = torch.from_numpy(so_h).cuda(), torch.from_numpy(wo_h).cuda()
    flags = torch.full((297,), 7, dtype=torch.uint8, device="cuda")
    for bad, scores in (("inf", torch.full((297,), np.inf)), ("a peak is inf", torch.cat([torch.rand(140) + 1, torch.full((157,), np.inf)]))):
        if bad != "inf":
            scores[139] = 1.0
            scores[3] = np.inf
        log(f"[threshold] {bad}")
        with pytest.raises(binding.EnovaError) as e:
            binding.enova_detect_threshold(det.handle, scores.float().cuda(), so, wo, 1, 297, 0.9, 1e-3, flags)
        assert e.value.status == binding.ENOVA_ENUMERIC
    short = np.array([0, 5], np.int64)                  # no window inside the prefix of two steps
    s2, w2 = torch.from_numpy(short).cuda(), torch.from_numpy(det.window_offsets(short)).cuda()
    with pytest.raises(binding.EnovaError) as e:
        binding.enova_detect_threshold(det.handle, torch.rand(2, device="cuda"), s2, w2, 1, 2, 0.9, 1e-3, flags[:2])
    assert e.value.status == binding.ENOVA_ESHAPE
    torch.cuda.synchronize()
    assert torch.all(flags == 7)
    det.close()
