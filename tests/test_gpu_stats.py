"""Reference statistics over metric counts, lengths and alignments at which their blocking changes:
against the oracle through ``enova_detect_ref_stats`` (one block per stream), and bit for bit against
the statistics a scoring call forms for itself (several blocks per stream where streams are few)."""
import numpy as np
import pytest

import oracle
from harness import log
from paper_2407_09486_amd import binding

pytestmark = pytest.mark.gpu


def _weights(W, M, H, dtype):
    rng = np.random.default_rng(3)
    D = W * M
    shapes = dict(w1=(H, D), b1=(H,), wmu=(2, H), bmu=(2,), wlv=(2, H), blv=(2,), wd1=(H, 2), bd1=(H,), wd2=(D, H),
                  bd2=(D,))
    w = {k: (rng.standard_normal(s) * 0.1).astype(np.float32) for k, s in shapes.items()}
    if dtype == "bf16":
        w["w1"] = (w["w1"].view(np.uint32) >> 16).astype(np.uint16)
    return w


# chunks of 16384 elements: one chunk, an exact number of them, one step more, more than the 32 at most;
# metric counts that divide 256, that do not, above 256 (several column groups), not a multiple of 4
@pytest.mark.parametrize("M,lengths,shift", [(8, [4096, 4098, 2, 1, 0, 70000], 0), (7, [300, 9364, 40001], 0),
                                             (1, [16384 * 2, 16384 * 2 + 3, 5], 1), (300, [40, 113, 1000], 0),
                                             (12, [20000, 37, 2731], 0), (16, [140000, 9], 1), (2, [33001], 0)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_statistics_over_blockings(M, lengths, shift, dtype):
    import torch
    log(f"[stats] M={M} lengths={lengths} shift={shift} {dtype}")
    rng = np.random.default_rng(M)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    x = (rng.standard_normal((int(offs[-1]), M)) * np.exp(rng.uniform(-2, 2, M)) + rng.uniform(-9, 9, M)).astype(np.float32)
    t = torch.from_numpy(x)
    if dtype == "bf16":
        t = t.to(torch.bfloat16)
        x = t.float().numpy()
    buf = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")   # shift: not 16-byte aligned
    buf[shift:] = t.reshape(-1).cuda()
    xd = buf[shift:].view(-1, M)
    W = 2
    det = binding.Detector(M, W, 1, 4, _weights(W, M, 4, dtype), latent=2, dtype=dtype)
    n = len(lengths)
    so = torch.from_numpy(offs).cuda()
    mean, std = torch.empty((n, M), device="cuda"), torch.empty((n, M), device="cuda")
    binding.enova_detect_ref_stats(det.handle, xd, so, n, mean, std)
    o_mean, o_std = oracle.ref_stats(x.astype(np.float64), offs, 0.5)
    np.testing.assert_allclose(mean.cpu().numpy(), o_mean, rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(std.cpu().numpy(), o_std, rtol=1e-6)
    wo_h = det.window_offsets(offs)
    wo, N = torch.from_numpy(wo_h).cuda(), int(wo_h[-1])
    own = det.score(xd, so, wo, N)
    given = det.score(xd, so, wo, N, mean, std)
    assert torch.equal(own[0], given[0]) and torch.equal(own[1], given[1])
    det.close()
