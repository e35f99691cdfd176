"""The sum of frames accumulates modulo 2^32 in every pixel by itself: sums that start just below 2^32 wrap, and their
neighbours hold their own counts, for detectors whose sums are added in pairs (even width) and one by one (odd width, a
sum off an 8-byte boundary).  Whole numbers, equal to the reference's."""
import numpy as np
import pytest
import torch

import paper_2104_06336_amd as stem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,shift", [(96, 64, 0), (96, 64, 1), (97, 64, 0), (300, 200, 0)],
                         ids=["pairs", "off 8 bytes", "odd width", "box inside"])
def test_each_pixel_wraps_alone(gpu, W, H, shift):
    print(f"\n[gpu] sum of frames past 2^32, {W}x{H} shift {shift}", flush=True)
    rng = np.random.default_rng(W + shift)
    F, C = 500, 200_000
    idx = rng.integers(0, W * H, size=C).astype(np.int32)
    off = np.linspace(0, C, F + 1).astype(np.int64)
    before = rng.integers(0, 2 ** 32, size=W * H, dtype=np.uint64)
    low = rng.random(W * H) < 0.7
    before[low] = 2 ** 32 - 1 - rng.integers(0, 30, size=int(low.sum()), dtype=np.uint64)
    buf = torch.zeros(W * H + 2, dtype=torch.int32, device="cuda")
    total = buf[shift:shift + W * H]
    total.copy_(torch.from_numpy(before.astype(np.uint32).view(np.int32)))
    mean = torch.zeros(W * H, dtype=torch.float32, device="cuda")
    d_idx, d_off = torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda()
    det, status = stem.Det(W, H, W // 2, H // 2, 1), stem.status_tensor()
    ref = before
    for f0, n in ((0, F // 2), (F // 2, F - F // 2), (0, F)):  # chunks of one acquisition, then it again
        stem.sum_frames(d_idx, d_off, f0, n, det, total, mean, d_status=status)
        counts = np.bincount(idx[off[f0]:off[f0 + n]], minlength=W * H).astype(np.uint64)
        ref = (ref + counts) % 2 ** 32
        assert np.array_equal(total.cpu().numpy().view(np.uint32).astype(np.uint64), ref)
        assert np.array_equal(mean.cpu().numpy(), (ref.astype(np.float64) / n).astype(np.float32))
    assert int(status.item()) == 0
    assert int(buf[W * H + 1].item()) == 0 and (shift == 0 or int(buf[0].item()) == 0)
