"""Binning workgroups of 128, 64 and 32 frames (by the number of kept pixels) at the edges of each: the last
number of pixels one workgroup holds and the first it does not, frame blocks that are not whole, whole
scans and row chunks, 8- and 16-bit counts, blocks of one and of several windows of events, and frames of
more than 255 events (16-bit counters in two passes).  The centre of mass of the same pass is compared
with the oracle's too.  The cube is compared with the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import paper_2104_06336_amd as stem
from oracle import eer as oeer

pytestmark = pytest.mark.gpu

W = 96


def _radius(n_k, bin_):
    """A radius that keeps at least n_k bins, as few as possible."""
    c = (np.arange(W // bin_) * bin_ + 0.5 * (bin_ - 1) - W // 2) ** 2
    d2 = np.sort((c[:, None] + c[None, :]).ravel())
    return float(np.sqrt(0.5 * (d2[n_k - 1] + d2[d2 > d2[n_k - 1]][0])))


# kept pixels asked for (the disk's symmetry gives up to 8 more), binning, scan
@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("n_k,bin_,scan", [(172, 4, (16, 48)), (184, 4, (32, 32)), (344, 3, (18, 30)),
                                           (352, 3, (64, 64)), (790, 2, (16, 36)), (804, 2, (32, 32))],
                         ids=lambda v: str(v) if not isinstance(v, tuple) else f"{v[0]}x{v[1]}")
def test_cube(gpu, n_k, bin_, scan, bits):
    print(f"\n[gpu] cube n_k {n_k} bin {bin_} scan {scan} bits {bits}", flush=True)
    r = _radius(n_k, bin_)
    kc, lut = oeer.bin_geometry(W, W, bin_, r)
    F = scan[0] * scan[1]
    rng = np.random.default_rng(n_k)
    for pile, most in ((0, 40), (300, 40), (0, 255)):
        n = rng.integers(0, most, size=F)  # up to 254: several windows per block, most not on a 16-byte line
        if pile:
            n[[0, F // 2, F - 1]] = pile  # past 255 events: the 16-bit counters
        off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
        idx = rng.integers(0, W * W, size=int(off[-1])).astype(np.int32)
        ref = oeer.bin_counts(idx, off, W, bin_, lut)
        det = stem.Det(W, W, W // 2, W // 2, bin_)
        sc = stem.Scan(scan[0], scan[1], 0.2)
        optics = stem.Optics.from_values(0.0196875, r, 1.27 / r, (0.0,) * 8)
        st = stem.SsbState(det, sc, optics, stem.Ssb(stem.STEM_FFT_FP32, 0, stem.STEM_G_RECOMPUTE, bits))
        assert st.n_k == len(kc)
        d_idx, d_off = torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda()
        for rows in (scan[0], 5):
            st.region(stem.STEM_REGION_D).fill_(77)
            com = torch.zeros(2 * F, dtype=torch.float64, device="cuda") if rows == 5 else None
            for y in range(0, scan[0], rows):
                st.accumulate(d_idx, d_off, y * scan[1], min(rows, scan[0] - y) * scan[1], com64=com)
            D = st.region(stem.STEM_REGION_D).view(torch.uint8 if bits == 8 else torch.int16).cpu().numpy()
            assert int(st.status.item()) == 0
            assert np.array_equal(D.reshape(len(kc), F).astype(np.int64), np.asarray(ref).astype(np.int64))
            if com is not None:
                cx, cy, *_ = oeer.com(idx, off, W, W)
                assert np.array_equal(com.cpu().numpy().reshape(2, F), np.stack([cx, cy]))
