"""Binning in several chunks of pixels by 64 frames a workgroup (more than 800 pixels, 2^13 to 2^16 frames) and by 128
(363 to 543 and more than 800 pixels past 2^16 frames), with and without the centre of mass of the same pass, 8- and
16-bit counts.  Bit for bit the oracle's."""
import numpy as np
import pytest
import torch

import paper_2104_06336_amd as stem
from oracle import eer as oeer

pytestmark = pytest.mark.gpu

W = 96


@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("r,bin_,scan", [(33.5, 2, (96, 90)), (36.0, 3, (270, 250)), (33.5, 2, (270, 250))],
                         ids=["64 frames", "128 frames, 3 chunks", "128 frames, 5 chunks"])
def test_chunks(gpu, r, bin_, scan, bits):
    print(f"\n[gpu] bin rule r {r} bin {bin_} scan {scan} bits {bits}", flush=True)
    kc, lut = oeer.bin_geometry(W, W, bin_, r)
    F = scan[0] * scan[1]
    rng = np.random.default_rng(F)
    n = rng.integers(0, 30, size=F)
    n[[1, F // 3]] = 300  # two workgroups with 16-bit counters
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    idx = rng.integers(0, W * W, size=int(off[-1])).astype(np.int32)
    ref = np.asarray(oeer.bin_counts(idx, off, W, bin_, lut)).astype(np.int64)
    det, sc = stem.Det(W, W, W // 2, W // 2, bin_), stem.Scan(scan[0], scan[1], 0.2)
    st = stem.SsbState(det, sc, stem.Optics.from_values(0.0196875, r, 1.27 / r, (0.0,) * 8),
                       stem.Ssb(stem.STEM_FFT_FP32, 0, stem.STEM_G_RECOMPUTE, bits))
    assert st.n_k == len(kc) and (363 <= st.n_k <= 543 if bin_ == 3 else 801 <= st.n_k <= 905)
    d_idx, d_off = torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda()
    com = torch.zeros(2 * F, dtype=torch.float64, device="cuda")
    for kw in ({}, {"com64": com}):
        st.region(stem.STEM_REGION_D).fill_(77)
        st.accumulate(d_idx, d_off, 0, F, **kw)
        D = st.region(stem.STEM_REGION_D).view(torch.uint8 if bits == 8 else torch.int16).cpu().numpy()
        assert int(st.status.item()) == 0
        assert np.array_equal(D.reshape(len(kc), F).astype(np.int64), ref)
    cx, cy, *_ = oeer.com(idx, off, W, W)
    assert np.array_equal(com.cpu().numpy().reshape(2, F), np.stack([cx, cy]))
