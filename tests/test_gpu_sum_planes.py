"""The fused sum's planes of partials where a scan has 257 column sets: five or three planes of workgroup sums with the
values written (from 100 pixels on, and below), the waves' own ten in one chunk of pixels without, three on the matrix
cores with few pixels and with several chunks.  T and the phase against the FP64 oracle (rel-L2 1e-5, BF16 1e-4: the
targets of every sum here), the number of planes as the state reports it."""
import pytest
import torch

import paper_2104_06336_amd as stem
from gen import C4_TRUE_ABERRATIONS, WORKLOADS, simulate

from helpers import gpu_ssb, oracle_ssb, rel_l2

pytestmark = pytest.mark.gpu

FP32, BF16 = stem.STEM_FFT_FP32, stem.STEM_DFT_BF16_SPLIT
STORE, RECOMPUTE = stem.STEM_G_STORE, stem.STEM_G_RECOMPUTE


@pytest.mark.parametrize("scan", [(1024, 512), (512, 1024)], ids=["1024x512", "512x1024"])
@pytest.mark.parametrize("bin_", [2, 4], ids=["more pixels", "fewer pixels"])
def test_planes(gpu, scan, bin_):
    wl = WORKLOADS["small"].replace(name=f"planes {scan}", scan=scan, bin=bin_, r_bf=12.0, mean_e=3.0)
    d = simulate(wl, device="cuda")
    d_idx, d_off = d.idx.contiguous(), d.off.contiguous()
    idx, off = d_idx.cpu().numpy(), d_off.cpu().numpy()
    ref = oracle_ssb(idx, off, wl, c=C4_TRUE_ABERRATIONS)
    n_k = len(ref["kc"])
    more = bin_ == 2
    assert 100 <= n_k < 140 if more else 20 <= n_k < 100
    for g_mode, prec, mib, planes, tol in ((STORE, FP32, 0, 5 if more else 3, 1e-5), (RECOMPUTE, FP32, 4096, 10, 1e-5),
                                           (RECOMPUTE, BF16, 4096, 3, 1e-4), (RECOMPUTE, FP32, 32, 3, 1e-5)):
        print(f"\n[gpu] planes {scan} n_k {n_k} mode {g_mode} precision {prec} scratch {mib}", flush=True)
        st, out = gpu_ssb(d_idx, d_off, wl, c=C4_TRUE_ABERRATIONS, g_mode=g_mode, precision=prec, scratch_mib=mib)
        assert out["status"] == 0
        assert st.stats()[1] == planes
        assert rel_l2(out["T"], ref["T"]) <= tol and rel_l2(out["phi"], ref["phi"]) <= tol
        del st
        torch.cuda.empty_cache()
