"""The longest padded row of the mixed-radix plans (3888 = 6.8.9.9, 4374 LDS elements, more than 4096's) in both
directions: the reconstruction in one call and by FINALIZE and REFOCUS after chunks, in both G modes, with and
without phase factors.  Against the FP64 oracle, rel-L2 1e-5 (the FP32 target of every transform here)."""
import numpy as np
import pytest
import torch

import paper_2104_06336_amd as stem
from gen import C4_TRUE_ABERRATIONS, WORKLOADS, simulate

from helpers import gpu_ssb, oracle_ssb, rel_l2

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("g_mode", [stem.STEM_G_STORE, stem.STEM_G_RECOMPUTE], ids=["store", "recompute"])
@pytest.mark.parametrize("scan", [(3888, 16), (16, 3888)], ids=["3888x16", "16x3888"])
def test_longest_row(gpu, scan, g_mode):
    print(f"\n[gpu] longest padded row {scan} mode {g_mode}", flush=True)
    wl = WORKLOADS["small"].replace(name=f"scan {scan}", scan=scan, bin=8, mean_e=20.0)
    d = simulate(wl, device="cuda")
    d_idx, d_off = d.idx.contiguous(), d.off.contiguous()
    idx, off = d_idx.cpu().numpy(), d_off.cpu().numpy()
    plain, ab = oracle_ssb(idx, off, wl), oracle_ssb(idx, off, wl, c=C4_TRUE_ABERRATIONS)
    for c, ref in (((0.0,) * 8, plain), (C4_TRUE_ABERRATIONS, ab)):
        _, out = gpu_ssb(d_idx, d_off, wl, c=c, g_mode=g_mode)
        assert out["status"] == 0
        assert rel_l2(out["T"], ref["T"]) <= TOL and rel_l2(out["phi"], ref["phi"]) <= TOL
    st, out = gpu_ssb(d_idx, d_off, wl, g_mode=g_mode, chunk_rows=max(1, scan[0] // 3), scratch_mib=1)
    assert rel_l2(out["T"], plain["T"]) <= TOL
    T = torch.zeros(wl.n_frames, dtype=torch.complex64, device="cuda")
    st.refocus(c=C4_TRUE_ABERRATIONS, T=T)
    assert int(st.status.item()) == 0
    assert rel_l2(T.cpu().numpy().reshape(scan), ab["T"]) <= TOL
