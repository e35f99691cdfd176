"""The mixed-radix transforms and the fused column sum at lengths that reach every radix, pass count and
edge of their plans: two to four passes, radices 2 to 16, both sides of the fused sum's change from 256
to 512 threads (2048), a fast length beside another one, fewer pixels than a workgroup takes at once,
16-bit counts, and chunks of pixels.  Against the FP64 oracle, rel-L2 1e-5 (the FP32 target of every
transform here)."""
import numpy as np
import pytest
import torch

import paper_2104_06336_amd as stem
from gen import C4_TRUE_ABERRATIONS, WORKLOADS, simulate
from oracle import ssb as ossb

from helpers import gpu_com, gpu_ssb, oracle_dpc, oracle_pruned, oracle_row_dft, oracle_ssb, rel_l2, state_pruned, state_X, structs

pytestmark = pytest.mark.gpu

TOL = 1e-5
# scan, bin, bits: 18 = 2.9, 50 = 5.10, 150 = 10.15, 36 = 4.9 / 6.6, 54 = 6.9, 240 = 15.16, 32 and 64 fast,
# 2250 and 3750 four passes or 512 threads, 2048 the last length of 256 threads
SCANS = [((18, 50), 4, 8), ((150, 36), 4, 16), ((32, 54), 2, 8), ((240, 64), 4, 8), ((2250, 16), 8, 8),
         ((16, 3750), 8, 16), ((2048, 20), 8, 8)]


@pytest.mark.parametrize("g_mode", [stem.STEM_G_STORE, stem.STEM_G_RECOMPUTE], ids=["store", "recompute"])
@pytest.mark.parametrize("scan,bin_,bits", SCANS, ids=[f"{s[0]}x{s[1]}" for s, _, _ in SCANS])
def test_plans(gpu, scan, bin_, bits, g_mode):
    print(f"\n[gpu] plans {scan} bin {bin_} bits {bits} mode {g_mode}", flush=True)
    wl = WORKLOADS["small"].replace(name=f"scan {scan}", scan=scan, bin=bin_, mean_e=20.0)
    d = simulate(wl, device="cuda")
    d_idx, d_off = d.idx.contiguous(), d.off.contiguous()
    idx, off = d_idx.cpu().numpy(), d_off.cpu().numpy()
    plain = oracle_ssb(idx, off, wl)
    n_k = len(plain["kc"])
    npair = int(ossb.ssb_sum(np.zeros((n_k,) + scan), plain["kc"], wl.step, wl.dk, wl.lam, wl.r_bf)[1].sum())
    th = np.random.default_rng(5).uniform(-0.3, 0.3, size=n_k).astype(np.float32)
    ab = oracle_ssb(idx, off, wl, c=C4_TRUE_ABERRATIONS, theta=th)
    for scratch in (0, 1):
        for c, theta, ref in (((0.0,) * 8, None, plain), (C4_TRUE_ABERRATIONS, th, ab)):
            st, out = gpu_ssb(d_idx, d_off, wl, c=c, theta=theta, g_mode=g_mode, d_bits=bits, scratch_mib=scratch)
            assert out["status"] == 0
            assert rel_l2(out["T"], ref["T"]) <= TOL and rel_l2(out["phi"], ref["phi"]) <= TOL
            assert st.stats()[0] == npair
        if g_mode == stem.STEM_G_STORE:
            assert rel_l2(state_X(st, wl), oracle_row_dft(plain["D"], wl)) <= TOL
            pg, poff = state_pruned(st)
            pg_ref, poff_ref = oracle_pruned(plain["G"], plain["kc"], wl)
            assert np.array_equal(poff, poff_ref) and rel_l2(pg, pg_ref) <= TOL
    g = gpu_com(d_idx, d_off, wl, phase=True)
    assert rel_l2(g["phase"], oracle_dpc(idx, off, wl)) <= TOL


@pytest.mark.parametrize("g_mode", [stem.STEM_G_STORE, stem.STEM_G_RECOMPUTE], ids=["store", "recompute"])
@pytest.mark.parametrize("scan", [(48, 80), (54, 64)], ids=["48x80", "54x64"])
def test_fit(gpu, scan, g_mode):
    """SSBPhase on accumulated events: the phase, then dL/dc and dL/dtheta against the oracle gradient, at the
    first coefficients (FINALIZE) and at others (from the stored values in STORE); 1e-4 per component, the
    tolerance of every adjoint here."""
    print(f"\n[gpu] fit {scan} mode {g_mode}", flush=True)
    wl = WORKLOADS["small"].replace(name=f"fit {scan}", scan=scan, bin=2, mean_e=20.0)
    d = simulate(wl, device="cuda")
    d_idx, d_off = d.idx.contiguous(), d.off.contiguous()
    idx, off = d_idx.cpu().numpy(), d_off.cpu().numpy()
    det, sc, optics = structs(wl)
    st = stem.SsbState(det, sc, optics, stem.Ssb(stem.STEM_FFT_FP32, 0, g_mode, 8, 1))
    st.accumulate(d_idx, d_off, 0, wl.n_frames)
    rng = np.random.default_rng(11)
    th = rng.uniform(-0.3, 0.3, size=st.n_k).astype(np.float32)
    for k in range(2):
        c = tuple(np.array(C4_TRUE_ABERRATIONS) * (1 + rng.uniform(-0.5, 0.5, size=8)))
        ct = torch.tensor(c, dtype=torch.float64, requires_grad=True)
        tt = torch.from_numpy(th).cuda().requires_grad_(True)
        phi = stem.SSBPhase.apply(ct, tt, st)
        (-torch.var(phi, unbiased=False)).backward()
        ref = oracle_ssb(idx, off, wl, c=c, theta=th)
        assert int(st.status.item()) == 0
        assert rel_l2(phi.detach().cpu().numpy(), ref["phi"]) <= TOL
        dco, dtho = ossb.ssb_adjoint(ref["G"], ref["kc"], ossb.neg_var_grad(ref["phi"]), wl.step, wl.dk, wl.lam,
                                     wl.r_bf, c, th)
        dc = ct.grad.numpy()
        assert np.all(np.abs(dc - dco) <= 1e-4 * np.abs(dco) + 1e-6 * np.max(np.abs(dco)))
        assert rel_l2(tt.grad.cpu().numpy(), dtho) <= 1e-4
