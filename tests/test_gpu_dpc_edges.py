"""DPC integration where the descent's geometric sum is not finite or has no terms: settings that diverge (mu = 5, so
|1 - mu q^2 / d| = 4 and 4^2000 overflows a double) on gradients that vanish at every frequency but q = 0, which is held at
zero, and no iterations at all on a gradient of NaN.  Step by step, Phi stays at exactly zero in all of them, so the phase
is zero.  (A constant's transform vanishes exactly only where the length is a power of two.)"""
import pytest
import torch

import paper_2104_06336_amd as stem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("com,mu,n_iter,scan", [(0.0, 5.0, 2000, (64, 64)), (0.0, 5.0, 2000, (48, 80)),
                                                (0.25, 5.0, 2000, (64, 64)), (float("nan"), 0.5, 0, (64, 64)),
                                                (float("nan"), 0.5, 0, (48, 80))])
def test_zero_phase(gpu, com, mu, n_iter, scan):
    print(f"\n[gpu] dpc of com {com}, mu {mu}, {n_iter} iterations, scan {scan}", flush=True)
    ny, nx = scan
    F = ny * nx
    det, sc = stem.Det(64, 64, 32, 32, 1), stem.Scan(ny, nx, 0.2)
    c64 = torch.full((2 * F,), com, dtype=torch.float64, device="cuda")
    phase = torch.full((F,), 7.0, device="cuda")
    ws = torch.empty(stem.com_dpc_workspace_bytes(sc), dtype=torch.uint8, device="cuda")
    idx, off = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(F + 1, dtype=torch.int64, device="cuda")
    status = stem.status_tensor()
    stem.com_dpc(idx, off, 0, 0, det, sc, stem.Optics.from_values(0.0196875, 10.0, 0.1, (0.0,) * 8),
                 stem.Dpc(mu, 0.0, 0.0, n_iter), com64=c64, phase=phase, ws=ws, d_status=status)
    assert int(status.item()) == 0
    assert torch.equal(phase, torch.zeros_like(phase))
