"""Validation of chunks that hold no event (no frames' events at all, empty frames between others) and of single events at
every place in a 16-byte line, with indices outside the detector beside them in the line, which are not reported."""
import pytest
import torch

import paper_2104_06336_amd as stem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("place", range(4))
def test_validate(gpu, place):
    print(f"\n[gpu] validation at place {place} of a line", flush=True)
    det = stem.Det(8, 8, 4, 4, 1)
    buf = torch.full((64,), 64, dtype=torch.int32, device="cuda")  # every entry past the detector
    for first in range(4):
        d_idx = buf[place:]
        e = 16 + first
        d_idx[e] = 63
        empty = torch.full((6,), e, dtype=torch.int64, device="cuda")
        one = torch.tensor([e, e, e + 1, e + 1], dtype=torch.int64, device="cuda")
        two = torch.tensor([e, e + 2], dtype=torch.int64, device="cuda")
        for off, want in ((empty, 0), (one, 0), (two, 2)):  # STEM_ERANGE: the second event is past the detector
            status = stem.status_tensor()
            stem.eer_load_csr(None, None, 0, off.numel() - 1, d_idx.numel(), det, d_idx, off, d_status=status)
            assert int(status.item()) == want
        d_idx[e] = 64
    # no events in the whole array: nothing of it is read, whatever it starts with
    off = torch.zeros(5, dtype=torch.int64, device="cuda")
    status = stem.status_tensor()
    stem.eer_load_csr(None, None, 0, 4, 0, det, buf[place:place + 1], off, d_status=status)
    assert int(status.item()) == 0
