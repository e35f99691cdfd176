"""The rule for the binning's frames per workgroup (host code of the built library, no GPU): a workgroup of less than
128 frames only where it takes fewer chunks of pixels, and for a large scan only where that is one chunk."""
import ctypes

import pytest

import paper_2104_06336_amd as stem

HOLDS = {128: 181, 64: 351, 32: 800}  # kept pixels a workgroup's counters hold


def _frames(n_k, n_frames):
    return stem.lib()._ZN4stem10bin_framesEil(n_k, ctypes.c_int64(n_frames))


@pytest.mark.parametrize("n_frames", [1, 64 * 64, 2 ** 13 + 1, 2 ** 15, 2 ** 15 + 1, 2 ** 16 + 1, 2 ** 18, 2 ** 18 + 1, 2 ** 20,
                                      4096 * 4096])
def test_fewer_chunks(n_frames):
    for n_k in range(1, 4097):
        fr = _frames(n_k, n_frames)
        chunks = {f: -(-n_k // h) for f, h in HOLDS.items()}
        assert fr in HOLDS
        if fr < 128:
            assert chunks[fr] < chunks[128] and chunks[fr] <= chunks[min(128, 2 * fr)], (n_k, n_frames)
            if n_frames > 2 ** 16:
                assert chunks[fr] == 1, (n_k, n_frames)
            if n_frames > 2 ** 18:
                assert n_k <= HOLDS[64] or chunks[128] >= 5, (n_k, n_frames)
