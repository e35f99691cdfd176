"""Every scan length the library accepts gets a launch from each kernel of the mixed-radix transforms: at least one
row (or pixel, or row pair) per workgroup, butterflies within a thread's registers, LDS within a compute
unit's 160 KB.  The plans and the row counts are the built library's own (host code, no GPU)."""
import ctypes

import paper_2104_06336_amd as stem

LDS = 160 * 1024
STATIC = 16 * 1024  # more than the static LDS beside the rows in any of the three kernels


class Pass(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int32) for k in ("r", "m", "ns", "off", "step", "rp", "rq", "wp")] + [
        ("mm", ctypes.c_uint32), ("mns", ctypes.c_uint32)]


class Plan(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int32) for k in ("n", "np", "ntw", "len")] + [("mn", ctypes.c_uint32), ("p", Pass * 6)]


def _lengths():
    def smooth(n):
        for p in (2, 3, 5):
            while n % p == 0:
                n //= p
        return n == 1
    return [n for n in range(16, 4097, 2) if smooth(n)]


def _lds(p, rows, stride):
    return 8 * ((p.ntw + 1) // 2 * 2 + max(rows * stride, 256))


def _fits(p, rows, threads, ept):
    """rows of every pass within the registers of the workgroup's threads"""
    return all(rows * p.p[s].m <= threads * max(1, ept // p.p[s].r) for s in range(p.np))


def test_every_accepted_length_has_a_launch():
    lib = stem.lib()
    ok, plan = lib._ZN4stem14scan_length_okEi, lib._ZN4stem8gen_planEiRNS_5GPlanE
    ok.restype = plan.restype = ctypes.c_bool
    gsum = lib._ZN4stem9gsum_rowsEiRNS_5GPlanE
    rows_of = lib._ZN4stem12gen_fft_rowsERKNS_5GPlanEl
    pairs_of = lib._ZN4stem10gen_x_rowsERKNS_5GPlanElRi
    lengths = _lengths()
    assert len(lengths) == 104 and {n for n in range(4098) if ok(n)} == set(lengths)
    for n in lengths:
        p = Plan()
        assert plan(n, ctypes.byref(p)) and p.n == n and p.len >= n
        # the fused column sum: 256 threads up to 2048, then 512; one last butterfly per thread
        q = Plan()
        rows, threads = gsum(n, ctypes.byref(q)), 512 if n > 2048 else 256
        last = q.p[q.np - 1]
        assert rows >= 1, n
        assert rows * last.m <= threads and _fits(q, rows, threads, 12 if last.r <= 12 else 16), n
        assert _lds(q, rows, q.len) + STATIC <= LDS, n
        for nrows in (2, 16, 256, 4096, 4096 * 4096):
            rows = rows_of(ctypes.byref(p), ctypes.c_int64(nrows))
            assert rows >= 1 and _fits(p, rows, 256, 30) and _lds(p, rows, p.len) + STATIC <= LDS, (n, nrows)
            stride = ctypes.c_int(0)
            lrb = pairs_of(ctypes.byref(p), ctypes.c_int64(nrows), ctypes.byref(stride))
            assert lrb >= 0 and stride.value >= p.len, (n, nrows)
            assert _fits(p, 1 << lrb, 512, 20) and _lds(p, 1 << lrb, stride.value) + STATIC <= LDS, (n, nrows)
