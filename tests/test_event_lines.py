"""The 16-byte lines that validation loads (csrc/geom.h, compiled for the host): every event lies in one of them, every
line holds an event, and an empty range, wherever it starts, loads none."""
import ctypes
import os
import subprocess

import pytest

import paper_2104_06336_amd.build_lib as build_lib

SOURCE = """
#include "geom.h"
extern "C" void lines(uint64_t base, int64_t e0, int64_t e1, int64_t* out) {
  const stem::Lines l = stem::lines_of((uintptr_t)base, e0, e1);
  out[0] = l.first;
  out[1] = l.n;
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("lines")
    src, so = os.path.join(d, "lines.hip"), os.path.join(d, "lines.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build_lib.HIPCC, *build_lib.FLAGS, "-shared", src, "-o", so], check=True, capture_output=True)
    fn = ctypes.CDLL(so).lines
    fn.restype = None
    fn.argtypes = [ctypes.c_uint64, ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]

    def call(base, e0, e1):
        out = (ctypes.c_int64 * 2)()
        fn(base, e0, e1, out)
        return out[0], out[1]
    return call


def test_lines_hold_events(lines):
    for base in (0x7F0000001000 + 4 * k for k in range(4)):  # an int32 array at any place in a line
        for e0 in list(range(9)) + [2 ** 31 + 1, 2 ** 33 + 2]:
            for n in range(1, 20):
                first, m = lines(base, e0, e0 + n)
                a = base + 4 * first
                assert a % 16 == 0 and a <= base + 4 * e0 < a + 16
                assert a + 16 * (m - 1) <= base + 4 * (e0 + n - 1) < a + 16 * m


def test_empty_range_loads_nothing(lines):
    for base in (0x7F0000001000 + 4 * k for k in range(4)):
        for e0 in range(9):
            assert lines(base, e0, e0)[1] == 0
