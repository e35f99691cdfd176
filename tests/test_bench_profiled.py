"""The kernels whose counted traffic bench.py reports are kernels of the built library under those names (a template
parameter that changes would drop them from the counters' summary without a word)."""
import subprocess

import bench
import paper_2104_06336_amd.build_lib as build_lib


def test_profiled_names_exist():
    out = subprocess.run(["nm", "-DC", build_lib.LIB], check=True, capture_output=True, text=True).stdout
    kernels = [line.split(" ", 2)[-1].removeprefix("void ") for line in out.splitlines() if "stem::k_" in line]
    for name in bench.PROFILED:
        assert any(k.startswith(name + "(") for k in kernels), name
