"""The host eigensolvers leave part of the CPUs to the rest of the process (CPU)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("cpus,threads", [("1", 1), ("2", 2), ("4", 3), ("8", 6), ("16", 12), ("64", 12), ("0", 1)])
def test_host_threads(cpus, threads):
    code = "import ctypes, sys; print(ctypes.CDLL(sys.argv[1])._ZN3bse12host_threadsEv())"
    lib = os.path.join(ROOT, "paper_2504_10096_amd", "libbse.so")
    out = subprocess.run([sys.executable, "-c", code, lib], capture_output=True, text=True, check=True,
                         env=dict(os.environ, OMP_NUM_THREADS=cpus)).stdout
    assert int(out) == threads
