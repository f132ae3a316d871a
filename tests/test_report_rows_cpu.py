"""Host checks of the reporting kernels at the far ends of the grids that
lbm_create takes (no GPU): tests/report_rows_check.cpp runs the addressing of
csrc/lattice.h for rows whose offsets pass 32 bits, tests/diag_launch_check.cpp
the size of the diagnostics' launch."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def run(source):
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "check")
        r = subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I",
                            os.path.join(ROOT, "paper_2112_08479_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                            "-o", exe, os.path.join(HERE, source)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        r = subprocess.run([exe], capture_output=True, text=True, timeout=240)
        assert r.returncode == 0 and "fails 0" in r.stdout, r.stdout[-2000:]


@pytest.mark.timeout(300)
def test_rows_beyond_32_bit_offsets():
    run("report_rows_check.cpp")


@pytest.mark.timeout(300)
def test_diagnostics_launch_size():
    run("diag_launch_check.cpp")
