"""Host check of the two-step kernel's addressing (no GPU).

tests/twostep_check.cpp runs csrc/twostep.h, which the kernel is built from, for
every tile, wave, lane and plane of ragged grids: bounds of every load, store
and LDS place, what the second step reads against the reference pull, every slot
stored once, and the split into chunks.
"""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2112_08479_amd", "csrc")


@pytest.mark.timeout(300)
def test_two_step_addressing():
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "twostep_check")
        r = subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC,
                            "-o", exe, os.path.join(HERE, "twostep_check.cpp")], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        r = subprocess.run([exe], capture_output=True, text=True, timeout=240)
        assert r.returncode == 0 and "fails 0" in r.stdout, r.stdout[-2000:]
