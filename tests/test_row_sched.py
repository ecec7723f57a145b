"""Work order of the one-row late kernels where heads are split over the XCDs
(csrc/wise_device.hpp): every row once, even shares.  Host code."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("/opt/rocm/bin/hipcc") is None, reason="no HIP compiler")
def test_every_row_once(tmp_path):
    exe = tmp_path / "sched"
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2609_27373_amd", "csrc"),
                    os.path.join(ROOT, "tests", "row_sched.cpp"), "-o", str(exe)], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", (res.returncode, res.stderr)
