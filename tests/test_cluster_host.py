"""The buffer sizes of a batch query that several workgroups run (fused.h),
built for the host: what one workgroup alone may write fits at every number of
workgroups."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1906_03420_amd", "csrc")
INC = os.path.join(os.path.dirname(HERE), "include")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_buffers_hold_what_one_workgroup_writes(tmp_path):
    exe = str(tmp_path / "cluster_check")
    cmd = [HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", INC, "-I", CSRC,
           os.path.join(HERE, "native", "cluster_check.hip"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]
