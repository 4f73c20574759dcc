"""The host side of handles and forward calls without a GPU: a driver that defines the HIP runtime calls itself
(tests/host/fake_hip_driver.cpp) and links the built library."""
import os
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


def test_host_side_of_forward_calls(tmp_path):
    lib = ROOT / "paper_1805_12549_amd" / "libcg_conv.so"
    hipcc = "/opt/rocm/bin/hipcc" if Path("/opt/rocm/bin/hipcc").exists() else shutil.which("hipcc")
    if hipcc is None or not lib.exists():
        pytest.skip("needs hipcc and the built library")
    exe = tmp_path / "fake_hip_driver"
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wall", "-rdynamic", "-I", str(ROOT / "include"),
           str(ROOT / "tests" / "host" / "fake_hip_driver.cpp"), "-L", str(lib.parent), "-lcg_conv",
           "-Wl,-rpath," + str(lib.parent), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, env=dict(os.environ))
    assert r.returncode == 0 and "host calls driver: ok" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
