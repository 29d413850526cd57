"""How the blocks of all heads are dealt to the XCDs, checked on the host: the functions that the kernels call."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_block_is_dealt_once_and_short_heads_evenly(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no ROCm toolchain")
    exe = str(tmp_path / "xcd_map")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "paper_2602_13515_amd", "csrc"),
                        "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "xcd_map", "driver.hip"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "every block once" in r.stdout, r.stdout[-2000:]
