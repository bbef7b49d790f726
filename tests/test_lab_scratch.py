"""The scratch of the label recovery on the CPU: over a sweep of sizes and workspace layouts its
arrays lie inside the workspace's shared region and apart, and the rows of U are shared out over
enough workgroups (one workgroup for a whole narrow factor made a call on 1e6 x 4 take 64 ms for 0.5)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_36074_amd")


def test_label_scratch_layout(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("ROCm toolchain not found")
    if not os.path.exists(os.path.join(PKG, "libnlr.so")):
        from paper_2609_36074_amd import _build
        _build.build()
    exe = str(tmp_path / "driver")
    res = subprocess.run([hipcc, "-xhip", "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only",
                          "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                          os.path.join(ROOT, "tests", "lab_scratch_driver.cpp"), "-o", exe,
                          "-L", PKG, "-lnlr", f"-Wl,-rpath,{PKG}"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
