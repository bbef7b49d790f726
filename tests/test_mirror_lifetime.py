"""A context's pinned mirror outlives every kernel that writes it: nlr_api.cpp run on the CPU against
a HIP runtime of the driver's own, which notes launches that will write the mirror and checks that
the stream has been waited for before the memory is freed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_36074_amd")


def test_mirror_is_not_written_after_destroy(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("ROCm toolchain not found")
    if not os.path.exists(os.path.join(PKG, "libnlr.so")):
        from paper_2609_36074_amd import _build
        _build.build()
    exe = str(tmp_path / "driver")
    res = subprocess.run([hipcc, "-xhip", "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only",
                          "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                          os.path.join(ROOT, "tests", "mirror_driver.cpp"), "-o", exe, "-rdynamic",
                          "-L", PKG, "-lnlr", f"-Wl,-rpath,{PKG}"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "all checks passed" in res.stdout, res.stdout + res.stderr
