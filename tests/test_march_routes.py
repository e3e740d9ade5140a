"""Which march a frame or a batch takes (``tests/sanitize/route_driver.cpp``,
the library's host code over the host-memory HIP stand-in, CPU only)."""
import os
import shutil

import pytest


def test_routes(tmp_path):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("g++ or the HIP headers are missing")
    from test_sanitizers import FLAGS, ROOT, SAN, _check, _run
    csrc = os.path.join(ROOT, "paper_2501_01628_amd", "csrc")
    exe = str(tmp_path / "route_driver")
    rc, log = _run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", csrc, *FLAGS, "-ffp-contract=off",
                    os.path.join(SAN, "route_driver.cpp"), os.path.join(csrc, "api.cpp"),
                    os.path.join(csrc, "tet_build.cpp"), "-o", exe], str(tmp_path))
    assert rc == 0, log[-4000:]
    rc, log = _run([exe], str(tmp_path))
    _check(rc, log)
    assert "OK: 0 failed expectations" in log
