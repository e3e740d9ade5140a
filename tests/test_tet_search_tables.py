"""The tetrahedral search's float32 planes and cell heads (``tet_build.cpp``)
against brute force (``tests/sanitize/tet_search_driver.cpp``), built with the
host sanitizers (CPU only)."""
import os
import shutil

import pytest


def test_search_tables_against_brute_force(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ is missing")
    from test_sanitizers import FLAGS, ROOT, SAN, _check, _run
    csrc = os.path.join(ROOT, "paper_2501_01628_amd", "csrc")
    exe = str(tmp_path / "tet_search_driver")
    rc, log = _run(["g++", "-std=c++17", *FLAGS, "-ffp-contract=off", "-I", csrc,
                    os.path.join(SAN, "tet_search_driver.cpp"), os.path.join(csrc, "tet_build.cpp"), "-o", exe],
                   str(tmp_path))
    assert rc == 0, log[-4000:]
    rc, log = _run([exe], str(tmp_path))
    _check(rc, log)
    assert "OK: 0 failed expectations" in log
