"""A call that the device memory cap refuses is never counted as holding what it was
refused, not even for a moment in which another thread's call could be refused for it
(tests/native/cap_check.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_1811_03510_amd import ccs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_refused_bytes_are_never_counted(tmp_path):
    ccs.lib()  # raises where the library is not built
    exe = str(tmp_path / "cap_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-o", exe, os.path.join(ROOT, "tests", "native", "cap_check.cpp"),
                    "-ldl"], check=True, capture_output=True, text=True)
    r = subprocess.run([exe, str(ccs.LIB_PATH)], capture_output=True, text=True, timeout=120)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stdout + r.stderr
