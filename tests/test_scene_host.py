"""The host side of scene creation when the system refuses memory or threads
(tests/native/scene_host_check.cpp): it throws and leaves nothing behind, or builds the
same scene on fewer threads; it never ends the process."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_03510_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_refused_memory_and_threads(tmp_path):
    exe = str(tmp_path / "scene_host_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-pthread", "-o", exe,
                    os.path.join(ROOT, "tests", "native", "scene_host_check.cpp"),
                    *(os.path.join(CSRC, f) for f in ("scene_host.cpp", "bvh_build.cpp", "refit_plan.cpp")), "-ldl"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout[-3000:], r.stderr[-3000:])
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert "0 failure(s)" in r.stdout
