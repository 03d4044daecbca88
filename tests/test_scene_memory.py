"""What a scene holds on the device: no more than it needs with a refit level by level
(the CPU part carries the compact refit plan out, tests/native/refit_words_check.cpp), so
that a cap on device memory that admits such a scene admits this one."""
import os
import shutil
import subprocess

import pytest

from paper_1811_03510_amd import scenes as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_words_under_sanitizers(tmp_path):
    exe = str(tmp_path / "refit_words_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-o", exe, os.path.join(ROOT, "tests", "native", "refit_words_check.cpp"),
                    os.path.join(ROOT, "paper_1811_03510_amd", "csrc", "refit_plan.cpp")],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout[-3000:], r.stderr[-3000:])
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert "0 failure(s)" in r.stdout


def level_by_level(n, local):
    """Nodes of 64 B, records of 256 B, both orders of the patches, the parents of records and nodes, the nodes by depth,
    256 queue counters; in patch frames 48 B a record and the staging of creation's refit."""
    nodes = max(1, n) if n <= 1 else n - 1
    words = 4 * (4 * nodes if n else 1) + 64 * n + 2 * max(1, n) + max(1, n) + 2 * nodes + 256
    return 4 * words + (4 * 12 * n + 4 * 60 * n if local else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("local", [False, True], ids=["world", "local"])
@pytest.mark.parametrize("n", [0, 1, 2, 3, 5, 64, 65, 512, 70000])
def test_scene_fits_where_level_by_level_does(n, local, monkeypatch):
    torch = pytest.importorskip("torch")
    from paper_1811_03510_amd import ccs
    w = S.config1(8, 8)
    cp, types = (w.cp, w.types) if n <= 512 else S.instanced_scene(n // 500, extent=8.0)
    cp, types = torch.from_numpy(cp[:n]).cuda(), torch.from_numpy(types[:n]).cuda()
    monkeypatch.setenv("CCS_MAX_DEVICE_BYTES", str(ccs.device_bytes_in_use() + level_by_level(n, local)))
    scene = ccs.Scene(cp, types, 8, local_frames=local)
    assert scene.info()["n_patches"] == n
    scene.close()
