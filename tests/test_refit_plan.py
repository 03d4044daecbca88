"""The refit's work plan (host) under the address and undefined-behaviour sanitizers
(tests/native/refit_plan_check.cpp), and the refit on the GPU at the edges of its
workgroups: the same points again leave every node box as the builder made it."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_03510_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_plan_under_sanitizers(tmp_path):
    exe = str(tmp_path / "refit_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-pthread", "-o", exe,
                    os.path.join(ROOT, "tests", "native", "refit_plan_check.cpp"), os.path.join(CSRC, "bvh_build.cpp"),
                    os.path.join(CSRC, "refit_plan.cpp")], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    print(r.stdout[-3000:], r.stderr[-3000:])
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert "0 failure(s)" in r.stdout and "runtime error" not in r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("local", [False, True], ids=["world", "local"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130, 512, 5000, 70000])
def test_refit_to_the_same_points_keeps_every_box(n, local):
    """Hits and the count of visited nodes per ray as before the refit (a box too large or too small changes it), in
    frame 0 and in a frame that was moved elsewhere in between."""
    torch = pytest.importorskip("torch")
    from paper_1811_03510_amd import ccs
    if n <= 512:
        w = S.config1(64, 64)
        cp, types, rays = w.cp[:n], w.types[:n], np.concatenate([w.primary, w.diffuse])
    else:
        cp, types = S.instanced_scene(n // 500, extent=8.0)
        rays = S.surface_bounce_rays(cp, types, 8, (0.0, -30.0, 9.0), 20000)
    cp, rays = torch.from_numpy(cp).cuda(), torch.from_numpy(rays).cuda()
    scene = ccs.Scene(cp, torch.from_numpy(types).cuda(), 8, local_frames=local)
    h0, c0 = scene.intersect_counted(rays)
    scene.set_frames(2)
    moved = (cp * 1.25 + 0.5).contiguous()
    for frame in (0, 1):
        for points in (moved, cp):
            scene.refit_frame(frame, points)
        (h,), c = scene.intersect_batched([(frame, rays, None)], counted=True)
        torch.cuda.synchronize()
        assert torch.equal(h.view(torch.int32), h0.view(torch.int32)) and torch.equal(c, c0)
    assert (c0[:, 0] > 0).any()
    scene.close()
