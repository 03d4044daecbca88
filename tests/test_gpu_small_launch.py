"""Launches whose rays run on 16 lanes each, from the start (small launches) or at
the end of a wave, against the counting kernel, which keeps every ray on one lane
to its end: hits bitwise equal at the edges of the launch rules (rays per wave,
rays on 16 lanes against one, rays by position against the queue)."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ccs():
    from paper_1811_03510_amd import ccs as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


@pytest.fixture(scope="module")
def rays(c1):
    """270,000 torus rays, both classes mixed in a seeded order, inactive and invalid ones among them."""
    extra = S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, 240000, seed=77)
    r = np.concatenate([c1.primary, c1.diffuse, extra])[:270000]
    r = r[S.choose(5, len(r), len(r))[np.argsort(S.uniform(6, len(r)), kind="stable")]].copy()
    r[7::997, 7] = -1.0             # inactive
    r[11::1013, 0] = np.nan         # not traced
    r[13::1009, 7] = 3.0            # short
    r[17::1019, 4:7] *= [1, 1, 0]   # a zero direction component
    return torch.from_numpy(r).cuda()


def equal(ccs, scene, rays, n, parts=1):
    want, _ = scene.intersect_counted(rays[:n])
    if parts == 1:
        got = scene.intersect(rays[:n])
    else:  # uneven batches, an empty one among them
        cut = sorted({0, n // 7, n // 7, n // 2, n})
        got = torch.cat(scene.intersect_batched([(0, rays[a:b], None) for a, b in zip([0] + cut, cut + [n])]))
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert n < 500 or (ccs.hit_ids(got) != ccs.NO_HIT).any()


@pytest.mark.parametrize("local,depth,learned", [(True, 12, False), (False, 12, False), (True, 1, False),
                                                 (True, 18, False), (False, 17, False), (True, 12, True),
                                                 (False, 9, True)])
def test_small_launches_match_one_lane_per_ray(ccs, c1, rays, local, depth, learned):
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), depth, local_frames=local)
    if learned:
        scene.set_policy(torch.from_numpy(S.mlp_init()).cuda())
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = [1, 2, 3, 4, 5, 63, 65, 1000, 16 * cus, 20 * cus + 1, 40 * cus + 1, 64 * cus, 64 * cus + 1, 8 * 16 * cus + 1,
             8 * 64 * cus + 1, 12 * 64 * cus, 12 * 64 * cus + 1, 270000]
    for n in sizes:
        if n <= len(rays):
            equal(ccs, scene, rays, n)
    for n in (7, 5001, 64 * cus, 100003):
        equal(ccs, scene, rays, n, parts=4)
    for waves in (1, 2):  # few resident waves: the small launch's rays no longer fit at once
        scene.set_launch(waves_per_cu=waves)
        for n in (1, 4 * waves * cus, 4 * waves * cus + 1, 64 * waves * cus + 5):
            equal(ccs, scene, rays, n)
    scene.close()


def test_small_launches_of_frames_and_tiny_scenes(ccs, c1, rays):
    cp = torch.from_numpy(c1.cp).cuda()
    scene = ccs.Scene(cp, torch.from_numpy(c1.types).cuda(), 12, local_frames=True)
    scene.set_frames(3)
    for f in range(3):
        scene.refit_frame(f, torch.from_numpy(S.animate(c1.cp, f, 3)).cuda())
    for n in (10, 4000, 30000):
        batches = [(f, rays[f * n:(f + 1) * n], None) for f in (2, 0, 1)]
        want, _ = scene.intersect_batched(batches, counted=True)
        got = scene.intersect_batched(batches)
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g.view(torch.int32), w.view(torch.int32))
    scene.close()
    for n_patches in (0, 1, 2):
        scene = ccs.Scene(cp[:n_patches], torch.from_numpy(c1.types[:n_patches]).cuda(), 6)
        for n in (1, 500, 20000):
            want, _ = scene.intersect_counted(rays[:n])
            got = scene.intersect(rays[:n])
            torch.cuda.synchronize()
            assert torch.equal(got.view(torch.int32), want.view(torch.int32))
        scene.close()


def test_small_launches_under_capture(ccs, c1, rays):
    """Captured launches (by position, 16 lanes a ray, and through the queue) replayed with eager work between."""
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), 12, local_frames=True)
    sizes = (1000, 40000, 250000)
    want = [scene.intersect_counted(rays[:n])[0] for n in sizes]
    hits = [torch.empty((n, 4), device="cuda") for n in sizes]
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for n, h in zip(sizes, hits):
            scene.intersect(rays[:n], h)
    for _ in range(3):
        for h in hits:
            h.fill_(7.0)
        scene.intersect(rays[:5000])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for h, w in zip(hits, want):
            assert torch.equal(h.view(torch.int32), w.view(torch.int32))
    scene.close()
