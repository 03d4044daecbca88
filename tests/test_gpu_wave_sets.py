"""Launches whose rays are taken by position, in pairs that go round the waves of a set
of 32: every ray is traced once at the edges of lanes a wave, pairs and sets, against
a launch over all rays that takes them from the queue."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,local", [(12, True), (9, False), (18, True)])
def test_every_ray_once(c1, depth, local):
    from paper_1811_03510_amd import ccs
    extra = S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, 200000, seed=13)
    rays = torch.from_numpy(np.concatenate([c1.primary, c1.diffuse, extra])).cuda()
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), depth, local_frames=local)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    fits = scene.get_launch()["waves_per_cu"] * cus * 64
    assert len(rays) > fits
    whole = scene.intersect(rays).view(torch.int32)
    solo, spread = 96 * cus, 8 * cus
    for n in (solo + 1, solo + 2, solo + 15, solo + 17, solo + 511, solo + 513, 16 * spread - 1, 16 * spread + 1,
              17 * spread + 3, 33 * spread - 1, 64 * spread, 64 * spread + 1, fits - 1, fits):
        hits = torch.full((n + 1, 4), -5.0, device="cuda")
        scene.intersect(rays[:n], hits[:n])
        torch.cuda.synchronize()
        assert torch.equal(hits[:n].view(torch.int32), whole[:n]), n
        assert (hits[n] == -5.0).all()
    scene.close()
