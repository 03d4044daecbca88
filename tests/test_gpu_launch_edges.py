"""The largest launch of a wave per ray and the smallest beyond it, with all resident
waves and with few, against the counting kernel, which keeps every ray on one lane."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,local,learned", [(12, True, False), (9, False, False), (18, True, False), (12, True, True)])
def test_edges_of_a_wave_per_ray(c1, depth, local, learned):
    from paper_1811_03510_amd import ccs
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), depth, local_frames=local)
    if learned:
        scene.set_policy(torch.from_numpy(S.mlp_init()).cuda())
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    edge = (160 if learned else 96) * cus
    extra = S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, edge, seed=19)
    rays = torch.from_numpy(np.concatenate([c1.primary[:edge // 2], extra])[:edge + 1]).cuda()
    for waves in (0, 1, 2, 5):
        scene.set_launch(waves_per_cu=waves)
        for n in ({edge - 1, edge, edge + 1} if waves == 0 else {waves * cus - 1, waves * cus, waves * cus + 1}):
            want, _ = scene.intersect_counted(rays[:n])
            hits = torch.full((n + 1, 4), -5.0, device="cuda")
            scene.intersect(rays[:n], hits[:n])
            torch.cuda.synchronize()
            assert torch.equal(hits[:n].view(torch.int32), want.view(torch.int32)), (waves, n)
            assert (hits[n] == -5.0).all()
    scene.close()
