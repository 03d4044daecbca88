"""Batches of several kinds in one launch from the queue, listed in either order: every
ray's hit has the bits it has in a launch of its own."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("learned", [False, True], ids=["closest", "learned"])
def test_listing_changes_no_hit(c1, learned):
    from paper_1811_03510_amd import ccs
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), 12, local_frames=True)
    if learned:
        scene.set_policy(torch.from_numpy(S.mlp_init()).cuda())
    secondary = S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, 210001, seed=31)
    parts = [torch.from_numpy(np.ascontiguousarray(r)).cuda()
             for r in (c1.primary[:10007], c1.diffuse[:5003], secondary[:0], secondary)]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert sum(len(r) for r in parts) > scene.get_launch()["waves_per_cu"] * cus * 64  # through the queue
    alone = [scene.intersect(r) for r in parts]
    for order in ((0, 1, 2, 3), (3, 2, 1, 0), (2, 3, 0, 1)):
        hits = [torch.full((len(r), 4), 5.0, device="cuda") for r in parts]
        scene.intersect_batched([(0, parts[k], hits[k]) for k in order])
        torch.cuda.synchronize()
        for h, a in zip(hits, alone):
            assert torch.equal(h.view(torch.int32), a.view(torch.int32)), order
    scene.close()
