"""Records by a lane per node and by blocks of rays, at the edges between the two forms:
a ray's rows and labels have the bits they have in a launch of a few rays."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,local,per_cu", [(3, True, 160), (4, False, 160), (12, True, 160), (16, False, 160),
                                                (17, True, 240), (20, False, 240)])
def test_rows_at_the_edges_of_the_forms(c1, depth, local, per_cu):
    from paper_1811_03510_amd import ccs
    edge = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    extra = S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, edge, seed=23)
    rays = torch.from_numpy(np.concatenate([c1.primary[:4000], extra])[:edge + 65]).cuda()
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), depth, local_frames=local)
    hits = scene.intersect(rays)
    few = [scene.record(rays[k:k + 999], hits[k:k + 999]) for k in range(0, len(rays), 999)]
    want_f, want_y = torch.cat([f for f, _ in few]), torch.cat([y for _, y in few])
    assert (want_y != 255).any() and (want_y == 255).any()
    for n in (1, 63, edge - 1, edge, edge + 1, edge + 63, edge + 65):
        f = torch.full((n * depth + 1, 16), 7.0, device="cuda")
        y = torch.full((n * depth + 1,), 9, dtype=torch.uint8, device="cuda")
        ccs._check(ccs.lib().ccs_policy_record(scene._h, ccs._ptr(rays), ccs._ptr(hits), n, ccs._ptr(f), ccs._ptr(y),
                                               ccs._stream(None)))
        torch.cuda.synchronize()
        assert torch.equal(f[:-1].view(torch.int32), want_f.view(-1, 16)[:n * depth].view(torch.int32)), n
        assert torch.equal(y[:-1], want_y.view(-1)[:n * depth]), n
        assert (f[-1] == 7.0).all() and y[-1] == 9
    scene.close()
