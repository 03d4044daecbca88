"""Learned order on a wave per ray (launches of at most 160 rays per compute unit) and for
a wave's last ray: the ray's node, pending siblings, preferred v-half and network inputs
in scalars.  Hits bitwise those of the counting kernel, one lane per ray, for networks
that always agree, always differ and mix, in patch and world frames, at leaf depths 1 to 16."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,local", [(1, True), (2, False), (7, True), (12, True), (12, False), (16, True)])
@pytest.mark.parametrize("net", ["init", "random", "zero"])
def test_matches_one_lane_per_ray(c1, depth, local, net):
    from paper_1811_03510_amd import ccs
    theta = S.mlp_init()
    if net == "random":
        theta = (np.random.default_rng(depth).normal(size=theta.shape) * 0.7).astype(np.float32)
    elif net == "zero":
        theta = np.zeros_like(theta)
    rays = np.concatenate([c1.diffuse, S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, 44000, seed=31)])
    rays = np.ascontiguousarray(rays[::-1]).copy()
    rays[5::701, 7] = -1.0
    rays = torch.from_numpy(rays).cuda()
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), depth, local_frames=local)
    scene.set_policy(torch.from_numpy(theta).cuda())
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (1, 700, 160 * cus, 160 * cus + 1):
        want, _ = scene.intersect_counted(rays[:n])
        hits = torch.full((n + 1, 4), -5.0, device="cuda")
        scene.intersect(rays[:n], hits[:n])
        torch.cuda.synchronize()
        assert torch.equal(hits[:n].view(torch.int32), want.view(torch.int32)), n
        assert (hits[n] == -5.0).all()
    scene.close()
