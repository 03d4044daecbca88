"""Records of the ordering network at the edges of their blocks (16 rays a block up to
40,960 rays, 64 beyond, the nodes of the rays that hit dealt to 256 lanes): a ray's rows
do not depend on the rays beside it, blocks of misses and of hits among them."""
import numpy as np
import pytest

from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rays(c1):
    r = S.surface_bounce_rays(c1.cp, c1.types, 12, c1.eye, 41100, seed=5).copy()
    r[200:300, 7] = -1.0  # a run of rays that are not traced
    return torch.from_numpy(r).cuda()


@pytest.mark.parametrize("depth,local", [(12, True), (1, True), (20, True), (16, False)])
def test_rows_do_not_depend_on_the_block(c1, rays, depth, local):
    from paper_1811_03510_amd import ccs
    scene = ccs.Scene(torch.from_numpy(c1.cp).cuda(), torch.from_numpy(c1.types).cuda(), depth, local_frames=local)
    hits = scene.intersect(rays)
    traced = hits[:, 1].view(torch.int32) != -1
    order = torch.argsort(traced.int(), descending=True, stable=True)  # all hits, then all misses
    f, y = scene.record(rays, hits)
    assert (y != 255).any() and (y.view(-1, depth)[~traced] == 255).all() and (f.view(-1, depth, 16)[~traced] == 0).all()
    assert (f[y == 255] == 0).all()

    def check(pick):
        n = len(pick)
        g, z = scene.record(rays[pick].contiguous(), hits[pick].contiguous())
        assert torch.equal(g.view(n, depth, 16).view(torch.int32), f.view(-1, depth, 16)[pick].view(torch.int32))
        assert torch.equal(z.view(n, depth), y.view(-1, depth)[pick])

    for n in (1, 15, 16, 17, 64, 65, 40959, 40960, 40961, 41023, 41025):
        check(torch.arange(n, device="cuda"))
    check(order)
    check(order[:30000])
    check(order.flip(0))
    scene.close()
