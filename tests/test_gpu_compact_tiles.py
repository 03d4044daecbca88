"""Compaction in one launch (more than 2,097,152 rays, tiles of 8192 whose places come
from the tiles before them): the edges of the last tile and of a look-back's 64 tiles
against numpy, in a workspace of earlier words at an odd word, and replayed graphs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILE, FROM = 8192, 256 * 8192


def level(n, share):
    rng = np.random.default_rng(n)
    keep = rng.random(n) < share
    keep[-1] = share > 0
    rays = rng.normal(size=(n, 8)).astype(np.float32)
    rays[:, 3] = 0.0
    rays[:, 7] = np.where(keep, np.inf, -1.0)
    return rays, keep


@pytest.mark.parametrize("n", [FROM, FROM + 1, FROM + 511, FROM + TILE - 1, FROM + TILE, FROM + TILE + 1,
                               FROM + 64 * TILE + 7])
@pytest.mark.parametrize("share", [0.0, 0.03, 1.0])
def test_tiles(n, share):
    from paper_1811_03510_amd import ccs
    rays, keep = level(n, share)
    dev, words = torch.from_numpy(rays).cuda(), ccs.compact_work_words(n)
    out = torch.full((n, 8), 5.0, device="cuda")
    index = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    work = torch.full((words + 3,), -9, dtype=torch.int32, device="cuda")
    m = int(keep.sum())
    for at in (0, 1):
        ccs.compact_rays(dev, out, index, work[at:at + words])
        torch.cuda.synchronize()
        assert int(work[at].item()) == m and (work[at + words:].cpu().numpy() == -9).all()
    assert np.array_equal(index[:m].cpu().numpy(), np.flatnonzero(keep).astype(np.int32))
    assert np.array_equal(out[:m].cpu().numpy().view(np.uint32), rays[keep].view(np.uint32))
    assert (out[m:] == 5.0).all() and (index[m:] == -7).all()


def test_tiles_in_a_replayed_graph():
    from paper_1811_03510_amd import ccs
    n = FROM + 5 * TILE + 3
    sets = [level(n, share) for share in (0.4, 0.1, 0.8)]
    dev = torch.from_numpy(sets[0][0]).cuda()
    out, index = torch.empty_like(dev), torch.empty(n, dtype=torch.int32, device="cuda")
    work = torch.empty(ccs.compact_work_words(n), dtype=torch.int32, device="cuda")
    ccs.compact_rays(dev, out, index, work)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ccs.compact_rays(dev, out, index, work)
    for rays, keep in sets + sets[:1]:
        dev.copy_(torch.from_numpy(rays))
        graph.replay()
        torch.cuda.synchronize()
        m = int(keep.sum())
        assert int(work[0].item()) == m
        assert np.array_equal(index[:m].cpu().numpy(), np.flatnonzero(keep).astype(np.int32))
        assert np.array_equal(out[:m].cpu().numpy().view(np.uint32), rays[keep].view(np.uint32))
