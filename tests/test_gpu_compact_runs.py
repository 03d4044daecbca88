"""Ray compaction at the edges of its split (256 rays a wave's run, 128 a load step,
four runs a block, 2048 blocks, beyond which a run grows), against numpy, with
nothing written behind the kept rays or the count's workspace."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FULL = 2048 * 4 * 256


@pytest.mark.parametrize("n", [2, 31, 33, 127, 129, 256, 511, 513, 1023, 1025, 4 * 256 * 7 + 129, FULL, FULL + 1,
                               2 * FULL + 300])
@pytest.mark.parametrize("share", [0.0, 0.02, 0.6, 1.0])
def test_runs(n, share):
    from paper_1811_03510_amd import ccs
    rng = np.random.default_rng(n)
    rays = rng.normal(size=(n, 8)).astype(np.float32)
    keep = rng.random(n) < share
    rays[:, 3] = 0.0
    rays[:, 7] = np.where(keep, np.inf, -1.0)
    dev = torch.from_numpy(rays).cuda()
    words = ccs.compact_work_words(n)
    out = torch.full((n + 3, 8), 5.0, device="cuda")
    index = torch.full((n + 3,), -7, dtype=torch.int32, device="cuda")
    work = torch.full((words + 2,), -9, dtype=torch.int32, device="cuda")
    for _ in range(2):  # a workspace of an earlier call
        ccs.compact_rays(dev, out, index, work)
    torch.cuda.synchronize()
    m = int(work[0].item())
    assert m == int(keep.sum()) and (work[words:].cpu().numpy() == -9).all()
    assert np.array_equal(index[:m].cpu().numpy(), np.flatnonzero(keep).astype(np.int32))
    assert np.array_equal(out[:m].cpu().numpy().view(np.uint32), rays[keep].view(np.uint32))
    assert (out[m:] == 5.0).all() and (index[m:] == -7).all()
