"""A batch that solves over the grey levels holds no workspace of the
per-voxel passes until a setter asks for it; from then on it gives what it
gave with the workspace made at creation."""
import numpy as np
import pytest

from phantom import PhantomParams, phantom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import _lib
    _lib.load()
    return torch.device("cuda:0")


def test_memory_of_a_new_batch(dev):
    """2^30 voxels: the tables of the per-voxel tiles would take 28 MB."""
    import torch
    from paper_1601_00072_amd import FCMBatch
    print("CASE batch memory", flush=True)
    x = torch.randint(0, 256, (1 << 30,), dtype=torch.uint8, device=dev)
    with FCMBatch(x[:1000], [1000], [dict(n_clusters=4, max_iter=3)]) as b:  # the runtime's own first allocations
        b.solve()
        b.set_tiling(2)
        b.solve()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    with FCMBatch(x, [1 << 24] * 64, [dict(n_clusters=4, max_iter=3)] * 64) as b:
        held = before - torch.cuda.mem_get_info()[0]
        b.set_tiling(2)
        tiled = before - torch.cuda.mem_get_info()[0]
    print("bytes held", held, "with tiles", tiled, flush=True)
    assert held <= 14 << 20 and tiled >= 28 << 20


@pytest.mark.parametrize("setter", ["tiling", "block", "tail"])
def test_tiles_made_late(dev, setter):
    """Solves over the levels, then with tiles: the bits of a batch that had
    its tiles set before its first solve; labels on both routes."""
    import torch
    from paper_1601_00072_amd import FCMBatch
    print("CASE tiles made late", setter, flush=True)
    sizes = [1, 40, 33000, 70001, 300000]
    flat = phantom(PhantomParams(shape=(99, 64, 64), seed=3)).ravel()[:sum(sizes)].copy()
    d = torch.from_numpy(flat).to(dev)
    params = [dict(n_clusters=2 + i, m=(2.0, 1.5, 2.5)[i % 3]) for i in range(len(sizes))]

    def tile(b):
        if setter == "tiling":
            b.set_tiling(1)
        elif setter == "block":
            b.set_block(256)
        else:
            b.set_tail_tiling(2, 1)

    with FCMBatch(d, sizes, params) as b:
        tile(b)
        want = b.solve()
        lab_want = b.labels().cpu().numpy()
    with FCMBatch(d, sizes, params) as b:
        first = b.solve()
        lab_levels = b.labels().cpu().numpy()
        start = 0
        for r, n in zip(first, sizes):
            lut = np.argmin(np.abs(np.arange(256.0)[:, None] - r.centroids[None, :]), axis=1).astype(np.uint8)
            assert np.array_equal(lab_levels[start:start + n], lut[flat[start:start + n]])
            start += n
        tile(b)
        for _ in range(2):
            got = b.solve()
            for r, q in zip(got, want):
                assert r.iters == q.iters and r.J == q.J and np.array_equal(r.centroids, q.centroids)
            assert np.array_equal(b.labels().cpu().numpy(), lab_want)
        assert b.timeline(4).shape == (got[4].passes + 1,)
