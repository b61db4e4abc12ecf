"""Labels outside the counted classes, scattered over the image (an "ignore"
label): exact counts at the sizes of a word, and a cost that does not grow
with their number."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch.device("cuda:0")


@pytest.mark.parametrize("n_pred,n_truth", [(1, 1), (2, 16), (16, 2), (4, 8), (3, 5), (6, 5)])
def test_every_byte_value_in_every_place(dev, n_pred, n_truth):
    """All 65,536 pairs of byte values, at all four places of a word (the
    neighbours in range or not), against numpy."""
    import torch
    from paper_1601_00072_amd import confusion
    print("CASE confusion bytes", n_pred, n_truth, flush=True)
    a, b = np.meshgrid(np.arange(256, dtype=np.uint8), np.arange(256, dtype=np.uint8))
    for place in range(4):
        for fill in ((0, 0), (n_pred - 1, n_truth - 1), (255, 255)):
            p, t = (np.full((65536, 4), f, np.uint8) for f in fill)
            p[:, place], t[:, place] = a.ravel(), b.ravel()
            p, t = p.ravel(), t.ravel()
            ok = (p < n_pred) & (t < n_truth)
            want = np.zeros(n_pred * n_truth + 1, np.int64)
            np.add.at(want, p[ok].astype(int) * n_truth + t[ok], 1)
            want[-1] = np.count_nonzero(~ok)
            got = confusion(torch.from_numpy(p).to(dev), torch.from_numpy(t).to(dev), n_pred, n_truth)
            assert np.array_equal(got.cpu().numpy(), want), (place, fill)


def test_cost_of_scattered_labels(dev):
    """30 % of the labels outside cost no more than 0.1 % (3 % allowed; one
    voxel at a time where a word holds one took 5.6 % more)."""
    import torch
    from paper_1601_00072_amd import confusion
    print("CASE confusion cost", flush=True)
    n = 1 << 24
    p, t = (torch.randint(0, 4, (n,), device=dev, dtype=torch.uint8) for _ in range(2))
    few, many = t.clone(), t.clone()
    r = torch.rand(n, device=dev)
    few[r < 0.001] = 255
    many[r < 0.3] = 255
    best = [1e9, 1e9]
    for _ in range(10):
        for i, q in enumerate((few, many)):
            for _ in range(3):
                confusion(p, q, 4, 4)
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(20):
                confusion(p, q, 4, 4)
            e1.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], e0.elapsed_time(e1))
    assert best[1] <= 1.03 * best[0], best
