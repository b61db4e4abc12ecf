"""Confusion counts taken four voxels at a time: words whose labels are all in
range, words with one label outside (at the limit, 127, 128, 255), and label
counts at the edge of the small table -- exact against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pred,n_truth", [(1, 1), (4, 4), (8, 4), (2, 16), (16, 2), (16, 3)])
@pytest.mark.parametrize("share", [0.0, 0.02, 0.5])
def test_words(n_pred, n_truth, share):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import confusion
    print("CASE confusion words", n_pred, n_truth, share, flush=True)
    rng = np.random.default_rng(n_pred * 100 + n_truth)
    n = 70007
    p, t = rng.integers(0, n_pred, n), rng.integers(0, n_truth, n)
    for a, lim in ((p, n_pred), (t, n_truth)):
        out = rng.random(n) < share
        a[out] = rng.choice([lim, 127, 128, 255], int(out.sum()))
    p, t = p.astype(np.uint8), t.astype(np.uint8)
    want = np.zeros(n_pred * n_truth + 1, np.int64)
    ok = (p < n_pred) & (t < n_truth)
    np.add.at(want, p[ok].astype(int) * n_truth + t[ok], 1)
    want[-1] = np.count_nonzero(~ok)
    for off in (0, 3):
        pd = torch.zeros(n + 16, dtype=torch.uint8, device="cuda:0")[off:off + n]
        pd.copy_(torch.from_numpy(p))
        got = confusion(pd, torch.from_numpy(t).to("cuda:0"), n_pred, n_truth).cpu().numpy()
        assert np.array_equal(got, want)
