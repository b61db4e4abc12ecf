"""Histograms of instances of very different sizes (a list of blocks) and of
many small ones (a wave each): exact counts against numpy through both entry
points, the starts of a batch that counts them, and the time of an uneven
call against that of its parts."""
import ctypes
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UNEVEN = [3_000_001] + [4097] * 70 + [1, 16, 17, 31] + [40_000] * 3


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import _lib
    _lib.load()
    return torch.device("cuda:0")


def bytes_of(sizes, lead=3, seed=5):
    rng = np.random.default_rng(seed)
    x = rng.integers(0, 256, sum(sizes) + lead, dtype=np.uint8)
    x[::3] = 7
    return x


def noalloc(x, sizes):
    import torch
    from paper_1601_00072_amd import _lib as L
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    out = torch.full((len(sizes), 256), -1.0, dtype=torch.float32, device=x.device)
    rc = L.load().fcm_histogram_noalloc(ctypes.c_void_p(x.data_ptr()), off.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                                        len(sizes), ctypes.c_void_p(out.data_ptr()),
                                        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    return out


@pytest.mark.parametrize("sizes", [
    UNEVEN, UNEVEN[::-1], [5] * 40 + [2_000_000] + [5] * 40, [100] * 900 + [700_000, 1, 900_000] + [3] * 100,
    [16384 * 30] + [16384] * 64 + [16385] * 64,
    [1] * 512, [1 + (37 * i) % 1024 for i in range(1000)], [1024] * 511, [1024] * 515, [4096] * 511, [4096] * 513, [1 + (37 * i) % 4096 for i in range(1000)], [4096] * 600 + [4097]],
    ids=lambda s: f"{len(s)}-{s[0]}-{max(s)}")
def test_counts(dev, sizes):
    import torch
    from paper_1601_00072_amd import histogram
    print("CASE histogram split", len(sizes), "largest", max(sizes), flush=True)
    x = bytes_of(sizes)
    d = torch.from_numpy(x).to(dev)[3:]
    got = [histogram(d, sizes).cpu().numpy() for _ in range(2)]
    if len(sizes) <= 1024:
        got += [noalloc(d, sizes).cpu().numpy() for _ in range(2)]
    off = 3
    for i, n in enumerate(sizes):
        want = (np.bincount(x[off:off + n], minlength=256).astype(np.float64) / n).astype(np.float32)
        assert all(np.array_equal(g[i], want) for g in got), i
        off += n


def test_batch_starts(dev):
    """A batch's learned starts come from the same histograms."""
    import torch
    from paper_1601_00072_amd import MLP, FCMBatch, histogram
    print("CASE batch starts", flush=True)
    sizes = UNEVEN
    d = torch.from_numpy(bytes_of(sizes)).to(dev)[3:].clone()
    with MLP(3, seed=4) as net, FCMBatch(d, sizes, [dict(n_clusters=3)] * len(sizes)) as b:
        want = net.warm_centroids(histogram(d, sizes)).cpu().numpy()
        for _ in range(2):
            b.set_start(net)
            b.solve()
            for i, w in enumerate(want):
                v0 = b.trajectory(i, 0)[0]
                assert np.array_equal(v0, w) or not np.all(np.isfinite(w))


def test_uneven_call_costs_its_parts(dev):
    """One large volume among many small slices: not more than three times the two parts' own calls."""
    import torch
    from paper_1601_00072_amd import histogram
    print("CASE uneven histogram time", flush=True)
    big, small = [1 << 26], [4096] * 5000
    x = torch.randint(0, 256, (sum(big) + sum(small),), dtype=torch.uint8, device=dev)

    def best(view, sizes):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            histogram(view, sizes)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    parts = best(x[:1 << 26], big) + best(x[1 << 26:], small)
    assert best(x, big + small) <= 3.0 * parts
