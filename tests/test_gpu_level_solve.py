"""The default solve (persistent driver, launch left to the library), which
runs over the grey levels: block edges of the count, both ways of merging the
counts, unaligned inputs, every start, steps, and changes of driver between
steps, against the level-regrouped FP64 oracle at FP64 tolerances (both sides
sum 256 levels in FP64; only the order differs)."""
import numpy as np
import pytest

from oracle import fcm_hist
from phantom import PhantomParams, phantom
from tests.test_gpu_levels import check

pytestmark = pytest.mark.gpu

SHARE = 16384  # voxels per block of the count


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import _lib
    _lib.load()
    return torch.device("cuda:0")


def place(dev, x, offset):
    import torch
    buf = torch.zeros(x.size + offset + 16, dtype=torch.uint8, device=dev)
    buf[offset:offset + x.size] = torch.from_numpy(x).to(dev)
    return buf[offset:offset + x.size]


def data(n, seed=1):
    return phantom(PhantomParams(shape=(-(-n // 4096), 64, 64), seed=seed)).ravel()[:n].copy()


@pytest.mark.parametrize("n", [4096, 16 * 512 - 1, SHARE, SHARE + 1, 2 * SHARE + 17, 17 * SHARE - 3, 256 * SHARE + 5])
@pytest.mark.parametrize("offset,C,m", [(0, 4, 2.0), (5, 8, 2.0), (15, 2, 1.5), (1, 3, 2.5)])
def test_sizes(dev, n, offset, C, m):
    from paper_1601_00072_amd import FCM
    print("CASE level solve n", n, "offset", offset, "C", C, "m", m, flush=True)
    x = data(n)
    xt = place(dev, x, offset)
    with FCM(xt, C, m=m) as f:
        r = f.solve()
        check(x, C, r, [f.trajectory(t) for t in range(r.iters + 1)], f.labels().cpu().numpy(), m=m)
        for _ in range(3):                 # counters and ticket are left as they were found
            f.solve_async()
        again, _ = f.result()
    assert again.iters == r.iters and np.array_equal(again.centroids, r.centroids) and again.J == r.J


@pytest.mark.parametrize("values", [[0], [255], [0, 255], [7, 7, 9], list(range(256))])
def test_few_levels(dev, values):
    """Levels at both ends of the range, one level, all levels."""
    from paper_1601_00072_amd import FCM
    print("CASE level solve values", values[:4], flush=True)
    x = np.resize(np.array(values, dtype=np.uint8), 70001)
    with FCM(place(dev, x, 3), 2) as f:
        r = f.solve()
        check(x, 2, r, [f.trajectory(t) for t in range(r.iters + 1)], f.labels().cpu().numpy())
    assert (r.lo, r.hi) == (min(values), max(values))


@pytest.mark.parametrize("drivers", [(2, 0), (0, 2), (1, 2, 0, 2)])
def test_driver_changes_between_steps(dev, drivers):
    """A level launch continues what per-voxel passes left, and the other way
    round: the per-voxel passes work in FP32 (1e-5), and labels are exact."""
    from paper_1601_00072_amd import FCM
    print("CASE drivers", drivers, flush=True)
    x = data(50000)
    ora = fcm_hist.solve(fcm_hist.histogram(x), 4, 2.0, 1e-5, 300)
    with FCM(place(dev, x, 0), 4) as f:
        for i, d in enumerate(drivers):
            f.set_tuning(driver=d)
            r = f.iterate(2) if i + 1 < len(drivers) else f.solve()
        assert r.status == 0 and abs(r.iters - ora.T) <= 1 and r.passes == r.iters + 1
        for t in range(min(r.iters, ora.T) + 1):
            v = f.trajectory(t)[0]
            assert np.max(np.abs(v - ora.v[t]) / np.maximum(np.abs(ora.v[t]), 1.0)) <= 1e-5
        lab = f.labels().cpu().numpy()
    assert np.array_equal(lab, fcm_hist.level_labels(ora.v[ora.T])[x])


@pytest.mark.parametrize("init", [[1e20, 10.0, 50.0], [-3.0e38, 0.0, 3.0e38]])
def test_start_out_of_fp32_range(dev, init):
    """A start whose squared distances overflow FP32 ends as it does in the
    per-voxel pass: non-finite objective at iteration 0."""
    from paper_1601_00072_amd import FCM
    print("CASE start out of range", init, flush=True)
    x = place(dev, data(20000), 0)
    with FCM(x, 3, init=init) as f:
        r = f.solve()
    with FCM(x, 3, init=init) as f:
        f.set_tuning(driver=2, grid=4)
        ref = f.solve()
    assert r.status == ref.status == -5 and r.iters == ref.iters == 0


def test_autotune_keeps_the_library_choice(dev):
    """The launch left to the library is a candidate of its own."""
    from paper_1601_00072_amd import FCM
    print("CASE autotune", flush=True)
    x = data(300000)
    with FCM(place(dev, x, 0), 4) as f:
        f.autotune(reps=1)
        r = f.solve()
        ora = fcm_hist.solve(fcm_hist.histogram(x), 4, 2.0, 1e-5, 300)
        assert r.status == 0 and np.max(np.abs(r.centroids - ora.v[ora.T])) <= 1e-3


def test_batch_tiles(dev):
    """Instances of one tile, of exactly one, and of many, aligned and not, all
    cluster counts and fuzziness classes, one launch; repeated, then with the
    caller's tiles (per-voxel passes) and back to the same bits."""
    import torch
    from paper_1601_00072_amd import FCMBatch
    print("CASE level batch", flush=True)
    sizes = [1, 17, 4096, SHARE - 1, SHARE, SHARE + 1, 2 * SHARE + 31, 9 * SHARE + 5, 300001, 3 * SHARE]
    items = []
    for i, n in enumerate(sizes):
        p = dict(n_clusters=2 + i % 7, m=[2.0, 1.5, 2.5][i % 3], eps=1e-5)
        if i == 6:
            p["init"] = [10.0 + 20.0 * k for k in range(p["n_clusters"])]
        items.append((data(n, seed=20 + i), p))
    flat = np.concatenate([x for x, _ in items])
    params = [p for _, p in items]
    x = place(dev, flat, 3)
    with FCMBatch(x, sizes, params) as b:
        for turn in range(2):
            res = b.solve()
            lab = b.labels().cpu().numpy()
            start = 0
            for i, ((xi, p), r) in enumerate(zip(items, res)):
                if np.unique(xi).size > p["n_clusters"]:
                    traj = [b.trajectory(i, t) for t in range(r.iters + 1)]
                    check(xi, p["n_clusters"], r, traj, lab[start:start + xi.size], m=p["m"], init=p.get("init"))
                us = b.timeline(i)
                assert us.shape == (r.passes + 1,) and us[0] >= 0.0 and np.all(np.diff(us) >= 0.0)
                start += xi.size
            if turn:
                for r, q in zip(res, first):
                    assert r.iters == q.iters and r.J == q.J and np.array_equal(r.centroids, q.centroids)
            first = res
        b.set_tiling(4, 0)
        tiled = b.solve()
    with FCMBatch(x, sizes, params) as b:
        b.set_tiling(4, 0)
        again = b.solve()
    for r, q, t in zip(tiled, again, first):
        assert r.iters == q.iters and np.array_equal(r.centroids, q.centroids)
        if r.iters == t.iters and r.status == 0:
            assert np.max(np.abs(r.centroids - t.centroids)) <= 1e-2
