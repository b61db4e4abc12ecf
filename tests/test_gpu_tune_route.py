"""The autotuner and the two routes of a solve: a default object (over the grey
levels) is not moved to the per-voxel passes by choices that were made for
per-voxel objects, in this process or in a file, its own choice is the level
solve and is taken again from the file, and what is reported reproduces it.
The route shows in the bits of the result."""
import os
import shutil

import numpy as np
import pytest

from phantom import PhantomParams, phantom

pytestmark = pytest.mark.gpu

SHIPPED = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1601_00072_amd",
                       "tuning_mi355x.txt")


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import _lib
    _lib.load()
    return torch.device("cuda:0")


def same(a, b):
    return a.iters == b.iters and a.J == b.J and np.array_equal(a.centroids, b.centroids)


def voxels(dev, shape, seed=2):
    import torch
    return torch.from_numpy(phantom(PhantomParams(shape=shape, seed=seed)).ravel()).to(dev)


@pytest.mark.parametrize("m", [2.0, 2.5])
def test_handle_after_a_per_voxel_one(dev, tmp_path, m):
    from paper_1601_00072_amd import FCM
    print("CASE autotune route, m", m, flush=True)
    x = voxels(dev, (3, 80, 96))
    cache = tmp_path / "tune.txt"
    with FCM(x, 5, m=m) as f:
        ref = f.solve()
        assert f.tuning["grid"] == 0
        f.set_tuning(**f.tuning)                # a record that was read changes nothing
        f.reset()
        assert same(f.solve(), ref)
    with FCM(x, 5, m=m) as f:
        f.set_tuning(driver=2, grid=4)
        assert f.tuning["grid"] == 4
        slow, _ = f.autotune(cache=cache, reps=1)
        assert slow["grid"] > 0 and not same(f.solve(), ref)
    lines = cache.read_text().splitlines()
    assert len(lines) == 1
    with FCM(x, 5, m=m) as f:
        tun, ms = f.autotune(cache=cache, reps=3)
        assert tun == f.tuning and (tun["driver"], tun["grid"], tun["exchange"]) == (2, 0, 0)
        assert same(f.solve(), ref)
    lines = cache.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split("\t")[2].split()[:2] == ["2", "0"]
    with FCM(x, 5, m=m) as f:                   # its own choice, taken again
        assert f.autotune(cache=cache, reps=1) == (tun, pytest.approx(ms))
        assert same(f.solve(), ref)
    with FCM(x, 5, m=m) as f:
        f.set_tuning(**tun)
        assert same(f.solve(), ref)
    with FCM(x, 5, m=m) as f:                   # and the per-voxel one's
        f.set_tuning(driver=2, grid=4)
        assert f.autotune(cache=cache, reps=1)[0] == slow
    assert len(cache.read_text().splitlines()) == 2


def test_handle_with_the_shipped_file(dev, tmp_path):
    """Its lines are per-voxel choices: they go to per-voxel handles alone."""
    from paper_1601_00072_amd import FCM
    print("CASE shipped file", flush=True)
    x = voxels(dev, (64, 128, 128)).repeat(64)
    cache = tmp_path / "tune.txt"
    shutil.copy(SHIPPED, cache)
    with FCM(x, 4) as f:
        ref = f.solve()
        f.autotune(cache=cache, reps=3)
        assert f.tuning["grid"] == 0 and same(f.solve(), ref)
    with FCM(x, 4) as f:
        f.set_tuning(driver=2, grid=4)
        tun, ms = f.autotune(cache=cache, reps=1)
        assert (tun["grid"], tun["exchange"], ms) == (512, 3, pytest.approx(1.56017))


def test_histogram_driver_keeps_its_own(dev, tmp_path):
    from paper_1601_00072_amd import FCM
    print("CASE histogram driver", flush=True)
    x = voxels(dev, (3, 50, 60))
    cache = tmp_path / "tune.txt"
    with FCM(x, 3) as f:
        f.set_tuning(driver=3)
        assert f.autotune(cache=cache, reps=3)[0]["driver"] == 3
    with FCM(x, 3) as f:
        assert f.autotune(cache=cache, reps=3)[0]["driver"] == 2
    assert len(cache.read_text().splitlines()) == 2


def test_batch_after_a_tiled_one(dev, tmp_path):
    from paper_1601_00072_amd import FCMBatch
    print("CASE batch autotune route", flush=True)
    x = voxels(dev, (9, 64, 64))
    sizes, params = [4096] * 9, [dict(n_clusters=2 + i % 5) for i in range(9)]
    cache = tmp_path / "tune.txt"

    def all_same(a, b):
        return all(same(p, q) for p, q in zip(a, b))

    with FCMBatch(x, sizes, params) as b:
        ref = b.solve()
    with FCMBatch(x, sizes, params) as b:
        b.set_tiling()
        slow = b.autotune(cache=cache, reps=1)
        assert not all_same(b.solve(), ref)
    assert len(cache.read_text().splitlines()) == 1
    for turn in range(2):                       # tuned, then taken from the record
        with FCMBatch(x, sizes, params) as b:
            ms = b.autotune(cache=cache, reps=3)[3]
            assert all_same(b.solve(), ref)
        assert turn == 0 or ms == pytest.approx(first)
        first = ms
    lines = cache.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split("\t")[2].split()[1] == "0"
    with FCMBatch(x, sizes, params) as b:
        b.set_tiling()
        assert b.autotune(cache=cache, reps=1)[:3] == slow[:3]
        assert not all_same(b.solve(), ref)
