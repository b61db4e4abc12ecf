"""The level solve (default tuning) where its result must not depend on how
the solve was reached: queries before it, steps, other routes' launches."""
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


def volume(dev, shape=(5, 64, 64), seed=1):
    import torch
    return torch.from_numpy(phantom(PhantomParams(shape=shape, seed=seed)).ravel()).to(dev)


@pytest.mark.parametrize("init", [[1e20, 10.0, 50.0], [-3.0e38, 0.0, 3.0e38], [10.0, 50.0, 1.9e19]])
@pytest.mark.parametrize("first", ["none", "centroids", "iterate", "labels"])
def test_start_out_of_range_after_a_query(dev, init, first):
    """A start whose squared distances overflow FP32 is reported as the
    per-voxel pass reports it (status, iteration 0, J and delta NaN), also
    when the start was read or labelled before the solve."""
    from paper_1601_00072_amd import FCM
    print("CASE start out of range", init, "after", first, flush=True)
    x = volume(dev)
    got = []
    for kw in ({}, dict(driver=2, grid=4)):
        with FCM(x, 3, init=init) as f:
            if kw:
                f.set_tuning(**kw)
            v0 = np.asarray(init, np.float32).astype(np.float64)
            if first == "centroids":
                assert np.array_equal(f.centroids(), v0)
            elif first == "iterate":
                assert f.iterate(0).status == 2
            elif first == "labels":
                f.labels()
            r = f.solve()
            v, d, J = f.trajectory(0)
            assert np.array_equal(v, v0) and np.isnan(d) and np.isnan(J)
            got.append((r.status, r.iters, r.passes))
            assert np.isnan(r.J) and np.isnan(r.delta) and np.array_equal(r.centroids, v0)
    assert got[0] == got[1] == (-5, 0, 1)


def test_batch_start_out_of_range(dev):
    from paper_1601_00072_amd import FCMBatch
    print("CASE batch start out of range", flush=True)
    x = volume(dev)
    n = x.numel()
    with FCMBatch(x, [n // 2, n - n // 2], [dict(n_clusters=3, init=[1e20, 10.0, 50.0]), dict(n_clusters=3)]) as b:
        a, ok = b.solve()
    assert a.status == -5 and a.iters == 0 and a.passes == 1 and np.isnan(a.J) and np.isnan(a.delta)
    assert ok.status == 0 and np.isfinite(ok.J)


TINY, DEFAULT = 1e-8, 5.0  # wait limits in seconds: about one clock tick (every wait gives up), the library's own


def test_pending_wait_limit_is_reported_behind_a_level_solve(dev):
    """An asynchronous per-voxel solve whose waits give up is reported by the
    next fcm_solve_wait also when a level solve was enqueued behind it; the
    handle then recovers on both routes."""
    import torch
    from paper_1601_00072_amd import FCM
    from paper_1601_00072_amd.api import FcmError
    print("CASE pending abort, then a level solve", flush=True)
    x = volume(dev, (64, 128, 128), 2)
    lab = torch.empty_like(x)
    with FCM(x, 4) as f:
        ref = f.solve()
        f.set_tuning(driver=2, launch=1, grid=256)
        f.set_wait_limit(TINY)
        f.solve_async(lab)
        f.set_wait_limit(DEFAULT)
        f.set_tuning(driver=2)
        f.solve_async(lab)
        with pytest.raises(FcmError) as e:
            f.result()
        assert e.value.status == -3
        f.solve_async(lab)
        r, _ = f.result()
        assert r.status == 0 and r.J == ref.J and np.array_equal(r.centroids, ref.centroids)
        f.set_tuning(driver=2, launch=1, grid=256)
        f.solve_async(lab)
        r, _ = f.result()
        assert r.status == 0 and np.max(np.abs(r.centroids - ref.centroids) / ref.centroids) <= 1e-4


def test_solve_behind_a_pending_wait_limit(dev):
    """The synchronous level solve behind such a launch runs again from its start, as the per-voxel one does."""
    from paper_1601_00072_amd import FCM
    print("CASE pending abort, then a synchronous level solve", flush=True)
    x = volume(dev, (64, 128, 128), 2)
    with FCM(x, 4) as f:
        ref = f.solve()
        f.set_tuning(driver=2, launch=1, grid=256)
        f.set_wait_limit(TINY)
        f.solve_async()
        f.set_wait_limit(DEFAULT)
        f.set_tuning(driver=2)
        f.reset()
        r = f.solve()
        assert f.set_wait_limit(0) == 1
    assert r.status == 0 and r.J == ref.J and np.array_equal(r.centroids, ref.centroids)


@pytest.mark.parametrize("captured", ["voxels", "levels"])
def test_captured_solve_and_the_other_route(dev, captured):
    """A graph of one route's asynchronous solve, replayed after solves of the
    other route and on new contents of the input: the result read is the
    replayed solve's."""
    import torch
    from paper_1601_00072_amd import FCM
    print("CASE captured", captured, flush=True)
    a, b = volume(dev, (64, 128, 128), 2), volume(dev, (64, 128, 128), 5)
    x, lab = a.clone(), torch.empty_like(a)
    routes = {"voxels": dict(driver=2, launch=1, grid=64, exchange=1), "levels": dict(driver=2, exchange=0)}
    other = "levels" if captured == "voxels" else "voxels"
    want = {}
    for name, src in (("a", a), ("b", b)):
        with FCM(src, 4) as f:
            f.set_tuning(**routes[captured])
            want[name] = f.solve()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s), FCM(x, 4) as f:
        f.set_tuning(**routes[captured])
        f.solve_async(lab)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            f.solve_async(lab)
        f.set_tuning(**routes[other])
        for turn in range(3):
            for name, src in (("b", b), ("a", a)):
                x.copy_(a if name == "b" else b)
                f.reset()
                f.solve()                  # the other route, on other contents
                f.solve_async(lab)
                assert f.result()[0].J != want[name].J
                x.copy_(src)
                g.replay()
                r, _ = f.result()
                assert r.J == want[name].J and r.iters == want[name].iters
                assert np.array_equal(r.centroids, want[name].centroids)
                assert np.array_equal(f.trajectory(r.iters)[0], r.centroids)


TWINS = [[40.0, 40.0, 110.0], [110.5, 40.5, 40.5], [40.5, 110.0, 150.0, 40.5], [7.25, 7.25],
         [0.0, 0.0, 0.0, 110.0, 110.0, 150.0, 150.0, 255.0], [0.5, 0.5, 0.5, 110.5, 110.5, 150.5, 150.5, 255.0],
         [110.5, 0.5, 110.5, 255.0, 0.5, 150.5, 0.5]]


def extended(h, init, m, T):
    """Iterations 0..T in 80-bit arithmetic: (v, J) of each."""
    L = np.longdouble
    g = np.nonzero(h)[0]
    c, g, v = h[g].astype(L), g.astype(L), np.array(init, dtype=L)
    out = []
    for _ in range(T + 1):
        d = abs(g[:, None] - v[None, :])
        zero = d == 0
        d[zero] = 1
        u = d ** (-2 / (L(m) - 1))
        on = zero.any(axis=1)
        u[on] = zero[on]
        a = c[:, None] * (u / u.sum(axis=1, keepdims=True)) ** L(m)
        out.append((v, (a * (g[:, None] - v[None, :]) ** 2).sum()))
        v = (a * g[:, None]).sum(axis=0) / a.sum(axis=0)
    return out


def check_equal_centroids(h, init, m, r, tr):
    """Equal start centroids stay equal to the last bit, and every iteration
    matches the FP64 oracle (which treats them alike too) at FP64 tolerances,
    beside the oracle's own distance from 80-bit arithmetic (3.9e-11 of J in
    the one case that passes a saddle for 280 iterations)."""
    from oracle import fcm_hist
    T = max(r.iters, 1)
    ora, ext = fcm_hist.solve(h, len(init), m, 0.0, T, v0=np.asarray(init, np.float64)), extended(h, init, m, T)
    for t, (v, d, J) in enumerate(tr):
        for k in range(len(init)):
            assert v[k] == v[init.index(init[k])]
        off = np.abs(ora.v[t] - ext[t][0])
        assert np.all(np.abs(v - ora.v[t]) <= 1e-10 * np.maximum(np.abs(ora.v[t]), 1.0) + off)
        assert abs(J - ora.J[t]) <= 1e-11 * ora.J[t] + abs(ora.J[t] - ext[t][1])
        assert t == 0 or abs(d - ora.delta[t]) <= 1e-11 + 10 * off.max()
    assert ora.delta[r.iters] < 1e-5 + 1e-11 + 10 * off.max()


@pytest.mark.parametrize("m", [2.0, 1.5, 2.5])
@pytest.mark.parametrize("init", TWINS)
def test_equal_centroids_in_steps(dev, init, m):
    """Start centroids that are equal, on grey levels and between them: single
    steps, larger ones and the whole solve give the same bits."""
    from oracle import fcm_hist
    from paper_1601_00072_amd import FCM
    print("CASE equal centroids", init, "m", m, flush=True)
    x = volume(dev, (16, 64, 64), 4)
    got = []
    for k in (1, 3, 1000):
        with FCM(x, len(init), m=m, init=init) as f:
            r = f.iterate(k)
            while r.status == 2:
                r = f.iterate(k)
            got.append((r, [f.trajectory(t) for t in range(r.iters + 1)]))
    ref, tr = got[0]
    for r, t in got[1:]:
        assert r.iters == ref.iters and r.J == ref.J and r.delta == ref.delta
        for a, b in zip(t, tr):
            assert np.array_equal(a[0], b[0]) and a[2] == b[2] and (a[1] == b[1] or np.isnan(a[1]))
    check_equal_centroids(fcm_hist.histogram(x.cpu().numpy()), init, m, ref, tr)


def test_equal_centroids_in_a_batch(dev):
    import torch
    from oracle import fcm_hist
    from paper_1601_00072_amd import FCMBatch
    print("CASE equal centroids, batch", flush=True)
    x = volume(dev, (16, 64, 64), 4)
    items = [(init, m) for init in TWINS for m in (2.0, 1.5, 2.5)]
    with FCMBatch(torch.cat([x] * len(items)), [x.numel()] * len(items),
                  [dict(n_clusters=len(init), m=m, init=init) for init, m in items]) as b:
        res = b.solve()
        trs = [[b.trajectory(i, t) for t in range(r.iters + 1)] for i, r in enumerate(res)]
    h = fcm_hist.histogram(x.cpu().numpy())
    for (init, m), r, tr in zip(items, res, trs):
        assert r.status == 0
        check_equal_centroids(h, init, m, r, tr)


@pytest.mark.parametrize("C,m", [(2, 2.0), (4, 1.5), (8, 2.5), (8, 3.0)])
@pytest.mark.parametrize("n", [1, 100, 65537])
def test_one_level(dev, C, m, n):
    """All centroids on the only grey level present: converged in two passes with J = 0."""
    import torch
    from paper_1601_00072_amd import FCM
    print("CASE one level C", C, "m", m, "n", n, flush=True)
    x = torch.full((n,), 77, dtype=torch.uint8, device=dev)
    with FCM(x, C, m=m) as f:
        r = f.solve()
        assert (r.status, r.iters, r.passes, r.J, r.delta) == (0, 1, 2, 0.0, 0.0)
        assert np.array_equal(r.centroids, np.full(C, 77.0)) and not f.labels().any()
