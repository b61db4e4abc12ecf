"""Results read column by column equal those read record by record (host only)."""
import numpy as np

from paper_1601_00072_amd import _lib as L
from paper_1601_00072_amd import api


def test_columns_equal_records():
    rng = np.random.default_rng(0)
    out = (L.FcmResult * 7)()
    for i, r in enumerate(out):
        r.iters, r.passes, r.status, r.n_clusters = i, i + 1, (0, 1, -5)[i % 3], 2 + i
        r.delta, r.J, r.kernel_ms, r.lo, r.hi = (float("nan") if i == 0 else 0.1 * i), 1e9 * i, 0.5 * i, i, 255 - i
        for k in range(8):
            r.centroids[k] = rng.uniform(0, 255)
    got = api._results(out)
    assert len(got) == 7
    for a, r in zip(got, out):
        b = api._result(r)
        for f in ("iters", "passes", "status", "J", "kernel_ms", "lo", "hi"):
            assert getattr(a, f) == getattr(b, f) and type(getattr(a, f)) is type(getattr(b, f))
        assert a.delta == b.delta or (np.isnan(a.delta) and np.isnan(b.delta))
        assert a.centroids.dtype == np.float64 and np.array_equal(a.centroids, b.centroids)
        a.centroids[0] = -1.0            # the caller's own copy
        assert r.centroids[0] != -1.0
