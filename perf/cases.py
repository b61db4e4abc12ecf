"""Performance cases: the work that users of the library have it do, through its public Python entry points.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw(rng)`` more of the same ranges,
``prepare(case, seed)`` what a program holds before the call, ``run(state)`` one pass, ``work(case)`` the bytes
and operations that a pass cannot do without, and ``exact(case, seed)`` the outputs in 64 bits by plain numpy
and torch.

Inputs are brain-like phantoms made on the GPU: nested ellipses (ellipsoids) of four tissues with a smooth
multiplicative bias field and additive Gaussian noise, clipped to 8 bits, as the repository's own workloads.

Outputs of a solve are the label image, the centroids and the objective.  The library evaluates memberships in
FP32 by contract and stores centroids and objective in doubles, so both are returned as the FP32 values that
they carry.  The iteration count and the last membership change are left out: whether the change falls below
eps at iteration T or T + 1 is decided by the rounding of the centroids (the test-suite compares both in a
band), and the centroids of two neighbouring iterations agree far below the bound of their type.
"""
import math

import numpy as np
import torch

DEV = "cuda:0"
MEANS = (0.0, 40.0, 110.0, 150.0)
AXES = ((0.90, 0.85, 0.90), (0.72, 0.66, 0.72), (0.55, 0.45, 0.50))


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _solve(name, shape, C, m=2.0, eps=1e-5, how="handle", offset=0, kahan=False, given=False, sigma=8.0, bias=0.1):
    c = {"kind": "solve", "d": shape[0], "h": shape[1], "w": shape[2], "C": C, "m": m, "eps": eps, "how": how,
         "offset": offset, "kahan": kahan, "given": given, "sigma": sigma, "bias": bias}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small slice through the one-call entry point: what a script that segments a picture does, a new
        # solver each time (the paper's smallest point, 40 KB)
        _solve("slice_once", (1, 200, 200), 4, how="once"),
        # slices one after another on a solver that is kept (interactive use): latency of one solve and its labels
        _solve("slice_kept", (1, 256, 256), 4),
        # the same at the paper's stopping rule, compensated cross-block sums, a given start and an input that is not
        # aligned (a crop of a larger buffer)
        _solve("slice_crop", (1, 333, 517), 3, eps=0.005, offset=7, kahan=True, given=True),
        # a 1 MB volume (the paper's largest point) in a serving loop: solves and labels enqueued back to back
        _solve("volume_1m_async", (64, 128, 128), 4, how="async"),
        # a brain volume of the usual atlas size, more clusters and another fuzziness, waited for
        _solve("volume_7m_c8", (181, 217, 181), 8, m=2.5, sigma=3.0, bias=0.2),
        # the largest single volume, solve and labels enqueued, then the result read
        _solve("volume_67m", (256, 512, 512), 4, how="queued", sigma=9.0, bias=0.2),
        # a series of equal slices solved together
        {"name": "batch_series", "kind": "batch", "count": 64, "slices": 64, "lo": 256, "hi": 256, "C_lo": 4, "C_hi": 4,
         "eps": 1e-5},
        # the mixed batch: slices of side 64..512 and some cubes, 3 to 8 clusters each
        {"name": "batch_mixed", "kind": "batch", "count": 512, "slices": 496, "lo": 64, "hi": 512, "C_lo": 3, "C_hi": 8,
         "eps": 1e-5},
        # a slice solved from the network's start centroids
        {"name": "warm_slice", "kind": "warm", "d": 1, "h": 256, "w": 256, "C": 4, "sigma": 6.0, "bias": 0.1},
        # one epoch of training of the network on histograms of slices
        {"name": "train_epoch", "kind": "train", "count": 2048, "batch": 256, "C": 4, "epochs": 1},
        # start centroids for many slices: their histograms, then inference
        {"name": "starts_1024", "kind": "starts", "count": 1024, "side": 256, "C": 4},
        # segmentation quality of a large volume: confusion counts and Dice per tissue
        {"name": "dice_67m", "kind": "dice", "d": 256, "h": 512, "w": 512, "C": 4, "offset": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["batch"] * 2 + ["warm", "train", "starts", "dice"])
    if kind == "solve":
        C = rng.choice([2, 3, 4, 4, 4, 5, 6, 8])
        m = rng.choice([2.0, 2.0, 2.0, 1.5, 2.5, 3.0])
        how = rng.choice(["once", "handle", "handle", "async", "queued"])
        if rng.random() < 0.5:
            shape = (1, _log_int(rng, 64, 1024), _log_int(rng, 64, 1024))
        else:
            shape = (_log_int(rng, 20, 181), _log_int(rng, 64, 320), _log_int(rng, 64, 320))
        return _solve(None, shape, C, m=m, eps=rng.choice([1e-5, 1e-5, 1e-4, 0.005]), how=how,
                      offset=rng.choice([0, 0, 1, 5, 13]), kahan=rng.random() < 0.2, given=rng.random() < 0.2,
                      sigma=round(rng.uniform(3.0, 10.0), 2), bias=round(rng.uniform(0.0, 0.2), 3))
    if kind == "batch":
        lo = _log_int(rng, 64, 256)
        hi = _log_int(rng, lo, 512)
        C_lo = rng.randint(3, 5)
        count = _log_int(rng, 2, 400)
        return {"kind": "batch", "count": count, "slices": count - rng.randint(0, count // 32), "lo": lo, "hi": hi,
                "C_lo": C_lo, "C_hi": rng.randint(C_lo, 8), "eps": rng.choice([1e-5, 1e-4])}
    if kind == "warm":
        shape = (1, _log_int(rng, 100, 700), _log_int(rng, 100, 700)) if rng.random() < 0.7 else (
            _log_int(rng, 20, 128), 128, _log_int(rng, 64, 160))
        return {"kind": "warm", "d": shape[0], "h": shape[1], "w": shape[2], "C": 4, "sigma": round(rng.uniform(3.0, 10.0), 2),
                "bias": round(rng.uniform(0.0, 0.2), 3)}
    if kind == "train":
        return {"kind": "train", "count": _log_int(rng, 100, 3000), "batch": rng.choice([32, 64, 100, 256, 512]),
                "C": rng.choice([3, 4, 4, 6]), "epochs": 1}
    if kind == "starts":
        return {"kind": "starts", "count": _log_int(rng, 1, 1500), "side": _log_int(rng, 64, 256), "C": rng.choice([3, 4, 4, 5])}
    return {"kind": "dice", "d": _log_int(rng, 1, 128), "h": _log_int(rng, 64, 512), "w": _log_int(rng, 64, 512),
            "C": rng.choice([3, 4, 4, 6, 9]), "offset": rng.choice([0, 0, 3])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _phantom(shape, sigma, bias, gen, rs):
    """uint8 image of `shape` (d, h, w) on the GPU, and its tissue labels."""
    d, h, w = shape
    scale = 1.0 + 0.2 * (rs.random_sample(3) - 0.5)
    shift = rs.random_sample(3) - 0.5
    jit = [m * (1.0 + 0.1 * (rs.random_sample() - 0.5)) for m in MEANS]
    ax = [torch.linspace(-1, 1, s, device=DEV) if s > 1 else torch.zeros(1, device=DEV) for s in (w, h, d)]
    cs = [torch.cos(math.pi / 2 * a + float(p)) for a, p in zip(ax, shift)]
    field = cs[2].view(d, 1, 1) * cs[1].view(1, h, 1) * cs[0].view(1, 1, w)
    field = 1.0 + bias * field / field.abs().max()
    label = torch.zeros((d, h, w), dtype=torch.uint8, device=DEV)
    for k, axes in enumerate(AXES):
        r = [(a / float(s * e)) ** 2 for a, s, e in zip(ax, axes, scale)]
        label[(r[2].view(d, 1, 1) + r[1].view(1, h, 1) + r[0].view(1, 1, w)) <= 1.0] = k + 1
    img = torch.tensor(jit, dtype=torch.float32, device=DEV)[label.long()] * field
    img += sigma * torch.randn((d, h, w), device=DEV, generator=gen)
    return img.round_().clamp_(0, 255).to(torch.uint8), label


def _generators(seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) & 0x7FFFFFFF)
    return gen, np.random.RandomState(int(seed) & 0x7FFFFFFF)


def _placed(img, offset):
    """The image as a flat view `offset` bytes into a buffer of its own."""
    buf = torch.empty(img.numel() + offset + 16, dtype=torch.uint8, device=DEV)
    x = buf[offset:offset + img.numel()]
    x.copy_(img.reshape(-1))
    return x


def _solve_input(case, seed):
    gen, rs = _generators(seed)
    img, _ = _phantom((case["d"], case["h"], case["w"]), case["sigma"], case["bias"], gen, rs)
    x = _placed(img, case.get("offset", 0))
    init = None
    if case.get("given"):
        init = [float(v) for v in np.linspace(5.0, 160.0, case["C"]) + rs.uniform(-3.0, 3.0, case["C"])]
    return x, init


def _batch_input(case, seed):
    gen, rs = _generators(seed)
    mix = np.random.RandomState(case["count"])  # the sizes and cluster counts belong to the case, the voxels to the seed
    flat, sizes, Cs = [], [], []
    for i in range(case["count"]):
        side = int(mix.randint(case["lo"], case["hi"] + 1))
        shape = (1, side, side)
        if i >= case["slices"]:
            side = int(mix.randint(96, 161))
            shape = (side, side, side)
        img, _ = _phantom(shape, float(rs.uniform(3.0, 10.0)), float(rs.uniform(0.0, 0.2)), gen, rs)
        flat.append(img.reshape(-1))
        sizes.append(img.numel())
        Cs.append(int(mix.randint(case["C_lo"], case["C_hi"] + 1)))
    return torch.cat(flat), sizes, Cs


def _histograms(count, C, rs):
    """Normalised histograms of mixtures of C tissues, and their means / 255 (float64)."""
    g = np.arange(256)[None, None, :]
    mean = np.sort(rs.uniform(0.0, 200.0, (count, C)), axis=1) + 6.0 * np.arange(C)
    width = rs.uniform(4.0, 12.0, (count, C))
    share = rs.dirichlet(np.full(C, 4.0), count)
    dens = (share[:, :, None] / width[:, :, None] * np.exp(-0.5 * ((g - mean[:, :, None]) / width[:, :, None]) ** 2)).sum(1)
    hist = np.floor(65536 * dens / dens.sum(1, keepdims=True) + rs.random_sample((count, 256)))
    return hist / hist.sum(1, keepdims=True), mean / 255.0


def _network(C):
    """Parameters of a 256 -> 128 -> 64 -> C network that places centroids sensibly: random hidden layers and an
    output layer fitted by least squares (always the same, as a network that was trained once)."""
    rs = np.random.RandomState(20 + C)
    # first layer: smooth functions of the grey level, so that the hidden units see where the mass of a histogram lies
    g = np.arange(256)[:, None] / 255.0
    W1 = 2.0 * np.cos(math.pi * (rs.uniform(0.0, 6.0, (1, 128)) * g + rs.uniform(0.0, 2.0, (1, 128))))
    b1 = rs.normal(0.0, 0.3, 128)
    W2 = rs.normal(0.0, math.sqrt(2.0 / 128), (128, 64))
    b2 = rs.normal(0.0, 0.3, 64)
    h, t = _histograms(4000, C, rs)
    a = np.maximum(np.maximum(h @ W1 + b1, 0.0) @ W2 + b2, 0.0)
    A = np.concatenate([a, np.ones((len(a), 1))], axis=1)
    sol = np.linalg.solve(A.T @ A + 1e-1 * np.eye(65), A.T @ t)
    return np.concatenate([v.ravel() for v in (W1, b1, W2, b2, sol[:64], sol[64])]).astype(np.float32)


def _untrained(C):
    """He-initialised parameters: where a training starts."""
    rs = np.random.RandomState(40 + C)
    parts = []
    for rows, cols in ((256, 128), (128, 64), (64, C)):
        parts += [rs.normal(0.0, math.sqrt(2.0 / rows), rows * cols), np.zeros(cols)]
    return np.concatenate(parts).astype(np.float32)


def _dice_input(case, seed):
    gen, rs = _generators(seed)
    img, truth = _phantom((case["d"], case["h"], case["w"]), 8.0, 0.1, gen, rs)
    edges = torch.linspace(20.0, 140.0, case["C"] - 1, device=DEV)
    pred = torch.bucketize(img.float(), edges).to(torch.uint8)
    return _placed(pred, case["offset"]), truth.reshape(-1)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    from paper_1601_00072_amd import FCM, MLP, FCMBatch
    s = {"case": case}
    kind = case["kind"]
    if kind == "solve":
        s["x"], s["init"] = _solve_input(case, seed)
        if case["how"] != "once":
            s["labels"] = torch.empty_like(s["x"])
            s["fcm"] = FCM(s["x"], case["C"], m=case["m"], eps=case["eps"], init=s["init"], kahan_only=case["kahan"])
    elif kind == "batch":
        x, sizes, Cs = _batch_input(case, seed)
        s["x"], s["labels"] = x, torch.empty_like(x)
        s["batch"] = FCMBatch(x, sizes, [{"n_clusters": C, "eps": case["eps"]} for C in Cs])
    elif kind == "warm":
        s["x"], _ = _solve_input(case, seed)
        s["labels"] = torch.empty_like(s["x"])
        s["fcm"] = FCM(s["x"], case["C"])
        s["net"] = MLP(case["C"])
        s["net"].set_params(_network(case["C"]))
    elif kind == "train":
        _, rs = _generators(seed)
        h, t = _histograms(case["count"], case["C"], rs)
        s["hist"] = torch.from_numpy(h.astype(np.float32)).to(DEV)
        s["target"] = torch.from_numpy(t.astype(np.float32)).to(DEV)
        s["net"] = MLP(case["C"])
        s["theta"] = _untrained(case["C"])
    elif kind == "starts":
        gen, rs = _generators(seed)
        n = case["side"] ** 2
        s["x"] = torch.cat([_phantom((1, case["side"], case["side"]), 6.0, 0.1, gen, rs)[0].reshape(-1)
                            for _ in range(case["count"])])
        s["sizes"] = [n] * case["count"]
        s["net"] = MLP(case["C"])
        s["net"].set_params(_network(case["C"]))
    else:
        s["pred"], s["truth"] = _dice_input(case, seed)
    return s


def _found(res, labels):
    return {"labels": labels, "centroids": res.centroids.astype(np.float32), "J": np.float32(res.J)}


def run(s):
    from paper_1601_00072_amd import confusion, dice, histogram, solve
    case = s["case"]
    kind = case["kind"]
    if kind == "solve":
        if case["how"] == "once":
            res, labels = solve(s["x"], case["C"], m=case["m"], eps=case["eps"], init=s["init"], kahan_only=case["kahan"])
            return _found(res, labels)
        f = s["fcm"]
        if case["how"] in ("async", "queued"):
            f.solve_async(s["labels"])
            return {"labels": s["labels"]} if case["how"] == "async" else _found(f.result()[0], s["labels"])
        f.reset()
        res = f.solve()
        return _found(res, f.labels(s["labels"]))
    if kind == "batch":
        res = s["batch"].solve()
        s["batch"].labels(s["labels"])
        return {"labels": s["labels"], "centroids": np.concatenate([r.centroids for r in res]).astype(np.float32),
                "J": np.array([r.J for r in res], dtype=np.float32)}
    if kind == "warm":
        res, _, _ = s["fcm"].solve_warm(s["net"])
        return _found(res, s["fcm"].labels(s["labels"]))
    if kind == "train":
        s["net"].set_params(s["theta"])
        losses = s["net"].train(s["hist"], s["target"], epochs=case["epochs"], batch=case["batch"], lr=1e-3, seed=3)
        return {"params": s["net"].params(), "losses": losses.astype(np.float32)}
    if kind == "starts":
        hist = histogram(s["x"], s["sizes"])
        return {"hist": hist, "starts": s["net"].warm_centroids(hist)}
    counts = confusion(s["pred"], s["truth"], case["C"], 4)
    return {"counts": counts, "dice": dice(counts, case["C"], 4)}


def _voxels(case):
    if case["kind"] == "starts":
        return case["count"] * case["side"] ** 2
    if case["kind"] == "batch":
        lo, hi = case["lo"], case["hi"]
        return case["slices"] * (lo * lo + lo * hi + hi * hi) / 3.0 + (case["count"] - case["slices"]) * 128 ** 3
    return case["d"] * case["h"] * case["w"]


def work(case):
    """The voxels read once and the labels written once; a membership evaluation over the 256 grey levels per
    iteration is all the arithmetic that 8-bit data need, so it counts as nothing beside the bytes."""
    kind = case["kind"]
    if kind == "train":
        params = 256 * 128 + 128 + 128 * 64 + 64 + 64 * case["C"] + case["C"]
        steps = -(-case["count"] // case["batch"]) * case["epochs"]
        return {"bytes": 4.0 * (case["count"] * case["epochs"] * (256 + case["C"]) + 6 * params * steps),
                "flops": 6.0 * params * case["count"] * case["epochs"]}
    if kind == "starts":
        return {"bytes": float(_voxels(case) + 4 * 256 * case["count"]), "flops": 2.0 * 41000 * case["count"]}
    return {"bytes": 2.0 * _voxels(case), "flops": 0.0}


# ---------------------------------------------------------------------------
# 64-bit values, in plain numpy and torch
# ---------------------------------------------------------------------------

def _memberships(x, v, m):
    d = np.abs(x[:, None] - v[None, :])
    zero = d == 0.0
    d[zero] = 1.0
    w = (d.min(axis=1, keepdims=True) / d) ** (2.0 / (m - 1.0))
    rows = zero.any(axis=1)
    w[rows] = zero[rows]
    return w / w.sum(axis=1, keepdims=True)


def _fcm64(counts, C, m, eps, v0=None, max_iter=300):
    """Algorithm 1 over the grey levels present (every voxel sum regroups by level): v^T and J^T."""
    g = np.nonzero(counts)[0]
    x, c = g.astype(np.float64), counts[g].astype(np.float64)
    lo, hi = x[0], x[-1]
    v = np.asarray(v0 if v0 is not None else [lo + k * (hi - lo) / (C - 1) for k in range(C)], dtype=np.float64)
    v = v.astype(np.float32).astype(np.float64)
    before, t = None, 0
    while True:
        u = _memberships(x, v, m)
        a = c[:, None] * u ** m
        J = float((a * (x[:, None] - v[None, :]) ** 2).sum())
        if t >= max_iter or (before is not None and np.abs(u - before).max() < eps):
            return v, J
        den = a.sum(axis=0)
        v = np.where(den > 0.0, (a * x[:, None]).sum(axis=0) / np.where(den > 0.0, den, 1.0), v)
        before, t = u, t + 1


def _counts(x):
    h = np.zeros(256, dtype=np.int64)
    for part in x.split(1 << 24):
        h += torch.bincount(part.int(), minlength=256).cpu().numpy()
    return h


def _network64(theta, h, C):
    p, o = theta.astype(np.float64), 0
    W = []
    for rows, cols in ((256, 128), (1, 128), (128, 64), (1, 64), (64, C), (1, C)):
        W.append(p[o:o + rows * cols].reshape(rows, cols))
        o += rows * cols
    z1 = np.maximum(h @ W[0] + W[1], 0.0)
    z2 = np.maximum(z1 @ W[2] + W[3], 0.0)
    return W, z1, z2, z2 @ W[4] + W[5]


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        if case["how"] == "async":
            return None  # labels alone: whole numbers
        x, init = _solve_input(case, seed)
        v, J = _fcm64(_counts(x), case["C"], case["m"], case["eps"], init)
        return {"labels": None, "centroids": v, "J": np.float64(J)}
    if kind == "batch":
        x, sizes, Cs = _batch_input(case, seed)
        found = [_fcm64(_counts(p), C, 2.0, case["eps"]) for p, C in zip(x.split(sizes), Cs)]
        return {"labels": None, "centroids": np.concatenate([v for v, _ in found]), "J": np.array([J for _, J in found])}
    if kind == "starts":
        gen, rs = _generators(seed)
        h = np.stack([_counts(_phantom((1, case["side"], case["side"]), 6.0, 0.1, gen, rs)[0].reshape(-1))
                      for _ in range(case["count"])]).astype(np.float64)
        return {"hist": h / h.sum(axis=1, keepdims=True), "starts": None}  # the network runs in BF16 by contract
    if kind == "dice":
        pred, truth = _dice_input(case, seed)
        n = np.zeros((case["C"], 4))
        for p, t in zip(pred.split(1 << 24), truth.split(1 << 24)):
            n += torch.bincount(p.int() * 4 + t.int(), minlength=4 * case["C"]).cpu().numpy().reshape(case["C"], 4)
        both = np.array([n[k, k] if k < case["C"] else 0.0 for k in range(4)])
        own = np.array([n[k].sum() if k < case["C"] else 0.0 for k in range(4)])
        with np.errstate(invalid="ignore"):
            return {"counts": None, "dice": 2.0 * both / (own + n.sum(axis=0))}
    if kind == "train" and case["batch"] >= case["count"] and case["epochs"] == 1:
        _, rs = _generators(seed)
        h, t = _histograms(case["count"], case["C"], rs)
        h, t = h.astype(np.float32).astype(np.float64), t.astype(np.float32).astype(np.float64)
        _, _, _, y = _network64(_untrained(case["C"]), h, case["C"])
        return {"params": None, "losses": np.array([((y - t) ** 2).mean()])}
    return None  # a minibatch's order is the library's own; a warm start runs through BF16
