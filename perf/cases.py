"""The calls that a user of the layout library makes, as cases to be timed and compared.

Kinds of case (one public call or the short sequence of calls that a program makes in one go):

* ``fuzzy``      kNN lists -> fuzzy union B on the device (``umap_fuzzy_graph_device``);
* ``fit``        a whole layout: create from B, the random start and every epoch, copy out, destroy;
* ``epochs``     a handle that is kept: the next epochs from its present layout, copy out (a program that takes a run
                 in pieces and looks at the layout in between);
* ``refine``     B with new weights and the layout of an earlier run: create, set the embedding, the last epochs;
* ``transform``  new points against a frozen layout: create from host arrays, every epoch, copy out;
* ``trust``      T(k) of a layout of points (``umap_trustworthiness``).

Graphs: up to 100,000 vertices the exact kNN graph of clustered points in the order in which a data set lists them
(random); beyond, a window kNN graph (k of the 128 nearest ids, distances a running sum of exponential steps), either
in its own order (neighbours have close ids) or with the vertices shuffled, as they are in most data sets.
"""

from __future__ import annotations

import math

import torch

from paper_2008_00325_amd import umap_layout as U

# a and b of Phi at spread 1, min_dist 0.1
PHI_A, PHI_B = 1.5769436359405518, 0.8950607180595398
DEV = "cuda"
MAX_POINTS = 100_000   # exact kNN of points up to here, window graphs beyond


def listed() -> list[dict]:
    return [
        # the smallest data sets (2,000 points, the shape of the digits / blobs experiments): latency and launches
        dict(name="fuzzy_2k", kind="fuzzy", n=2000, k=15, order="random"),
        # the input side at a million points, vertices in the order of the data set
        dict(name="fuzzy_1m", kind="fuzzy", n=1_000_000, k=15, order="random"),
        # a whole small layout from host arrays, 500 epochs as small sets get
        dict(name="fit_2k", kind="fit", n=2000, k=15, dim=2, epochs=500, neg=5, order="random", host=True),
        # a whole layout of an MNIST-sized set
        dict(name="fit_70k", kind="fit", n=70_000, k=15, dim=2, epochs=200, neg=5, order="random", host=False),
        # the benchmark's workload: a million vertices in local order, ingest and 200 epochs
        dict(name="fit_1m", kind="fit", n=1_000_000, k=15, dim=2, epochs=200, neg=5, order="local", host=False),
        # a million vertices in the order of the data set: neighbours anywhere in the table
        dict(name="epochs_1m_shuffled", kind="epochs", n=1_000_000, k=15, dim=2, epochs=200, neg=5, order="random",
             steps=20),
        # more neighbours and three output dimensions (the k = 30 workload)
        dict(name="epochs_1m_k30_3d", kind="epochs", n=1_000_000, k=30, dim=3, epochs=200, neg=5, order="local",
             steps=20),
        # a layout made for clustering, ten output dimensions, ragged size
        dict(name="epochs_200k_10d", kind="epochs", n=200_003, k=15, dim=10, epochs=200, neg=5, order="random",
             steps=20),
        # the graph of an earlier layout with new weights: ingest and the last epochs
        dict(name="refine_777k", kind="refine", n=777_777, k=15, dim=2, epochs=200, neg=5, order="random", steps=10),
        # inference: 50,003 new points against a million-row layout
        dict(name="transform_50k", kind="transform", n=50_003, n_table=1_000_000, k=15, dim=2, epochs=100, neg=5),
        # the quality measure on a small and on an image-like set
        dict(name="trust_5k", kind="trust", n=5003, d=64, k=15, dim=2),
        dict(name="trust_70k", kind="trust", n=70_000, d=784, k=15, dim=2),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["fuzzy", "fuzzy", "fit", "fit", "epochs", "epochs", "refine", "transform", "trust", "trust"])
    k = rng.choice([5, 10, 15, 15, 15, 20, 30])
    dim = rng.choice([2, 2, 2, 2, 3, 3, 5, 8, 10, 16])
    neg = rng.choice([5, 5, 5, 5, 3, 8, 10])
    order = rng.choice(["random", "random", "local"])
    if kind == "fuzzy":
        return dict(kind=kind, n=_log_int(rng, 1000, 1_000_000), k=k, order=order)
    if kind == "fit":
        n = _log_int(rng, 1000, 200_000)
        return dict(kind=kind, n=n, k=k, dim=dim, epochs=500 if n <= 10_000 else 200, neg=neg, order=order,
                    host=rng.random() < 0.3)
    if kind == "epochs":
        return dict(kind=kind, n=_log_int(rng, 10_000, 1_000_000), k=k, dim=dim, epochs=200, neg=neg, order=order,
                    steps=20)
    if kind == "refine":
        return dict(kind=kind, n=_log_int(rng, 10_000, 1_000_000), k=k, dim=rng.choice([2, 2, 3]), epochs=200, neg=neg,
                    order=order, steps=10)
    if kind == "transform":
        return dict(kind=kind, n=_log_int(rng, 100, 100_000), n_table=_log_int(rng, 2000, 1_000_000), k=k,
                    dim=rng.choice([2, 2, 2, 3, 8]), epochs=rng.choice([30, 100]), neg=neg)
    n = _log_int(rng, 2000, 50_000)
    return dict(kind="trust", n=n, d=_log_int(rng, 16, 784), k=rng.choice([5, 15, 15, 15, 30]),
                dim=rng.choice([2, 2, 2, 3, 10]))


# ---- inputs ---------------------------------------------------------------


def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _points_knn(n: int, k: int, g: torch.Generator) -> tuple[torch.Tensor, torch.Tensor]:
    """Exact kNN (self excluded) of points in 50-D around 10 centres, in random order; Euclidean distances ascending."""
    c = 4.0 * torch.randn(10, 50, generator=g, device=DEV)
    scale = 0.5 + torch.rand(10, 1, generator=g, device=DEV)
    lab = torch.randint(0, 10, (n,), generator=g, device=DEV)
    x = c[lab] + scale[lab] * torch.randn(n, 50, generator=g, device=DEV)
    sq = (x * x).sum(1)
    ids = torch.empty(n, k, dtype=torch.int32, device=DEV)
    dist = torch.empty(n, k, dtype=torch.float32, device=DEV)
    step = max(1, (1 << 28) // n)
    for s in range(0, n, step):
        t = min(n, s + step)
        d2 = sq[s:t, None] + sq[None, :] - 2.0 * (x[s:t] @ x.T)
        d2[torch.arange(t - s, device=DEV), torch.arange(s, t, device=DEV)] = math.inf
        v, i = torch.topk(d2, k, dim=1, largest=False, sorted=True)
        ids[s:t] = i.int()
        dist[s:t] = v.clamp_min(0.0).sqrt()
    return ids, dist


def _window_picks(lo: torch.Tensor, hi: torch.Tensor, centre: torch.Tensor, k: int, g: torch.Generator,
                  self_too: bool) -> torch.Tensor:
    """k distinct ids per row within 64 of `centre` and inside [lo, hi); the centre itself only with self_too."""
    off = torch.arange(-64, 65, device=DEV)
    if not self_too:
        off = off[off != 0]
    key = torch.rand(centre.numel(), off.numel(), generator=g, device=DEV)
    cand = centre[:, None] + off[None, :]
    key[(cand < lo) | (cand >= hi)] = 2.0
    pick = torch.topk(key, k, dim=1, largest=False, sorted=True).indices
    return torch.gather(cand, 1, pick)


def _window_knn(n: int, k: int, order: str, g: torch.Generator) -> tuple[torch.Tensor, torch.Tensor]:
    ids = torch.empty(n, k, dtype=torch.int32, device=DEV)
    for s in range(0, n, 1 << 18):
        rows = torch.arange(s, min(n, s + (1 << 18)), device=DEV)
        ids[rows] = _window_picks(0, n, rows, k, g, False).int()
    step = -torch.log1p(-torch.rand(n, k, generator=g, device=DEV))
    dist = torch.cumsum(step, 1)
    if order == "random":
        p = torch.randperm(n, generator=g, device=DEV)
        ids2, dist2 = torch.empty_like(ids), torch.empty_like(dist)
        ids2[p] = p[ids.long()].int()
        dist2[p] = dist
        ids, dist = ids2, dist2
    return ids.contiguous(), dist.contiguous()


def _knn(case: dict, g: torch.Generator) -> tuple[torch.Tensor, torch.Tensor]:
    if case["n"] <= MAX_POINTS and case["order"] == "random":
        return _points_knn(case["n"], case["k"], g)
    return _window_knn(case["n"], case["k"], case["order"], g)


def _memberships(dist: torch.Tensor) -> torch.Tensor:
    """exp(-max(0, d - rho) / sigma) in 64 bits: rho the row's least positive distance, sigma by bisection (start 1,
    doubled while unbounded, at most 64 steps, stop within 1e-5 of log2 k), at least 1e-3 of the mean distance."""
    n, k = dist.shape
    d = dist.double()
    rho = torch.where(d > 0, d, math.inf).min(1).values
    found = torch.isfinite(rho)
    rho = torch.where(found, rho, 0.0)
    x = (d - rho[:, None]).clamp_min(0.0)
    lo = torch.zeros(n, dtype=torch.float64, device=DEV)
    hi = torch.full_like(lo, math.inf)
    s = torch.ones_like(lo)
    done = torch.zeros(n, dtype=torch.bool, device=DEV)
    target = math.log2(k)
    for _ in range(64):
        f = torch.exp(-x / s[:, None]).sum(1)
        done |= (f - target).abs() < 1e-5
        if bool(done.all()):
            break
        up = f > target
        hi = torch.where(up & ~done, s, hi)
        lo = torch.where(~up & ~done, s, lo)
        s = torch.where(done, s, torch.where(torch.isinf(hi), 2.0 * s, 0.5 * (lo + hi)))
    floor = torch.where(found, 1e-3 * d.mean(1), 1e-3 * d.mean())
    return torch.exp(-x / torch.maximum(s, floor)[:, None])


def _union(ids: torch.Tensor, dist: torch.Tensor) -> tuple[torch.Tensor, torch.Tensor, torch.Tensor]:
    """rows, cols and values (64 bits) of B = A + A^T - A o A^T in 2 n k slots: (i, j) in slot i k + s, (j, i) in slot
    n k + i k + s, or a placeholder (i, i, 0) there when row j lists i itself."""
    n, k = ids.shape
    m = _memberships(dist).reshape(-1)
    i = torch.arange(n, device=DEV).repeat_interleave(k)
    j = ids.reshape(-1).long()
    key, perm = torch.sort(i * n + j)
    rev = j * n + i
    pos = torch.searchsorted(key, rev).clamp_max(key.numel() - 1)
    mutual = key[pos] == rev
    back = torch.where(mutual, m[perm[pos]], 0.0)
    b = m + back - m * back
    rows = torch.cat([i, torch.where(mutual, i, j)]).int()
    cols = torch.cat([j, i]).int()
    return rows, cols, torch.cat([b, torch.where(mutual, 0.0, b)])


def _graph(case: dict, g: torch.Generator) -> tuple[torch.Tensor, torch.Tensor, torch.Tensor]:
    rows, cols, vals = _union(*_knn(case, g))
    return rows, cols, vals.float()


def _curve(n: int, dim: int, g: torch.Generator) -> torch.Tensor:
    """A layout in which close ids lie close together: a closed curve through [-10, 10]^dim with some noise."""
    t = torch.arange(n, device=DEV)[:, None] / n * (2.0 * math.pi)
    f = torch.arange(1, dim + 1, device=DEV)[None, :] * 3.0 + 4.0
    return (9.0 * torch.sin(t * f + f) + 0.1 * torch.randn(n, dim, generator=g, device=DEV)).float().contiguous()


def _transform_inputs(case: dict, g: torch.Generator):
    n, m, k = case["n"], case["n_table"], case["k"]
    anchor = torch.randint(0, m, (n,), generator=g, device=DEV)
    cols = _window_picks(0, m, anchor, k, g, True).int().reshape(-1)
    rows = torch.arange(n, device=DEV, dtype=torch.int32).repeat_interleave(k)
    vals = 0.05 + 0.95 * torch.rand(n * k, generator=g, device=DEV)
    return _curve(m, case["dim"], g), rows, cols, vals


def _trust_inputs(case: dict, g: torch.Generator) -> tuple[torch.Tensor, torch.Tensor]:
    """Image-like points in [0, 1]^d on a noisy surface over `dim` latent coordinates, and the latent coordinates with
    some noise as their layout (neighbourhoods mostly kept)."""
    n, d, dim = case["n"], case["d"], case["dim"]
    z = torch.randn(n, dim, generator=g, device=DEV) + 4.0 * torch.randn(10, dim, generator=g, device=DEV)[
        torch.randint(0, 10, (n,), generator=g, device=DEV)]
    w = torch.randn(dim, d, generator=g, device=DEV) / math.sqrt(dim)
    ph = torch.rand(d, generator=g, device=DEV) * 2.0 * math.pi
    x = 0.4 + 0.5 * torch.sin(0.3 * (z @ w) + ph) + 0.05 * torch.randn(n, d, generator=g, device=DEV)
    y = z + 0.05 * torch.randn(n, dim, generator=g, device=DEV)
    return x.clamp(0.0, 1.0).float().contiguous(), y.float().contiguous()


def _run_seed(seed: int) -> int:
    return (int(seed) * 0x9E3779B97F4A7C15 + 1) & ((1 << 63) - 1)


def prepare(case: dict, seed: int) -> dict:
    g = _gen(seed)
    kind, n = case["kind"], case["n"]
    st = dict(case, seed=_run_seed(seed))
    if kind == "fuzzy":
        st["ids"], st["dist"] = _knn(case, g)
        m = 2 * n * case["k"]
        st["rows"] = torch.empty(m, dtype=torch.int32, device=DEV)
        st["cols"] = torch.empty(m, dtype=torch.int32, device=DEV)
        st["vals"] = torch.empty(m, dtype=torch.float32, device=DEV)
    elif kind in ("fit", "refine", "epochs"):
        coo = _graph(case, g)
        if case.get("host"):
            st["coo"] = tuple(t.cpu().numpy() for t in coo)
        else:
            st["coo"] = coo
            st["out"] = torch.empty(n, case["dim"], dtype=torch.float32, device=DEV)
        if kind in ("refine", "epochs"):
            st["start"] = (20.0 * torch.rand(n, case["dim"], generator=g, device=DEV) - 10.0).cpu().numpy()
        if kind == "epochs":
            st["h"] = _create_device(st)
            U.umap_layout_set_embedding(st["h"], st["start"])
            del st["coo"], st["start"]
    elif kind == "transform":
        table, rows, cols, vals = _transform_inputs(case, g)
        st["table"], st["coo"] = table.cpu().numpy(), tuple(t.cpu().numpy() for t in (rows, cols, vals))
    else:
        st["x"], st["y"] = _trust_inputs(case, g)
    return st


def _create_device(st: dict) -> U.Handle:
    r, c, v = st["coo"]
    return U.umap_layout_create_device(st["n"], st["dim"], r, c, v, r.numel(), PHI_A, PHI_B, st["epochs"], st["neg"])


def run(st: dict):
    kind = st["kind"]
    if kind == "fuzzy":
        U.umap_fuzzy_graph_device(st["n"], st["k"], st["ids"], st["dist"], st["rows"], st["cols"], st["vals"])
        return st["rows"], st["cols"], st["vals"]
    if kind == "trust":
        return U.umap_trustworthiness(st["x"], st["y"], st["k"])
    if kind == "transform":
        with U.umap_transform_create(st["n"], st["table"], *st["coo"], PHI_A, PHI_B, st["epochs"], st["neg"]) as h:
            U.umap_layout_run(h, st["seed"])
            return U.umap_layout_get(h)
    if kind == "epochs":
        U.umap_layout_run_epochs(st["h"], st["seed"], st["epochs"] - st["steps"], st["epochs"])
        U.umap_layout_get_device(st["h"], st["out"])
        return st["out"]
    if kind == "refine":
        with _create_device(st) as h:
            U.umap_layout_set_embedding(h, st["start"])
            U.umap_layout_run_epochs(h, st["seed"], st["epochs"] - st["steps"], st["epochs"])
            U.umap_layout_get_device(h, st["out"])
        return st["out"]
    if st["host"]:
        with U.umap_layout_create(st["n"], st["dim"], *st["coo"], PHI_A, PHI_B, st["epochs"], st["neg"]) as h:
            U.umap_layout_run(h, st["seed"])
            return U.umap_layout_get(h)
    with _create_device(st) as h:
        U.umap_layout_run(h, st["seed"])
        U.umap_layout_get_device(h, st["out"])
    return st["out"]


# ---- what a pass cannot do without ------------------------------------------


def work(case: dict) -> dict:
    kind, n, k = case["kind"], case["n"], case["k"]
    if kind == "fuzzy":
        # lists read once, COO written once; a few evaluations of k exponentials per row
        return {"bytes": 8.0 * n * k + 24.0 * n * k, "flops": 20.0 * 2.0 * n * k}
    if kind == "trust":
        d, dim = case["d"], case["dim"]
        return {"bytes": 4.0 * n * (d + dim), "flops": float(n) * n * (d + 3 * dim)}   # each pair of points once
    dim, neg = case["dim"], case["neg"]
    if kind == "transform":
        kept, moved, steps, ingest = 1.0 * n * k, 0.53, case["epochs"], 12.0 * n * k + 4.0 * case["n_table"] * dim
    else:
        # about 1.78 of the n k neighbours survive as edges of the union; an edge is sampled in 0.29 of the epochs
        kept, moved = 1.78 * n * k, 0.29
        steps = case.get("steps", case["epochs"])
        ingest = 0.0 if kind == "epochs" else 24.0 * n * k
    updates = kept * moved * steps * (1 + neg)
    # per epoch: eps of every edge, the tail of a sampled one, the layout read and written
    stream = steps * (4.0 * kept + 4.0 * kept * moved + 8.0 * n * dim)
    return {"bytes": ingest + stream, "flops": updates * (5.0 * dim + 10.0)}


def tolerance(case: dict):
    kind = case["kind"]
    if kind in ("fit", "transform"):
        # hundreds of epochs of a chaotic iteration: another rounding anywhere ends in another layout.  The library's
        # contract is that the sums are exact and the layout is a function of the seed, bit for bit.
        return "exact"
    if kind == "fuzzy":
        return {"rel": 1e-7}
    if kind == "trust":
        return {"rel": 2.5e-7}
    # single epochs in 32 bits (measured 1e-7 to 1e-6 off 64 bits); a pair that nearly meets moves a coordinate further
    return {"rel": 4e-6, "max": 0.05}


# ---- the same in 64 bits, in plain torch ----------------------------------


def _philox(c0, c1, c2, c3, key: int):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    mask = 0xFFFFFFFF
    k0, k1 = key & mask, (key >> 32) & mask
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # modulo 2^64: the words of the product are read out below
        c0, c1, c2, c3 = (((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask)
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _exact_epochs(rows, cols, eps, y, table, first: int, last: int, n_epochs: int, neg: int, key: int) -> torch.Tensor:
    """Epochs first .. last - 1 from layout y over edges sorted by (row, col); table: the frozen layout of a transform,
    None for a fit."""
    e_all = torch.arange(rows.numel(), device=DEV)
    eps64 = eps.double()

    def periods(m: int):
        return torch.floor((m / eps64).float())    # a 64-bit quotient rounded once more is the 32-bit quotient

    for ep in range(first, last):
        act = periods(ep + 1) > periods(ep)
        i, j, e = rows[act], cols[act], e_all[act]
        src = y if table is None else table
        diff = y[i] - src[j]
        d2 = (diff * diff).sum(1, keepdim=True)
        p = d2 ** PHI_B
        c = torch.where(d2 > 0, -2.0 * PHI_A * PHI_B * p / (d2 * (1.0 + PHI_A * p)), 0.0)
        total = torch.zeros_like(y)
        total.index_add_(0, i, (2.0 if table is None else 1.0) * (c * diff).clamp(-4.0, 4.0))
        for r in range(neg):
            if r % 4 == 0:
                w = _philox(e & 0xFFFFFFFF, e >> 32, torch.full_like(e, ep), torch.full_like(e, 0x4E470000 | (r >> 2)), key)
            v = (w[r % 4] * src.shape[0]) >> 32
            diff = y[i] - src[v]
            if table is None:
                diff = torch.where((v == i)[:, None], 0.0, diff)
            d2 = (diff * diff).sum(1, keepdim=True)
            c = 2.0 * PHI_B / ((1e-3 + d2) * (1.0 + PHI_A * d2 ** PHI_B))
            total.index_add_(0, i, (c * diff).clamp(-4.0, 4.0))
        y = y + (1.0 - ep / n_epochs) * total
    return y


def _kept(rows, cols, vals, n_cols: int, n_epochs: int, fit: bool):
    ok = (vals > 0) & ((rows != cols) if fit else True)
    rows, cols, vals = rows[ok].long(), cols[ok].long(), vals[ok]
    w_max = vals.max()
    ok = vals >= w_max / n_epochs
    rows, cols, vals = rows[ok], cols[ok], vals[ok]
    o = torch.argsort(rows * n_cols + cols)
    return rows[o], cols[o], (w_max.double() / vals[o].double()).float()


def exact(case: dict, seed: int):
    g = _gen(seed)
    kind, n, key = case["kind"], case["n"], _run_seed(seed)
    if kind == "fuzzy":
        return None, None, _union(*_knn(case, g))[2]
    if kind in ("epochs", "refine"):
        rows, cols, eps = _kept(*_graph(case, g), n, case["epochs"], True)
        y = (20.0 * torch.rand(n, case["dim"], generator=g, device=DEV) - 10.0).double()
        first, last = case["epochs"] - case["steps"], case["epochs"]
        return _exact_epochs(rows, cols, eps, y, None, first, last, case["epochs"], case["neg"], key)
    if kind == "trust":
        x, y = _trust_inputs(case, g)
        return _exact_trust(x.double(), y.double(), case["k"])
    return None   # a whole run: chaotic, 64 bits end in another layout


def _exact_trust(x: torch.Tensor, y: torch.Tensor, k: int) -> float:
    n = x.shape[0]
    nx, pen = (x * x).sum(1), 0
    step = max(1, (1 << 27) // n)
    for s in range(0, n, step):
        t = min(n, s + step)
        i, own = torch.arange(t - s, device=DEV), torch.arange(s, t, device=DEV)
        dy = torch.zeros(t - s, n, dtype=torch.float64, device=DEV)
        for q in range(y.shape[1]):
            dy += (y[s:t, q, None] - y[None, :, q]) ** 2
        dy[i, own] = math.inf
        nbr = torch.topk(dy, k, dim=1, largest=False).indices
        dx = nx[s:t, None] + nx[None, :] - 2.0 * (x[s:t] @ x.T)
        dx[i, own] = math.inf
        thr = torch.gather(dx, 1, nbr)
        for q in range(k):
            rank = (dx < thr[:, q, None]).sum(1) + 1
            pen += int((rank - k).clamp_min(0).sum())
    return 1.0 - 2.0 / (n * k * (2.0 * n - 3.0 * k - 1.0)) * pen
