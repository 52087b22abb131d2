"""Trustworthiness where its tiles and pieces change: panels of 128 points, 32
features per step, 8 or 16 thresholds at a time.  Points on a lattice of small
integers, many of them repeated, have exact fp32 distances with ties
everywhere, so the GPU's ranks must equal the oracle's one for one; generic
points agree within the swaps that fp32 cannot tell apart.  The fp32 kernels
that run where the points' bf16 parts do not fit are held to the same."""

import sys

import numpy as np
import pytest

import oracle as O
from paper_2008_00325_amd import umap_layout as U

pytestmark = pytest.mark.gpu


def case(msg):
    print(f"[gpu case] {msg}", flush=True)
    sys.stdout.flush()


def _both(monkeypatch, X, Y, k):
    import torch

    torch.cuda.set_device(0)
    x, y = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    monkeypatch.setenv("UMAP_LAYOUT_FAULT", "pairs")    # however few points
    pairs = U.umap_trustworthiness(x, y, k)
    monkeypatch.setenv("UMAP_LAYOUT_FAULT", "split")
    plain = U.umap_trustworthiness(x, y, k)
    monkeypatch.delenv("UMAP_LAYOUT_FAULT")
    assert U.umap_trustworthiness(x, y, k) in (pairs, plain)
    return pairs, plain


SHAPES = [(5, 1, 1, 1), (127, 31, 3, 7), (128, 32, 2, 8), (129, 33, 2, 9), (256, 64, 16, 16), (257, 5, 1, 17),
          (383, 100, 2, 32), (385, 7, 3, 33), (640, 17, 2, 64), (1500, 3, 2, 15)]


@pytest.mark.parametrize("n,d,dim,k", SHAPES)
def test_lattice_ranks_equal_the_oracle(monkeypatch, n, d, dim, k):
    rng = np.random.default_rng(n * 7 + d)
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32)
    X[rng.integers(0, n, n // 4)] = X[rng.integers(0, n, n // 4)]
    Y = rng.standard_normal((n, dim)).astype(np.float32)   # the oracle takes ties of the embedding in any order
    case(f"lattice n {n} d {d} dim {dim} k {k}")
    want = O.trustworthiness(X, Y, k)
    for got in _both(monkeypatch, X, Y, k):
        assert abs(got - want) <= 1e-12


@pytest.mark.parametrize("n,d,k", [(32640, 3, 5), (32641, 7, 17), (33001, 96, 5)])
def test_long_rows_of_tiles_equal_the_fp32_kernels(monkeypatch, n, d, k):
    """Runs of four tiles, with 255, 256 and 258 panels (runs that end at the last
    panel, one, two and three tiles before): both kernels' distances are exact on a lattice, so that the ranks are the
    same."""
    rng = np.random.default_rng(n + d)
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32)
    X[rng.integers(0, n, n // 4)] = X[rng.integers(0, n, n // 4)]
    Y = rng.standard_normal((n, 2)).astype(np.float32)
    case(f"runs n {n} d {d} k {k}")
    pairs, plain = _both(monkeypatch, X, Y, k)
    assert abs(pairs - plain) <= 1e-12


def test_more_blocks_than_one_launch_holds(monkeypatch):
    """11,584 panels: runs of four tiles would take more than 2^24 blocks of 256
    threads, the most that a launch holds, so the runs are longer."""
    n = 11_584 * 128 - 5
    rng = np.random.default_rng(8)
    X = rng.integers(-40, 41, size=(n, 3)).astype(np.float32)
    Y = np.concatenate([X[:, :1] + rng.standard_normal((n, 1)), rng.standard_normal((n, 1))], axis=1).astype(np.float32)
    case(f"grid limit n {n}")
    pairs, plain = _both(monkeypatch, X, Y, 2)
    assert 0.0 < pairs < 1.0 and abs(pairs - plain) <= 1e-12


@pytest.mark.parametrize("n,d,dim,k", [(1001, 40, 2, 15), (2049, 300, 3, 5), (1500, 784, 2, 30)])
def test_scales_of_features(monkeypatch, n, d, dim, k):
    """Features of very different scales (all three parts of a value matter)."""
    rng = np.random.default_rng(n)
    Z = rng.standard_normal((n, dim))
    X = (np.sin(Z @ rng.standard_normal((dim, d))) * 10.0 ** rng.integers(-4, 5, size=d)).astype(np.float32)
    Y = (Z + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    case(f"scales n {n} d {d} dim {dim} k {k}")
    want = O.trustworthiness(X, Y, k)
    # a pair that fp32 distances order differently moves T by 2 / (n k (2n - 3k - 1)); a hundred of n k are allowed
    for got in _both(monkeypatch, X, Y, k):
        assert abs(got - want) <= 200.0 / (n * k * (2.0 * n - 3.0 * k - 1.0))


def test_far_and_non_finite_embedding():
    """Embedding coordinates whose squared distances overflow are ranked by
    index; non-finite ones are refused."""
    import torch

    n, k = 300, 15
    rng = np.random.default_rng(1)
    X = rng.standard_normal((n, 6)).astype(np.float32)
    Y = rng.standard_normal((n, 2)).astype(np.float32)
    Y[7] = 1e30
    Y[200] = -3e38
    with np.errstate(over="ignore"):
        D = ((Y[:, None, :] - Y[None, :, :]) ** 2).sum(-1)
    assert np.isinf(D[7]).sum() == n - 1
    case("embedding with overflowing distances")
    t = U.umap_trustworthiness(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), k)
    np.fill_diagonal(D, np.nan)
    nbr = np.argsort(np.where(np.isnan(D), np.inf, D) + 0.0, axis=1, kind="stable")
    nbr = np.stack([r[r != i][:k] for i, r in enumerate(nbr)])
    DX = ((X[:, None, :].astype(np.float64) - X[None, :, :]) ** 2).sum(-1)
    np.fill_diagonal(DX, np.inf)
    rank = np.argsort(np.argsort(DX, axis=1, kind="stable"), axis=1, kind="stable") + 1
    pen = np.maximum(np.take_along_axis(rank, nbr, axis=1) - k, 0).sum()
    want = 1.0 - 2.0 / (n * k * (2.0 * n - 3.0 * k - 1.0)) * pen
    assert abs(t - want) <= 4.0 / (n * k * (2.0 * n - 3.0 * k - 1.0))
    Y[3] = np.nan
    with pytest.raises(U.UmapLayoutError) as ei:
        U.umap_trustworthiness(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), k)
    assert ei.value.code == U.UMAP_E_INVAL


@pytest.mark.parametrize("n,d,k", [(300, 6, 5), (1000, 40, 15), (515, 33, 40)])
@pytest.mark.parametrize("what", ["inf", "-inf", "nan", "far", "inf and nan", "all far"])
def test_far_and_non_finite_points(monkeypatch, n, d, k, what):
    """Input points that are not finite, or whose squared norms or distances leave
    fp32's range, give the ranks of the fp32 kernels."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Y = X[:, :2] + 0.1 * rng.standard_normal((n, 2)).astype(np.float32)
    if "inf" in what:
        X[7, d // 2] = np.float32(what.split()[0])
        X[n - 1, 0] = np.inf
    if "nan" in what:
        X[130, 1] = np.nan
    if what == "far":
        X[5] = 1e19          # distances overflow, no coordinate does
        X[n - 2, 2] = 3e38
        X[9, 0] = 4.7e18     # a finite norm close to the limit
    if what == "all far":
        X *= np.float32(3e18)
    case(f"points {what} n {n} d {d} k {k}")
    pairs, plain = _both(monkeypatch, X, Y, k)
    assert pairs == plain
    if what != "all far":    # a few points out of place, nothing else
        ok = X.copy()
        ok[~(np.abs(X) < 1e10).all(axis=1)] = 50.0
        assert abs(pairs - O.trustworthiness(ok, Y, k)) <= 10.0 / n


@pytest.mark.parametrize("n,d,dim,k", [(700, 1, 1, 5), (1003, 2, 2, 15), (900, 3, 3, 30), (1500, 8, 2, 15), (1201, 15, 4, 8),
                                       (2000, 16, 2, 16)])
@pytest.mark.parametrize("scaled", [False, True])
def test_few_features_equal_the_fp32_kernels(monkeypatch, n, d, dim, k, scaled):
    """Up to 16 features the pairs' products are the fp32 kernels', term by term."""
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    if scaled:
        X *= (10.0 ** rng.uniform(-3, 3, d)).astype(np.float32)
    Y = np.resize(X, (n, dim)) + (0.1 * rng.standard_normal((n, dim))).astype(np.float32)
    case(f"few features n {n} d {d} dim {dim} k {k} scaled {scaled}")
    pairs, plain = _both(monkeypatch, X, Y, k)
    assert pairs == plain


@pytest.mark.parametrize("d", [17, 32, 33, 300, 784])
def test_ranks_are_not_biased(monkeypatch, d):
    """Sums cut off toward zero make every dot product of non-negative features too
    small, and T too large, at every draw.  Over eight draws of image-like points the
    mean of T's distance from 64-bit sums is within four of its standard errors of
    zero, or as near as the fp32 kernels'."""
    import torch

    n, k = 6000, 15
    off = []
    for seed in range(8):
        g = torch.Generator(device="cuda").manual_seed(100 * d + seed)
        z = torch.randn(n, 2, generator=g, device="cuda")
        w = torch.randn(2, d, generator=g, device="cuda")
        x = (0.4 + 0.5 * torch.sin(0.3 * z @ w + 6.0 * torch.rand(d, generator=g, device="cuda"))
             + 0.05 * torch.randn(n, d, generator=g, device="cuda")).clamp(0, 1).contiguous()
        y = (z + 0.05 * torch.randn(n, 2, generator=g, device="cuda")).contiguous()
        case(f"bias d {d} seed {seed}")
        t = U.umap_trustworthiness(x, y, k)
        x64, y64 = x.double(), y.double()
        nx, own = (x64 * x64).sum(1), torch.arange(n, device="cuda")
        dy = (y64[:, None, 0] - y64[None, :, 0]) ** 2 + (y64[:, None, 1] - y64[None, :, 1]) ** 2
        dy[own, own] = np.inf
        nbr = torch.topk(dy, k, dim=1, largest=False).indices
        dx = nx[:, None] + nx[None, :] - 2.0 * (x64 @ x64.T.contiguous())
        dx[own, own] = np.inf
        thr = torch.gather(dx, 1, nbr)
        pen = sum(int(((dx < thr[:, q, None]).sum(1) + 1 - k).clamp_min(0).sum()) for q in range(k))
        unit = 2.0 / (n * k * (2.0 * n - 3.0 * k - 1.0))
        monkeypatch.setenv("UMAP_LAYOUT_FAULT", "split")
        plain = U.umap_trustworthiness(x, y, k)
        monkeypatch.delenv("UMAP_LAYOUT_FAULT")
        off.append(((t - (1.0 - unit * pen)) / unit, (plain - (1.0 - unit * pen)) / unit))
    pairs, plain = np.array(off).T
    print("units off:", np.round(pairs), "fp32 kernels", np.round(plain), flush=True)
    assert abs(pairs.mean()) <= abs(plain.mean()) + 4.0 * pairs.std(ddof=1) / np.sqrt(pairs.size)
