"""One-launch epochs (the draw launch applies the negative samples itself)
against the one-thread-per-vertex kernel, bit for bit, on both sides of each
line of the rule that chooses them: table size by row width, and the work of
an epoch (24M terms: edges x (1 + neg_rate))."""

import sys

import numpy as np
import pytest

from paper_2008_00325_amd import synth
from paper_2008_00325_amd import umap_layout as U

pytestmark = pytest.mark.gpu

A_DEF, B_DEF = 1.577, 0.895


def case(msg):
    print(f"[gpu case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def torch_device_first():
    import torch

    torch.cuda.init()
    torch.cuda.set_device(0)


def _both_kernels(h, E, N, what):
    out = []
    for kernel in (0, 1):
        case(f"{what}: kernel {kernel}")
        U.umap_layout_set_kernel(h, kernel)
        U.umap_layout_set_embedding(h, E)
        U.umap_layout_run_epochs(h, 77, N // 2, N // 2 + 2)
        st = U.umap_layout_stats(h)
        assert st["overflow_redone"] == 0
        out.append((U.umap_layout_get(h), st["active_edges"]))
    assert out[0][1] == out[1][1] > 0
    assert np.array_equal(out[0][0].view(np.uint32), out[1][0].view(np.uint32))


# (vertices, components, mean degree, neg_rate)
FITS = [
    (2_001, 1, 9, 5), (2_001, 2, 9, 0), (2_001, 3, 9, 12), (4_097, 12, 7, 8), (4_097, 13, 7, 4), (4_097, 16, 7, 5),
    (786_432, 2, 6, 5),      # 6 MB: the last 2-component table of one launch by size, 28M terms
    (786_433, 2, 6, 5),      # beyond: record filing
    (367_001, 5, 12, 5), (367_002, 5, 12, 5),          # around 7 MB (367,001.6 rows), 26M terms
    (1_100_000, 16, 4, 5),   # 70 MB and 26M terms: record filing at 16 components
    (1_100_000, 16, 3, 5),   # 20M terms: one launch
]


@pytest.mark.parametrize("n,dim,deg,R", FITS)
def test_fit_one_launch_bits(n, dim, deg, R):
    r, c, v = synth.random_symmetric_coo(n, deg, seed=n % 1000 + dim)
    N = 20
    with U.umap_layout_create(n, dim, r, c, v, A_DEF, B_DEF, N, R) as h:
        _both_kernels(h, synth.embedding_state(n, dim, 5, 10.0), N, f"fit {n} x {dim}, degree {deg}, R {R}")


# (new points, table rows, components, neighbours, neg_rate)
TRANSFORMS = [
    (5_000, 130, 2, 3, 5),           # more new points than table rows
    (63, 1_000_000, 3, 15, 5),       # a table of four ranges, one launch by work
    (257, 200_000, 10, 15, 9),
    (300_001, 1_000_000, 2, 15, 5),  # 27M terms: record filing
    (300_001, 700_000, 3, 15, 5),
]


@pytest.mark.parametrize("n_new,n_table,dim,k,R", TRANSFORMS)
def test_transform_one_launch_bits(n_new, n_table, dim, k, R):
    r, c, v = synth.transform_graph(n_new, n_table, k)
    T = synth.embedding_state(n_table, dim, 6, 10.0)
    N = 20
    with U.umap_transform_create(n_new, T, r, c, v, A_DEF, B_DEF, N, R) as h:
        _both_kernels(h, synth.embedding_state(n_new, dim, 7, 10.0), N,
                      f"transform of {n_new} points on {n_table} x {dim}, k {k}, R {R}")


def test_row_ranges_on_both_sides_of_the_work_line():
    """Row ranges of one handle below and above 24M terms give the rows of the
    whole epoch (786,433 x 2: record filing for all rows, one launch for a share)."""
    n, N, R = 786_433, 20, 5
    r, c, v = synth.random_symmetric_coo(n, 7, seed=3)
    E = synth.embedding_state(n, 2, 8, 10.0)
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, N, R) as h:
        U.umap_layout_set_embedding(h, E)
        U.umap_layout_run_epochs(h, 4, 9, 10)
        full = U.umap_layout_get(h)
        for r0, r1 in ((0, 600_000), (600_000, n), (n - 1, n)):
            case(f"rows [{r0}, {r1})")
            U.umap_layout_set_rows(h, r0, r1)
            U.umap_layout_set_embedding(h, E)
            U.umap_layout_run_epochs(h, 4, 9, 10)
            got = U.umap_layout_get(h)
            assert np.array_equal(got[r0:r1].view(np.uint32), full[r0:r1].view(np.uint32))
            assert np.array_equal(got[:r0].view(np.uint32), E[:r0].view(np.uint32))
            assert np.array_equal(got[r1:].view(np.uint32), E[r1:].view(np.uint32))


def _banded(n, per_row, reach, far, seed):
    """Tails within `reach` rows of their rows, `far` random edges besides."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n, dtype=np.int64), per_row)
    j = i + rng.integers(1, reach + 1, i.size)
    i, j = i[j < n], j[j < n]
    e = np.sort(rng.integers(0, n, size=(2, far)), axis=0)
    key = np.unique(np.concatenate([i * n + j, (e[0] * n + e[1])[e[0] != e[1]]]))
    lo, hi = (key // n).astype(np.int32), (key % n).astype(np.int32)
    v = rng.uniform(0.05, 1.0, lo.size).astype(np.float32)
    return np.r_[lo, hi], np.r_[hi, lo], np.r_[v, v]


# every way the draw kernel reads a fit's tails, in one launch and with records (from 786,433 x 2 on and 27M terms)
@pytest.mark.parametrize("n,per_row", [(300_001, 2), (800_003, 4)])
@pytest.mark.parametrize("reach,far,what", [(64, 0, "16-bit tails and halo"), (64, 1, "halo, one far edge"),
                                            (3_000, 0, "16-bit tails, no halo"), (200_000, 0, "neither")])
@pytest.mark.parametrize("dim", [1, 2, 3])
def test_tail_reading_bits(n, per_row, reach, far, what, dim):
    r, c, v = _banded(n, per_row, reach, 40 * far, seed=n % 1000 + reach)
    N = 20
    with U.umap_layout_create(n, dim, r, c, v, A_DEF, B_DEF, N, 5) as h:
        _both_kernels(h, synth.embedding_state(n, dim, 9, 10.0), N, f"{what}: {n} x {dim}")
