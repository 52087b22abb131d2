"""The device ingest against a sort on the host, bit for bit, at the sizes where
it changes: buckets of 2^8 to 2^14 rows (16,384-row buckets are counted in two
parts), rows longer than a workgroup sorts together (512 entries), many entries
in one bucket, empty rows and buckets, pruned entries, and a bipartite graph.
And what it refuses: an entry without its reverse, or with another value there,
wherever it stands; duplicates in short and long rows."""

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


def _expected(n, r, c, v, N, bipartite=False):
    keep = v > 0 if bipartite else (v > 0) & (r != c)
    w_max = v[keep].max()
    keep &= v >= w_max / np.float32(N)
    r, c, v = r[keep], c[keep], v[keep]
    o = np.lexsort((c, r))
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int64)
    return row_ptr, c[o], w_max / v[o]


def _check(h, n, r, c, v, N, bipartite=False):
    want = _expected(n, r, c, v, N, bipartite)
    got = U.umap_layout_get_graph(h)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    st = U.umap_layout_stats(h)
    assert st["max_degree"] == np.diff(want[0]).max() and st["nnz_kept"] == want[1].size


def _hubs(n, hubs, degree, seed, rest=None):
    """`hubs` vertices joined to `degree` others each, and a sparse rest."""
    rng = np.random.default_rng(seed)
    lo, hi = [], []
    for q in range(hubs):
        h = int(rng.integers(0, n))
        t = rng.choice(n, size=degree, replace=False)
        t = t[t != h]
        lo.append(np.minimum(h, t))
        hi.append(np.maximum(h, t))
    e = rng.integers(0, n, size=(2, 2 * n if rest is None else rest))
    e = e[:, e[0] != e[1]]
    lo.append(e.min(0))
    hi.append(e.max(0))
    key = np.unique(np.concatenate(lo).astype(np.int64) * n + np.concatenate(hi))
    lo, hi = (key // n).astype(np.int32), (key % n).astype(np.int32)
    v = (rng.random(lo.size) * 0.98 + 0.004).astype(np.float32)   # some below w_max / N
    p = rng.permutation(2 * lo.size)
    return np.r_[lo, hi][p], np.r_[hi, lo][p], np.r_[v, v][p]


# (vertices, mean degree)
@pytest.mark.parametrize("n,deg", [(1, 0), (2, 1), (31, 30), (32, 20), (33, 5), (256, 12), (257, 12), (8191, 6),
                                   (262_143, 5), (262_145, 5), (1_048_577, 3), (9_000_001, 1)])
def test_random_graphs(n, deg):
    r, c, v = synth.random_symmetric_coo(n, deg, seed=n % 997) if deg else (np.zeros(0, np.int32),) * 2 + (
        np.zeros(0, np.float32),)
    # entries that are dropped: zeros, negative values, self loops
    extra = np.arange(min(n, 50), dtype=np.int32)
    r, c = np.r_[r, extra, extra], np.r_[c, extra, (extra + 1) % n]
    v = np.r_[v, np.full(extra.size, 5.0, np.float32), np.where(extra % 2, 0.0, -1.0).astype(np.float32)]
    case(f"random graph n {n} degree {deg}")
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, 50, 5) as h:
        if deg:
            _check(h, n, r, c, v, 50)
        else:
            assert U.umap_layout_stats(h)["nnz_kept"] == 0


@pytest.mark.parametrize("n,hubs,degree", [(700, 3, 511), (700, 3, 512), (700, 40, 513), (5_000, 2, 4_999),
                                           (300_000, 12, 20_000)])
def test_hub_graphs(n, hubs, degree):
    r, c, v = _hubs(n, hubs, degree, seed=degree)
    case(f"n {n}, {hubs} hubs of degree {degree}")
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, 200, 5) as h:
        _check(h, n, r, c, v, 200)


@pytest.mark.parametrize("n_new,n_table,k", [(3, 40_000, 9_000), (400, 90_000, 700), (300_001, 130, 3)])
def test_bipartite(n_new, n_table, k):
    rng = np.random.default_rng(k)
    if k > n_table // 16:
        cols = np.stack([rng.permutation(n_table)[:k] for _ in range(n_new)])
    else:
        start, step = rng.integers(0, n_table, (n_new, 1)), rng.integers(1, n_table // k, (n_new, 1))
        cols = (start + step * np.arange(k)) % n_table
    rows = np.repeat(np.arange(n_new, dtype=np.int32), k)
    p = rng.permutation(rows.size)
    r, c = rows[p], cols.ravel().astype(np.int32)[p]
    v = rng.uniform(0.001, 1.0, rows.size).astype(np.float32)
    case(f"bipartite {n_new} x {n_table}, {k} entries per row")
    with U.umap_transform_create(n_new, synth.embedding_state(n_table, 2, 1), r, c, v, A_DEF, B_DEF, 100, 5) as h:
        _check(h, n_new, r, c, v, 100, bipartite=True)


def test_asymmetric_and_duplicate_entries():
    n = 3_000
    r, c, v = _hubs(n, 4, 900, seed=9)
    v = np.maximum(v, np.float32(0.1))
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, 200, 5):
        pass
    deg = np.bincount(r, minlength=n)
    long_rows, short_rows = np.flatnonzero(deg > 512), np.flatnonzero(deg < 20)
    picks = [np.flatnonzero(np.isin(r, long_rows) & np.isin(c, short_rows) & (r < c))[0],
             np.flatnonzero(np.isin(r, long_rows) & np.isin(c, short_rows) & (r > c))[-1],
             np.flatnonzero(np.isin(c, long_rows) & np.isin(r, short_rows) & (r < c))[3],
             np.flatnonzero(np.isin(c, long_rows) & np.isin(r, short_rows) & (r > c))[-4],
             np.flatnonzero(np.isin(r, short_rows) & np.isin(c, short_rows) & (r < c))[5],
             np.flatnonzero(np.isin(r, short_rows) & np.isin(c, short_rows) & (r > c))[6]]
    for e in picks:
        case(f"entry {e} ({r[e]}, {c[e]}): missing, another value, listed twice")
        gone = np.delete(np.arange(r.size), e)
        other = v.copy()
        other[e] = np.nextafter(v[e], np.float32(1))
        for rr, cc, vv, code in ((r[gone], c[gone], v[gone], U.UMAP_E_ASYMMETRIC), (r, c, other, U.UMAP_E_ASYMMETRIC),
                                 (np.r_[r, r[e]], np.r_[c, c[e]], np.r_[v, v[e]], U.UMAP_E_INVAL)):
            with pytest.raises(U.UmapLayoutError) as ei:
                U.umap_layout_create(n, 2, rr, cc, vv, A_DEF, B_DEF, 200, 5)
            assert ei.value.code == code
    # as many entries above the diagonal as below, none with its reverse
    a = picks[4]
    far = np.flatnonzero(np.isin(r, short_rows) & np.isin(c, short_rows) & (r < c) & (r != r[a]))[9]
    back = np.flatnonzero((r == c[far]) & (c == r[far]))[0]
    gone = np.delete(np.arange(r.size), [a, back])
    with pytest.raises(U.UmapLayoutError) as ei:
        U.umap_layout_create(n, 2, r[gone], c[gone], v[gone], A_DEF, B_DEF, 200, 5)
    assert ei.value.code == U.UMAP_E_ASYMMETRIC


def test_entries_up_to_the_last_31_bit_number():
    """2^31 - 2 entries, all kept: the passes over entries end within one step of
    2^31, where 32-bit signed entry numbers would wrap.  A ring of 11.5M vertices
    joined to 93 on each side."""
    import ctypes

    import torch

    m = 93
    n = (2**31 - 2) // (2 * m)
    nnz = 2 * m * n
    assert nnz == 2**31 - 2
    if torch.cuda.mem_get_info()[0] < 130 * 2**30:
        pytest.skip("needs 130 GiB of device memory")
    case(f"ring of {n} vertices, {nnz} entries")
    off = torch.cat([torch.arange(-m, 0), torch.arange(1, m + 1)]).to("cuda", torch.int32)
    r, c = (torch.empty(n, 2 * m, dtype=torch.int32, device="cuda") for _ in range(2))
    v = (1.0 - 0.005 * off.abs().float()).repeat(n)
    r[:] = torch.arange(n, dtype=torch.int32, device="cuda")[:, None]
    torch.add(r, off[None, :], out=c)
    c[c < 0] += n
    c[c >= n] -= n
    h = U.umap_layout_create_device(n, 2, r, c, v, nnz, A_DEF, B_DEF, 2, 0)
    del r, c, v
    torch.cuda.empty_cache()
    with h:
        st = U.umap_layout_stats(h)
        assert st["nnz_kept"] == nnz and st["max_degree"] == 2 * m
        row_ptr, col = np.empty(n + 1, np.int64), np.empty(nnz, np.int32)
        assert U.lib().umap_layout_get_graph(h.ptr, row_ptr.ctypes.data_as(ctypes.c_void_p),
                                             col.ctypes.data_as(ctypes.c_void_p), None, None) == U.UMAP_OK
    assert np.array_equal(row_ptr, 2 * m * np.arange(n + 1, dtype=np.int64))
    col = col.reshape(n, 2 * m)
    off = np.r_[np.arange(-m, 0), np.arange(1, m + 1)].astype(np.int32)
    step = 1 << 20
    for a in range(0, n, step):
        print(f"[gpu case] rows from {a}", flush=True)
        want = np.arange(a, min(n, a + step), dtype=np.int32)[:, None] + off[None, :]
        if a == 0 or a + step >= n:
            want = np.sort(want % n, axis=1)
        assert np.array_equal(col[a:a + step], want)


@pytest.mark.parametrize("n", [2**29 + 5, 3 * 2**29 + 77])
def test_more_rows_than_one_grid_dimension(n):
    """Blocks of 32 rows that need a second grid dimension (from 2^29 rows on), and
    bucket counters beyond 64 KB of LDS (from 2^30 rows on)."""
    import torch

    if torch.cuda.mem_get_info()[0] < 160 * 2**30:
        pytest.skip("needs 160 GiB of device memory")
    rng = np.random.default_rng(3)
    ends = np.r_[np.arange(40), n // 2 + np.arange(40), n - 1 - np.arange(40), rng.integers(0, n, 1000)]
    key = np.unique(np.sort(rng.permutation(np.r_[ends, ends]).reshape(-1, 2), axis=1).astype(np.int64) @ [n, 1])
    lo, hi = key // n, key % n
    lo, hi = lo[lo != hi].astype(np.int32), hi[lo != hi].astype(np.int32)
    v = rng.uniform(0.6, 1.0, lo.size).astype(np.float32)
    r, c, v = np.r_[lo, hi], np.r_[hi, lo], np.r_[v, v]
    case(f"{n} rows")
    with U.umap_layout_create_device(n, 1, *(torch.from_numpy(x).cuda() for x in (r, c, v)), r.size, A_DEF, B_DEF, 2,
                                     1) as h:
        row_ptr, col, eps = U.umap_layout_get_graph(h)
        st = U.umap_layout_stats(h)
    o = np.lexsort((c, r))
    assert np.array_equal(col, c[o]) and np.array_equal(eps, v.max() / v[o])
    rows, count = np.unique(r, return_counts=True)
    assert st["max_degree"] == count.max() and st["nnz_kept"] == r.size
    at, a = 0, 0
    for b, m in zip(rows.tolist() + [n], count.tolist() + [0]):   # row_ptr is constant from one row's end to the next
        assert (row_ptr[a:b + 1] == at).all(), (a, b)
        at, a = at + m, b + 1
    assert a == n + 1


@pytest.mark.parametrize("n,hub", [(300, 0), (1_100, 0), (9_001, 9_000)])
def test_asymmetric_entries_in_every_piece(n, hub):
    """Blocks of rows with more than 4,096 entries (4 rows of a complete graph of
    1,100, 32 rows with a hub of 9,000) are checked in pieces: one entry changed or
    taken out anywhere in them is found."""
    if hub:
        lo, hi = np.zeros(hub, np.int32), np.arange(1, hub + 1, dtype=np.int32)
    else:
        lo, hi = np.triu_indices(n, 1)
    r, c = np.r_[lo, hi].astype(np.int32), np.r_[hi, lo].astype(np.int32)
    v = np.random.default_rng(n).uniform(0.5, 1.0, lo.size).astype(np.float32)
    v = np.r_[v, v]
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, 50, 5) as h:
        _check(h, n, r, c, v, 50)
    half = lo.size
    for e in (0, half // 5, half // 2, half - 1, half, half + half // 3, 2 * half - 1):
        case(f"n {n}, entry ({r[e]}, {c[e]})")
        other = v.copy()
        other[e] = np.nextafter(v[e], np.float32(1))
        gone = np.delete(np.arange(r.size), e)
        for rr, cc, vv in ((r, c, other), (r[gone], c[gone], v[gone])):
            with pytest.raises(U.UmapLayoutError) as ei:
                U.umap_layout_create(n, 2, rr, cc, vv, A_DEF, B_DEF, 50, 5)
            assert ei.value.code == U.UMAP_E_ASYMMETRIC


@pytest.mark.parametrize("n,hubs,degree", [(300_000, 3, 65_000), (300_000, 5, 90_000), (9_000_001, 2, 140_000)])
def test_buckets_taken_in_chunks(n, hubs, degree):
    """Buckets of more than 65,536 entries (those of a hub) are counted and filed by
    several workgroups, 32,768 entries each; in buckets of 16,384 rows in two parts."""
    r, c, v = _hubs(n, hubs, degree, seed=degree, rest=400_000)
    case(f"n {n}, {hubs} hubs of degree {degree}")
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, 200, 5) as h:
        _check(h, n, r, c, v, 200)


@pytest.mark.parametrize("n_new,k", [(1, 65_536), (1, 65_537), (2, 131_072), (40, 90_000)])
def test_few_rows_taken_in_chunks(n_new, k):
    n_table = 200_000
    rng = np.random.default_rng(k)
    c = np.concatenate([rng.permutation(n_table)[:k] for _ in range(n_new)]).astype(np.int32)
    r = np.repeat(np.arange(n_new, dtype=np.int32), k)
    v = rng.uniform(0.001, 1.0, r.size).astype(np.float32)
    p = rng.permutation(r.size)
    r, c, v = r[p], c[p], v[p]
    case(f"bipartite {n_new} x {n_table}, {k} entries per row")
    with U.umap_transform_create(n_new, synth.embedding_state(n_table, 2, 1), r, c, v, A_DEF, B_DEF, 100, 5) as h:
        _check(h, n_new, r, c, v, 100, bipartite=True)


@pytest.mark.parametrize("n,deg", [(200, 127), (200, 128), (257, 140), (258, 200), (1_003, 500), (1_003, 520)])
def test_dense_graphs(n, deg):
    """Blocks of 4 rows from 128 entries per row on: circulant graphs of `deg` entries
    per row (one more where n is even and deg odd), and rows of 513 and more."""
    i, half = np.arange(n), deg // 2
    lo = np.concatenate([i] * half + ([i[: n // 2]] if deg % 2 else []))
    hi = np.concatenate([(i + q) % n for q in range(1, half + 1)] + ([i[: n // 2] + n // 2] if deg % 2 else []))
    v = np.random.default_rng(n).uniform(0.001, 1.0, lo.size).astype(np.float32)
    p = np.random.default_rng(deg).permutation(2 * lo.size)
    r, c, v = np.r_[lo, hi][p].astype(np.int32), np.r_[hi, lo][p].astype(np.int32), np.r_[v, v][p]
    case(f"circulant n {n}, {deg} entries per row")
    with U.umap_layout_create(n, 2, r, c, v, A_DEF, B_DEF, 400, 5) as h:
        _check(h, n, r, c, v, 400)
