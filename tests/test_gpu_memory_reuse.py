"""Device blocks kept between handles and calls: a handle that gets memory of
earlier ones (larger, smaller, of another kind) gives the bits of a first
run, also from several threads on streams of their own, and what is kept is
bounded."""

import sys
import threading

import numpy as np
import pytest

from paper_2008_00325_amd import synth
from paper_2008_00325_amd import umap_layout as U

pytestmark = pytest.mark.gpu

A_DEF, B_DEF = 1.577, 0.895
SIZES = [(3_000, 8, 2), (200_000, 6, 2), (3_001, 9, 5), (60_000, 12, 16), (500, 4, 3), (201_000, 6, 2)]


def case(msg):
    print(f"[gpu case] {msg}", flush=True)
    sys.stdout.flush()


def _graphs():
    return [synth.random_symmetric_coo(n, deg, seed=q) for q, (n, deg, _) in enumerate(SIZES)]


def _layout(graph, n, dim, stream):
    import torch

    with torch.cuda.stream(stream):
        r, c, v = (torch.from_numpy(x).cuda() for x in graph)
        out = torch.empty(n, dim, dtype=torch.float32, device="cuda")
    stream.synchronize()
    with U.umap_layout_create_device(n, dim, r, c, v, r.numel(), A_DEF, B_DEF, 30, 5, stream=stream) as h:
        U.umap_layout_run(h, 5)
        U.umap_layout_get_device(h, out)
    return out.cpu().numpy().view(np.uint32)


def test_reused_blocks_give_the_same_bits():
    import torch

    torch.cuda.set_device(0)
    graphs = _graphs()
    first = []
    for q, (n, _, dim) in enumerate(SIZES):
        case(f"first run of {n} x {dim}")
        first.append(_layout(graphs[q], n, dim, torch.cuda.Stream()))
    wrong = []

    def worker(seed):
        order = np.random.default_rng(seed).permutation(3 * len(SIZES)) % len(SIZES)
        stream = torch.cuda.Stream()
        x = torch.randn(700, 20, device="cuda")
        y = x[:, :2].contiguous()
        torch.cuda.synchronize()
        t0 = U.umap_trustworthiness(x, y, 10, stream=stream)
        for q in order:
            n, _, dim = SIZES[q]
            if not np.array_equal(_layout(graphs[q], n, dim, stream), first[q]):
                wrong.append((seed, int(q)))
            if U.umap_trustworthiness(x, y, 10, stream=stream) != t0:
                wrong.append((seed, "trustworthiness"))

    case("three threads, mixed sizes")
    threads = [threading.Thread(target=worker, args=(s,)) for s in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_kept_memory_is_bounded():
    import torch

    torch.cuda.synchronize()
    empty = np.zeros(0, np.int32)
    held = []
    for n in (10_000_000, 20_000_000, 30_000_000, 40_000_000, 50_000_000):
        case(f"handle of {n} rows")
        before = torch.cuda.mem_get_info()[0]
        with U.umap_layout_create(n, 4, empty, empty, np.zeros(0, np.float32), A_DEF, B_DEF, 10, 5) as h:
            U.umap_layout_init(h, 1)
        held.append(before - torch.cuda.mem_get_info()[0])
    assert sum(held) <= (4 << 30) + (64 << 20)
    # and given back as other sizes are asked for
    small = np.array([0, 1], np.int32)
    before = torch.cuda.mem_get_info()[0]
    for _ in range(80):
        with U.umap_layout_create(2, 1, small, small[::-1].copy(), np.ones(2, np.float32), A_DEF, B_DEF, 3, 5):
            pass
    assert sum(held) > 1 << 30 and torch.cuda.mem_get_info()[0] >= before + sum(held) - (64 << 20)


def _empty_handle(n):
    empty = np.zeros(0, np.int32)
    return U.umap_layout_create(n, 4, empty, empty, np.zeros(0, np.float32), A_DEF, B_DEF, 10, 5)


def test_kept_memory_is_given_back_when_asked():
    import torch

    torch.cuda.synchronize()
    U.umap_layout_destroy(None)
    base = torch.cuda.mem_get_info()[0]
    h = _empty_handle(15_000_000)
    size = base - torch.cuda.mem_get_info()[0]
    assert size > 1 << 30
    h.close()
    assert base - torch.cuda.mem_get_info()[0] >= size // 2   # kept
    U.umap_layout_destroy(None)
    assert base - torch.cuda.mem_get_info()[0] <= 64 << 20
    with _empty_handle(1000) as h:                            # and the library goes on
        U.umap_layout_init(h, 1)


def test_a_handle_does_not_hold_much_more_than_it_needs():
    import torch

    torch.cuda.synchronize()
    U.umap_layout_destroy(None)
    base = torch.cuda.mem_get_info()[0]
    with _empty_handle(6_000_000):
        U.umap_layout_destroy(None)
        need = base - torch.cuda.mem_get_info()[0]
    U.umap_layout_destroy(None)
    _empty_handle(10_000_000).close()                         # leaves a block of 10/6 of that
    with _empty_handle(6_000_000):
        U.umap_layout_destroy(None)
        assert base - torch.cuda.mem_get_info()[0] <= need + need // 8 + (64 << 20)


def test_host_failure_in_every_call_with_scratch(monkeypatch):
    """A C++ exception that is no HIP failure ends as a status code."""
    import torch

    ids = torch.tensor([[1], [0]], dtype=torch.int32, device="cuda")
    dist = torch.ones(2, 1, device="cuda")
    i4, v4 = torch.empty(4, dtype=torch.int32, device="cuda"), torch.empty(4, device="cuda")
    x = torch.randn(40, 3, device="cuda")
    y = x[:, :2].contiguous()
    monkeypatch.setenv("UMAP_LAYOUT_FAULT", "host")
    for call in (lambda: U.umap_fuzzy_graph_device(2, 1, ids, dist, i4, i4, v4), lambda: U.umap_trustworthiness(x, y, 3),
                 lambda: _empty_handle(10)):
        with pytest.raises(U.UmapLayoutError) as ei:
            call()
        assert ei.value.code == U.UMAP_E_NOMEM
    monkeypatch.delenv("UMAP_LAYOUT_FAULT")
    assert 0.0 <= U.umap_trustworthiness(x, y, 3) <= 1.0


def test_small_calls_after_one_that_does_not_fit():
    """An allocation that fails leaves no error behind for the next call's launches."""
    import torch

    empty = np.zeros(0, np.int32)
    free = torch.cuda.mem_get_info()[0]
    with pytest.raises(U.UmapLayoutError) as ei:
        U.umap_layout_create(2**31 - 1, 16, empty, empty, np.zeros(0, np.float32), A_DEF, B_DEF, 10, 5)
    assert ei.value.code == U.UMAP_E_NOMEM
    x = torch.randn(400, 3, device="cuda")
    y = x[:, :2].contiguous()
    assert 0.0 <= U.umap_trustworthiness(x, y, 3) <= 1.0
    with _empty_handle(1000) as h:
        U.umap_layout_run(h, 1)
    assert torch.cuda.mem_get_info()[0] >= free - (64 << 20)
