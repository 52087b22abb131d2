"""Launch sizes at the limits of what the calls accept, on the host: a launch has
fewer than 2^32 work-items per grid dimension and its blocks cover the work."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GRID_ITEMS = 2**32


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("sizes") / "launch_sizes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2008_00325_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "launch_sizes.cpp"), "-o", exe], check=True, timeout=120)

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        return [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]

    return ask


def test_pair_ranks_fit_a_launch(sizes):
    # 11,583 / 11,584 panels: 2^24 blocks of four tiles; the last: more than the points that the embedding's
    # neighbours are found of (a wavefront per point)
    panels = [1, 2, 255, 256, 547, 11_583, 11_584, 20_000, 524_288]
    got = sizes([f"pairs {m}" for m in panels])
    for m, (span, blocks, threads) in zip(panels, got):
        assert span >= 1 and blocks * threads < GRID_ITEMS
        if m <= 20_000:
            assert blocks == sum(-(-q // span) for q in range(1, m + 1))
    assert [s for s, _, _ in got][:7] == [1, 1, 4, 4, 4, 4, 8]


def test_row_blocks_fit_a_launch(sizes):
    # blocks of 32 rows of up to 2^31 - 1 rows: beyond 2^29 rows one dimension does not hold them
    rows = [1, 32, 33, 2**29 - 32, 2**29 - 31, 2**29, 2**30 + 77, 2**31 - 1]
    for n, (x, y) in zip(rows, sizes([f"grid {-(-n // 32)}" for n in rows])):
        assert x * 256 < GRID_ITEMS and y < 2**16
        assert -(-n // 32) <= x * y < -(-n // 32) + y
        assert (y == 1) == (n <= 2**29 - 32)


def test_halo_rule(sizes):
    """A far edge or a tenth of them does not cost a large local graph its halo."""
    kept = 26_700_000
    asked = {(kept, kept, 1_000_000, 2): 1, (kept - 2, kept, 1_000_000, 2): 1, (9 * kept // 10, kept, 1_000_000, 1): 1,
             (kept // 10, kept, 1_000_000, 2): 1, (kept // 17, kept, 1_000_000, 2): 0, (0, kept, 1_000_000, 2): 0,
             (kept, kept, 131_072, 2): 1, (kept, kept, 131_071, 2): 0, (0, 0, 1_000_000, 2): 0}
    got = sizes([f"halo {near} {k} {n} {dim}" for near, k, n, dim in asked])
    assert [g for (g,) in got] == list(asked.values())


def test_few_points_are_ranked_row_by_row(sizes):
    asked = {(500, 8, 64): 0, (500, 784, 15): 0, (2_000, 300, 64): 0, (2_584, 8, 15): 0, (2_585, 8, 15): 1, (2_000, 784, 64): 1,
             (500, 300, 5): 0, (501, 300, 5): 1, (250, 784, 8): 1, (5_003, 64, 15): 1, (70_000, 784, 15): 1}
    got = sizes([f"ranks {n} {d} {k}" for n, d, k in asked])
    assert [g for (g,) in got] == list(asked.values())
