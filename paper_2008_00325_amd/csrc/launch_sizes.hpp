// launch_sizes.hpp -- how many workgroups a call takes, as plain functions of its
// sizes (no HIP types: they are also compiled and checked on the host alone).
#pragma once

#include <stdint.h>

namespace ul {

// A launch's work-items per grid dimension must stay below 2^32.
constexpr int64_t kGridItems = (int64_t)1 << 32;

// A grid of at least `blocks` blocks of `threads` threads: one dimension where that
// many fit, else two (block blockIdx.y * x + blockIdx.x; those past the last have no work).
struct Grid2 {
    uint32_t x, y;
};
constexpr Grid2 grid2(int64_t blocks, int64_t threads)
{
    const int64_t most = (kGridItems - 1) / threads;
    const int64_t y = (blocks + most - 1) / most;
    return Grid2{(uint32_t)((blocks + y - 1) / y), (uint32_t)y};
}

// ---- ranks of the trustworthiness: blocks of 256 threads over pairs of panels ----
constexpr int64_t kPairThreads = 256;

// Blocks take `span` column tiles of one row panel, from the diagonal on: for the
// last m panels ceil(1 / span) + .. + ceil(m / span) blocks.
constexpr int64_t panel_blocks(int64_t m, int64_t span)
{
    const int64_t q = m / span, r = m % span;
    return span * q * (q + 1) / 2 + r * (q + 1);
}

// Column tiles per block: about 4096 blocks where the points allow it (two are
// resident per CU), a row panel's counts and operands being shared by the tiles of
// a block, but at most 4, so that the last blocks do not run alone for long.  ms per
// call with 1 / 2 / 4 / 8 / 16 tiles per block, k = 15: 5,003 x 64 0.23 / 0.22 / 0.30 /
// 0.47 / 0.81, 16,000 x 64 1.01 / 0.99 / 0.99 / 1.20 / 1.52, 32,640 x 64 3.41 / 3.28 /
// 3.27 / 3.38 / 3.62, 32,640 x 784 7.50 / 7.57 / 7.76 / 8.08 / 8.76, 70,000 x 64 13.9 /
// 13.2 / 12.9 / 13.0 / 13.1, 70,000 x 784 32.6 / 32.4 / 32.7 / 33.1 / 33.9.  Longer where that
// many blocks would not fit one launch (from 1,482,625 points on).
constexpr int64_t panel_span(int64_t panels)
{
    int64_t span = panels * (panels + 1) / 2 / 4096;
    span = span < 1 ? 1 : span > 4 ? 4 : span;
    while (span < panels && panel_blocks(panels, span) * kPairThreads >= kGridItems) span *= 2;
    return span;
}

// Whether the ranks come from every pair once, in tiles of 128 x 128, rather than from
// the fp32 kernel, which takes them row by row: a tile's counting is a long chain (the longer
// the more neighbours) that few tiles do not hide, while the fp32 kernel's time grows
// with the features.  us per call, pairs / fp32: k = 15, 500 x 8 152 / 79, 2,048 x 8 135 /
// 96, 2,560 x 64 152 / 128, 3,072 x 64 154 / 141, 2,048 x 300 176 / 162, 2,560 x 300 184 / 201,
// 1,024 x 784 243 / 233, 1,280 x 784 248 / 252; k = 64, 500 x 8 481 / 176, 2,560 x 64 399 /
// 401, 2,560 x 300 459 / 523, 1,536 x 784 629 / 636; k = 5, 2,048 x 64 90 / 78, 2,560 x 64
// 92 / 99, 640 x 300 103 / 109, 250 x 784 130 / 193.
constexpr bool pairs_pay(int64_t n, int32_t d, int32_t k)
{
    return n + (k <= 8 ? 7 : 2) * (int64_t)d > 2600;
}

// ---- draw kernel at 1-2 components ----
// Whether the 64 rows on each side of a wave's own are staged for the tails that lie
// there: `near` of `kept` tails are within 64 rows of theirs.  A staged row is an LDS
// read instead of a gather, for more LDS per workgroup.  us per epoch at 2 components
// without / with (k = 15 graphs in local order, a share of the tails anywhere): 1M
// vertices, all near 574 / 567, 1 % far 589 / 583, 50 % 670 / 657, 90 % 722 / 715, 95 %
// 726 / 723, 98 % 726 / 726; 500,000 201 / 197, 50 % far 229 / 225; 140,000 to 300,000
// the same; 40,000 18.9 / 19.6, 20,000 11.1 / 11.7 (there the table is in every L2).
constexpr bool halo_pays(int64_t near, int64_t kept, int64_t n, int32_t dim)
{
    return kept > 0 && 16 * near >= kept && n * dim * (int64_t)sizeof(float) >= (int64_t)1 << 20;
}

}  // namespace ul
