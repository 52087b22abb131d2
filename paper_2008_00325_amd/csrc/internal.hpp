// internal.hpp -- launchers shared between the host API and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout_device.hpp"

namespace ul {

// Sets the thread-local message read by umap_layout_last_error; returns code.
int set_error(int code, const char *msg);

// Flags raised by the ingest kernels.
enum PrepFlag : unsigned {
    kBadIndex = 1u,
    kBadValue = 2u,
    kDuplicate = 4u,
    kAsymmetric = 8u,
    kWide = 16u,   // a tail's offset from its row needs more than 16 bits (no error)
};

// Device-resident scalars of the ingest.
struct PrepScalars {
    unsigned flags;
    unsigned wmax_bits;   // bits of the largest kept candidate weight (> 0)
    int max_degree;
    int n_long;           // rows of the long-row list
    int n_sym;            // pieces of sym_list
    int n_heavy;          // chunks of buckets with more than
    int heavy_above;      //   this many entries
    int unused;
    unsigned long long near;   // tails within kHalo of their row
    long long up_minus_low;    // entries above minus entries below the diagonal
};

// Work split of the wavefront epoch kernels: wave w owns the whole rows
// [part[w], part[w+1]), chosen so that consecutive waves cover about C units
// of (edges + row_weight * rows), C = wave_cost(total units) <= kWaveCost.  The
// row weight bounds the rows of a wave (and so its LDS accumulator) by
// rows_cap; long waves amortise the per-wave set-up and commit, and C shrinks
// (by halves, down to kMinWaveCost) until a graph gives at least
// kTargetWaves waves, so that small graphs still fill the chip.
constexpr int kWaveCost = 8192;
constexpr int kMinWaveCost = 256;
constexpr int64_t kTargetWaves = 4096;
__host__ __device__ constexpr int row_weight(int dim) { return 32 * (dim > 2 ? dim : 2); }
__host__ __device__ constexpr int rows_cap(int dim) { return kWaveCost / row_weight(dim) + 1; }
inline int64_t wave_cost(int64_t total_units)
{
    int64_t c = kWaveCost;
    while (c > kMinWaveCost && total_units / c < kTargetWaves) c >>= 1;
    return c;
}
// Most waves any graph of at most `total_units` gets (wave_cost grows with the
// total, so a smaller total never needs more than 2 kTargetWaves).
inline int64_t max_wave_count(int64_t total_units)
{
    const int64_t big = total_units / kWaveCost;
    return (big > 2 * kTargetWaves ? big : 2 * kTargetWaves) + 2;
}

// ---- ingest (kernels_prep.hip) ----
struct PrepBuffers {
    // inputs (device)
    const int32_t *rows;
    const int32_t *cols;
    const float *vals;
    int64_t nnz;
    int64_t n;          // rows
    int64_t n_cols;     // columns are in [0, n_cols); n unless bipartite
    bool bipartite;     // rows and columns are different vertex sets (no self loops, no symmetry)
    int32_t n_epochs;
    // scratch (device); nb = bucket_count(n, nnz); the first three one after the other
    uint32_t *bucket_n;   // bucket_counters(n, nnz): candidates per bucket, a cache line apart
    PrepScalars *scalars;
    int32_t *lstart;      // n
    uint32_t *cursor;     // bucket_counters(n, nnz)
    int32_t *first;       // kSubs nb + 1
    int32_t *heavy_first; // nb + 1
    uint32_t *kept_n;     // nb
    int32_t *kfirst;      // nb + 1
    int2 *pair;           // nnz entries (col, value bits) by bucket, later in (row, col) order
    uint16_t *lrow;       // nnz, their rows in the bucket
    int2 *pair_rows;      // nnz, by row
    int32_t *rp32;        // n + 1, row_ptr in 32 bits
    int32_t *long_rows;   // long_row_slots(nnz)
    int2 *sym_list;       // symmetry_slots(nnz): (block of rows, piece)
    int32_t *block_max;   // row_blocks(n, nnz), per-block parts of the scalars
    int32_t *block_near;  // row_blocks(n, nnz)
    int32_t *block_diff;  // row_blocks(n, nnz)
    // outputs (device)
    int64_t *row_ptr;   // n + 1
    int32_t *col;       // nnz (capacity)
    float *eps;         // nnz (capacity)
    int16_t *col16;     // nnz (capacity), col - row; null when bipartite
};

// An entry's bucket is counted and filled in one of kSubs parts, by its tile, so
// that the workgroups of one XCD (tiles are dealt round-robin) share counters
// with each other only.
constexpr int kSubs = 8;
int64_t bucket_count(int64_t n, int64_t nnz);
int64_t bucket_counters(int64_t n, int64_t nnz);
int64_t row_blocks(int64_t n, int64_t nnz);
int64_t long_row_slots(int64_t nnz);
int64_t symmetry_slots(int64_t nnz);
hipError_t launch_prep(const PrepBuffers &B, hipStream_t s);
// Waves over rows [r0, r1) (0 <= r0 < r1); n_waves = ceil(units / cost) for
// the units (edges + row_weight x rows) of the range.
hipError_t launch_partition(const int64_t *row_ptr, int64_t r0, int64_t r1, int32_t dim, int64_t cost,
                            int32_t *part, WaveDesc *desc, int64_t n_waves, uint8_t *head, hipStream_t s);
hipError_t launch_zero_u64(unsigned long long *p, int64_t count, hipStream_t s);
// ---- layout (kernels_layout.hip) ----
hipError_t launch_init(float *E, int64_t n, int32_t dim, uint64_t seed, hipStream_t s);
hipError_t launch_init_transform(const int64_t *row_ptr, const int32_t *col, const float *eps, const float *T,
                                 int64_t n, int32_t dim, float *E, hipStream_t s);
// Graph-side arrays of the epoch kernels.
struct WaveGraph {
    const int64_t *row_ptr;   // n + 1
    const int32_t *col;       // kept edges, sorted by (row, col)
    const float *eps;         // epochs per sample of each edge
    const uint8_t *head;      // row of each edge relative to its wave's first row
    const int32_t *part;      // n_waves + 1 wave boundaries (rows)
    const WaveDesc *desc;     // n_waves: the same and the waves' edges, one 16-byte load per wave
    int64_t n_waves;
    // negative samples are filed by vertex-table range: P = 2^lg_phases ranges
    int32_t n_phases;
    int32_t lg_phases;
    uint32_t *rec;            // records ((row in wave) << 24 | offset in range), slots by record_offset
    int32_t *rec_count;       // P x n_waves
    unsigned *overflow;       // set when a record did not fit its range slot
    int64_t cap_limit;        // < 0: none; else record slots per range are cut to it (failure injection)
    long long *delta;         // n x dim fixed-point partial sums between launches
    const int16_t *col16;     // col - row in 16 bits (a fit whose tails all fit), else null
    int32_t one_launch;       // the draw launch applies the negative samples itself (no records, no range launches)
    int32_t halo;             // rows around a wave's own are staged for the tails (see halo_pays)
};

// First record slot of wave w (edges from e0): every wave gets
// 1.25 x neg_rate x its edges + 256 x P slots, split evenly over the P table
// ranges.  A range of a wave gets more than its share of a wave's draws only
// with vanishing probability (the ranges split uniform random words); a draw
// that finds its range full raises the overflow flag and the epochs are redone
// by the one-thread-per-vertex kernel.
__host__ __device__ inline int64_t record_offset(int64_t w, int64_t e0, int32_t neg_rate, int32_t n_phases)
{
    return (5 * (int64_t)neg_rate * e0 + 3) / 4 + (int64_t)256 * n_phases * w;
}

// At most this many table ranges (phases) per epoch.
constexpr int kMaxPhases = 16;
// The range count trades the gathers' L2 hit rate (a range of about 2 MB
// stays resident in one XCD's 4 MB L2 next to the streamed edge data) against
// the cost of each further range: one more launch and one more round trip of
// the n x dim int64 partial sums.  Measured on 1M and 5M vertices with 2 to 16
// components, the best count is 4 up to about 2.5M vertices and 8 at 5M,
// whatever the row width, and never more than a 2 MB range needs.
constexpr int64_t kPhaseTableBytes = 2 << 20;
constexpr int64_t kPhaseRows = 2500000;
// A table of one range never files records (see one_launch_epoch for the
// tables of several ranges that do not either).
constexpr int64_t kOneRangeBytes = 6 << 20;
constexpr int64_t kOneRangeBytesWide = 4 << 20;
constexpr int32_t kOneRangeMaxDim = 13;
// log2 of the number of ranges for a table of n vertices x dim: 0 up to
// kOneRangeBytes (kOneRangeBytesWide from 9 to kOneRangeMaxDim components);
// else min(the ranges that bring a range down to kPhaseTableBytes, 4 ranges per
// kPhaseRows vertices rounded up to a power of two), at most kMaxPhases.
int32_t phase_log2(int64_t n, int32_t dim);

// Whether an epoch over `edges` edges runs as one launch, in which the draw
// kernel gathers and applies each negative sample itself, instead of filing
// records for one launch per table range.  One launch saves the records (4
// bytes written and read per sample), the partial sums and P launches of at
// least 7 us; the range launches gather from a slice that stays in L2.  Two
// lines, both measured on MI355X (us per epoch, one launch / range launches):
//  * by table size, because wide rows pay more per partial sum and record
//    while a gather is one L2 request at any width: window graphs of k = 15 in
//    local order, 2 components 6 MB 240 / 256, 8 MB 413 / 323; 3 components
//    6 MB 173 / 199, 8 MB 302 / 262; 5 components 6 MB 129 / 163, 8 MB 202 /
//    200; 8 components 12 MB 214 / 252, 20 MB 402 / 408 (shuffled 459 / 433);
//    10 components 12 MB 211 / 242, 20 MB 394 / 400 (454 / 424); 13 components
//    20 MB 330 / 376 (382 / 383); 16 components 20 MB 213 / 364, 64 MB 748 /
//    1048;
//  * by work, because the saved launches do not shrink with it: transforms of
//    100K points with 15 edges (9M terms) on 1M x 2 47 / 73, 5M x 2 80 / 117,
//    1M x 3 65 / 72; an eighth of the rows of the 1M window graph (20M terms)
//    in 2-D 54 / 76, 3-D 71 / 80; 300K points (27M terms) 129 / 132, 231 / 198
//    and 180 / 146.
constexpr int64_t kOneLaunchTerms = 24000000;
inline bool one_launch_epoch(int64_t n_table, int32_t dim, int64_t edges, int32_t neg_rate)
{
    const int64_t mb = dim <= 3 ? 6 : dim <= 5 ? 7 : dim <= 10 ? 16 : dim <= 13 ? 20 : 64;
    return n_table * dim * (int64_t)sizeof(float) <= mb << 20 || edges * (1 + (int64_t)neg_rate) <= kOneLaunchTerms;
}

hipError_t launch_epoch(int kernel, int32_t dim, const EpochArgs &A, const WaveGraph &G, hipStream_t s);
// One asynchronous epoch, in place on A.E_next (A.E must be the same buffer).
hipError_t launch_epoch_hogwild(int32_t dim, const EpochArgs &A, const WaveGraph &G, hipStream_t s);
// Count slots one epoch of `kernel` writes (one per wave).
int64_t count_slots(int kernel, int64_t n, int64_t n_waves);
// out[r] = sum of counts[r * stride + 0 .. slots) for r < rows.
hipError_t launch_reduce_counts(const int32_t *counts, int64_t stride, int64_t slots, int32_t rows,
                                unsigned long long *out, hipStream_t s);
// *out = a[0] + ... + a[n - 1].
hipError_t launch_sum_u64(const unsigned long long *a, int64_t n, unsigned long long *out, hipStream_t s);
// Epochs whose per-wave counts are kept before they are summed.
constexpr int kCountRing = 256;
hipError_t launch_debug_active(const float *eps, int64_t nnz, int32_t epoch, uint8_t *out, hipStream_t s);
hipError_t launch_debug_negatives(uint32_t n, uint64_t seed, int32_t epoch, int64_t e_first, int64_t count,
                                  int32_t neg_rate, uint32_t *out, hipStream_t s);
hipError_t launch_probe_copy(const void *src, void *dst, int64_t bytes, hipStream_t s);
hipError_t launch_probe_gather(const void *table, int64_t entries, int64_t threads, int32_t iters, void *out,
                               hipStream_t s);

// ---- trustworthiness (kernels_trust.hip) ----
// The ranks come from the points split into bf16 parts, or packed as they are up to
// 16 features (trust_split_bytes; 0 beyond kTrustSplitBytes), every pair once, or
// from fp32 products of X itself, every pair twice (split null).
constexpr int64_t kTrustSplitBytes = (int64_t)16 << 30;
int64_t trust_padded(int64_t n);
size_t trust_split_bytes(int64_t n, int32_t d);
// Scratch, with np = trust_padded(n): split (or null), nx[np], nbr[np k],
// thr[np k], cnt[np k] (slot s of point i at s np + i), sum[1] and flags[1]
// (both zeroed by the caller).  With kTrustFarPoint raised the sum is not to be
// used: some point is too far out for the split points' ranks (split null: it is
// never raised).
enum TrustFlag : unsigned { kTrustBadEmbedding = 1u, kTrustFarPoint = 2u };
hipError_t launch_trustworthiness(const float *X, int64_t n, int32_t d, const float *Y, int32_t dim, int32_t k,
                                  void *split, float *nx, int32_t *nbr, float *thr, int32_t *cnt,
                                  unsigned long long *sum, unsigned *flags, hipStream_t s);

// ---- fuzzy graph (kernels_graph.hip) ----
// Scratch: rho_sigma[n] (rho_i, sigma_i) and flags[1] (zeroed by the caller).
hipError_t launch_fuzzy_graph(int64_t n, int32_t k, const int32_t *ids, const float *dists, int32_t *rows,
                              int32_t *cols, float *vals, double2 *rho_sigma, unsigned *flags, hipStream_t s);

}  // namespace ul
