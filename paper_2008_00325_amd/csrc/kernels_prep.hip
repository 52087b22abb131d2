// kernels_prep.hip -- device ingest of the COO graph B (sparse-data handling
// section: the COO list is sorted by row and indexed by a CSR row pointer).
//
// Steps (all on the handle's stream, one host synchronisation at the end):
//   1. k_check: indices and values checked, w_max = the largest weight of a
//      candidate edge (val > 0, row != col; a bipartite graph -- new points to a
//      frozen table -- keeps row == col, which are different vertices there),
//      candidates counted per bucket of 2^lg consecutive rows
//   2. k_bucket_scatter: the candidates filed by bucket, a tile of 8K entries at
//      a time, so that a bucket gets runs of a tile's entries
//   3. k_bucket_rows: one workgroup per bucket drops what lies below
//      w_max / n_epochs, counts its rows in LDS and files the rest by row; buckets
//      of many entries (hubs) in chunks, by k_heavy_rows before and after it
//   4. k_row_sort: 32 rows at a time (4 in dense graphs) sorted by column in LDS
//      (rank sort; equal columns flag a duplicate); row_ptr, col, eps = w_max / val
//      and the tails as 16-bit offsets written.  Rows of more than kLongRow entries
//      by k_long_row_sort, a stable radix sort, one workgroup per row
//   5. k_symmetry (not for a bipartite graph): each kept (i, j, v) must have
//      a (j, i) with bit-equal v
//   6. wave partition for the epoch kernel
//
// Entries move in runs: a count and a scatter with one global atomic and three
// 4-byte stores per entry at random rows took 1343 us on a shuffled graph of
// 777,777 rows (23.3M entries), where steps 2 and 3 take 163 and 202; a rank sort
// from memory and a pass for the offsets 470 us, step 4 271.  (1M rows in local
// order: 836 -> 110 + 231 us, 470 -> 368 us.)  Steps 3 and 4 are bound by the
// latency of a workgroup's chain of loads, step 2 by its streams.
#include "internal.hpp"
#include "launch_sizes.hpp"

namespace ul {


// rows in [0, n), columns in [0, n_cols); bipartite: row and column index
// different vertex sets
struct IngestShape {
    uint32_t n, n_cols;
    int32_t bipartite;
};

__device__ __forceinline__ bool candidate(int32_t r, int32_t c, float v, IngestShape sh)
{
    return (uint32_t)r < sh.n && (uint32_t)c < sh.n_cols && (sh.bipartite || r != c) && v > 0.0f && isfinite(v);
}

__device__ __forceinline__ float keep_threshold(const PrepScalars *S, int32_t n_epochs)
{
    return __uint_as_float(S->wmax_bits) / (float)n_epochs;
}

__device__ __forceinline__ unsigned wave_or(unsigned v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v |= __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ unsigned wave_max(unsigned v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor(v, off));
    return v;
}

// Slot of the calling lane in the counter ctr[key], with one atomic add per
// run of consecutive lanes that hold the same key (inactive lanes end a run):
// the counter's old value plus the lane's rank in its run.  Kernel-built
// graphs list a row's entries together, so runs are long.  Every lane of the
// wave must call it.
__device__ __forceinline__ int32_t run_atomic_add(int32_t *ctr, int32_t key, bool active)
{
    const int lane = (int)lane_id();
    const int32_t prev = __shfl_up(key, 1);
    const unsigned long long act = __ballot(active);
    const bool prev_act = lane > 0 && ((act >> (lane - 1)) & 1ull);
    const bool head = active && !(prev_act && prev == key);
    const unsigned long long heads = __ballot(head);
    const unsigned long long le = (2ull << lane) - 1ull;   // lanes 0 .. lane
    int32_t base = 0;
    if (head) {
        const unsigned long long above = (heads | ~act) & ~le;
        const int end = above ? __builtin_ctzll(above) : 64;
        base = atomicAdd(&ctr[key], end - lane);
    }
    const unsigned long long hm = heads & le;
    const int h = hm ? 63 - __builtin_clzll(hm) : lane;
    return __shfl(base, h) + lane - h;
}

// Buckets of consecutive rows: 2^lg rows each, at least kSortRows (the rows of a
// k_row_sort block lie in one bucket) and at most 2^16 (an entry's row in its
// bucket is a 16-bit number), about kBuckets of them where that allows.  2^8 rows
// or more, unless there are then fewer buckets than workgroups fit the chip and they
// get more than kBucketEntries entries each (a complete graph of 300 vertices: k_bucket_rows
// 77 -> 12 us; 20,000 rows of 1,000: 467 -> 219; where there are more buckets, finer ones
// only cost: 100,000 rows of 120 1048 -> 1105 us in all).
constexpr int kSortRows = 32;
constexpr int kBuckets = 1024;
constexpr int kMinBucketLg = 5, kFewBucketLg = 8, kMaxBucketLg = 16;
constexpr int64_t kBucketEntries = 16384;
constexpr int kFewBuckets = 512;
// counters of buckets lie a cache line apart: workgroups add to all of them
constexpr int kPad = 32;
constexpr int kTileThreads = 1024;
constexpr int kTileItems = 8;
constexpr int kTile = kTileThreads * kTileItems;
// rows of a bucket counted in LDS at a time
constexpr int kBucketRows = 8192;

int32_t bucket_lg(int64_t n, int64_t nnz)
{
    int32_t lg = kFewBucketLg;
    while (lg < kMaxBucketLg && (n >> lg) >= kBuckets) ++lg;
    while (lg > kMinBucketLg && (n >> (lg - 1)) < kFewBuckets && (nnz << lg) > kBucketEntries * n) --lg;
    return lg;
}
int64_t bucket_count(int64_t n, int64_t nnz)
{
    const int32_t lg = bucket_lg(n, nnz);
    return (n + ((int64_t)1 << lg) - 1) >> lg;
}
int64_t bucket_counters(int64_t n, int64_t nnz) { return kPad * kSubs * bucket_count(n, nnz); }
// Rows of a block of k_row_sort and k_symmetry: kSortRows, or kSortRowsDense in
// graphs of long rows, where those fill a block and more blocks the chip (a complete
// graph of 300 vertices: k_row_sort 179 us with 32 rows, now 30; 100,000 rows of 120,
// which have blocks enough, 175).
constexpr int kSortRowsDense = 4;
constexpr int64_t kDenseRow = 128;
int32_t sort_rows(int64_t n, int64_t nnz) { return nnz >= kDenseRow * n ? kSortRowsDense : kSortRows; }
int64_t row_blocks(int64_t n, int64_t nnz) { return (n + sort_rows(n, nnz) - 1) / sort_rows(n, nnz); }

// Buckets of many entries (those of hubs) are counted and filed in chunks by
// workgroups of their own: a bucket of more than kHeavyEntries entries that also
// has more than its part of the work were the chip to share all entries (two
// workgroups per CU are resident).
constexpr int64_t kHeavyEntries = 65536;
constexpr uint32_t kHeavyChunk = 32768;
constexpr int32_t kHeavyShare = 256;
int64_t heavy_chunks(int64_t nnz) { return nnz > kHeavyEntries ? nnz / kHeavyChunk + kHeavyShare : 0; }
// counter of part `sub` of bucket b
__device__ __forceinline__ int64_t counter_at(int32_t sub, int32_t b, int32_t nb) { return ((int64_t)sub * nb + b) * kPad; }

__global__ __launch_bounds__(kTileThreads) void k_check(const int32_t *__restrict__ rows,
                                                        const int32_t *__restrict__ cols,
                                                        const float *__restrict__ vals, int64_t nnz, IngestShape sh,
                                                        int32_t lg, int32_t nb, uint32_t *__restrict__ bucket_n,
                                                        PrepScalars *S)
{
    extern __shared__ int32_t s_n[];   // nb counters
    __shared__ unsigned s_flags, s_max;
    for (int32_t b = threadIdx.x; b < nb; b += kTileThreads) s_n[b] = 0;
    if (threadIdx.x == 0) s_flags = s_max = 0;
    __syncthreads();
    unsigned flags = 0, mx = 0;
    // the grid is a multiple of kSubs: a block's tiles are of one part
    for (int64_t t0 = (int64_t)blockIdx.x * kTile; t0 < nnz; t0 += (int64_t)gridDim.x * kTile) {
        int32_t r[kTileItems], c[kTileItems];
        float v[kTileItems];
#pragma unroll
        for (int q = 0; q < kTileItems; ++q) {
            const int64_t t = t0 + q * kTileThreads + threadIdx.x;
            const bool in = t < nnz;
            r[q] = in ? rows[t] : 0;
            c[q] = in ? cols[t] : 0;
            v[q] = in ? vals[t] : 0.0f;   // 0: not a candidate
        }
#pragma unroll
        for (int q = 0; q < kTileItems; ++q) {
            if ((uint32_t)r[q] >= sh.n || (uint32_t)c[q] >= sh.n_cols) flags |= kBadIndex;   // (0, 0) past the end is none
            if (!isfinite(v[q])) flags |= kBadValue;
            const bool cand = candidate(r[q], c[q], v[q], sh);
            if (cand) mx = max(mx, __float_as_uint(v[q]));  // positive floats order as integers
            run_atomic_add(s_n, cand ? r[q] >> lg : 0, cand);
        }
    }
    flags = wave_or(flags);
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) {
        if (flags) atomicOr(&s_flags, flags);
        if (mx) atomicMax(&s_max, mx);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_flags) atomicOr(&S->flags, s_flags);
        if (s_max) atomicMax(&S->wmax_bits, s_max);
    }
    for (int32_t b = threadIdx.x; b < nb; b += kTileThreads)
        if (s_n[b]) atomicAdd(&bucket_n[counter_at(blockIdx.x % kSubs, b, nb)], (uint32_t)s_n[b]);
}

// Exclusive scan of get(0) .. get(count - 1) by one workgroup: put(t, the sum
// before t) for t < count; returns the total.  s_wave: kTileThreads / 64 words.
template <typename Get, typename Put>
__device__ __forceinline__ int32_t scan_loop(int32_t count, int32_t *s_wave, Get get, Put put)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int32_t carry = 0;
    for (int32_t base = 0; base < count; base += kTileThreads) {
        const int32_t t = base + tid;
        const int32_t v = t < count ? get(t) : 0;
        int32_t x = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        if (lane == 63) s_wave[wv] = x;
        __syncthreads();
        int32_t before = 0, total = 0;
#pragma unroll
        for (int k = 0; k < kTileThreads / 64; ++k) {
            before += k < wv ? s_wave[k] : 0;
            total += s_wave[k];
        }
        if (t < count) put(t, carry + before + x - v);
        carry += total;
        __syncthreads();
    }
    return carry;
}

// The candidates' counters (bucket b, part sub: b kSubs + sub in this order) ->
// first[t], the entries before each, and the cursors that start there; then the
// chunks of the heavy buckets: heavy_first[b] = chunks of the buckets before b.
__global__ __launch_bounds__(kTileThreads) void k_bucket_starts(const uint32_t *__restrict__ in, int32_t nb,
                                                                int32_t *__restrict__ first,
                                                                uint32_t *__restrict__ cursor,
                                                                int32_t *__restrict__ heavy_first, PrepScalars *S)
{
    __shared__ int32_t s_wave[kTileThreads / 64];
    __shared__ int32_t s_large;
    const int32_t count = kSubs * nb;
    if (threadIdx.x == 0) s_large = 0;
    __syncthreads();
    const int32_t total = scan_loop(
        count, s_wave,
        [&](int32_t t) {
            const int32_t v = (int32_t)in[counter_at(t % kSubs, t / kSubs, nb)];
            if (v > kHeavyEntries / kSubs) s_large = 1;   // its bucket may be heavy
            return v;
        },
        [&](int32_t t, int32_t before) {
            first[t] = before;
            cursor[counter_at(t % kSubs, t / kSubs, nb)] = (uint32_t)before;
        });
    if (threadIdx.x == 0) first[count] = total;
    __syncthreads();   // s_large, first
    int32_t chunks = 0;
    int32_t above = INT32_MAX;   // no bucket is heavy
    if (s_large) {
        above = max((int32_t)kHeavyEntries, total / kHeavyShare);
        chunks = scan_loop(
            nb, s_wave,
            [&](int32_t b) {
                const int32_t m = first[(b + 1) * kSubs] - first[b * kSubs];
                return m > above ? (int32_t)(((uint32_t)m + kHeavyChunk - 1) / kHeavyChunk) : 0;
            },
            [&](int32_t b, int32_t before) { heavy_first[b] = before; });
    }
    if (threadIdx.x == 0) {
        heavy_first[nb] = chunks;
        S->n_heavy = chunks;
        S->heavy_above = above;
    }
}

// kfirst[b] = kept entries of the buckets before b
__global__ __launch_bounds__(kTileThreads) void k_kept_starts(const uint32_t *__restrict__ kept_n, int32_t nb,
                                                              int32_t *__restrict__ kfirst)
{
    __shared__ int32_t s_wave[kTileThreads / 64];
    const int32_t total = scan_loop(nb, s_wave, [&](int32_t b) { return (int32_t)kept_n[b]; },
                                    [&](int32_t b, int32_t before) { kfirst[b] = before; });
    if (threadIdx.x == 0) kfirst[nb] = total;
}

// A tile of entries filed by bucket: ranks in LDS counters, one reservation per
// tile and bucket (in the counters of the tile's XCD: 226 -> 164 us).
__global__ __launch_bounds__(kTileThreads) void k_bucket_scatter(const int32_t *__restrict__ rows,
                                                                 const int32_t *__restrict__ cols,
                                                                 const float *__restrict__ vals, int64_t nnz,
                                                                 IngestShape sh, int32_t lg, int32_t nb,
                                                                 uint32_t *__restrict__ cursor,
                                                                 int2 *__restrict__ pair, uint16_t *__restrict__ lrow)
{
    extern __shared__ int32_t s_n[];   // nb counters, then the tile's first slots
    for (int32_t b = threadIdx.x; b < nb; b += kTileThreads) s_n[b] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kTile;
    int32_t r[kTileItems], c[kTileItems], rank[kTileItems];
    float v[kTileItems];
#pragma unroll
    for (int q = 0; q < kTileItems; ++q) {
        const int64_t t = base + q * kTileThreads + threadIdx.x;
        const bool in = t < nnz;
        r[q] = in ? rows[t] : 0;
        c[q] = in ? cols[t] : 0;
        v[q] = in ? vals[t] : 0.0f;   // 0: not a candidate
    }
#pragma unroll
    for (int q = 0; q < kTileItems; ++q) {
        const bool cand = candidate(r[q], c[q], v[q], sh);
        const int32_t slot = run_atomic_add(s_n, cand ? r[q] >> lg : 0, cand);
        rank[q] = cand ? slot : -1;
    }
    __syncthreads();
    for (int32_t b = threadIdx.x; b < nb; b += kTileThreads) {
        const int32_t m = s_n[b];
        if (m) s_n[b] = (int32_t)atomicAdd(&cursor[counter_at(blockIdx.x % kSubs, b, nb)], (uint32_t)m);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kTileItems; ++q) {
        if (rank[q] < 0) continue;
        const uint32_t p = (uint32_t)(s_n[r[q] >> lg] + rank[q]);
        pair[p] = make_int2(c[q], __float_as_int(v[q]));
        lrow[p] = (uint16_t)(r[q] & ((1 << lg) - 1));
    }
}

// The entries [c0, c1) of a bucket whose rows lie in [a, a + m) of it and which are
// kept, counted per row (s_n[row - a]).  Entry numbers are unsigned: a step beyond
// the last entry may pass 2^31.
constexpr int kEntriesAhead = 8;   // loads of a thread in flight
__device__ __forceinline__ void count_entries(const int2 *__restrict__ pair, const uint16_t *__restrict__ lrow,
                                              uint32_t c0, uint32_t c1, int32_t a, int32_t m, float thresh,
                                              int32_t *s_n)
{
    for (; c0 < c1; c0 += kEntriesAhead * kTileThreads) {
        uint32_t q[kEntriesAhead];
        float v[kEntriesAhead];
#pragma unroll
        for (int u = 0; u < kEntriesAhead; ++u) {
            const uint32_t e = c0 + u * kTileThreads + threadIdx.x;
            q[u] = 0xFFFFFFFFu;
            if (e < c1) {
                q[u] = (uint32_t)lrow[e] - (uint32_t)a;
                v[u] = __int_as_float(pair[e].y);
            }
        }
#pragma unroll
        for (int u = 0; u < kEntriesAhead; ++u)
            if (q[u] < (uint32_t)m && v[u] >= thresh) atomicAdd(&s_n[q[u]], 1);
    }
}

// The same entries moved to out[s_n[row - a]++].
__device__ __forceinline__ void file_entries(const int2 *__restrict__ pair, const uint16_t *__restrict__ lrow,
                                             uint32_t c0, uint32_t c1, int32_t a, int32_t m, float thresh, int32_t *s_n,
                                             int2 *__restrict__ out)
{
    for (; c0 < c1; c0 += kEntriesAhead * kTileThreads) {
        uint32_t q[kEntriesAhead];
        int2 p[kEntriesAhead];
#pragma unroll
        for (int u = 0; u < kEntriesAhead; ++u) {
            const uint32_t e = c0 + u * kTileThreads + threadIdx.x;
            q[u] = 0xFFFFFFFFu;
            if (e < c1) {
                q[u] = (uint32_t)lrow[e] - (uint32_t)a;
                p[u] = pair[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kEntriesAhead; ++u)
            if (q[u] < (uint32_t)m && __int_as_float(p[u].y) >= thresh) out[atomicAdd(&s_n[q[u]], 1)] = p[u];
    }
}

__device__ __forceinline__ int32_t bucket_rows(int64_t row0, int64_t n, int32_t lg)
{
    return (int32_t)(n - row0 < ((int64_t)1 << lg) ? n - row0 : (int64_t)1 << lg);
}

// One workgroup per bucket: its kept entries counted per row in LDS and filed by
// row into `out`, from the bucket's first slot on.  lstart[row] = the row's
// first entry counted from there, kept_n[bucket] = its kept entries.  Buckets of
// more rows than the counters hold take them kBucketRows at a time.  A heavy
// bucket's rows were counted by k_heavy_rows<false> (in lstart), which files them
// afterwards from `rcursor` on.
__global__ __launch_bounds__(kTileThreads) void k_bucket_rows(const int2 *__restrict__ pair,
                                                              const uint16_t *__restrict__ lrow,
                                                              const int32_t *__restrict__ first, int64_t n, int32_t lg,
                                                              int32_t n_epochs, const PrepScalars *S,
                                                              int2 *__restrict__ out, int32_t *__restrict__ lstart,
                                                              int32_t *__restrict__ rcursor,
                                                              uint32_t *__restrict__ kept_n)
{
    __shared__ int32_t s_n[kBucketRows];
    __shared__ int32_t s_wave[kTileThreads / 64];
    const int tid = threadIdx.x;
    const float thresh = keep_threshold(S, n_epochs);
    const uint32_t e0 = first[blockIdx.x * kSubs], e1 = first[(blockIdx.x + 1) * kSubs];
    const bool heavy = e1 - e0 > (uint32_t)S->heavy_above;
    const int64_t row0 = (int64_t)blockIdx.x << lg;
    const int32_t rows = bucket_rows(row0, n, lg);
    int32_t done = 0;   // kept entries of the rows before
    if (heavy) {        // (a loop of its own: in the other it cost registers and 14 us at 1M rows)
        done = scan_loop(rows, s_wave, [&](int32_t t) { return lstart[row0 + t]; },
                         [&](int32_t t, int32_t before) {
                             lstart[row0 + t] = before;
                             rcursor[row0 + t] = before;
                         });
    } else {
        for (int32_t a = 0; a < rows; a += kBucketRows) {
            const int32_t m = rows - a < kBucketRows ? rows - a : kBucketRows;
            for (int32_t t = tid; t < m; t += kTileThreads) s_n[t] = 0;
            __syncthreads();
            count_entries(pair, lrow, e0, e1, a, m, thresh, s_n);
            __syncthreads();
            const int32_t before = done;
            done += scan_loop(m, s_wave, [&](int32_t t) { return s_n[t]; },
                              [&](int32_t t, int32_t x) {
                                  s_n[t] = before + x;
                                  lstart[row0 + a + t] = before + x;
                              });
            file_entries(pair, lrow, e0, e1, a, m, thresh, s_n, out + e0);
            __syncthreads();
        }
    }
    if (tid == 0) kept_n[blockIdx.x] = (uint32_t)done;
}

// The chunks of the heavy buckets, in strides over the grid.  Counting: their kept
// entries per row added to row_n[row].  FILE: slots reserved from row_n[row] on (the
// row's first entry in the bucket), one atomic per chunk and row, and the entries
// filed there.  (A bucket taken by one
// workgroup whatever its entries: 19.5M edges with 1/x-distributed ends 8.3 ms, now 0.25
// in all three kernels; 200 rows of 50,000 16.8 ms, now 0.19.)
template <bool FILE>
__global__ __launch_bounds__(kTileThreads) void k_heavy_rows(const int2 *__restrict__ pair,
                                                             const uint16_t *__restrict__ lrow,
                                                             const int32_t *__restrict__ first,
                                                             const int32_t *__restrict__ heavy_first, int64_t n,
                                                             int32_t lg, int32_t nb, int32_t n_epochs,
                                                             const PrepScalars *S, int32_t *__restrict__ row_n,
                                                             int2 *__restrict__ out)
{
    __shared__ int32_t s_n[kBucketRows];
    const int tid = threadIdx.x;
    const int32_t items = S->n_heavy;
    const float thresh = keep_threshold(S, n_epochs);
    for (int32_t item = blockIdx.x; item < items; item += gridDim.x) {
        // bucket b: the last with heavy_first[b] <= item (light ones have no chunks)
        int32_t lo = 0, hi = nb - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (heavy_first[mid] <= item) lo = mid; else hi = mid - 1;
        }
        const uint32_t e0 = first[lo * kSubs], e1 = first[(lo + 1) * kSubs];
        const uint32_t c0 = e0 + (uint32_t)(item - heavy_first[lo]) * kHeavyChunk;
        const uint32_t c1 = e1 - c0 > kHeavyChunk ? c0 + kHeavyChunk : e1;
        const int64_t row0 = (int64_t)lo << lg;
        const int32_t rows = bucket_rows(row0, n, lg);
        for (int32_t a = 0; a < rows; a += kBucketRows) {
            const int32_t m = rows - a < kBucketRows ? rows - a : kBucketRows;
            for (int32_t t = tid; t < m; t += kTileThreads) s_n[t] = 0;
            __syncthreads();
            count_entries(pair, lrow, c0, c1, a, m, thresh, s_n);
            __syncthreads();
            for (int32_t t = tid; t < m; t += kTileThreads)
                if (s_n[t]) s_n[t] = atomicAdd(&row_n[row0 + a + t], s_n[t]);
            __syncthreads();
            if (FILE) {
                file_entries(pair, lrow, c0, c1, a, m, thresh, s_n, out + e0);
                __syncthreads();
            }
        }
    }
}

// Rows longer than this are sorted by k_long_row_sort: the rank sort reads a
// row once per entry, deg^2 LDS reads in all.
constexpr int32_t kLongRow = 512;
constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kRowTile = 1024;   // entries of consecutive rows in LDS at a time (8 blocks per CU)

// Entries that a block of k_symmetry takes at a time.
constexpr int32_t kSymEntries = 4096;
__host__ __device__ inline int32_t symmetry_pieces(int32_t entries)
{
    return entries > kSymEntries ? (int32_t)(((int64_t)entries + kSymEntries - 1) / kSymEntries) : 1;
}

// What k_row_sort and k_long_row_sort write, beside the row pointers.
struct SortedRows {
    int32_t *col;
    float *eps;
    int2 *pair;        // (col, value bits): the symmetry check's copy
    int16_t *col16;    // col - row (null: bipartite)
};

// ROWS rows per block.  src: the rows' entries in any order, from
// first[bucket kSubs] + lstart[row] on; out: in (row, col) order.  Rank sort: an
// entry's slot is the number of smaller columns in its row, read from LDS four
// at a time (the rows are padded to multiples of four there); the entries are
// put in order in LDS and written in runs.  A slot left empty is a duplicate.
// (26.7M entries, 1M rows: 475 us reading the row entry by entry and writing
// each entry at its slot, 446 us with 16 rows per block, now 375.)
template <int ROWS>
__global__ __launch_bounds__(256) void k_row_sort(const int2 *__restrict__ src, const int32_t *__restrict__ first,
                                                  const int32_t *__restrict__ kfirst,
                                                  const int32_t *__restrict__ lstart, int64_t n, int32_t lg,
                                                  PrepScalars *S, int64_t *__restrict__ row_ptr,
                                                  int32_t *__restrict__ rp32, int32_t *__restrict__ long_rows,
                                                  int32_t *__restrict__ block_near, int32_t *__restrict__ block_max,
                                                  int2 *__restrict__ sym_list, SortedRows out)
{
    __shared__ __align__(16) int32_t s_col[kRowTile + 4 * ROWS];   // columns by padded row
    __shared__ int2 s_out[kRowTile];
    __shared__ uint8_t s_row[kRowTile];
    __shared__ int32_t s_start[ROWS + 1], s_pad[ROWS + 1];
    __shared__ unsigned s_flags, s_near;
    __shared__ int32_t s_piece;
    const int tid = threadIdx.x;
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t r0 = block * ROWS;
    if (r0 >= n) return;   // the last row of a grid of two dimensions
    const int nr = (int)(n - r0 < ROWS ? n - r0 : ROWS);
    const int64_t b = r0 >> lg;
    const int32_t dst = kfirst[b];
    const int2 *const in = src + first[b * kSubs];
    const float w_max = __uint_as_float(S->wmax_bits);
    // the rows' first entries, as uniform values (scalar loads) and in LDS
    int32_t ustart[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) ustart[k] = k < nr ? lstart[r0 + k] : INT32_MAX;
    if (tid <= nr) {
        const int64_t r = r0 + tid;
        // past the last row of a bucket: the bucket's kept entries
        const int32_t st = r < n && (tid < nr || (r >> lg) == b) ? lstart[r] : kfirst[b + 1] - dst;
        s_start[tid] = st;
        if (tid < nr || r == n) {
            row_ptr[r] = (int64_t)dst + st;
            rp32[r] = dst + st;
        }
    }
    if (tid == 0) s_flags = s_near = 0;
    __syncthreads();
    static_assert(ROWS < 64, "a lane per row");
    if (tid < 64) {
        const int32_t len = tid < nr ? s_start[tid + 1] - s_start[tid] : 0;
        // the rows' places in s_col
        int32_t x = (len + 3) & ~3;
#pragma unroll
        for (int off = 1; off < 2 * ROWS; off <<= 1) {
            const int32_t y = __shfl_up(x, off);
            if (tid >= off) x += y;
        }
        if (tid <= nr) s_pad[tid] = x - ((len + 3) & ~3);
        const unsigned mx = wave_max((unsigned)len);
        if (tid == 0) block_max[block] = (int32_t)mx;
        if (len > kLongRow) long_rows[atomicAdd(&S->n_long, 1)] = (int32_t)(r0 + tid);
    }
    // the symmetry check's pieces of these entries but the first
    const int32_t more = out.col16 ? symmetry_pieces(s_start[nr] - s_start[0]) - 1 : 0;
    if (more > 0) {
        if (tid == 0) s_piece = atomicAdd(&S->n_sym, more);
        __syncthreads();
        for (int32_t t = tid; t < more; t += 256) sym_list[s_piece + t] = make_int2((int)block, t + 1);
    }
    unsigned flags = 0, near = 0;
    for (int a = 0; a < nr;) {
        const int32_t t0 = s_start[a];
        if (s_start[a + 1] - t0 > kLongRow) {   // k_long_row_sort
            ++a;
            continue;
        }
        int z = a + 1;   // rows [a, z) together
        while (z < nr && s_start[z + 1] - t0 <= kRowTile && s_start[z + 1] - s_start[z] <= kLongRow) ++z;
        const int32_t m = s_start[z] - t0;
        // a thread's entries are tid, tid + 256, ..
        constexpr int kItems = kRowTile / 256;
        int2 p[kItems];
        int row[kItems];
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            const int32_t t = u * 256 + tid;
            if (t < m) p[u] = in[t0 + t];
        }
        __syncthreads();   // s_pad
        const int32_t pad0 = s_pad[a];
        for (int32_t t = tid; t < s_pad[z] - pad0; t += 256) s_col[t] = INT32_MAX;
        for (int32_t t = tid; t < m; t += 256) s_out[t] = make_int2(-1, 0);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            if (u * 256 >= m) break;
            const int32_t t = u * 256 + tid;
            // the last row that starts at or before t (it is not empty)
            int r = -1;
#pragma unroll
            for (int k = 0; k < ROWS; ++k) r += ustart[k] - t0 <= t;
            row[u] = r;
            if (t < m) s_col[s_pad[r] - pad0 + t - (s_start[r] - t0)] = p[u].x;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            const int32_t t = u * 256 + tid;
            if (t < m) {
                const int32_t rs = s_start[row[u]] - t0;
                const int quads = (s_start[row[u] + 1] - s_start[row[u]] + 3) >> 2;
                const int4 *const rc = reinterpret_cast<const int4 *>(&s_col[s_pad[row[u]] - pad0]);
                int32_t rank = 0;
#pragma unroll 4
                for (int q = 0; q < quads; ++q) {
                    const int4 c = rc[q];
                    rank += (c.x < p[u].x) + (c.y < p[u].x) + (c.z < p[u].x) + (c.w < p[u].x);
                }
                s_out[rs + rank] = p[u];
                s_row[t] = (uint8_t)row[u];   // the same entries of the row in any order
            }
        }
        __syncthreads();
        for (int32_t t = tid; t < m; t += 256) {
            const int2 q = s_out[t];
            if (q.x < 0) flags |= kDuplicate;
            const int32_t o = dst + t0 + t;
            const float v = __int_as_float(q.y);
            out.col[o] = q.x;
            out.eps[o] = w_max / v;
            if (out.col16) {
                const int64_t d = (int64_t)q.x - (r0 + s_row[t]);
                out.pair[o] = q;
                out.col16[o] = (int16_t)d;
                if (d < INT16_MIN || d > INT16_MAX) flags |= kWide;
                near += d >= -kHalo && d <= kHalo;
            }
        }
        __syncthreads();
        a = z;
    }
    flags = wave_or(flags);
    if ((tid & 63) == 0 && flags) atomicOr(&s_flags, flags);
    if (near) atomicAdd(&s_near, near);
    __syncthreads();
    if (tid == 0) {
        // (most blocks of a shuffled graph raise kWide: look before adding)
        if (s_flags && (s_flags & ~*(volatile unsigned *)&S->flags)) atomicOr(&S->flags, s_flags);
        block_near[block] = (int32_t)s_near;
    }
}

// One workgroup per long row (the grid takes the list in strides): a
// least-significant-digit radix sort of the row's (column, slot) pairs by
// column, 4-bit digits, each pass stable (the digit's global offset from a
// counting sweep, then chunks of 1024 entries in order, each entry placed
// after the earlier entries of its digit: rank in its wavefront by ballot,
// wavefront offsets in LDS).  The pairs move between two buffers inside the
// row's own segment: (col, eps), eps holding the slot as an int, and the two
// halves of the row's `pair` segment.  An even number of passes leaves the
// result in (col, eps); then eps, pair and the offsets are written in sorted
// order and equal neighbours flag a duplicate.
__global__ __launch_bounds__(kSortThreads) void k_long_row_sort(const int2 *__restrict__ src,
                                                                const int32_t *__restrict__ first,
                                                                const int32_t *__restrict__ kfirst,
                                                                const int32_t *__restrict__ lstart, int64_t n,
                                                                int32_t lg, int32_t passes,
                                                                const int32_t *__restrict__ long_rows, PrepScalars *S,
                                                                SortedRows out)
{
    __shared__ int32_t s_hist[16];
    __shared__ int32_t s_wcnt[kSortWaves][16];
    __shared__ int32_t s_woff[kSortWaves][16];
    const int tid = threadIdx.x, wv = tid / 64, lane = tid % 64;
    const float w_max = __uint_as_float(S->wmax_bits);
    const int32_t n_long = S->n_long;
    for (int32_t item = blockIdx.x; item < n_long; item += gridDim.x) {
        const int64_t r = long_rows[item];
        const int64_t b = r >> lg;
        const int32_t ls = lstart[r];
        const int32_t le = r + 1 < n && ((r + 1) >> lg) == b ? lstart[r + 1] : kfirst[b + 1] - kfirst[b];
        const int64_t L = le - ls;
        const int2 *const in = src + first[b * kSubs] + ls;
        const int64_t rs = (int64_t)kfirst[b] + ls;
        int32_t *const spare = reinterpret_cast<int32_t *>(out.pair + rs);
        int32_t *const key[2] = {out.col + rs, spare};
        int32_t *const idx[2] = {reinterpret_cast<int32_t *>(out.eps) + rs, spare + L};
        for (int64_t t = tid; t < L; t += kSortThreads) {
            key[0][t] = in[t].x;
            idx[0][t] = (int32_t)t;
        }
        __syncthreads();
        for (int32_t pass = 0; pass < passes; ++pass) {
            const int from = pass & 1, to = from ^ 1;
            const int shift = 4 * pass;
            if (tid < 16) s_hist[tid] = 0;
            __syncthreads();
            for (int64_t t = tid; t < L; t += kSortThreads) atomicAdd(&s_hist[((uint32_t)key[from][t] >> shift) & 15u], 1);
            __syncthreads();
            if (tid == 0) {
                int32_t run = 0;
                for (int d = 0; d < 16; ++d) {
                    const int32_t c = s_hist[d];
                    s_hist[d] = run;   // first slot of digit d
                    run += c;
                }
            }
            __syncthreads();
            for (int64_t c0 = 0; c0 < L; c0 += kSortThreads) {
                const int64_t t = c0 + tid;
                const bool valid = t < L;
                const int32_t k = valid ? key[from][t] : 0;
                const int32_t ix = valid ? idx[from][t] : 0;
                const int d = valid ? (int)(((uint32_t)k >> shift) & 15u) : 16;
                int rank = 0;
                for (int v = 0; v < 16; ++v) {
                    const unsigned long long m = __ballot(d == v);
                    if (d == v) rank = (int)lanes_below(m);
                    if (lane == 0) s_wcnt[wv][v] = __popcll(m);
                }
                __syncthreads();
                if (tid < 16) {
                    int32_t run = s_hist[tid];
                    for (int w = 0; w < kSortWaves; ++w) {
                        s_woff[w][tid] = run;
                        run += s_wcnt[w][tid];
                    }
                    s_hist[tid] = run;
                }
                __syncthreads();
                if (valid) {
                    const int32_t pos = s_woff[wv][d] + rank;
                    key[to][pos] = k;
                    idx[to][pos] = ix;
                }
                __syncthreads();
            }
        }
        unsigned flags = 0, near = 0;
        for (int64_t t = tid; t < L; t += kSortThreads) {
            const int32_t c = key[0][t];
            const float v = __int_as_float(in[idx[0][t]].y);
            if (t > 0 && key[0][t - 1] == c) flags |= kDuplicate;
            out.eps[rs + t] = w_max / v;
            if (out.col16) {
                const int64_t d = (int64_t)c - r;
                out.pair[rs + t] = make_int2(c, __float_as_int(v));
                out.col16[rs + t] = (int16_t)d;
                if (d < INT16_MIN || d > INT16_MAX) flags |= kWide;
                near += d >= -kHalo && d <= kHalo;
            }
        }
        flags = wave_or(flags);
        if (lane == 0 && flags) atomicOr(&S->flags, flags);
        if (near) atomicAdd(&S->near, (unsigned long long)near);
        __syncthreads();
    }
}

// The kept graph is symmetric if every (i, j, v) with i < j has its (j, i, v) and
// there are as many entries above the diagonal as below it (no entry is listed
// twice): half the lookups.  A wave takes 64 consecutive entries at a time;
// those above the diagonal are looked up by 16 lanes together, four per load,
// in the first entries of row j, which is sorted, so that its entries below
// the diagonal come first: 16 entries a round, three rounds, and what is not
// decided then by a binary search.  The random lines of the rows bound it on a
// shuffled graph: 2559 us on 20.8M edges with one binary search per lane and
// entry, now 486 (26.7M edges in local order 693 -> 274).  Rows of more than
// kLookupRow entries go to the binary search at once, which reads the columns
// alone.
// A block takes up to kSymEntries entries of its rows; the further
// pieces of long or dense rows are listed by k_row_sort and taken by blocks of
// their own, so that no block has a long row to itself: 9M edges of a complete
// graph of 3,000 vertices, where each block had 32 rows, 4444 us, now 500; 19.5M
// edges with 1/x-distributed ends 29.5 ms, now 0.48.
constexpr uint32_t kLookupRow = 96;
__global__ __launch_bounds__(256) void k_symmetry(const int2 *__restrict__ pair, const int32_t *__restrict__ col,
                                                  const int32_t *__restrict__ rp32, int64_t n, int32_t rows,
                                                  int64_t row_blocks,
                                                  int32_t more_blocks, const int2 *__restrict__ sym_list,
                                                  PrepScalars *S, int32_t *__restrict__ block_diff)
{
    // After a duplicate the in-row sort leaves some slots unwritten; the
    // graph is rejected anyway, so skip the check rather than read them.
    if (S->flags & (kDuplicate | kBadIndex | kBadValue)) return;
    constexpr int kG = 16;        // lanes per lookup
    constexpr int kRounds = 3;
    constexpr int kAhead = 8;     // loads in flight
    __shared__ int32_t s_start[kSortRows + 1];
    __shared__ int4 s_list[4][64];   // (first entry, end of row, i, value bits)
    __shared__ int s_diff;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= row_blocks + more_blocks) return;   // the last row of a grid of two dimensions
    const bool first_piece = block < row_blocks;
    // the first piece of the block's own rows, or the listed pieces in strides
    const int64_t items = first_piece ? 1 : S->n_sym;
    int64_t item = first_piece ? 0 : block - row_blocks;
    if (item >= items) return;
    if (tid == 0) s_diff = 0;
    bool bad = false;
    int diff = 0;   // entries above the diagonal minus entries below
    const int group = lane / kG, part = lane % kG;
    do {
        const int2 p0 = first_piece ? make_int2((int)block, 0) : sym_list[item];
        const int64_t r0 = (int64_t)p0.x * rows;
        const int nr = (int)(n - r0 < rows ? n - r0 : rows);
        __syncthreads();   // the last piece's rows are done with
        if (tid <= nr) s_start[tid] = rp32[r0 + tid];
        __syncthreads();
        // entry numbers are unsigned: steps beyond a row's or the last entry may pass 2^31
        const uint32_t a0 = (uint32_t)s_start[0] + (uint32_t)p0.y * kSymEntries;
        const uint32_t a1 = s_start[nr];
        const uint32_t e1 = a1 - a0 > (uint32_t)kSymEntries ? a0 + kSymEntries : a1;
        for (uint32_t c0 = a0 + wv * 64; c0 < e1; c0 += 256) {
            const uint32_t e = c0 + lane;
            const bool in = e < e1;
            int2 p = make_int2(0, 0);
            int32_t i = 0;
            if (in) {
                p = pair[e];
                int lo = 0, hi = nr - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if ((uint32_t)s_start[mid] <= e) lo = mid; else hi = mid - 1;
                }
                i = (int32_t)(r0 + lo);
            }
            bool open = in && p.x > i;   // still to be found
            diff += in ? (open ? 1 : -1) : 0;
            uint32_t at = 0, re = 0;
            if (open) {
                at = rp32[p.x];
                re = rp32[p.x + 1];
            }
            bool late = open && re - at > kLookupRow;   // for the binary search
            open = open && !late;
            for (int round = 0; round < kRounds; ++round) {
                const unsigned long long m = __ballot(open);
                if (m == 0) break;
                const int cnt = __popcll(m);
                const int mine = (int)lanes_below(m);   // place in the list
                if (open) s_list[wv][mine] = make_int4((int)at, (int)re, i, p.y);
                wave_sync();
                unsigned long long hit = 0;
                for (int s0 = 0; s0 < cnt; s0 += 4 * kAhead) {
                    int4 w[kAhead];
                    int2 q[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (s0 + 4 * u >= cnt) break;
                        const int s = s0 + 4 * u + group;
                        w[u] = s_list[wv][s < cnt ? s : 0];
                        q[u] = make_int2(-1, 0);
                        const uint32_t x = (uint32_t)w[u].x + part;
                        if (s < cnt && x < (uint32_t)w[u].y) q[u] = pair[x];
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (s0 + 4 * u >= cnt) break;
                        const unsigned long long h = __ballot(q[u].x == w[u].z && q[u].y == w[u].w);   // column -1 is none
                        if ((mine >> 2) == (s0 >> 2) + u) hit = h;
                    }
                }
                if (open) {
                    at += kG;
                    if ((hit >> (kG * (mine & 3))) & ((1ull << kG) - 1ull)) open = false;
                    else if (at >= re) {
                        open = false;
                        bad = true;
                    }
                }
                wave_sync();   // the list is written again
            }
            if (open || late) {
                uint32_t lo = at, hi = re;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (col[mid] < i) lo = mid + 1; else hi = mid;
                }
                if (lo >= re) bad = true;
                else {
                    const int2 q = pair[lo];
                    bad |= q.x != i || q.y != p.y;
                }
            }
        }
        item += first_piece ? 1 : more_blocks;
    } while (item < items);
    if (diff) atomicAdd(&s_diff, diff);
    if (__ballot(bad) != 0 && lane == 0) atomicOr(&S->flags, (unsigned)kAsymmetric);
    __syncthreads();
    if (tid == 0) {
        if (first_piece) block_diff[block] = s_diff;
        else if (s_diff) atomicAdd(reinterpret_cast<unsigned long long *>(&S->up_minus_low), (unsigned long long)(long long)s_diff);
    }
}

// The blocks' largest rows and partial sums into the scalars (diff null:
// bipartite).  Thousands of workgroups adding to one line would wait for each
// other: 62,500 of them took 200 us of the sort and the symmetry check each.
__global__ __launch_bounds__(256) void k_prep_sums(const int32_t *__restrict__ mx, const int32_t *__restrict__ near,
                                                   const int32_t *__restrict__ diff, int64_t count, PrepScalars *S)
{
    if (S->flags & (kDuplicate | kBadIndex | kBadValue)) diff = nullptr;   // the check did not run
    int64_t a = 0, d = 0;
    unsigned m = 0;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < count; t += (int64_t)gridDim.x * 256) {
        m = max(m, (unsigned)mx[t]);
        a += near[t];
        if (diff) d += diff[t];
    }
    m = wave_max(m);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        d += __shfl_xor(d, off);
    }
    if ((threadIdx.x & 63) == 0) {
        if (m) atomicMax(&S->max_degree, (int)m);
        if (a) atomicAdd(&S->near, (unsigned long long)a);
        if (d) atomicAdd(reinterpret_cast<unsigned long long *>(&S->up_minus_low), (unsigned long long)d);
    }
}

static int64_t grid_for(int64_t items)
{
    int64_t b = (items + 255) / 256;
    if (b > 256 * 32) b = 256 * 32;
    return b < 1 ? 1 : b;
}

int64_t long_row_slots(int64_t nnz) { return nnz / (kLongRow + 1); }
int64_t symmetry_slots(int64_t nnz) { return nnz / kSymEntries; }

hipError_t launch_prep(const PrepBuffers &B, hipStream_t s)
{
    const IngestShape sh{(uint32_t)B.n, (uint32_t)B.n_cols, B.bipartite ? 1 : 0};
    const int32_t lg = bucket_lg(B.n, B.nnz);
    const int32_t nb = (int32_t)bucket_count(B.n, B.nnz);
    const size_t lds = sizeof(int32_t) * (size_t)nb;
    const int64_t tiles = (B.nnz + kTile - 1) / kTile;
    const int64_t heavy = heavy_chunks(B.nnz) < 1024 ? heavy_chunks(B.nnz) : 1024;
    // the bucket counters, the scalars and, for heavy buckets, the rows' counts start
    // at zero (the cursors at the scan); they lie one after the other
    char *const zero_end = heavy ? reinterpret_cast<char *>(B.lstart + B.n) : reinterpret_cast<char *>(B.scalars + 1);
    hipError_t e = launch_zero_u64(reinterpret_cast<unsigned long long *>(B.bucket_n),
                                   (zero_end - reinterpret_cast<char *>(B.bucket_n) + 7) / 8, s);
    if (e != hipSuccess) return e;
    if (tiles > 0) {
        // every block adds its counters to all buckets' once: two rounds of blocks
        const int64_t g = tiles < 1024 ? (tiles + kSubs - 1) / kSubs * kSubs : 1024;
        hipLaunchKernelGGL(k_check, dim3((unsigned)g), dim3(kTileThreads), lds, s, B.rows, B.cols, B.vals, B.nnz, sh, lg,
                           nb, B.bucket_n, B.scalars);
    }
    hipLaunchKernelGGL(k_bucket_starts, dim3(1), dim3(kTileThreads), 0, s, B.bucket_n, nb, B.first, B.cursor,
                       B.heavy_first, B.scalars);
    if (tiles > 0)
        hipLaunchKernelGGL(k_bucket_scatter, dim3((unsigned)tiles), dim3(kTileThreads), lds, s, B.rows, B.cols, B.vals,
                           B.nnz, sh, lg, nb, B.cursor, B.pair, B.lrow);
    // (the rows' cursors of heavy buckets: rp32, which the row sort writes)
    if (heavy)
        hipLaunchKernelGGL((k_heavy_rows<false>), dim3((unsigned)heavy), dim3(kTileThreads), 0, s, B.pair, B.lrow, B.first,
                           B.heavy_first, B.n, lg, nb, B.n_epochs, B.scalars, B.lstart, B.pair_rows);
    hipLaunchKernelGGL(k_bucket_rows, dim3((unsigned)nb), dim3(kTileThreads), 0, s, B.pair, B.lrow, B.first, B.n, lg,
                       B.n_epochs, B.scalars, B.pair_rows, B.lstart, B.rp32, B.kept_n);
    if (heavy)
        hipLaunchKernelGGL((k_heavy_rows<true>), dim3((unsigned)heavy), dim3(kTileThreads), 0, s, B.pair, B.lrow, B.first,
                           B.heavy_first, B.n, lg, nb, B.n_epochs, B.scalars, B.rp32, B.pair_rows);
    hipLaunchKernelGGL(k_kept_starts, dim3(1), dim3(kTileThreads), 0, s, B.kept_n, nb, B.kfirst);
    const SortedRows out{B.col, B.eps, B.pair, B.col16};
    const int32_t per_block = sort_rows(B.n, B.nnz);
    const int64_t blocks = row_blocks(B.n, B.nnz);
    const Grid2 rg = grid2(blocks, 256);
    auto *const sort = per_block == kSortRows ? k_row_sort<kSortRows> : k_row_sort<kSortRowsDense>;
    hipLaunchKernelGGL(sort, dim3(rg.x, rg.y), dim3(256), 0, s, B.pair_rows, B.first, B.kfirst, B.lstart, B.n, lg,
                       B.scalars, B.row_ptr, B.rp32, B.long_rows, B.block_near, B.block_max, B.sym_list, out);
    const int64_t max_long = long_row_slots(B.nnz);
    if (max_long > 0) {
        int32_t passes = 0;   // 4-bit digits of the largest column, rounded up to an even count
        for (int64_t top = B.n_cols - 1; top > 0; top >>= 4) ++passes;
        passes += passes & 1;
        hipLaunchKernelGGL(k_long_row_sort, dim3((unsigned)(max_long < 512 ? max_long : 512)), dim3(kSortThreads), 0, s,
                           B.pair_rows, B.first, B.kfirst, B.lstart, B.n, lg, passes, B.long_rows, B.scalars, out);
    }
    if (!B.bipartite) {
        const int64_t more = symmetry_slots(B.nnz) < 1024 ? symmetry_slots(B.nnz) : 1024;
        const Grid2 sg = grid2(blocks + more, 256);
        hipLaunchKernelGGL(k_symmetry, dim3(sg.x, sg.y), dim3(256), 0, s, B.pair, B.col, B.rp32, B.n, per_block,
                           blocks, (int32_t)more, B.sym_list, B.scalars, B.block_diff);
    }
    const int64_t g = (blocks + 1023) / 1024;
    hipLaunchKernelGGL(k_prep_sums, dim3((unsigned)(g < 64 ? g : 64)), dim3(256), 0, s, B.block_max, B.block_near,
                       B.bipartite ? nullptr : B.block_diff, blocks, B.scalars);
    return hipGetLastError();
}

// part[w] = first row r with row_ptr[r] + wgt * r >= w * cost, for
// w < n_waves; part[n_waves] = n.  A wave then holds at most
// cost / wgt + 1 <= rows_cap(dim) rows (cost rises by >= wgt per row) and
// about cost edges unless its last row alone is longer.
// Waves over rows [r0, r1): part[w] is the first row r >= r0 whose units
// (edges and row weights from r0 up to r) reach w x cost; part[n_waves] = r1.
__global__ void k_partition(const int64_t *__restrict__ row_ptr, int64_t r0, int64_t r1, int32_t wgt, int64_t cost,
                            int32_t *__restrict__ part, int64_t n_waves)
{
    const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w > n_waves) return;
    if (w == n_waves) {
        part[w] = (int32_t)r1;
        return;
    }
    const int64_t target = row_ptr[r0] + (int64_t)wgt * r0 + w * cost;
    int64_t lo = r0, hi = r1;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (row_ptr[mid] + (int64_t)wgt * mid >= target) hi = mid; else lo = mid + 1;
    }
    part[w] = (int32_t)lo;
}

// head[e] = row of edge e minus the first row of its wave (< rows_cap <= 256).
// One thread per row of [r0, r1): its wave is the last w with part[w] <= row.
__global__ void k_head_local(const int64_t *__restrict__ row_ptr, int64_t r0, int64_t r1,
                             const int32_t *__restrict__ part, int64_t n_waves, WaveDesc *__restrict__ desc,
                             uint8_t *__restrict__ head)
{
    const int64_t w0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w0 < n_waves) {
        const int32_t a = part[w0], b = part[w0 + 1];
        const int64_t ea = row_ptr[a], eb = row_ptr[b];
        desc[w0] = WaveDesc{a, b - a, (int32_t)ea, (int32_t)(eb - ea)};
    }
    const int64_t r = r0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= r1) return;
    int64_t lo = 0, hi = n_waves - 1;
    while (lo < hi) {
        int64_t mid = (lo + hi + 1) >> 1;
        if (part[mid] <= r) lo = mid; else hi = mid - 1;
    }
    const uint8_t h = (uint8_t)(r - part[lo]);
    for (int64_t e = row_ptr[r]; e < row_ptr[r + 1]; ++e) head[e] = h;
}

hipError_t launch_partition(const int64_t *row_ptr, int64_t r0, int64_t r1, int32_t dim, int64_t cost,
                            int32_t *part, WaveDesc *desc, int64_t n_waves, uint8_t *head, hipStream_t s)
{
    if (cost < 1 || cost > kWaveCost || r0 < 0 || r1 <= r0 || n_waves < 1) return hipErrorInvalidValue;
    static_assert(rows_cap(1) <= 256 && rows_cap(16) <= 256, "head offsets must fit in a byte");
    int64_t blocks = (n_waves + 1 + 255) / 256;
    hipLaunchKernelGGL(k_partition, dim3((unsigned)blocks), dim3(256), 0, s, row_ptr, r0, r1, row_weight(dim), cost,
                       part, n_waves);
    const int64_t threads = r1 - r0 > n_waves ? r1 - r0 : n_waves;
    hipLaunchKernelGGL(k_head_local, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, row_ptr, r0, r1, part,
                       n_waves, desc, head);
    return hipGetLastError();
}

__global__ void k_zero_u64(unsigned long long *p, int64_t count)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += stride) p[t] = 0;
}

hipError_t launch_zero_u64(unsigned long long *p, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_u64, dim3((unsigned)grid_for(count)), dim3(256), 0, s, p, count);
    return hipGetLastError();
}

}  // namespace ul
