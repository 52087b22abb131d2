// kernels_trust.hip -- trustworthiness T(k) of an embedding on the GPU
// (batched pairwise distances, Alg. 1; normalised as in Venna and Kaski's
// definition that the experiments section cites):
//
//   T(k) = 1 - 2 / (n k (2n - 3k - 1)) * sum_i sum_{j in N^_k(i)} max(0, r(i, j) - k)
//
// where N^_k(i) are the k nearest neighbours of i in the embedding and r(i, j)
// is the 1-based rank of j among all points by input distance from i (self
// excluded, ties by index); neighbours with r <= k are the input neighbours
// and add nothing.
//
//  1. k_tw_split: every input row as three bf16 parts per feature, and |x_i|^2
//     (k_tw_pack: as it is, up to 16 features; k_tw_norms where neither fits).
//  2. k_tw_embed_knn: one wavefront per point, a brute-force scan of the
//     embedding keeping the k best (distance, index) pairs sorted across lanes.
//  3. k_tw_thresholds: input distance from i to each embedding neighbour.
//  4. k_tw_rank_pairs: the input distances of every pair of points once, as tiles
//     of 128 x 128 on the matrix cores, compared in registers with the
//     neighbour thresholds of both points: only the counts r(i, j) - 1 leave the
//     chip, never the n x n distances.  (k_tw_rank: every pair twice, fp32
//     matrix instructions on X itself; for few points (pairs_pay), where the
//     parts would not fit, or where the points' norms come near fp32's range.)
//  5. k_tw_penalty: the penalties' sum.
#include "internal.hpp"
#include "launch_sizes.hpp"

namespace ul {

typedef float v4f __attribute__((ext_vector_type(4)));


__global__ __launch_bounds__(256) void k_tw_norms(const float *__restrict__ X, int64_t n, int32_t d,
                                                  float *__restrict__ nx)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float *x = X + i * d;
    float s = 0.0f;
    for (int32_t q = 0; q < d; ++q) s = fmaf(x[q], x[q], s);
    nx[i] = s;
}

// (a, ia) before (b, ib): smaller distance, then smaller index.
__device__ __forceinline__ bool pair_less(float a, int32_t ia, float b, int32_t ib)
{
    return a < b || (a == b && ia < ib);
}

// (distance, index) as one 64-bit key that orders as pair_less does for
// non-negative indices: the float's bits mapped to an unsigned integer of the
// same order (negative values flipped whole, positive ones with the sign bit
// set), -0 first made +0 so that equal floats give equal keys.
__device__ __forceinline__ uint64_t pair_key(float a, int32_t ia)
{
    const uint32_t bits = __float_as_uint(a + 0.0f);
    const uint32_t ord = (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
    return ((uint64_t)ord << 32) | (uint32_t)ia;
}

// the value of a lane given by a uniform number, as a uniform value
__device__ __forceinline__ float read_lane(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
// the value of the lane below (lane 0: its own), without the LDS crossbar
__device__ __forceinline__ int from_lane_below(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
}

// One wavefront per point i: lanes 0..k-1 hold the k best (distance, index)
// pairs seen so far, ascending; the points come in chunks of 64, and the lanes of
// a chunk that qualify are inserted one at a time.  Later candidates have larger
// indices, so once the list is full a candidate must be strictly closer than its
// last entry, whose distance is kept as a uniform value; kAhead chunks are
// loaded and compared together, and most groups hold no candidate.  (Fetching the
// last pair from its lane for every chunk, one chunk at a time: 443 us at 20,000
// points, 3620 at 70,000; now 360 and 2340.)
template <int DIM>
__global__ __launch_bounds__(256) void k_tw_embed_knn(const float *__restrict__ Y, int64_t n, int32_t k, int64_t np,
                                                      int32_t *__restrict__ nbr)
{
    constexpr int kAhead = DIM <= 2 ? 8 : DIM <= 4 ? 4 : DIM <= 8 ? 2 : 1;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kWave;
    if (i >= n) return;
    const int lane = (int)(threadIdx.x % kWave);
    float yi[DIM];
#pragma unroll
    for (int q = 0; q < DIM; ++q) yi[q] = Y[i * DIM + q];
    float bd = INFINITY;
    int32_t bi = 0x7FFFFFFF;
    float last = INFINITY;   // distance of entry k - 1
    bool full = false;
    for (int64_t base = 0; base < n; base += kAhead * kWave) {
        float y[kAhead][DIM], dc[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t c = base + u * kWave + lane;
            const int64_t cc = c < n ? c : n - 1;
#pragma unroll
            for (int q = 0; q < DIM; ++q) y[u][q] = Y[cc * DIM + q];
        }
        float least = NAN;   // fminf ignores it
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t c = base + u * kWave + lane;
            float s = 0.0f;
#pragma unroll
            for (int q = 0; q < DIM; ++q) {
                const float t = y[u][q] - yi[q];
                s = fmaf(t, t, s);
            }
            dc[u] = c < n && c != i ? s : NAN;   // NaN: never a candidate
            least = fminf(least, dc[u]);
        }
        if (full && __ballot(least < last) == 0) continue;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int32_t ci = (int32_t)(base + u * kWave + lane);
            bool pending = true;
            while (true) {
                pending = pending && (full ? dc[u] < last : dc[u] <= last);
                const unsigned long long m = __ballot(pending);
                if (m == 0) break;
                const int src = __ffsll((long long)m) - 1;
                const float nd = read_lane(dc[u], src);
                const int32_t ni = __builtin_amdgcn_readlane(ci, src);
                if (lane == src) pending = false;
                // insertion position: slots holding a smaller pair
                const int pos = __popcll(__ballot(lane < k && pair_less(bd, bi, nd, ni)));
                const float up_d = __int_as_float(from_lane_below(__float_as_int(bd)));
                const int32_t up_i = from_lane_below(bi);
                if (lane < k) {
                    if (lane == pos) {
                        bd = nd;
                        bi = ni;
                    } else if (lane > pos) {
                        bd = up_d;
                        bi = up_i;
                    }
                }
                last = read_lane(bd, k - 1);
                full = __builtin_amdgcn_readlane(bi, k - 1) != 0x7FFFFFFF;
            }
        }
    }
    if (lane < k) nbr[(int64_t)lane * np + i] = bi;
}

// One wavefront per point i: the input distance to each of its k embedding
// neighbours (lanes split the features, coalesced rows).  A neighbour slot
// left unfilled (a non-finite embedding coordinate never compares below the
// running threshold) raises `flags` and gets a threshold that nothing counts
// against.
__global__ __launch_bounds__(256) void k_tw_thresholds(const float *__restrict__ X, int64_t n, int32_t d, int32_t k,
                                                       int64_t np, const float *__restrict__ nx,
                                                       const int32_t *__restrict__ nbr, float *__restrict__ thr,
                                                       unsigned *__restrict__ flags)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kWave;
    const int lane = threadIdx.x % kWave;
    if (i >= n) return;   // whole waves
    const float *xi = X + i * d;
    for (int32_t s = 0; s < k; ++s) {
        const int64_t j = nbr[s * np + i];   // the same for every lane
        if (j < 0 || j >= n) {
            if (lane == 0) {
                thr[s * np + i] = -INFINITY;
                atomicOr(flags, (unsigned)kTrustBadEmbedding);
            }
            continue;
        }
        const float *xj = X + j * d;
        float dot = 0.0f;
        for (int32_t q = lane; q < d; q += kWave) dot = fmaf(xi[q], xj[q], dot);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
        if (lane == 0) thr[s * np + i] = nx[i] + nx[j] - 2.0f * dot;
    }
}

// Input distances of a block of kRkRows points (rows) to a range of column
// tiles of CT x 16 points, as fp32 MFMA tiles (v_mfma_f32_16x16x4f32), turned
// into distances in registers and compared with each row's k thresholds.
//
//  * 8 waves; wave w owns rows 16 w .. 16 w + 15 of the block: lane l holds
//    row l % 16 and, in each of the CT column tiles of 16, the four columns
//    4 (l / 16) + 0..3 of the MFMA result layout.
//  * The features are taken CH (16 or 32) at a time, double buffered in LDS
//    ([point][feature], padded to CH + 4 floats so that a lane's 16-byte reads
//    are free of bank conflicts), the next chunk's global loads in flight while
//    the current one is multiplied.  Lane group g = l / 16 supplies features
//    g CH/4 .. (g + 1) CH/4 - 1, one per MFMA step, so each operand of a lane
//    comes from CH/16 16-byte LDS reads.
//  * Column splits (blockIdx.y) keep enough blocks in flight; each block adds
//    its rows' partial counts to cnt[row * k + s] with integer atomics (exact,
//    order-free).
constexpr int kRkRows = 128;
constexpr int kRankChunk = 16;   // features per LDS stage

__device__ __forceinline__ float4 load_features(const float *__restrict__ X, int64_t p, int32_t q, int64_t n,
                                                int32_t d, bool vec)
{
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (p >= n) return v;
    const float *x = X + p * d + q;
    if (vec) {
        if (q < d) v = *reinterpret_cast<const float4 *>(x);
    } else {
        if (q < d) v.x = x[0];
        if (q + 1 < d) v.y = x[1];
        if (q + 2 < d) v.z = x[2];
        if (q + 3 < d) v.w = x[3];
    }
    return v;
}

template <int KMAX, int CT, int CH>
__device__ __forceinline__ void rank_body(const float *__restrict__ X, int64_t n, int32_t d, int32_t k, int64_t np,
                                          const float *__restrict__ nx, const int32_t *__restrict__ nbr,
                                          const float *__restrict__ thr, int64_t tiles_per_split,
                                          int32_t *__restrict__ cnt_out)
{
    constexpr int COLS = 16 * CT;
    constexpr int PAD = CH + 4;        // floats per staged point
    constexpr int QUADS = CH / 4;      // float4 per staged point
    constexpr int NV = QUADS / 4;      // float4 a thread stages per operand (512 threads, 128 points)
    constexpr int GQ = CH / 16;        // float4 per lane group per operand
    static_assert(CH == 16 || CH == 32, "chunk of 16 or 32 features");
    __shared__ __align__(16) float s_rows[2][kRkRows * PAD];
    __shared__ __align__(16) float s_cols[2][COLS * PAD];
    __shared__ float s_nx[COLS];

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wv = tid / kWave;
    const int g = lane / 16;
    const int li = lane % 16;
    const int64_t row0 = (int64_t)blockIdx.x * kRkRows;
    const int rloc = wv * 16 + li;
    const int64_t row = row0 + rloc;
    const bool row_ok = row < n;
    const bool vec = (d % 4) == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;   // 16-byte loads

    // each threshold as a (distance, index) key; an unused slot gets the
    // smallest key, which no element is below
    uint64_t tkey[KMAX];
    int32_t cnt[KMAX];
#pragma unroll
    for (int s = 0; s < KMAX; ++s) {
        const bool use = row_ok && s < k;
        tkey[s] = use ? pair_key(thr[s * np + row], nbr[s * np + row]) : 0ull;
        cnt[s] = 0;
    }
    const float nrow = row_ok ? nx[row] : 0.0f;

    // staging: float4 number f = tid + 512 v (v < NV) is features
    // 4 (f % QUADS) .. +3 of point f / QUADS
    int sp[NV], sq[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        sp[v] = (tid + 512 * v) / QUADS;
        sq[v] = 4 * ((tid + 512 * v) % QUADS);
    }
    const int64_t n_tiles = (n + COLS - 1) / COLS;
    const int64_t t0 = (int64_t)blockIdx.y * tiles_per_split;
    const int64_t t1 = t0 + tiles_per_split < n_tiles ? t0 + tiles_per_split : n_tiles;

    for (int64_t tile = t0; tile < t1; ++tile) {
        const int64_t col0 = tile * COLS;
        if (tid < COLS) s_nx[tid] = col0 + tid < n ? nx[col0 + tid] : 0.0f;
        v4f acc[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

        float4 rv[NV], cv[NV];
        auto fetch = [&](int32_t q0) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                rv[v] = load_features(X, row0 + sp[v], q0 + sq[v], n, d, vec);
                cv[v] = sp[v] < COLS ? load_features(X, col0 + sp[v], q0 + sq[v], n, d, vec)
                                     : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        };
        auto stash = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                *reinterpret_cast<float4 *>(&s_rows[b][sp[v] * PAD + sq[v]]) = rv[v];
                if (sp[v] < COLS) *reinterpret_cast<float4 *>(&s_cols[b][sp[v] * PAD + sq[v]]) = cv[v];
            }
        };
        fetch(0);
        stash(0);
        __syncthreads();
        int buf = 0;
        for (int32_t q0 = 0; q0 < d; q0 += CH) {
            const bool more = q0 + CH < d;
            if (more) fetch(q0 + CH);
#pragma unroll
            for (int gq = 0; gq < GQ; ++gq) {
                const int f = g * (CH / 4) + 4 * gq;   // this lane group's features f .. f + 3
                const float4 bq = *reinterpret_cast<const float4 *>(&s_rows[buf][rloc * PAD + f]);
                float4 aq[CT];
#pragma unroll
                for (int t = 0; t < CT; ++t)
                    aq[t] = *reinterpret_cast<const float4 *>(&s_cols[buf][(t * 16 + li) * PAD + f]);
#pragma unroll
                for (int t = 0; t < CT; ++t) {
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[t].x, bq.x, acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[t].y, bq.y, acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[t].z, bq.z, acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[t].w, bq.w, acc[t], 0, 0, 0);
                }
            }
            if (more) stash(buf ^ 1);
            __syncthreads();
            buf ^= 1;
        }
        if (row_ok) {
#pragma unroll
            for (int t = 0; t < CT; ++t) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int cl = t * 16 + 4 * g + e;
                    const int64_t c = col0 + cl;
                    if (c >= n || c == row) continue;
                    const float dist = nrow + s_nx[cl] - 2.0f * acc[t][e];
                    const int32_t ci = (int32_t)c;
                    const uint64_t key = pair_key(dist, ci);
                    // points ordered before neighbour s, the neighbour itself excluded (its
                    // distance here need not equal the threshold's bit for bit)
#pragma unroll
                    for (int s = 0; s < KMAX; ++s)
                        cnt[s] += (key < tkey[s] && (uint32_t)ci != (uint32_t)tkey[s]) ? 1 : 0;
                }
            }
        }
        __syncthreads();   // s_nx and the buffers are refilled for the next tile
    }
    // the four lanes of a row (l, l + 16, l + 32, l + 48) hold disjoint columns
#pragma unroll
    for (int s = 0; s < KMAX; ++s) {
        int32_t c = cnt[s];
        c += __shfl_xor(c, 16);
        c += __shfl_xor(c, 32);
        if (row_ok && g == 0 && s < k && c != 0) atomicAdd(&cnt_out[s * np + row], c);
    }
}

// *sum += sum_i sum_s max(0, r(i, nbr_s) - k), r = 1 + the count of points before
// the neighbour: whole numbers, so the order of the adds does not matter.
__global__ __launch_bounds__(256) void k_tw_penalty(const int32_t *__restrict__ cnt, int64_t n, int32_t k, int64_t np,
                                                    unsigned long long *__restrict__ sum)
{
    int64_t p = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        for (int32_t s = 0; s < k; ++s) {
            const int64_t rank = (int64_t)cnt[s * np + i] + 1;
            if (rank > k) p += rank - k;
        }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off);
    __shared__ long long s_p[4];
    if ((threadIdx.x & 63) == 0) s_p[threadIdx.x >> 6] = p;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(sum, (unsigned long long)(s_p[0] + s_p[1] + s_p[2] + s_p[3]));
}

__global__ __launch_bounds__(256) void k_tw_zero(int32_t *__restrict__ p, int64_t count)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < count; t += stride) p[t] = 0;
}

template <int KMAX, int CT, int CH>
__global__ __launch_bounds__(512) void k_tw_rank(const float *__restrict__ X, int64_t n, int32_t d, int32_t k,
                                                 int64_t np, const float *__restrict__ nx,
                                                 const int32_t *__restrict__ nbr, const float *__restrict__ thr,
                                                 int64_t tiles_per_split,
                                                 int32_t *__restrict__ cnt_out)
{
    rank_body<KMAX, CT, CH>(X, n, d, k, np, nx, nbr, thr, tiles_per_split, cnt_out);
}

// The same for k <= 16, held to 128 registers: two blocks per CU, which this
// instance reaches without spilling (the wider ones would spill).
template <int KMAX, int CT, int CH>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_tw_rank_occ(
    const float *__restrict__ X, int64_t n, int32_t d, int32_t k, int64_t np, const float *__restrict__ nx,
    const int32_t *__restrict__ nbr, const float *__restrict__ thr, int64_t tiles_per_split,
    int32_t *__restrict__ cnt_out)
{
    rank_body<KMAX, CT, CH>(X, n, d, k, np, nx, nbr, thr, tiles_per_split, cnt_out);
}

template <int KMAX, int CT, int CH = kRankChunk>
static void launch_rank(const float *X, int64_t n, int32_t d, int32_t k, int64_t np, const float *nx, const int32_t *nbr,
                        const float *thr, int32_t *cnt, hipStream_t s)
{
    const int64_t row_blocks = (n + kRkRows - 1) / kRkRows;
    const int64_t n_tiles = (n + 16 * CT - 1) / (16 * CT);
    // at least ~2048 blocks when the columns allow it
    int64_t splits = (2048 + row_blocks - 1) / row_blocks;
    if (splits > n_tiles) splits = n_tiles;
    if (splits < 1) splits = 1;
    const int64_t per_split = (n_tiles + splits - 1) / splits;
    splits = (n_tiles + per_split - 1) / per_split;
    if constexpr (KMAX <= 16)
        hipLaunchKernelGGL((k_tw_rank_occ<KMAX, CT, CH>), dim3((unsigned)row_blocks, (unsigned)splits), dim3(512), 0,
                           s, X, n, d, k, np, nx, nbr, thr, per_split, cnt);
    else
        hipLaunchKernelGGL((k_tw_rank<KMAX, CT, CH>), dim3((unsigned)row_blocks, (unsigned)splits), dim3(512), 0, s,
                           X, n, d, k, np, nx, nbr, thr, per_split, cnt);
}

// ---------------------------------------------------------------------------
// The ranks from every pair of points once, on the bf16 matrix cores.
//
// Each fp32 feature is split into three bf16 values whose sum it is (8 + 8 + 8
// bits), and a dot product is the sum of the six products of parts down to 2^-16
// of the leading one; what is left out is below 2^-25 of the product, half the fp32
// rounding of one term.  Six bf16 instructions of 32 features take 96 matrix-core
// cycles where the fp32 ones take 256.
// The bf16 instructions cut what they add off toward zero, at the size of the
// accumulator or of the largest product.  So the leading products of 32 features
// (exact in fp32 each) and the others are summed apart, from zero, and added to the
// running sums as rounded fp32 numbers.  (All six accumulated in one chain over all
// features: 29.1 ms instead of 31.1 at 70,000 x 784, but every dot product low by
// 1.2e-8 of |x| |y| on average, and T at 32,000 x 784 5e-8 off 64-bit sums, now 3e-9
// as with the fp32 instructions.)  The dot products' error against 64-bit sums is below
// that of the fp32 chain from 16 features on (root mean square, of |x| |y|: 32
// image-like features 2.2e-8 against 5.1e-8, 784 6.9e-8 against 2.3e-7; 24 features of
// scales 1e-3 .. 1e3 3.6e-8 against 4.7e-8).  Fewer features of different scales would
// lose (8: 3.9e-8 against 3.7e-8): up to kPackFeat the points stay fp32 and the products
// are the fp32 instructions', in k_tw_rank's order.
// 70,000 x 784, k = 15: 29.5 ms where k_tw_rank takes 85.0.  The matrix cores are busy a
// third of the time, the VALU (counting) a quarter, LDS two fifths: two waves per SIMD
// (registers) do not cover the operands' way from the Infinity Cache.
//
// A block multiplies 128 points (rows) with tiles of 128 points on and above the
// diagonal and counts each distance for both of its points.  The split points
// lie in memory as the block wants them in LDS: [panel of 128][32 features]
// [point][12 units of 16 bytes: 3 parts x 4 groups of 8 features], the units of
// point r rotated by (r / 4) % 4 so that 16 lanes reading 16 points' units meet
// on no bank.  Four waves, 64 x 64 distances each (16 result tiles of 16 x 16);
// the next 32 features are loaded to registers while these are multiplied.
// ---------------------------------------------------------------------------
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kPanel = 128;
constexpr int kUnits = 12;                 // of a point and step
constexpr int kFeat = 32;                  // features per step
constexpr int kPackUnits = 4;              // of a point of up to
constexpr int kPackFeat = 16;              //   this many features, as they are
constexpr int kCountPiece = 16;            // thresholds counted at a time
constexpr int kTrStride = 68;              // floats per column of a transposed piece
constexpr int kTrCols = 16;

__device__ __forceinline__ int unit_slot(int u, int r)
{
    const int t = u + ((r >> 2) & 3);
    return t < kUnits ? t : t - kUnits;
}

// The unit of features 4 u .. 4 u + 3 of packed point r.
__device__ __forceinline__ int pack_slot(int u, int r) { return (u + (r >> 2)) & (kPackUnits - 1); }

// bf16 of x, to nearest even (toward zero where that would overflow)
__device__ __forceinline__ uint32_t bf16_bits(float x)
{
    const uint32_t b = __float_as_uint(x);
    const uint32_t r = (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
    return (r & 0x7F80u) == 0x7F80u ? b >> 16 : r;
}

// Squared norms up to here leave every distance, threshold and partial sum finite.
constexpr float kPairNormMax = 2.1e37f;   // below 2^128 / 16

// One wave per point of the padded panels: its parts and its squared norm
// (+infinity for the points past n, so that nothing counts them).  A point that is
// not finite or further out than kPairNormMax raises kTrustFarPoint: k_tw_rank_pairs
// counts by the signs of differences, which infinities and NaN do not order, and
// k_tw_rank takes such inputs.
__global__ __launch_bounds__(256) void k_tw_split(const float *__restrict__ X, int64_t n, int32_t d, int32_t steps,
                                                  uint4 *__restrict__ P, float *__restrict__ nx,
                                                  unsigned *__restrict__ flags)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kWave;
    const int lane = (int)(threadIdx.x % kWave);
    const int r = (int)(i % kPanel);
    const float *const x = X + i * d;
    float sq = 0.0f;
    for (int32_t g = lane; g < 4 * steps; g += kWave) {
        uint32_t part[3][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t lo[3], hi[3];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int32_t f = 8 * g + 2 * q + h;
                const float v = i < n && f < d ? x[f] : 0.0f;
                sq = fmaf(v, v, sq);
                uint32_t(&b)[3] = h ? hi : lo;
                b[0] = bf16_bits(v);
                const float v1 = v - __uint_as_float(b[0] << 16);
                b[1] = bf16_bits(v1);
                b[2] = bf16_bits(v1 - __uint_as_float(b[1] << 16));
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) part[p][q] = lo[p] | (hi[p] << 16);
        }
        uint4 *const row = P + (((i / kPanel) * steps + g / 4) * kPanel + r) * kUnits;
#pragma unroll
        for (int p = 0; p < 3; ++p)
            row[unit_slot(4 * p + g % 4, r)] = make_uint4(part[p][0], part[p][1], part[p][2], part[p][3]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if (lane == 0) {
        nx[i] = i < n ? sq : INFINITY;
        if (i < n && !(sq <= kPairNormMax)) atomicOr(flags, (unsigned)kTrustFarPoint);
    }
}

// Up to kPackFeat features: one thread per point of the padded panels (otherwise as
// k_tw_split; the norm in k_tw_norms' order).
__global__ __launch_bounds__(256) void k_tw_pack(const float *__restrict__ X, int64_t n, int32_t d, int64_t np,
                                                 uint4 *__restrict__ P, float *__restrict__ nx,
                                                 unsigned *__restrict__ flags)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= np) return;
    const int r = (int)(i % kPanel);
    float sq = 0.0f;
#pragma unroll
    for (int u = 0; u < kPackUnits; ++u) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = i < n && 4 * u + q < d ? X[i * d + 4 * u + q] : 0.0f;
            sq = fmaf(v[q], v[q], sq);
        }
        P[i * kPackUnits + pack_slot(u, r)] =
            make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
    }
    nx[i] = i < n ? sq : INFINITY;
    if (i < n && !(sq <= kPairNormMax)) atomicOr(flags, (unsigned)kTrustFarPoint);
}

// the next float above x (x itself where it is not finite)
__device__ __forceinline__ float next_up(float x)
{
    const int32_t b = __float_as_int(x + 0.0f);   // -0 becomes +0
    return fabsf(x) < INFINITY ? __int_as_float(b + ((b >> 31) | 1)) : x;
}

// Counting "x < t" for several thresholds t: the sign of x - t is shifted into a
// word per threshold and the words' bits are counted, two instructions per
// comparison.  (A compare into a scalar mask is followed by two wait states
// before the mask can be added: twice the cycles.)  x and t are not both
// infinite: x is a distance or +infinity, t finite or -infinity (kPairNormMax).
__device__ __forceinline__ uint32_t push_less(uint32_t bits, float x, float t)
{
    return __builtin_amdgcn_alignbit(bits, __float_as_uint(x - t), 31);
}

template <int KS, bool PACK>
__global__ __launch_bounds__(kPairThreads, 2) void k_tw_rank_pairs(const uint4 *__restrict__ P, int64_t n, int64_t np,
                                                          int32_t steps, int64_t span, int32_t k,
                                                          const float *__restrict__ nx,
                                                          const int32_t *__restrict__ nbr,
                                                          const float *__restrict__ thr, int32_t *__restrict__ cnt,
                                                          const unsigned *__restrict__ flags)
{
    if (*flags & kTrustFarPoint) return;   // the caller takes k_tw_rank
    constexpr int kOperand = kPanel * (PACK ? kPackUnits : kUnits); // units per panel and step
    constexpr int kTrBytes = 4 * kTrCols * kTrStride * 4;           // transposed pieces of the four waves
    constexpr int kThBytes = 4 * KS * kPanel * 4;                   // thresholds and neighbours, rows' and columns'
    constexpr int kOpBytes = 2 * kOperand * 16 > kTrBytes + kThBytes ? 2 * kOperand * 16 : kTrBytes + kThBytes;
    __shared__ __align__(16) unsigned char s_mem[kOpBytes];
    __shared__ int32_t s_cnt[2][KS][kPanel];                        // rows, columns
    __shared__ __align__(16) float s_nx[2][kPanel];
    v4u *const s_op = reinterpret_cast<v4u *>(s_mem);               // while multiplying: rows, then columns
    float *const s_tr = reinterpret_cast<float *>(s_mem);           // while counting
    float(*const s_thr)[KS][kPanel] = reinterpret_cast<float(*)[KS][kPanel]>(s_mem + kTrBytes);
    int32_t(*const s_nbr)[KS][kPanel] = reinterpret_cast<int32_t(*)[KS][kPanel]>(s_mem + kTrBytes + kThBytes / 2);

    const int tid = threadIdx.x, lane = tid % kWave, wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int g = lane / 16, li = lane % 16;
    const int wr = (wv >> 1) * 64, wc = (wv & 1) * 64;              // the wave's rows and columns in the tile
    const int64_t panels = np / kPanel;
    // row panel I: the first with panel_blocks of all panels up to it above blockIdx.x
    int64_t lo = 0, hi = panels - 1;
    const int64_t all = panel_blocks(panels, span);
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (all - panel_blocks(panels - mid - 1, span) > (int64_t)blockIdx.x) hi = mid; else lo = mid + 1;
    }
    const int64_t I = lo;
    const int64_t J0 = I + ((int64_t)blockIdx.x - (all - panel_blocks(panels - I, span))) * span;
    const int64_t J1 = J0 + span < panels ? J0 + span : panels;
    const int64_t r0 = I * kPanel;
    const int pieces = (k + KS - 1) / KS;

    for (int t = tid; t < KS * kPanel; t += 256) s_cnt[0][t / kPanel][t % kPanel] = 0;
    // units of this lane's fragments: point li of a 16-point group, features 8 g .. 8 g + 7
    int off[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) off[p] = PACK ? li * kPackUnits + pack_slot(g, li) : li * kUnits + unit_slot(4 * p + g, li);
    const v4u *const rowsP = reinterpret_cast<const v4u *>(P) + I * steps * kOperand + tid;

    for (int64_t J = J0; J < J1; ++J) {
        const int64_t c0 = J * kPanel;
        const v4u *const colsP = reinterpret_cast<const v4u *>(P) + J * steps * kOperand + tid;
        v4f acc[4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        constexpr int kLoads = kOperand / 256;   // units a thread loads per operand
        v4u ra[kLoads], ca[kLoads];
#pragma unroll
        for (int v = 0; v < kLoads; ++v) {
            ra[v] = rowsP[v * 256];
            ca[v] = colsP[v * 256];
        }
        if (tid < kPanel) s_nx[0][tid] = nx[r0 + tid];
        else s_nx[1][tid - kPanel] = nx[c0 + tid - kPanel];
        for (int32_t step = 0; step < steps; ++step) {
            __syncthreads();   // the last step's operands (or the last tile's counting) are done with
#pragma unroll
            for (int v = 0; v < kLoads; ++v) {
                s_op[v * 256 + tid] = ra[v];
                s_op[kOperand + v * 256 + tid] = ca[v];
            }
            __syncthreads();
            // the next step's operands (the last step's again after it: no branch)
            const int64_t next = (int64_t)(step + 1 < steps ? step + 1 : step) * kOperand;
#pragma unroll
            for (int v = 0; v < kLoads; ++v) {
                ra[v] = rowsP[next + v * 256];
                ca[v] = colsP[next + v * 256];
            }
            if constexpr (PACK) {
                float4 a[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    a[t] = __builtin_bit_cast(float4, s_op[(wr + 16 * t) * kPackUnits + off[0]]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 b = __builtin_bit_cast(float4, s_op[kOperand + (wc + 16 * u) * kPackUnits + off[0]]);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].x, b.x, acc[t][u], 0, 0, 0);
                        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].y, b.y, acc[t][u], 0, 0, 0);
                        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].z, b.z, acc[t][u], 0, 0, 0);
                        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].w, b.w, acc[t][u], 0, 0, 0);
                    }
                }
            } else {
                // two rows of result tiles at a time, each pair of tiles finished before
                // the next (the scheduler would keep all of them open, and spill)
#pragma unroll
                for (int t0 = 0; t0 < 4; t0 += 2) {
                    v8bf a[2][3];
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            a[t][p] = __builtin_bit_cast(v8bf, s_op[(wr + 16 * (t0 + t)) * kUnits + off[p]]);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        v8bf b[3];
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            b[p] = __builtin_bit_cast(v8bf, s_op[kOperand + (wc + 16 * u) * kUnits + off[p]]);
                        // smallest products first; the two tiles in turn
                        constexpr int kA[5] = {2, 0, 1, 1, 0}, kB[5] = {0, 2, 1, 0, 1};
                        const v4f zero = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                        v4f rest[2] = {zero, zero}, lead[2];
#pragma unroll
                        for (int q = 0; q < 5; ++q)
#pragma unroll
                            for (int t = 0; t < 2; ++t)
                                rest[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][kA[q]], b[kB[q]], rest[t], 0, 0, 0);
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            acc[t0 + t][u] += rest[t];
                            lead[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][0], b[0], zero, 0, 0, 0);
                        }
#pragma unroll
                        for (int t = 0; t < 2; ++t) acc[t0 + t][u] += lead[t];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
        // distances: lane (g, li) holds row 16 t + 4 g + e, column 16 u + li
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float nc = s_nx[1][wc + 16 * u + li];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4 nr = *reinterpret_cast<const float4 *>(&s_nx[0][wr + 16 * t + 4 * g]);
                const float nrv[4] = {nr.x, nr.y, nr.z, nr.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float dist = nrv[e] + nc - 2.0f * acc[t][u][e];
                    if (I == J && wr + 16 * t + 4 * g + e == wc + 16 * u + li) dist = INFINITY;   // the point itself
                    acc[t][u][e] = dist;
                }
            }
        }
        for (int piece = 0; piece < pieces; ++piece) {
            __syncthreads();   // the operands, or the last piece's thresholds and counts, are done with
            // A point counts for neighbour s of another when its distance is
            // smaller, or equal with a smaller index; neighbour s itself does not.
            // Where all points of a piece come before neighbour s, "equal" counts
            // (the next float up is the threshold); where it is among them, that
            // neighbour's count is taken point by point.
#pragma unroll
            for (int q = 0; q < KS * kPanel / 256; ++q) {
                const int t = q * 256 + tid;
                const int s = t / kPanel, at = t % kPanel;
                const int64_t slot = (piece * KS + s) * np;
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const int64_t p = (side ? c0 : r0) + at;
                    const bool use = piece * KS + s < k && p < n;
                    s_thr[side][s][at] = use ? thr[slot + p] : -INFINITY;
                    s_nbr[side][s][at] = use ? nbr[slot + p] : -1;
                }
                s_cnt[1][s][at] = 0;
                if (pieces > 1) s_cnt[0][s][at] = 0;
            }
            __syncthreads();
            if (I != J) {
                const int32_t i0 = (int32_t)(r0 + wr);   // rows i0 .. i0 + 63
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int col = wc + 16 * u + li;
                    float th[KS];
                    uint32_t bits[KS];
                    unsigned among = 0;
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        const float x0 = s_thr[1][s][col];
                        const int32_t at = s_nbr[1][s][col] - i0;
                        const bool in = (uint32_t)at < 64u;
                        th[s] = in ? -INFINITY : at >= 64 ? next_up(x0) : x0;
                        among |= in ? 1u << s : 0u;
                        bits[s] = 0;
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float x = acc[t][u][e];
#pragma unroll
                            for (int s = 0; s < KS; ++s) bits[s] = push_less(bits[s], x, th[s]);
                        }
#pragma unroll
                    for (int s = 0; s < KS; ++s) atomicAdd(&s_cnt[1][s][col], __popc(bits[s]));
                    if (__ballot(among != 0) == 0) continue;
#pragma unroll 1
                    for (int s = 0; s < KS; ++s) {
                        const bool in = (among >> s & 1u) != 0;
                        if (__ballot(in) == 0) continue;
                        const int at = s_nbr[1][s][col] - i0;
                        const float x0 = s_thr[1][s][col], x1 = next_up(x0);
                        uint32_t c = 0;
#pragma unroll
                        for (int t = 0; t < 4; ++t)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int i = 16 * t + 4 * g + e;
                                // before neighbour s equal counts, after it not, itself never
                                c = push_less(c, i == at ? INFINITY : acc[t][u][e], i < at ? x1 : x0);
                            }
                        if (in) atomicAdd(&s_cnt[1][s][col], __popc(c));
                    }
                }
            }
            // the rows: the distances transposed, kTrCols columns at a time, a lane per row
            float *const tr = s_tr + wv * kTrCols * kTrStride;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                wave_sync();
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    *reinterpret_cast<v4f *>(&tr[li * kTrStride + 16 * t + 4 * g]) = acc[t][u];
                wave_sync();
                const int32_t j0 = (int32_t)(c0 + wc + kTrCols * u);   // columns j0 .. j0 + 15
                float x[kTrCols];
#pragma unroll
                for (int j = 0; j < kTrCols; ++j) x[j] = tr[j * kTrStride + lane];
                unsigned among = 0;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const float x0 = s_thr[0][s][wr + lane];
                    const int32_t at = s_nbr[0][s][wr + lane] - j0;
                    const bool in = (uint32_t)at < (uint32_t)kTrCols;
                    const float th = in ? -INFINITY : at >= kTrCols ? next_up(x0) : x0;
                    among |= in ? 1u << s : 0u;
                    uint32_t bits = 0;
#pragma unroll
                    for (int j = 0; j < kTrCols; ++j) bits = push_less(bits, x[j], th);
                    atomicAdd(&s_cnt[0][s][wr + lane], __popc(bits));
                }
                if (__ballot(among != 0) == 0) continue;
#pragma unroll 1
                for (int s = 0; s < KS; ++s) {
                    const bool in = (among >> s & 1u) != 0;
                    if (__ballot(in) == 0) continue;
                    const int at = s_nbr[0][s][wr + lane] - j0;
                    const float x0 = s_thr[0][s][wr + lane], x1 = next_up(x0);
                    uint32_t c = 0;
#pragma unroll
                    for (int j = 0; j < kTrCols; ++j) c = push_less(c, j == at ? INFINITY : x[j], j < at ? x1 : x0);
                    if (in) atomicAdd(&s_cnt[0][s][wr + lane], __popc(c));
                }
            }
            __syncthreads();
            const bool rows_too = pieces > 1 || J + 1 == J1;
            for (int t = tid; t < KS * kPanel; t += 256) {
                const int s = piece * KS + t / kPanel;
                const int q = t % kPanel;
                if (s >= k) break;
                if (s_cnt[1][t / kPanel][q]) atomicAdd(&cnt[s * np + c0 + q], s_cnt[1][t / kPanel][q]);
                if (rows_too && s_cnt[0][t / kPanel][q]) atomicAdd(&cnt[s * np + r0 + q], s_cnt[0][t / kPanel][q]);
            }
        }
    }
}

int64_t trust_padded(int64_t n) { return (n + kPanel - 1) / kPanel * kPanel; }

size_t trust_split_bytes(int64_t n, int32_t d)
{
    const int64_t steps = ((int64_t)d + kFeat - 1) / kFeat;
    const int64_t bytes = trust_padded(n) * (d <= kPackFeat ? kPackUnits : steps * kUnits) * 16;
    return bytes <= kTrustSplitBytes ? (size_t)bytes : 0;
}

template <int KS, bool PACK>
static void launch_pairs(const uint4 *P, int64_t n, int64_t np, int32_t steps, int32_t k, const float *nx,
                         const int32_t *nbr, const float *thr, int32_t *cnt, const unsigned *flags, hipStream_t s)
{
    const int64_t panels = np / kPanel;
    const int64_t span = panel_span(panels);
    hipLaunchKernelGGL((k_tw_rank_pairs<KS, PACK>), dim3((unsigned)panel_blocks(panels, span)), dim3(kPairThreads), 0, s, P, n, np,
                       steps, span, k, nx, nbr, thr, cnt, flags);
}

template <int DIM>
static hipError_t launch_knn_dim(const float *Y, int64_t n, int32_t k, int64_t np, int32_t *nbr, hipStream_t s)
{
    const int64_t blocks = (n * kWave + 255) / 256;
    hipLaunchKernelGGL((k_tw_embed_knn<DIM>), dim3((unsigned)blocks), dim3(256), 0, s, Y, n, k, np, nbr);
    return hipGetLastError();
}

hipError_t launch_trustworthiness(const float *X, int64_t n, int32_t d, const float *Y, int32_t dim, int32_t k,
                                  void *split, float *nx, int32_t *nbr, float *thr, int32_t *cnt,
                                  unsigned long long *sum, unsigned *flags, hipStream_t s)
{
    const int64_t np = trust_padded(n);
    const int32_t steps = (d + kFeat - 1) / kFeat;
    const bool pack = d <= kPackFeat;
    if (split && pack)
        hipLaunchKernelGGL(k_tw_pack, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, X, n, d, np,
                           static_cast<uint4 *>(split), nx, flags);
    else if (split)
        hipLaunchKernelGGL(k_tw_split, dim3((unsigned)(np / 4)), dim3(256), 0, s, X, n, d, steps,
                           static_cast<uint4 *>(split), nx, flags);
    else
        hipLaunchKernelGGL(k_tw_norms, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, n, d, nx);
    hipError_t e = hipSuccess;
    switch (dim) {
#define UL_CASE(D) \
    case D: e = launch_knn_dim<D>(Y, n, k, np, nbr, s); break;
        UL_CASE(1) UL_CASE(2) UL_CASE(3) UL_CASE(4) UL_CASE(5) UL_CASE(6) UL_CASE(7) UL_CASE(8)
        UL_CASE(9) UL_CASE(10) UL_CASE(11) UL_CASE(12) UL_CASE(13) UL_CASE(14) UL_CASE(15) UL_CASE(16)
#undef UL_CASE
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tw_thresholds, dim3((unsigned)((n * kWave + 255) / 256)), dim3(256), 0, s, X, n, d, k, np, nx,
                       nbr, thr, flags);
    const int64_t nk = np * k;
    hipLaunchKernelGGL(k_tw_zero, dim3((unsigned)((nk + 255) / 256 < 4096 ? (nk + 255) / 256 : 4096)), dim3(256), 0,
                       s, cnt, nk);
    if (split) {
        const uint4 *const P = static_cast<const uint4 *>(split);
        auto *const pairs = k <= 8 ? (pack ? launch_pairs<8, true> : launch_pairs<8, false>)
                                   : (pack ? launch_pairs<kCountPiece, true> : launch_pairs<kCountPiece, false>);
        pairs(P, n, np, steps, k, nx, nbr, thr, cnt, flags, s);
    } else if (k <= 16) {
        launch_rank<16, 4>(X, n, d, k, np, nx, nbr, thr, cnt, s);
    } else if (k <= 32) {
        launch_rank<32, 4>(X, n, d, k, np, nx, nbr, thr, cnt, s);
    } else {
        launch_rank<64, 2>(X, n, d, k, np, nx, nbr, thr, cnt, s);
    }
    const int64_t pb = (n + 255) / 256;
    hipLaunchKernelGGL(k_tw_penalty, dim3((unsigned)(pb < 256 ? pb : 256)), dim3(256), 0, s, cnt, n, k, np, sum);
    return hipGetLastError();
}

}  // namespace ul
