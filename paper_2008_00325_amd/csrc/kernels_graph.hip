// kernels_graph.hip -- the input side of the layout: from kNN lists to the
// fuzzy union B (neighbourhood-weighting section, Eq. 1 and Eq. 2), in fp64.
//
//   k_smooth   one thread per vertex: rho_i, then sigma_i by bisection on
//              sum_j exp(-(d_ij - rho_i)+ / sigma) = log2 k
//   k_union    one lane per kNN entry (i, s): A_ij, the transposed value A_ji
//              where row j lists i, and B_ij = A_ij + A_ji - A_ij A_ji
//
// A row without a positive distance has memberships of 1 whatever its sigma
// (every (d_ij - rho_i)+ is 0), so its floor, 1e-3 of the mean distance of all
// rows, is never computed.
#include "internal.hpp"

namespace ul {

__device__ __forceinline__ double membership(double dist, double2 rs)
{
    double x = dist - rs.x;
    return exp(-(x > 0.0 ? x : 0.0) / rs.y);
}

// Rows of a block (one wavefront) of k_smooth, and the longest rows whose
// distances it keeps in registers and LDS; longer ones are read from memory.
constexpr int kSmoothRows = 64;
constexpr int kSmoothRegs = 64;

// sigma of one row.  The path of the fp64 bisection (start 1, doubled while
// unbounded, at most 64 steps, stop within 1e-5 of the target) is followed
// exactly, but most of its steps are decided without fp64 exponentials, which
// bound the kernel (1M rows of 15: 753 us with k fp64 exponentials and
// divisions in each of ~20 steps, now 100 us; 2,000 rows 73 -> 14 us):
//  * while the fp32 sum is further from the target than 1e-5 plus a bound of
//    its error, it decides.  Error: a term's argument carries four fp32
//    roundings and the hardware reciprocal's ulp (3.6e-7 relative, 0.37 of that
//    in the term at most) and the hardware exponential one ulp or so, below
//    4e-7 together, and each of the sum's k additions 6e-8 of the sum; the
//    bound takes at least twice the former and four times the latter.
//  * from there one fp64 evaluation gives f, f' and f'' at a step, and the steps
//    after it are decided by the parabola where its error bound allows:
//    |f'''| <= 1.01 k / s^3, so |error| <= 0.17 k (ds / s)^3, taken six times.
template <typename F32, typename F64>
__device__ __forceinline__ double bisect_sigma(int32_t k, F32 sum32, F64 eval64)
{
    const double target = log2((double)k);
    double lo = 0.0, hi = INFINITY, s = 1.0;
    auto step = [&](bool above) {
        if (above) hi = s; else lo = s;
        s = isinf(hi) ? 2.0 * s : 0.5 * (lo + hi);
    };
    const float t32 = (float)target, kf = (float)k;
    int it = 0;
    for (; it < 64; ++it) {
        const float f = sum32(1.44269504f * __builtin_amdgcn_rcpf((float)s));
        const float off = f - t32;
        if (!(fabsf(off) > 1.1e-5f + kf * (1e-6f + 2.5e-7f * f) + 1e-6f * t32)) break;
        step(off > 0.0f);
    }
    double sc = 0.0, fc = 0.0, gc = 0.0, hc = 0.0;   // f - target, f' and f'' / 2 at sc (sc = 0: none yet)
    for (; it < 64; ++it) {
        const double ds = s - sc, q = fabs(ds) / (s < sc ? s : sc);
        double off = fc + (gc + hc * ds) * ds;
        const double err = (double)k * (q * q * q) + 1e-10;
        const double mag = fabs(off);
        if (!(sc > 0.0 && (mag + err < 1e-5 || mag - err >= 1e-5))) {
            double f;
            eval64(s, f, gc, hc);
            off = f - target;
            sc = s;
            fc = off;
        }
        if (fabs(off) < 1e-5) break;
        step(off > 0.0);
    }
    return s;
}

// KR: distances per row kept in registers (k <= KR), 0: read from memory.
template <int KR>
__global__ __launch_bounds__(kSmoothRows) void k_smooth(const int32_t *__restrict__ ids, const float *__restrict__ d,
                                                        int64_t n, int32_t k, double2 *__restrict__ rho_sigma,
                                                        unsigned *flags)
{
    __shared__ float s_d[KR > 0 ? kSmoothRows * KR : 1];
    const int lane = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * kSmoothRows;
    const int rows = (int)(n - i0 < kSmoothRows ? n - i0 : kSmoothRows);
    const float *const db = d + i0 * k;
    const int32_t *const ib = ids + i0 * k;
    // the block's entries in order, coalesced: checks, and the distances to LDS
    unsigned bad = 0;
    if constexpr (KR > 0) {
        // k loads of each per lane, all in flight (one after the other cost a
        // block about 12 us)
        const uint32_t total = (uint32_t)(rows * k);
        float v[KR];
        int32_t id[KR];
#pragma unroll
        for (int q = 0; q < KR; ++q) {
            const uint32_t t = (uint32_t)(q * kSmoothRows + lane);
            v[q] = 0.0f;
            id[q] = 0;
            if (t < total) {
                v[q] = at32(db, t);
                id[q] = at32(ib, t);
            }
        }
#pragma unroll
        for (int q = 0; q < KR; ++q) {
            const uint32_t t = (uint32_t)(q * kSmoothRows + lane);
            if (!isfinite(v[q])) bad |= kBadValue;
            if ((uint32_t)id[q] >= (uint32_t)n) bad |= kBadIndex;
            if (t < total) s_d[t] = v[q];
        }
    } else {
        for (int64_t t = lane; t < (int64_t)rows * k; t += kSmoothRows) {
            if (!isfinite(db[t])) bad |= kBadValue;
            if ((uint32_t)ib[t] >= (uint32_t)n) bad |= kBadIndex;
        }
    }
    if (bad) atomicOr(flags, bad);
    __syncthreads();
    if (lane >= rows) return;
    const float *const di = KR > 0 ? s_d + lane * k : db + (int64_t)lane * k;
    double r = 0.0, sum = 0.0;
    bool found = false;
#pragma unroll 4
    for (int32_t j = 0; j < k; ++j) {
        const double dj = (double)di[j];
        sum += dj;
        if (dj > 0.0 && (!found || dj < r)) {
            r = dj;
            found = true;
        }
    }
    const float rf = (float)r;   // a distance: exact
    auto eval64 = [&](double s, double &f, double &g, double &h) {
        double su = 0.0, suu = 0.0;   // sums of u e^-u and u^2 e^-u, u = x / s
        f = 0.0;
#pragma unroll 4
        for (int32_t j = 0; j < k; ++j) {
            const double x = (double)di[j] - r;
            const double u = x > 0.0 ? x / s : 0.0;
            const double e = exp(-u);
            f += e;
            su += u * e;
            suu += u * u * e;
        }
        g = su / s;
        h = 0.5 * (suu - 2.0 * su) / (s * s);
    };
    double s;
    if constexpr (KR > 0) {
        float x[KR];
#pragma unroll
        for (int j = 0; j < KR; ++j) x[j] = j < k ? fmaxf(di[j] - rf, 0.0f) : INFINITY;   // exp2(-inf) = 0
        s = bisect_sigma(k, [&](float c) {
            float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < KR; ++j) a[j & 3] += __builtin_amdgcn_exp2f(-x[j] * c);
            return (a[0] + a[1]) + (a[2] + a[3]);
        }, eval64);
    } else {
        s = bisect_sigma(k, [&](float c) {
            float a = 0.0f;
            for (int32_t j = 0; j < k; ++j) a += __builtin_amdgcn_exp2f(-fmaxf(di[j] - rf, 0.0f) * c);
            return a;
        }, eval64);
    }
    const double floor_v = found ? 1e-3 * (sum / (double)k) : 0.0;
    rho_sigma[i0 + lane] = make_double2(r, s < floor_v ? floor_v : s);
}

// One lane per entry, 64 consecutive entries per wave.  Whether row j lists i
// is looked up by G lanes together, one id each, 64 / G rows per load: a row
// of 15 ids is one or two 128-byte lines, and these random lines bound the
// kernel on a shuffled graph.  (One lane reading its row id by id asked the
// L2 for the same lines k times, because the rows of the resident waves do not
// fit L1: 1M rows of 15 shuffled, 1808 us, now 494.)  kAhead loads are in
// flight at a time.
template <int G>
__global__ __launch_bounds__(256) void k_union(const int32_t *__restrict__ ids, const float *__restrict__ d, int64_t n,
                                               int32_t k, const double2 *__restrict__ rho_sigma,
                                               int32_t *__restrict__ rows, int32_t *__restrict__ cols,
                                               float *__restrict__ vals)
{
    constexpr int kRows = kWave / G;              // rows looked up per load
    constexpr int kAhead = G < 8 ? G : 8;
    const uint32_t nk = (uint32_t)(n * k);        // < 2^30
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    const int lane = (int)(threadIdx.x % kWave);
    const bool in = t < nk;
    const int32_t i = (int32_t)((in ? t : 0u) / (uint32_t)k);
    const int32_t j = in ? ids[t] : -1;
    const bool valid = (uint32_t)j < (uint32_t)n && j != i;
    const int32_t jv = valid ? j : -1;
    // entry e of the wave is looked up in step e / kRows by the lanes of group
    // e % kRows; the last match counts
    const int group = lane / G, part = lane % G;
    const int my_step = lane / kRows, my_group = lane % kRows;
    int32_t pos = -1;
    for (int32_t c0 = 0; c0 < k; c0 += G) {
        unsigned long long hit = 0;
#pragma unroll
        for (int s0 = 0; s0 < G; s0 += kAhead) {
            int32_t v[kAhead], want[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int e = (s0 + u) * kRows + group;
                const int32_t je = __shfl(jv, e);
                want[u] = __shfl(i, e);
                v[u] = -1;
                if (je >= 0 && c0 + part < k) v[u] = at32(ids, (uint32_t)je * (uint32_t)k + (uint32_t)(c0 + part));
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const unsigned long long m = __ballot(v[u] == want[u]);   // v = -1 never is one
                if (s0 + u == my_step) hit = m;
            }
        }
        const unsigned long long own = G == 64 ? hit : (hit >> (my_group * G)) & ((1ull << (G & 63)) - 1ull);
        if (own) pos = c0 + 63 - __builtin_clzll(own);
    }
    if (!in) return;
    float b = 0.0f;
    const bool mutual = valid && pos >= 0;
    if (valid) {
        const double aij = membership((double)d[t], rho_sigma[i]);
        double aji = 0.0;
        if (mutual) aji = membership((double)at32(d, (uint32_t)j * (uint32_t)k + (uint32_t)pos), rho_sigma[j]);
        b = (float)(aij + aji - aij * aji);
    }
    rows[t] = i;
    cols[t] = j;
    vals[t] = b;
    // the reverse orientation, unless row j lists i itself
    rows[nk + t] = mutual ? i : j;
    cols[nk + t] = i;
    vals[nk + t] = mutual ? 0.0f : b;
}

hipError_t launch_fuzzy_graph(int64_t n, int32_t k, const int32_t *ids, const float *dists, int32_t *rows,
                              int32_t *cols, float *vals, double2 *rho_sigma, unsigned *flags, hipStream_t s)
{
    const dim3 sg((unsigned)((n + kSmoothRows - 1) / kSmoothRows));
    if (k <= 8)
        hipLaunchKernelGGL((k_smooth<8>), sg, dim3(kSmoothRows), 0, s, ids, dists, n, k, rho_sigma, flags);
    else if (k <= 16)
        hipLaunchKernelGGL((k_smooth<16>), sg, dim3(kSmoothRows), 0, s, ids, dists, n, k, rho_sigma, flags);
    else if (k <= 32)
        hipLaunchKernelGGL((k_smooth<32>), sg, dim3(kSmoothRows), 0, s, ids, dists, n, k, rho_sigma, flags);
    else if (k <= kSmoothRegs)
        hipLaunchKernelGGL((k_smooth<kSmoothRegs>), sg, dim3(kSmoothRows), 0, s, ids, dists, n, k, rho_sigma, flags);
    else
        hipLaunchKernelGGL((k_smooth<0>), sg, dim3(kSmoothRows), 0, s, ids, dists, n, k, rho_sigma, flags);
    const dim3 ug((unsigned)((n * k + 255) / 256));
    if (k <= 8)
        hipLaunchKernelGGL((k_union<8>), ug, dim3(256), 0, s, ids, dists, n, k, rho_sigma, rows, cols, vals);
    else if (k <= 16)
        hipLaunchKernelGGL((k_union<16>), ug, dim3(256), 0, s, ids, dists, n, k, rho_sigma, rows, cols, vals);
    else if (k <= 32)
        hipLaunchKernelGGL((k_union<32>), ug, dim3(256), 0, s, ids, dists, n, k, rho_sigma, rows, cols, vals);
    else
        hipLaunchKernelGGL((k_union<64>), ug, dim3(256), 0, s, ids, dists, n, k, rho_sigma, rows, cols, vals);
    return hipGetLastError();
}

}  // namespace ul
