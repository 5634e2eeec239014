// pn_stats.hip -- the statistics of Sec. V over per-inspiral values on the
// GPU: equal-width and bivariate histograms, the Pearson coefficient, the
// Gaussian kernel density estimator with Silverman's bandwidth, and the
// Kolmogorov-Smirnov statistic against the uniform law.
//
// The number of partial sums of a reduction follows from the sizes of the call
// alone (at most kPart a component, of which the workspaces have room), and they
// are combined in a fixed order, so results do not depend on the device's size or
// on scheduling.  Histogram counts use integer atomics (order-free); the K-S
// statistic is a maximum.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include <rocprim/device/device_radix_sort.hpp>

#include "pn.h"

namespace pn {

int device_ready();   // pn_lib.hip: PN_OK when a gfx950 device is current

namespace {

constexpr int kBlock = 256;
constexpr int kPart = 512;          // most partial results per component
constexpr int kMaxComp = 16;

// ---------------------------------------------------------------------------
// histograms
// ---------------------------------------------------------------------------

// lo + k*step as a rounded product and then a rounded sum (contraction into
// a fused multiply-add is switched off here)
__device__ __forceinline__ double affine(double k, double step, double lo) {
#pragma clang fp contract(off)
    return k * step + lo;
}

// bin edge e_b = lo + b*step, e_nbins = hi
__device__ __forceinline__ double edge(int b, int nbins, double lo, double hi, double step) {
    return b == nbins ? hi : affine((double)b, step, lo);
}

// The bin of lo <= v <= hi: an estimate from the quotient (by the reciprocal
// istep of the bin width), corrected against the edges themselves where the
// quotient lies within 2^-10 of an integer.  That is enough while the
// rounding of the quotient and of the edges is below 2^-10 of a bin (near,
// from hist_near); otherwise every value is corrected.  (Correcting every
// value costs 240 instructions a pair of bins instead of about 35.)
__device__ __forceinline__ int bin_of(double v, int nbins, double lo, double hi, double step, double istep, bool near) {
    const double t = (v - lo) * istep;
    int b = (int)t;
    const double f = t - (double)b;
    if (near && f > 0x1p-10 && f < 1.0 - 0x1p-10) return b;
    b = b < 0 ? 0 : (b > nbins - 1 ? nbins - 1 : b);
    while (b > 0 && v < edge(b, nbins, lo, hi, step)) --b;
    while (b < nbins - 1 && v >= edge(b + 1, nbins, lo, hi, step)) ++b;
    return b;
}

// t has three roundings of a number up to nbins <= 4096; an edge has two, of
// numbers up to |lo| + |hi|
bool hist_near(double lo, double hi, double step) { return (std::fabs(lo) + std::fabs(hi)) * 0x1p-40 < step; }

__global__ void zero_i64(int64_t* p, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Blocks of 1024 threads count 4096 to 16,384 values each in LDS (more for
// samples beyond kHistBlocks blocks) and add their bins to the result with 64-bit
// global atomics.  Fewer values a block spread the counting over more of the
// chip, but the atomics of all blocks meet in the same few words, so a sample
// takes 64 blocks before they get more than 4096 values: 40,000 values in 79 x 79
// bins take 8 / 13 us with 4096 / 16,384 values a block, 3 x 2^20 values 20 / 16
// us, and 33 / 13 us in 20 bins (1024 blocks of 1024 values, one copy and every
// value corrected: 43 and 103 us).  A sample of up to kHistOne values is stored
// by one block without zeroing or atomics (5 us; a clearing launch is 3 us of 7).
constexpr int kHistBlock = 1024;
constexpr int kHistOne = 8192;
constexpr int kHistBlocks = 512;

// LDS copies of a histogram, chosen so that they fit 4096 counters: lanes
// next to each other count in different copies, since the few bins of a
// histogram otherwise make most lanes of a wave add to the same words.
int hist_copies(int nbins) {
    int r = 32;
    while (r > 1 && nbins * r > 4096) r /= 2;
    return r;
}

unsigned hist_blocks(int64_t n) {
    if (n <= kHistOne) return 1;
    const int64_t per = n / 64 < 4096 ? 4096 : (n / 64 > 16384 ? 16384 : n / 64), b = (n + per - 1) / per;
    return (unsigned)(b > kHistBlocks ? kHistBlocks : b);
}

// The next kHistAhead values of each thread, loaded together so that their
// latencies overlap; NaN, which no bin takes, beyond the end.
constexpr int kHistAhead = 4;
constexpr int kHistChunk = kHistAhead * kHistBlock;

__device__ __forceinline__ void hist_load(const double* __restrict__ x, int64_t n, int64_t i0, double (&v)[kHistAhead]) {
#pragma unroll
    for (int k = 0; k < kHistAhead; ++k) {
        const int64_t i = i0 + k * kHistBlock + threadIdx.x;
        v[k] = i < n ? x[i] : __builtin_nan("");
    }
}

__device__ __forceinline__ void hist_put(int64_t* at, unsigned count) {
    if (gridDim.x == 1) *at = (int64_t)count;
    else if (count) atomicAdd((unsigned long long*)at, (unsigned long long)count);
}

__global__ __launch_bounds__(kHistBlock) void hist_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                          int nbins, int copies, double lo, double hi, double step,
                                                          double istep, bool near, int64_t* __restrict__ counts) {
    extern __shared__ unsigned int sh[];
    const int c = blockIdx.y;
    for (int b = threadIdx.x; b < nbins * copies; b += kHistBlock) sh[b] = 0u;
    __syncthreads();
    const double* xc = x + (int64_t)c * ld;
    unsigned int* mine = sh + (threadIdx.x & (copies - 1));
    for (int64_t i0 = (int64_t)blockIdx.x * kHistChunk; i0 < n; i0 += (int64_t)gridDim.x * kHistChunk) {
        double v[kHistAhead];
        hist_load(xc, n, i0, v);
#pragma unroll
        for (int k = 0; k < kHistAhead; ++k)
            if (v[k] >= lo && v[k] <= hi) atomicAdd(&mine[bin_of(v[k], nbins, lo, hi, step, istep, near) * copies], 1u);
    }
    __syncthreads();
    // the copies of a bin, summed by as many lanes
    for (int k = threadIdx.x; k < nbins * copies; k += kHistBlock) {
        unsigned s = sh[k];
        for (int d = copies / 2; d > 0; d >>= 1) s += __shfl_xor(s, d);
        if ((k & (copies - 1)) == 0) hist_put(&counts[(int64_t)c * nbins + k / copies], s);
    }
}

__global__ __launch_bounds__(kHistBlock) void hist2d_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                            const double* __restrict__ y, int nbins, double lo,
                                                            double hi, double step, double istep, bool near,
                                                            int64_t* __restrict__ counts) {
    extern __shared__ unsigned int sh[];
    const int c = blockIdx.y;
    const int nb2 = nbins * nbins;
    for (int b = threadIdx.x; b < nb2; b += kHistBlock) sh[b] = 0u;
    __syncthreads();
    const double* xc = x + (int64_t)c * ld;
    const double* yc = y + (int64_t)c * ld;
    for (int64_t i0 = (int64_t)blockIdx.x * kHistChunk; i0 < n; i0 += (int64_t)gridDim.x * kHistChunk) {
        double u[kHistAhead], v[kHistAhead];
        hist_load(xc, n, i0, u);
        hist_load(yc, n, i0, v);
#pragma unroll
        for (int k = 0; k < kHistAhead; ++k)
            if (u[k] >= lo && u[k] <= hi && v[k] >= lo && v[k] <= hi)
                atomicAdd(&sh[bin_of(u[k], nbins, lo, hi, step, istep, near) * nbins +
                              bin_of(v[k], nbins, lo, hi, step, istep, near)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb2; b += kHistBlock) hist_put(&counts[(int64_t)c * nb2 + b], sh[b]);
}

// ---------------------------------------------------------------------------
// fixed-order block reductions
// ---------------------------------------------------------------------------

// v of another lane by a data-parallel move (0 in the rows that ROWS leaves out):
// a shuffle goes through the LDS, whose pipe the waves of a CU share (Pearson of
// 3 x 4,099 values 9.6 us with shuffles, 6.5 so; of 3 x 2^20 17.4 and 16 us)
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}

// sums over LANES (8, 16 or 64) lanes side by side, in each of them
template <int LANES, int K>
__device__ __forceinline__ void lane_sum(double (&v)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] += dpp<0xB1>(v[k]);                          // lanes 1, 0, 3, 2 of a quad
        v[k] += dpp<0x4E>(v[k]);                          // 2, 3, 0, 1
        v[k] += dpp<0x141>(v[k]);                         // 7 .. 0 of eight
        if (LANES > 8) v[k] += dpp<0x140>(v[k]);          // 15 .. 0 of a row
        if (LANES > 16) {
            v[k] += dpp<0x142, 0xa>(v[k]);                // lane 15 to the row after, for rows 1 and 3
            v[k] += dpp<0x143, 0xc>(v[k]);                // lane 31 to rows 2 and 3
            v[k] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v[k]), 63),
                                    __builtin_amdgcn_readlane(__double2loint(v[k]), 63));
        }
    }
}

// the sums of the waves of THREADS, in every thread, from each wave's in its lanes
template <int K, int THREADS>
__device__ __forceinline__ void block_add(double (&v)[K], double (*sh)[THREADS / 64]) {
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) sh[k][threadIdx.x >> 6] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] = 0.0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) v[k] += sh[k][w];
    }
}

// the sums over a block of THREADS, in every thread
template <int K, int THREADS>
__device__ __forceinline__ void block_sum(double (&v)[K], double (*sh)[THREADS / 64]) {
    lane_sum<64>(v);
    __syncthreads();
    block_add<K, THREADS>(v, sh);
}

__device__ __forceinline__ bool finite(double v) { return __builtin_isfinite(v); }
__device__ __forceinline__ double finite_or_zero(double v) { return finite(v) ? v : 0.0; }

__device__ __forceinline__ double block_max(double v, double* sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = __builtin_fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------------------
// Pearson: sums, then sums of the centred products.  Samples of one block
// (kPearOne values) take one launch; of larger ones, up to kPearParts blocks
// take chunks of kPearChunk values.  A wave keeps 64 x HOLD values in registers
// between its sums and its centred sums; the waves of a chunked block meet once,
// at its end.  The centred sums of two sets a, b about their own means combine
// to those about the mean of both with n_a n_b / (n_a + n_b) times the product
// of the differences of the means (Chan, Golub & LeVeque 1983), which loses no
// more than a second pass over memory would.  Values are centred about a pivot, their
// mean as rounded; the sum of what is centred gives the distance from the pivot
// to the mean, and the centred sums are corrected by n times its square (the
// two-pass form with a correction of the same paper).  Means stay pairs of a
// pivot and a distance where sets combine: means rounded at the size of a common
// offset cost the deviations the offset's digits (offset 10^9, deviation 0.5:
// 1e-9 of the deviations; with the pairs 1e-15).  Workspace:
// part[c][kPearParts].  Bound by launches and latency for small samples (3 x
// 4,099: four launches 12 us, one 6 us; 3 x 16,384: 18 and 9 us), by reading
// them for large ones (3 x 2^20: two passes 24 us, one 16 us; with three blocks
// on a CU, so that all 768 run at once).
// ---------------------------------------------------------------------------

constexpr int kPearBlock = 512;
constexpr int kPearParts = 256;
constexpr int kPearHold = 8;
constexpr int64_t kPearChunk = (int64_t)kPearBlock * kPearHold;
constexpr int kPearOneBlock = 1024;
constexpr int kPearKeep = 16;
constexpr int64_t kPearOne = (int64_t)kPearOneBlock * kPearKeep;

// a part: the mean of x and of y as a double and what that rounds off as a
// fraction of it (|fraction| <= 2^-53), the centred sums
struct PearPart {
    double mean[2];
    float rest[2];
    double cen[3];
};
static_assert(kPearParts * sizeof(PearPart) <= kPart * 3 * sizeof(double), "the parts fit the workspace");

// a set of n values: pivots, the means' distances from them, the centred sums
struct PearSet {
    double n, piv[2], d[2], cen[3];
};

__device__ __forceinline__ void pearson_out(int64_t n, double mx, double my, const double* v,
                                            double* __restrict__ out) {
    const double nm1 = (double)(n - 1);
    out[0] = mx;
    out[1] = my;
    out[2] = sqrt(v[0] / nm1);
    out[3] = sqrt(v[1] / nm1);
    out[4] = v[2] / sqrt(v[0] * v[1]);
}

// a wave's sums of its HOLD x 64 places
template <int HOLD>
__device__ __forceinline__ void pearson_sums(const double (&xv)[HOLD], const double (&yv)[HOLD], double (&m)[2]) {
    m[0] = m[1] = 0.0;
#pragma unroll
    for (int k = 0; k < HOLD; ++k) {
        m[0] += xv[k];
        m[1] += yv[k];
    }
    lane_sum<64>(m);
}

// the pivot from the sums, in = 1/n: rounded, the same for what is centred and
// for the set (no contraction with the subtraction)
__device__ __forceinline__ void pearson_pivot(const double (&m)[2], double in, PearSet& o) {
#pragma clang fp contract(off)
    o.piv[0] = m[0] * in;
    o.piv[1] = m[1] * in;
}

// a wave's centred sums xx, yy, xy, x and y of its cnt values
template <int HOLD>
__device__ __forceinline__ void pearson_centre(int cnt, const double (&xv)[HOLD], const double (&yv)[HOLD],
                                               const PearSet& p, double (&v)[5]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] = 0.0;
#pragma unroll
    for (int k = 0; k < HOLD; ++k) {
        if (k * 64 + lane < cnt) {
            const double dx = xv[k] - p.piv[0], dy = yv[k] - p.piv[1];
            v[0] += dx * dx;
            v[1] += dy * dy;
            v[2] += dx * dy;
            v[3] += dx;
            v[4] += dy;
        }
    }
    lane_sum<64>(v);
}

// the rest of the set from them.  Distances are 0 where a value or the pivot is
// infinite, and the sums not finite anyway; a correction that overflows belongs
// to sums that do.
__device__ __forceinline__ void pearson_settle(const double (&v)[5], double in, PearSet& o) {
    o.d[0] = finite_or_zero(v[3] * in);
    o.d[1] = finite_or_zero(v[4] * in);
    o.cen[0] = v[0] - finite_or_zero(v[3] * o.d[0]);
    o.cen[1] = v[1] - finite_or_zero(v[4] * o.d[1]);
    o.cen[2] = v[2] - finite_or_zero(v[3] * o.d[1]);
}

// a: a and b
__device__ __forceinline__ void pearson_join(PearSet& a, const PearSet& b) {
    // (from an infinite pivot on, distances from 0: infinities keep their sign)
    const double dx = (finite(a.piv[0]) ? b.piv[0] - a.piv[0] : b.piv[0]) + b.d[0] - a.d[0];
    const double dy = (finite(a.piv[1]) ? b.piv[1] - a.piv[1] : b.piv[1]) + b.d[1] - a.d[1];
    const double w = b.n / (a.n + b.n), f = a.n * w;
    a.cen[0] += b.cen[0] + f * dx * dx;
    a.cen[1] += b.cen[1] + f * dy * dy;
    a.cen[2] += b.cen[2] + f * dx * dy;
    a.d[0] += w * dx;
    a.d[1] += w * dy;
    a.n += b.n;
}

// the sets of WAVES waves, one a lane (n = 0: none), as one about the first
// one's pivot; plain: the means as sums of n times mean, for those that are not
// finite.  In each of WAVES lanes side by side.
template <int WAVES>
__device__ __forceinline__ void pearson_meet(const PearSet& p, const double (&base)[2], double (&d)[2],
                                             double (&plain)[2], double (&cen)[3]) {
    const bool any = p.n > 0.0;
    const double dx = any ? (p.piv[0] - base[0]) + p.d[0] : 0.0, dy = any ? (p.piv[1] - base[1]) + p.d[1] : 0.0;
    const double w = p.n * 0x1p-14;    // n times a mean may overflow where the mean of all does not
    double m[5] = {w * dx, w * dy, any ? w * (p.piv[0] + p.d[0]) : 0.0, any ? w * (p.piv[1] + p.d[1]) : 0.0, w};
    lane_sum<WAVES>(m);
    const double in = 1.0 / m[4];
    d[0] = m[0] * in; d[1] = m[1] * in;
    plain[0] = m[2] * in; plain[1] = m[3] * in;
    const double ex = any ? dx - d[0] : 0.0, ey = any ? dy - d[1] : 0.0;
    cen[0] = p.cen[0] + p.n * ex * ex;
    cen[1] = p.cen[1] + p.n * ey * ey;
    cen[2] = p.cen[2] + p.n * ex * ey;
    lane_sum<WAVES>(cen);
}

__global__ __launch_bounds__(kPearOneBlock) void pearson_one_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                                    const double* __restrict__ y,
                                                                    double* __restrict__ out) {
    constexpr int kWaves = kPearOneBlock / 64;
    __shared__ double sh[2][kWaves], sv[kWaves][5];
    const int c = blockIdx.x;
    const double* xc = x + (int64_t)c * ld;
    const double* yc = y + (int64_t)c * ld;
    // a row of 64 values a wave, then the next rows: small samples spread over the waves
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const double in = 1.0 / (double)n;
    double xv[kPearKeep], yv[kPearKeep], m[2], v[5];
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < kPearKeep; ++k) {
        const int r = (k * kWaves + wave) * 64, i = r + lane;
        xv[k] = i < n ? xc[i] : 0.0;
        yv[k] = i < n ? yc[i] : 0.0;
        cnt += n - r < 64 ? (n > r ? (int)(n - r) : 0) : 64;
    }
    // one pivot for the block: its waves have their sums of a few values at once
    pearson_sums(xv, yv, m);
    block_add<2, kPearOneBlock>(m, sh);
    PearSet p;
    pearson_pivot(m, in, p);
    pearson_centre(cnt, xv, yv, p, v);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 5; ++k) sv[wave][k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x >= kWaves) return;
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] = sv[threadIdx.x][k];
    lane_sum<kWaves>(v);
    pearson_settle(v, in, p);
    if (threadIdx.x == 0) pearson_out(n, p.piv[0] + p.d[0], p.piv[1] + p.d[1], p.cen, out + c * 5);
}

// the number of values in the chunks k, k + parts, .. of a block
__device__ __forceinline__ double pearson_count(int64_t n, int k, int parts) {
    const int64_t chunks = (n + kPearChunk - 1) / kPearChunk;
    const int64_t mine = (chunks - k + parts - 1) / parts;
    return (double)(mine * kPearChunk - ((chunks - 1) % parts == k ? chunks * kPearChunk - n : 0));
}

__global__ __launch_bounds__(kPearBlock, 6) void pearson_part_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                                     const double* __restrict__ y,
                                                                     PearPart* __restrict__ part) {
    constexpr int kWaves = kPearBlock / 64, kRow = 64 * kPearHold;
    __shared__ PearSet sh[kWaves];
    const int c = blockIdx.y;
    const double* xc = x + (int64_t)c * ld;
    const double* yc = y + (int64_t)c * ld;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (lane == 0) sh[wave] = PearSet{};
    for (int64_t i0 = blockIdx.x * kPearChunk + wave * kRow; i0 < n; i0 += gridDim.x * kPearChunk) {
        const int cnt = n - i0 < kRow ? (int)(n - i0) : kRow;
        double xv[kPearHold], yv[kPearHold];
#pragma unroll
        for (int k = 0; k < kPearHold; ++k) {
            const int i = k * 64 + lane;
            xv[k] = i < cnt ? xc[i0 + i] : 0.0;
            yv[k] = i < cnt ? yc[i0 + i] : 0.0;
        }
        PearSet q;
        double m[2], v[5];
        q.n = (double)cnt;
        const double in = 1.0 / q.n;
        pearson_sums(xv, yv, m);
        pearson_pivot(m, in, q);
        pearson_centre(cnt, xv, yv, q, v);
        pearson_settle(v, in, q);
        if (lane == 0) {
            // (the set so far is not kept in registers, which 24 waves a CU leave no more of)
            if (i0 >= kPearChunk * gridDim.x) {
                PearSet p = sh[wave];
                pearson_join(p, q);
                sh[wave] = p;
            } else {
                sh[wave] = q;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x >= kWaves) return;
    const PearSet p = sh[threadIdx.x];
    const double base[2] = {sh[0].piv[0], sh[0].piv[1]};
    double d[2], plain[2], cen[3];
    pearson_meet<kWaves>(p, base, d, plain, cen);
    if (threadIdx.x == 0) {
        PearPart& o = part[(int64_t)c * kPearParts + blockIdx.x];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            // the pivot and the distance as their sum and what it rounds off
            const double mean = base[k] + d[k], t = mean - base[k];
            const double rest = (base[k] - (mean - t)) + (d[k] - t);
            o.mean[k] = finite(mean) ? mean : plain[k];
            o.rest[k] = (float)finite_or_zero(rest / mean);
        }
        o.cen[0] = cen[0]; o.cen[1] = cen[1]; o.cen[2] = cen[2];
    }
}

__global__ __launch_bounds__(kPearParts) void pearson_final_kernel(int64_t n, int parts,
                                                                   const PearPart* __restrict__ part,
                                                                   double* __restrict__ out) {
    __shared__ double sh[4][kPearParts / 64];
    const int c = blockIdx.x;
    const bool mine = (int)threadIdx.x < parts;
    // the means' distances from the first part's, summed for the centred sums;
    // the plain sums for the mean itself (the first part's may be far from it)
    double d[2] = {0.0, 0.0}, m[4] = {0.0, 0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, base[2], nb = 0.0;
    const PearPart& first = part[(int64_t)c * kPearParts];
    base[0] = first.mean[0];
    base[1] = first.mean[1];
    if (mine) {
        const PearPart& o = part[(int64_t)c * kPearParts + threadIdx.x];
        nb = pearson_count(n, threadIdx.x, parts);
        const double w = nb / (double)n;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            d[k] = (o.mean[k] - base[k]) + o.mean[k] * (double)o.rest[k];
            m[k] = w * d[k];
            m[2 + k] = w * o.mean[k];
        }
        v[0] = o.cen[0]; v[1] = o.cen[1]; v[2] = o.cen[2];
    }
    block_sum<4, kPearParts>(m, sh);
    if (mine) {
        const double dx = d[0] - m[0], dy = d[1] - m[1];
        v[0] += nb * dx * dx;
        v[1] += nb * dy * dy;
        v[2] += nb * dx * dy;
    }
    block_sum<3, kPearParts>(v, sh);
    if (threadIdx.x == 0) pearson_out(n, m[2], m[3], v, out + c * 5);
}

// ---------------------------------------------------------------------------
// KDE: block (b, c, tile) takes one slice of the points and 256 grid points;
// partial sums part[c][b][g], combined in block order.
//
// With u = (g - x)/h and the grid step d = gstep/h, the 256 grid points of a
// tile are 16 segments of 16; segment i has its anchor at its 9th point, m_i =
// 16 (i - 8) steps from the tile's middle anchor, and the point j in -8 .. 7
// of the segment lies j steps from the anchor.  With v = u at the middle
// anchor and u_i = v + m_i d,
//   exp(-(u_i + j d)^2/2) = exp(-u_i^2/2) . exp(-v d)^j . exp(-(j^2/2 + m_i j) d^2),
// where the first factor depends on (i, x), the second on (j, x) and the
// third on (i, j) only: the sum over the points is the 16 x 16 product of the
// first two, taken by the FP64 matrix instruction four points at a time, and
// the third multiplies the finished sums.  The first factor, in turn, is formed
// by an exponential at one end of each group of four segments, the end nearer to
// the point, and a ratio from there outward:
//   exp(-(u + 16 s d)^2/2) = exp(-u^2/2) . exp(-16 s d u - 128 d^2),  s = +-1,
// the ratio shrinking by exp(-256 d^2) a segment.  That leaves two exponentials
// per (point, 64 grid points).  Bound by the FP64 units, which vector and
// matrix instructions share.
//
// The first factor is carried as 2^448 times its value.  Of a term that is a
// normal number, exp(-708) at least, the product of the first two is then at
// least exp(310 - 708 - 871 d^2) (j = 7, m_i = -128), which is normal too for
// d <= 0.59, and at most exp(310 + 1056 d^2) (j = -8), which leaves exp(30) for
// the sum over the points.  It is 0 beyond 46 h from the anchor, and the
// outermost anchors lie 128 d from the middle one: a point with |v d| > 46 d +
// 128 d^2, at most 72, has none, and v d is clamped to +-75.  With (hi - lo)/h .
// d <= 37 the second factor is at most exp(296) inside [lo, hi].  Other grids (a
// step coarse against the bandwidth, a bandwidth that is 0, negative or not a
// number, or one so large that the step is below 1e-290 of it, infinite ones
// among them: 65/d and the lanes beyond the end, with x at infinity, need a
// normal d) take one exponential per (point, grid point).  On 2^20 x 3 points and 201
// grid points that path takes 0.76 ms, the products with an
// exponential per (point, segment) 0.080 ms, these 0.073 ms.
// ---------------------------------------------------------------------------

__device__ __forceinline__ double kde_h(const double* sigma, int64_t stride, int c, double nfac) {
    return (1.06 * sigma[(int64_t)c * stride]) * nfac;
}

constexpr int kKdeTile = 256;       // grid points of a block
constexpr int kKdeRow = 18;         // LDS row of a point: 16 factors and padding
constexpr int kKdePoints = 32;      // points a wave takes at a time

__device__ __forceinline__ bool kde_products(double ih, double gstep, double span) {
    const double d = gstep * ih;
    return d >= 1e-290 && d <= 0.59 && (span * ih) * d <= 37.0;
}

// 2^(k + f): the polynomial interpolates 2^f on [-1/2, 1/2] at its Chebyshev
// nodes, formed in 50-digit arithmetic (largest error 3.2e-18).
__device__ __forceinline__ double exp2_parts(int k, double f) {
    double p = 4.455817908336064492979619e-10;
    p = __builtin_fma(p, f, 7.07419429728852100555915e-9);
    p = __builtin_fma(p, f, 1.017805708773394110461712e-7);
    p = __builtin_fma(p, f, 1.321543253591237616649419e-6);
    p = __builtin_fma(p, f, 1.525273384155677258925467e-5);
    p = __builtin_fma(p, f, 1.540353046372435420860299e-4);
    p = __builtin_fma(p, f, 1.333355814640647069705879e-3);
    p = __builtin_fma(p, f, 9.618129107587256668064659e-3);
    p = __builtin_fma(p, f, 5.550410866482162703948952e-2);
    p = __builtin_fma(p, f, 0.2402265069591015956717015);
    p = __builtin_fma(p, f, 0.6931471805599453092537366);
    p = __builtin_fma(p, f, 1.0);
    return __builtin_amdgcn_ldexp(p, k);
}

// 2^(t + kKdeScale) for t <= 0 (0 below t = -1523, NaN for NaN)
constexpr int kKdeScale = 448;

__device__ __forceinline__ double exp2_scaled(double t) {
    t = t < -1600.0 ? -1600.0 : t;
    const double k = __builtin_rint(t);
    return exp2_parts((int)k + kKdeScale, t - k);
}

typedef double double4_t __attribute__((ext_vector_type(4)));

// Chunks of 32 points are dealt to the waves of all blocks in turn; two lanes
// form a point's factors, lane p those of the segments and powers below the
// middle, lane 32 + p those above.
__device__ __forceinline__ void kde_block_products(int64_t n, const double* __restrict__ xc, double ih, double d,
                                                   double gmid, double* sh, int ngrid, int g0,
                                                   double* __restrict__ out) {
    constexpr double kLog2e = 1.44269504088896340736;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double (*first)[kKdeRow] = (double (*)[kKdeRow])sh + wave * 2 * kKdePoints;      // exp(-u_i^2/2)
    double (*power)[kKdeRow] = first + kKdePoints;                                    // exp(-v d)^j
    const int pt = lane & (kKdePoints - 1), half = lane / kKdePoints;
    // the ratio's exponent step u + step2 with both coefficients to twice the
    // precision, step2's integer apart: rounded alike for all points, they
    // would not average out
    const double step = -16.0 * d * kLog2e;
    const double steplo = __builtin_fma(-16.0 * d, kLog2e, -step) + (-16.0 * d) * 2.0355273740931033e-17;
    const double step2 = (8.0 * d) * step, step2i = __builtin_rint(step2), step2f = step2 - step2i;
    const double step2lo = __builtin_fma(8.0 * d, step, -step2) + (8.0 * d) * steplo;
    const double shrink = exp(-256.0 * d * d), far = 65.0 / d;
    const int64_t chunks = (n + kKdePoints - 1) / kKdePoints;
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    for (int64_t ch = (int64_t)blockIdx.x * (kBlock / 64) + wave; ch < chunks;
         ch += (int64_t)gridDim.x * (kBlock / 64)) {
        const int64_t i = ch * kKdePoints + pt;
        // beyond the end: a point at infinity, whose first factor is 0
        const double x = i < n ? xc[i] : __builtin_inf();
        const double v = (gmid - x) * ih;
        double a = v * d;
        a = __builtin_fmin(__builtin_fmax(a, -75.0), 75.0);
        // the powers -8 .. -1 or 0 .. 7
        const double b1 = exp(half ? -a : a);
        const double b2 = b1 * b1, b3 = b2 * b1, b4 = b2 * b2;
        double* r = &power[pt][8];
        const int s = half ? 1 : -1;
        r[s] = b1; r[2 * s] = b2; r[3 * s] = b3; r[4 * s] = b4;
        r[5 * s] = b4 * b1; r[6 * s] = b3 * b3; r[7 * s] = b4 * b3;
        r[half ? 0 : -8] = half ? 1.0 : b4 * b4;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int i0 = 8 * half + 4 * g;
            const double m0 = 16.0 * (double)(i0 - 8);
            const bool up = __builtin_fma(m0 + 24.0, d, v) >= 0.0;       // the group's middle is right of the point
            const double u = __builtin_fma(up ? m0 : m0 + 48.0, d, v);
            const double e0 = exp2_scaled((u * u) * (-0.5 * kLog2e));
            const double su = __builtin_fmin(up ? u : -u, far);          // beyond, e0 is 0
            const double k = __builtin_rint(__builtin_fma(su, step, step2f));
            double q = exp2_parts((int)k + (int)step2i, __builtin_fma(su, step, -k) + (step2f + __builtin_fma(su, steplo, step2lo)));
            const double e1 = e0 * q;
            q *= shrink;
            const double e2 = e1 * q;
            q *= shrink;
            double* f = &first[pt][up ? i0 : i0 + 3];
            const int t = up ? 1 : -1;
            f[0] = e0; f[t] = e1; f[2 * t] = e2; f[3 * t] = e2 * q;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int k = 0; k < kKdePoints / 4; ++k) {
            const int p = 4 * k + (lane >> 4);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(first[p][lane & 15], power[p][lane & 15], acc, 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // the four waves' products, summed in order: entry (i, j) is in lane
    // 16 (i % 4) + j, register i / 4
    __syncthreads();
    double* red = sh;
#pragma unroll
    for (int k = 0; k < 4; ++k) red[wave * 256 + (4 * k + (lane >> 4)) * 16 + (lane & 15)] = acc[k];
    __syncthreads();
    const int g = g0 + threadIdx.x;
    if (g < ngrid) out[g] = ((red[threadIdx.x] + red[256 + threadIdx.x]) + red[512 + threadIdx.x]) + red[768 + threadIdx.x];
}

__global__ __launch_bounds__(kBlock) void kde_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                     const double* __restrict__ sigma, int64_t sstride, double nfac,
                                                     int ngrid, double lo, double span, double gstep,
                                                     double* __restrict__ part) {
    __shared__ double2 sh[kBlock * kKdeRow / 2];
    const int c = blockIdx.y;
    const int g0 = blockIdx.z * kKdeTile;
    const double* xc = x + (int64_t)c * ld;
    const double ih = 1.0 / kde_h(sigma, sstride, c, nfac);
    double* out = part + ((int64_t)c * gridDim.x + blockIdx.x) * ngrid;
    if (kde_products(ih, gstep, span)) {
        kde_block_products(n, xc, ih, gstep * ih, affine((double)(g0 + 136), gstep, lo), (double*)sh, ngrid, g0,
                           out);
        return;
    }
    double* tile = (double*)sh;
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t j0 = (int64_t)blockIdx.x * per;
    const int64_t j1 = (j0 + per < n) ? j0 + per : n;
    // one grid point per thread; the block's slice of points is staged
    // through LDS
    const int g = g0 + threadIdx.x;
    const double xg = affine((double)g, gstep, lo);
    double acc = 0.0;
    for (int64_t t0 = j0; t0 < j1; t0 += kBlock) {
        const int64_t j = t0 + threadIdx.x;
        tile[threadIdx.x] = j < j1 ? xc[j] : 0.0;
        __syncthreads();
        const int cnt = (int)((j1 - t0) < kBlock ? (j1 - t0) : kBlock);
        for (int k = 0; k < cnt; ++k) {
            const double u = (xg - tile[k]) * ih;
            acc += exp(-0.5 * u * u);
        }
        __syncthreads();
    }
    if (g < ngrid) out[g] = acc;
}

// Sixteen grid points a block, sixteen threads over the partial sums of each
// (one thread a grid point left 201 threads with 512 dependent loads, 41 us).
__global__ __launch_bounds__(kBlock) void kde_final_kernel(int64_t n, const double* __restrict__ sigma, int64_t sstride,
                                                           double nfac, double sqrt2pi, int ngrid, int parts,
                                                           double span, double gstep, const double* __restrict__ part,
                                                           double* __restrict__ out) {
    __shared__ double sh[16][17];
    const int c = blockIdx.y;
    const int gl = threadIdx.x & 15, p = threadIdx.x >> 4;
    const int g = blockIdx.x * 16 + gl;
    double s = 0.0;
    if (g < ngrid)
        for (int b = p; b < parts; b += 16) s += part[((int64_t)c * parts + b) * ngrid + g];
    sh[p][gl] = s;
    __syncthreads();
    if (p != 0 || g >= ngrid) return;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += sh[k][gl];
    const double h = kde_h(sigma, sstride, c, nfac);
    const double ih = 1.0 / h;
    if (kde_products(ih, gstep, span)) {
        // the factor exp(-(j^2/2 + m_i j) d^2), its argument to about 32 digits
        const int i = (g % kKdeTile) >> 4, j = (g & 15) - 8;
        const double w = 0.5 * (double)(j * j) + (double)(16 * (i - 8) * j);
        const double d = gstep * ih;
        const double d2 = d * d, d2lo = __builtin_fma(d, d, -d2);
        const double e = w * d2, elo = __builtin_fma(w, d2, -e) + w * d2lo;
        const double f = exp(-e);
        s = __builtin_amdgcn_ldexp(s * __builtin_fma(-elo, f, f), -kKdeScale);
    }
    const double norm = 1.0 / (((double)n * h) * sqrt2pi);
    out[(int64_t)c * ngrid + g] = s * norm;
}

// Partial sums per component: enough blocks to fill the chip four deep (the
// blocks of a CU that fit its LDS), no more than give each wave two chunks of
// points; from the sizes alone, so that results do not depend on the device.
int kde_parts(int64_t n, int ncomp, int tiles) {
    const int64_t fill = 1024 / ((int64_t)ncomp * tiles);
    const int64_t two = (n + 2 * kKdePoints - 1) / (2 * kKdePoints);
    const int64_t need = (two + kBlock / 64 - 1) / (kBlock / 64);
    int64_t p = need < fill ? need : fill;
    p = p < 16 ? (need < 16 ? need : 16) : p;
    return (int)(p > kPart ? kPart : p);
}

// ---------------------------------------------------------------------------
// Kolmogorov-Smirnov against U[lo, hi].
//
// D needs the order of the values only where the empirical distribution may
// be furthest from F.  The values are counted in equal buckets of [lo, hi];
// with the counts below a bucket, its edges bound every deviation inside it
// from above and some deviation from below, and only the buckets whose upper
// bound reaches the largest lower bound (the candidates; a few per cent) are
// ranked, value by value.  Rounding is monotonic, so the bounds hold for the
// rounded deviations and D is that of the fully sorted sample, bit for bit.
//   ks_count, ks_sum   bucket counts, per block and summed
//   ks_scan            ranks, bounds, candidates (one block a component)
//   ks_collect         the candidates' values, each to its bucket's range
//   ks_split           where values cluster: below
//   ks_solve           ranks inside the candidates, the largest deviation, its p-value
// Bound by launches and latency up to 2^20 values: 3 x 2^20 took 0.69 ms by
// sorting (20 launches a component), 0.056 ms this way; samples of one block
// take one launch (ks_one).
//
// The bound works while a bucket holds far less of F than D ~ 1/sqrt(n); above
// kKsBucketMax values (2^22: 1/16384 against 4e-4) most buckets would be
// candidates, and a sorted copy serves, as it does for a workspace too small.
// ---------------------------------------------------------------------------

constexpr int64_t kKsBucketMax = (int64_t)1 << 22;
constexpr int kKsCount = 1024;           // threads of ks_count, ks_scan and ks_solve
constexpr int kKsPerBlock = 16384;       // values counted by one block
constexpr int kKsWave = 128;             // most values of a range that a wave ranks beside idle ones
constexpr int kKsBlock = 512;            // most values that a wave or a block ranks
constexpr int kKsBins = 1024;            // key bins of a refinement level
constexpr int kKsLevels = 7;             // 10 bits a level of the 64-bit key
constexpr unsigned kKsNone = 0xffffffffu;

// Values that cluster (scalar products of aligned spins, samples of a few
// values) put a large part of the sample into a few buckets, and a block that
// refines such a bucket reads it alone: 2^22 equal values took 6.4 ms, a sort
// 0.46.  Candidates with more than 1/16 of the sample (and 4096 values) are split
// by all blocks instead, as the sample is, but by values drawn from them:
// ks_scan sorts about 1000 of their values (splitters), ks_collect counts the
// others at and between the splitters, ks_split takes the deviations at the
// splitters, which are exact, and collects the values between two neighbours
// only where their bound exceeds the largest of those.  Ties are then splitters,
// and the rest is cut evenly however narrow the cluster: 0.12 ms.
constexpr int kKsHuge = 15;              // most such buckets
constexpr int kKsSplit = 1008;           // most splitters (with kKsHuge, a thread each)
constexpr unsigned kKsHugeMark = 0xffffff00u;
__host__ __device__ __forceinline__ int64_t ks_huge_min(int64_t n) { return n / 16 > 4096 ? n / 16 : 4096; }

// Places of one component's workspace, in 4-byte words from its start
// (256-byte aligned); buckets = 1024 .. 16384, about one for 16 values.
struct KsPlan {
    int buckets, blocks;
    int64_t count, slot, cand, part, split, list;       // word offsets
    int64_t bytes;
};

KsPlan ks_plan(int64_t n) {
    KsPlan p;
    p.buckets = 1024;
    while (p.buckets < 16384 && (int64_t)p.buckets * 16 < n) p.buckets *= 2;
    p.blocks = (int)((n + kKsPerBlock - 1) / kKsPerBlock);
    int64_t w = 64;                                      // header: KsView
    p.count = w; w += p.buckets + 64;                    // counts, then counts below (buckets + 1)
    p.slot = w; w += p.buckets;
    p.cand = w; w += p.buckets;
    p.part = w; w += (int64_t)p.buckets * p.blocks;
    p.split = w; w += 5 * kKsSplit + 2 * kKsHuge + 2;    // KsView
    p.list = w; w += 2 * n;
    p.bytes = (w * 4 + 255) / 256 * 256;
    return p;
}

struct KsView {
    unsigned* w;
    KsPlan p;
    __device__ unsigned long long* dmax() const { return (unsigned long long*)w; }
    __device__ unsigned* ncand() const { return w + 2; }
    __device__ unsigned* nhuge() const { return w + 3; }
    __device__ unsigned* nsub() const { return w + 4; }             // records at part(0)
    __device__ unsigned* done() const { return w + 5; }             // blocks of ks_solve
    // the huge buckets in order, the splitters below each (and all, at nhuge),
    // the number of values in those before it
    __device__ unsigned* huge_bucket() const { return w + 8; }
    __device__ unsigned* huge_split() const { return w + 8 + kKsHuge; }
    __device__ unsigned* huge_values() const { return w + 9 + 2 * kKsHuge; }
    // the S splitters, and counts: at them, between them (of bucket h: from
    // huge_split[h] + h), and the places of the latter already taken
    __device__ double* splitter() const { return (double*)(w + p.split); }
    __device__ unsigned* at_split() const { return w + p.split + 2 * kKsSplit; }
    __device__ unsigned* between() const { return at_split() + kKsSplit; }
    __device__ unsigned* taken() const { return between() + kKsSplit + kKsHuge; }
    __device__ unsigned* count() const { return w + p.count; }
    __device__ unsigned* slot() const { return w + p.slot; }
    __device__ unsigned* cand() const { return w + p.cand; }
    __device__ unsigned* part(int b) const { return w + p.part + (int64_t)b * p.buckets; }
    __device__ double* list() const { return (double*)(w + p.list); }
};
__device__ __forceinline__ KsView ks_view(void* ws, const KsPlan& p, int c) {
    return KsView{(unsigned*)((char*)ws + (int64_t)c * p.bytes), p};
}

// The bucket of v: not decreasing in v (each rounding is monotonic); values
// outside [lo, hi] go to the first and the last.
__device__ __forceinline__ int ks_bucket(double v, double lo, double scale, int buckets) {
    const double t = __builtin_fmin(__builtin_fmax((v - lo) * scale, 0.0), (double)(buckets - 1));
    return (int)t;
}

__device__ __forceinline__ double ks_F(double v, double lo, double w) { return (v - lo) / w; }
// the deviations at the value of rank i (from 0)
__device__ __forceinline__ double ks_up(int64_t i, double dn, double F) { return (double)(i + 1) / dn - F; }
__device__ __forceinline__ double ks_down(int64_t i, double dn, double F) { return F - (double)i / dn; }

// Values of F in bucket b lie between these (b / buckets is exact, ib =
// 1 / buckets; the factor covers the rounding of F and of the bucket's own
// product); the first and the last bucket also hold what lies outside [lo, hi].
__device__ __forceinline__ double ks_bucket_lo(int b, double ib) {
    return b == 0 ? -__builtin_inf() : ((double)b * ib) * (1.0 - 0x1p-48);
}
__device__ __forceinline__ double ks_bucket_hi(int b, int buckets, double ib) {
    return b == buckets - 1 ? __builtin_inf() : ((double)(b + 1) * ib) * (1.0 + 0x1p-48);
}

// t[k] += 1 from each lane that calls; lanes that agree with the first add once
__device__ __forceinline__ void lds_count(unsigned* t, int k) {
    const int k0 = __builtin_amdgcn_readfirstlane(k);
    const uint64_t same = __ballot(k == k0);
    if (k != k0) atomicAdd(&t[k], 1u);
    else if ((threadIdx.x & 63) == __ffsll((unsigned long long)same) - 1) atomicAdd(&t[k0], (unsigned)__popcll(same));
}

__global__ __launch_bounds__(kKsCount) void ks_count(int64_t n, int64_t ld, const double* __restrict__ x, double lo,
                                                     double scale, void* ws, KsPlan p) {
    extern __shared__ unsigned int sh[];
    const KsView v = ks_view(ws, p, blockIdx.y);
    const double* xc = x + (int64_t)blockIdx.y * ld;
    for (int b = threadIdx.x; b < p.buckets; b += kKsCount) sh[b] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) { *v.dmax() = 0ull; *v.done() = 0u; }
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * kKsPerBlock;
    const int64_t i1 = i0 + kKsPerBlock < n ? i0 + kKsPerBlock : n;
#pragma unroll 4
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kKsCount) atomicAdd(&sh[ks_bucket(xc[i], lo, scale, p.buckets)], 1u);
    __syncthreads();
    unsigned* out = v.part(blockIdx.x);
    for (int b = threadIdx.x; b < p.buckets; b += kKsCount) out[b] = sh[b];
}

// The counts of a bucket over the blocks, and for each block the sum of those
// before it: the place of its values among the bucket's.
__global__ __launch_bounds__(kBlock) void ks_sum(void* ws, KsPlan p) {
    const KsView v = ks_view(ws, p, blockIdx.y);
    const int b = blockIdx.x * kBlock + threadIdx.x;     // the buckets are a multiple of kBlock
    constexpr int kAhead = 16;                           // loads in flight
    unsigned s = 0;
    for (int k0 = 0; k0 < p.blocks; k0 += kAhead) {
        unsigned c[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) c[k] = k0 + k < p.blocks ? v.part(k0 + k)[b] : 0u;
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (k0 + k < p.blocks) {
                v.part(k0 + k)[b] = s;
                s += c[k];
            }
    }
    v.count()[b] = s;
}

// exclusive prefix sums over the block's threads, and the total
__device__ __forceinline__ unsigned block_scan(unsigned v, unsigned* sh, unsigned& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    unsigned before = 0, all = 0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) {
        before += k < wave ? sh[k] : 0u;
        all += sh[k];
    }
    __syncthreads();
    total = all;
    return before + inc - v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = __builtin_fmax(v, __shfl_xor(v, d));
    return v;
}

template <int PER>
__device__ __forceinline__ void store_words(unsigned* __restrict__ to, const unsigned* w) {
#pragma unroll
    for (int k = 0; k < PER; k += 4) {
        if (PER >= 4) {
            *(uint4*)(to + k) = make_uint4(w[k], w[k + 1 < PER ? k + 1 : 0], w[k + 2 < PER ? k + 2 : 0], w[k + 3 < PER ? k + 3 : 0]);
        } else {
#pragma unroll
            for (int j = 0; j < PER; ++j) to[j] = w[j];
        }
    }
}

// Ranks, bounds and candidates of one component, by one block: the counts
// become the counts below; `slots` receives each candidate's place in the list
// (kKsNone elsewhere), `cands` the candidates; returns their number.  PER =
// buckets / kKsCount.  The empirical distribution below a bucket is the count
// times 1/n, with a factor that covers the rounding against the quotient the
// deviations are formed with (four divisions a bucket, and single loads, took
// 37 us for 16,384 buckets, this 14 us).
template <int PER>
__device__ int ks_scan_block(int64_t n, unsigned* __restrict__ count, unsigned* __restrict__ slots,
                             unsigned* __restrict__ cursors, unsigned* __restrict__ cands, int buckets, unsigned* shu,
                             double* shd, unsigned* nhuge = nullptr, unsigned* huge = nullptr) {
    const int b0 = threadIdx.x * PER;
    const double in = 1.0 / (double)n, ib = 1.0 / buckets;       // the latter exact: a power of two
    constexpr double kDown = 1.0 - 0x1p-50, kUp = 1.0 + 0x1p-50;
    unsigned cnt[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; k += 4) {
        if (PER >= 4) {
            const uint4 q = *(const uint4*)(count + b0 + k);
            cnt[k] = q.x; cnt[k + 1 < PER ? k + 1 : 0] = q.y; cnt[k + 2 < PER ? k + 2 : 0] = q.z;
            cnt[k + 3 < PER ? k + 3 : 0] = q.w;
        } else {
#pragma unroll
            for (int j = 0; j < PER; ++j) cnt[j] = count[b0 + j];
        }
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) sum += cnt[k];
    unsigned total;
    const unsigned below0 = block_scan(sum, shu, total);
    // frac[k]: the empirical distribution below bucket b0 + k
    double frac[PER + 1];
    unsigned below = below0;
    frac[0] = (double)below * in;
    unsigned word[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        word[k] = below;
        below += cnt[k];
        frac[k + 1] = (double)below * in;
    }
    store_words<PER>(count + b0, word);
    if (threadIdx.x == kKsCount - 1) count[buckets] = below;
    // the largest lower bound: a bucket's last value lies below its upper edge,
    // its first above its lower edge
    double low = 0.0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (cnt[k]) {
            low = __builtin_fmax(low, frac[k + 1] * kDown - ks_bucket_hi(b0 + k, buckets, ib));
            low = __builtin_fmax(low, ks_bucket_lo(b0 + k, ib) - frac[k] * kUp);
        }
    }
    low = wave_max(low);
    if ((threadIdx.x & 63) == 0) shd[threadIdx.x >> 6] = low;
    __syncthreads();
    for (int k = 0; k < kKsCount / 64; ++k) low = __builtin_fmax(low, shd[k]);
    // candidates: where an upper bound reaches it
    unsigned mask = 0, vals = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (cnt[k] && (frac[k + 1] * kUp - ks_bucket_lo(b0 + k, ib) >= low ||
                       ks_bucket_hi(b0 + k, buckets, ib) - frac[k] * kDown >= low)) {
            mask |= 1u << k;
            vals += cnt[k];
        }
    }
    unsigned slot = block_scan(vals, shu, total);
    unsigned at = block_scan((unsigned)__popc(mask), shu, total);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const bool c = (mask >> k) & 1u;
        word[k] = c ? slot : kKsNone;
        if (c) {
            if (cursors) cursors[b0 + k] = slot;
            cands[at++] = b0 + k;
            slot += cnt[k];
            if (nhuge && cnt[k] > ks_huge_min(n)) huge[atomicAdd(nhuge, 1u)] = b0 + k;
        }
    }
    store_words<PER>(slots + b0, word);
    return (int)total;
}

// A place below n for each i, scattered so that it agrees with no period of the
// sample (a grid of parameters): places at a fixed distance found no value of a
// bucket that held all others.
__device__ __forceinline__ int64_t ks_scatter(unsigned i, int64_t n) {
    i = (i + 1u) * 0x9e3779b1u;
    i = (i ^ (i >> 15)) * 0x85ebca77u;
    i ^= i >> 13;
    return (int64_t)(((uint64_t)i * (uint64_t)n) >> 32);      // n <= 2^22
}

// The huge buckets' splitters, sorted by the block (bitonic, a value a thread):
// as many of their values as 16,384 places of the sample give, up to kKsSplit.
__device__ void ks_splitters(const KsView& v, int64_t n, const double* __restrict__ x, double lo, double scale, int nh,
                             const unsigned* huge, double* sh, unsigned* shn) {
    const int t = threadIdx.x;
    if (t == 0) *shn = 0u;
    unsigned rank = 0, before = 0;
    if (t < nh) {
        for (int h = 0; h < nh; ++h)
            if (huge[h] < huge[t]) {
                ++rank;
                before += v.count()[huge[h] + 1] - v.count()[huge[h]];
            }
        v.huge_bucket()[rank] = huge[t];
        v.huge_values()[rank] = before;
    }
    for (int i = t; i < 3 * kKsSplit + 2 * kKsHuge; i += kKsCount) v.at_split()[i] = 0u;
    __syncthreads();
    constexpr int kAhead = 4;
    for (int r = 0; r < 16; r += kAhead) {
        double u[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) u[k] = x[ks_scatter((unsigned)((r + k) * kKsCount + t), n)];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const unsigned b = ks_bucket(u[k], lo, scale, v.p.buckets);
            bool in = false;
            for (int h = 0; h < nh; ++h) in = in || huge[h] == b;
            const uint64_t mask = __ballot(in);
            unsigned at = 0;
            if (in && (t & 63) == __ffsll((unsigned long long)mask) - 1) at = atomicAdd(shn, (unsigned)__popcll(mask));
            if (mask != 0) at = __shfl(at, __ffsll((unsigned long long)mask) - 1) + __popcll(mask & ((1ull << (t & 63)) - 1));
            if (in && at < kKsSplit) sh[at] = u[k];
        }
        __syncthreads();
        const bool full = *shn >= kKsSplit;
        __syncthreads();
        if (full) break;
    }
    const int S = *shn < kKsSplit ? (int)*shn : kKsSplit;
    double u = t < S ? sh[t] : __builtin_inf();
    for (int k = 2; k <= kKsCount; k *= 2)
        for (int j = k / 2; j > 0; j /= 2) {
            double o;
            if (j < 64) {
                o = __shfl_xor(u, j);
            } else {
                __syncthreads();
                sh[t] = u;
                __syncthreads();
                o = sh[t ^ j];
            }
            u = ((t & j) == 0) == ((t & k) == 0) ? __builtin_fmin(u, o) : __builtin_fmax(u, o);
        }
    if (t < S) v.splitter()[t] = u;
    const unsigned b = ks_bucket(u, lo, scale, v.p.buckets);
    for (int h = 0; h < nh; ++h) {
        const int below = __syncthreads_count(t < S && b < v.huge_bucket()[h]);
        if (t == 0) v.huge_split()[h] = below;
    }
    if (t == 0) v.huge_split()[nh] = S;
}

__global__ __launch_bounds__(kKsCount) void ks_scan(int64_t n, int64_t ld, const double* __restrict__ x, double lo,
                                                    double scale, void* ws, KsPlan p) {
    __shared__ unsigned shu[kKsCount / 64];
    __shared__ double shd[kKsCount / 64];
    __shared__ unsigned nhuge, huge[kKsHuge];
    __shared__ double sample[kKsCount];
    const KsView v = ks_view(ws, p, blockIdx.x);
    if (threadIdx.x == 0) nhuge = 0u;
    __syncthreads();
    int total = 0;
    unsigned *c = v.count(), *s = v.slot(), *k = v.cand();
    switch (p.buckets / kKsCount) {
        case 1: total = ks_scan_block<1>(n, c, s, nullptr, k, p.buckets, shu, shd, &nhuge, huge); break;
        case 2: total = ks_scan_block<2>(n, c, s, nullptr, k, p.buckets, shu, shd, &nhuge, huge); break;
        case 4: total = ks_scan_block<4>(n, c, s, nullptr, k, p.buckets, shu, shd, &nhuge, huge); break;
        case 8: total = ks_scan_block<8>(n, c, s, nullptr, k, p.buckets, shu, shd, &nhuge, huge); break;
        default: total = ks_scan_block<16>(n, c, s, nullptr, k, p.buckets, shu, shd, &nhuge, huge); break;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        *v.ncand() = (unsigned)total;
        *v.nhuge() = nhuge;
        *v.nsub() = 0u;
    }
    if (nhuge > 0) ks_splitters(v, n, x + (int64_t)blockIdx.x * ld, lo, scale, (int)nhuge, huge, sample, shu);
}

// The number of the splitters below v (1024 of them, padded with infinity), for
// several values side by side.
template <int K>
__device__ __forceinline__ void ks_place(const double* spl, const double (&v)[K], int (&at)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) at[k] = 0;
#pragma unroll
    for (int step = 512; step > 0; step >>= 1)
#pragma unroll
        for (int k = 0; k < K; ++k) at[k] += spl[at[k] + step - 1] < v[k] ? step : 0;
}

// The candidates are a few per cent of the values: a word a bucket in LDS has
// the next place of the block's values of a candidate, and kKsNone for the
// others.  (Places handed out by global atomics met on the few candidates: 27 us
// for 3 x 2^20 values, this 8.)
__global__ __launch_bounds__(kKsCount) void ks_collect(int64_t n, int64_t ld, const double* __restrict__ x, double lo,
                                                       double scale, void* ws, KsPlan p) {
    extern __shared__ unsigned int sh[];
    __shared__ double spl[kKsCount];
    __shared__ unsigned bins[2 * kKsSplit + kKsHuge];
    const KsView v = ks_view(ws, p, blockIdx.y);
    const double* xc = x + (int64_t)blockIdx.y * ld;
    double* list = v.list();
    const int64_t i0 = (int64_t)blockIdx.x * kKsPerBlock + threadIdx.x;
    constexpr int kKeep = kKsPerBlock / kKsCount;
    double val[kKeep];
#pragma unroll
    for (int k = 0; k < kKeep; ++k) val[k] = i0 + k * kKsCount < n ? xc[i0 + k * kKsCount] : 0.0;
    for (int k = threadIdx.x; k < p.buckets; k += kKsCount) sh[k] = kKsNone;
    __syncthreads();
    const int ncand = (int)*v.ncand();
    const unsigned* before = v.part(blockIdx.x);
    for (int k = threadIdx.x; k < ncand; k += kKsCount) {
        const unsigned b = v.cand()[k];
        sh[b] = v.slot()[b] + before[b];
    }
    const int nh = (int)*v.nhuge();
    if (nh > 0) {
        __syncthreads();
        if ((int)threadIdx.x < nh) sh[v.huge_bucket()[threadIdx.x]] = kKsHugeMark + threadIdx.x;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kKeep; ++k) {
        const int b = ks_bucket(val[k], lo, scale, p.buckets);
        if (i0 + k * kKsCount < n && sh[b] < kKsHugeMark) list[atomicAdd(&sh[b], 1u)] = val[k];
    }
    if (nh == 0) return;
    const int S = (int)v.huge_split()[nh];
    spl[threadIdx.x] = (int)threadIdx.x < S ? v.splitter()[threadIdx.x] : __builtin_inf();
    for (int i = threadIdx.x; i < 2 * kKsSplit + kKsHuge; i += kKsCount) bins[i] = 0u;
    __syncthreads();
    // (read again: kept, they would cost half the occupancy)
    constexpr int kAhead = 2;
#pragma unroll 1
    for (int k0 = 0; k0 < kKeep; k0 += kAhead) {
        double u[kAhead];
        int at[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) u[k] = i0 + (k0 + k) * kKsCount < n ? xc[i0 + (k0 + k) * kKsCount] : 0.0;
        ks_place(spl, u, at);
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const unsigned h = sh[ks_bucket(u[k], lo, scale, p.buckets)] - kKsHugeMark;
            if (i0 + (k0 + k) * kKsCount < n && h < kKsHuge)
                lds_count(bins, at[k] < S && spl[at[k]] == u[k] ? at[k] : kKsSplit + at[k] + (int)h);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * kKsSplit + kKsHuge; i += kKsCount)
        if (bins[i]) atomicAdd(&v.at_split()[i], bins[i]);
}

// 64-bit keys that order as the values do
__device__ __forceinline__ uint64_t ks_key(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v == 0.0 ? 0.0 : v);      // -0 as 0
    return b ^ ((b >> 63) ? ~0ull : (1ull << 63));
}
__device__ __forceinline__ double ks_unkey(uint64_t k) {
    return __longlong_as_double((long long)(k ^ ((k >> 63) ? (1ull << 63) : ~0ull)));
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The largest deviation among m values l[0 .. m), which have the ranks r0 ..
// r0 + m - 1 of the sample, by counting; the wave's part of it: value e goes to
// lane e - e0 for e0 in steps of `stride` from first.  Equal values take their
// ranks in the order they lie.  The values are compared 64 at a time from the
// lanes that loaded them.
__device__ __forceinline__ double ks_ranked(const double* l, int m, int64_t r0, double dn, double lo, double w, int first,
                                            int stride) {
    const int lane = threadIdx.x & 63;
    m = __builtin_amdgcn_readfirstlane(m);
    first = __builtin_amdgcn_readfirstlane(first);
    double d = 0.0;
    if (m > 64) {                             // equal values: the first and the last rank
        const double v0 = l[0];
        int e = lane;
        while (e - lane < m && __ballot(e < m && l[e] != v0) == 0) e += 64;
        if (e - lane >= m) {
            const double F = ks_F(v0, lo, w);
            return __builtin_fmax(0.0, __builtin_fmax(ks_up(r0 + m - 1, dn, F), ks_down(r0, dn, F)));
        }
    }
    for (int e0 = first; e0 < m; e0 += stride) {
        const int e = e0 + lane;
        const double ve = e < m ? l[e] : 0.0;
        int rank = 0;
        for (int j0 = 0; j0 < m; j0 += 64) {
            const int mine = j0 + lane;
            const double vm = j0 == e0 ? ve : (mine < m ? l[mine] : 0.0);
            const int lim = m - j0 < 64 ? m - j0 : 64;
            // equal values of the 64 before come before, of the 64 after, after
            if (j0 < e0)
                for (int j = 0; j < lim; ++j) rank += lane_value(vm, j) <= ve ? 1 : 0;
            else if (j0 > e0)
                for (int j = 0; j < lim; ++j) rank += lane_value(vm, j) < ve ? 1 : 0;
            else
                for (int j = 0; j < lim; ++j) {
                    const double vj = lane_value(vm, j);
                    rank += (vj < ve || (vj == ve && j < lane)) ? 1 : 0;
                }
        }
        if (e < m) {
            const double F = ks_F(ve, lo, w);
            d = __builtin_fmax(d, __builtin_fmax(ks_up(r0 + rank, dn, F), ks_down(r0 + rank, dn, F)));
        }
    }
    return d;
}

// A bucket with more values than a wave ranks (values that cluster): the
// whole block refines it by key bins, 1024 a level, the bin with the largest
// upper bound first, until no bin's bound exceeds the deviation found; bins
// of up to kKsBlock values are ranked, bins of one repeated value have their
// largest deviations at their first and last rank.
struct KsRefine {
    unsigned below[kKsLevels][kKsBins + 1];
    unsigned done[kKsLevels][kKsBins / 32];
    uint64_t klo[kKsLevels], khi[kKsLevels];
    int64_t base[kKsLevels];
    int shift[kKsLevels];
    double vals[kKsBlock];
    unsigned later[kKsCount], nmid, nbig;
    unsigned long long k0, k1, pick;
    unsigned nvals;
    unsigned scan[kKsCount / 64];
    double red[kKsCount / 64];
};

// f(value) for the m values, a block's threads in turn, eight loads in flight
template <class F>
__device__ __forceinline__ void ks_each(const double* l, int m, F&& f) {
    constexpr int kAhead = 8;
    for (int i0 = threadIdx.x; i0 < m; i0 += kAhead * kKsCount) {
        double v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) v[k] = i0 + k * kKsCount < m ? l[i0 + k * kKsCount] : 0.0;
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (i0 + k * kKsCount < m) f(v[k]);
    }
}

// smallest and largest key of the values with keys in [a, b] (at least one)
__device__ __forceinline__ void ks_key_range(KsRefine& R, const double* l, int m, uint64_t a, uint64_t b) {
    __syncthreads();
    if (threadIdx.x == 0) { R.k0 = ~0ull; R.k1 = 0ull; }
    __syncthreads();
    unsigned long long k0 = ~0ull, k1 = 0ull;
    ks_each(l, m, [&](double v) {
        const uint64_t k = ks_key(v);
        if (k >= a && k <= b) {
            k0 = k < k0 ? k : k0;
            k1 = k > k1 ? k : k1;
        }
    });
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const unsigned long long o0 = __shfl_xor(k0, d), o1 = __shfl_xor(k1, d);
        k0 = o0 < k0 ? o0 : k0;
        k1 = o1 > k1 ? o1 : k1;
    }
    if ((threadIdx.x & 63) == 0 && k0 <= k1) {
        atomicMin(&R.k0, k0);
        atomicMax(&R.k1, k1);
    }
    __syncthreads();
}

// level lev: the values with keys in [R.k0, R.k1], the first of them of rank base
__device__ __forceinline__ void ks_build(KsRefine& R, int lev, const double* l, int m, int64_t base) {
    const uint64_t a = R.k0, b = R.k1;
    const int bits = 64 - __clzll((long long)(b - a));
    const int shift = bits > 10 ? bits - 10 : 0;
    for (int k = threadIdx.x; k <= kKsBins; k += kKsCount) R.below[lev][k] = 0u;
    if (threadIdx.x < kKsBins / 32) R.done[lev][threadIdx.x] = 0u;
    if (threadIdx.x == 0) { R.klo[lev] = a; R.khi[lev] = b; R.shift[lev] = shift; R.base[lev] = base; }
    __syncthreads();
    ks_each(l, m, [&](double v) {
        const uint64_t k = ks_key(v);
        if (k >= a && k <= b) lds_count(R.below[lev], (int)((k - a) >> shift));
    });
    __syncthreads();
    unsigned total;
    const unsigned before = block_scan(R.below[lev][threadIdx.x], R.scan, total);      // kKsCount == kKsBins
    R.below[lev][threadIdx.x] = before;
    if (threadIdx.x == 0) R.below[lev][kKsBins] = total;
    __syncthreads();
}

__device__ __forceinline__ double block_max_all(KsRefine& R, double v) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) R.red[threadIdx.x >> 6] = v;
    __syncthreads();
    for (int k = 0; k < kKsCount / 64; ++k) v = __builtin_fmax(v, R.red[k]);
    return v;
}

__device__ __forceinline__ double ks_refine(KsRefine& R, const double* l, int m, int64_t r0, double dn, double lo, double w) {
    double best = 0.0;
    ks_key_range(R, l, m, 0ull, ~0ull);
    if (R.k0 == R.k1) {                       // equal values
        const double F = ks_F(ks_unkey(R.k0), lo, w);
        return __builtin_fmax(0.0, __builtin_fmax(ks_up(r0 + m - 1, dn, F), ks_down(r0, dn, F)));
    }
    int lev = 0;
    ks_build(R, 0, l, m, r0);
    while (lev >= 0) {
        // the open bin with the largest upper bound (the lowest of equal ones)
        const int b = threadIdx.x;
        const unsigned b0 = R.below[lev][b], b1 = R.below[lev][b + 1];
        const uint64_t ka = R.klo[lev] + ((uint64_t)b << R.shift[lev]);
        uint64_t kb = ka + (((uint64_t)1 << R.shift[lev]) - 1);
        if (kb > R.khi[lev] || kb < ka) kb = R.khi[lev];
        double ub = -1.0;
        if (b1 > b0 && !((R.done[lev][b >> 5] >> (b & 31)) & 1u))
            ub = __builtin_fmax(__builtin_fmax(ks_up(R.base[lev] + b1 - 1, dn, ks_F(ks_unkey(ka), lo, w)),
                                               ks_down(R.base[lev] + b0, dn, ks_F(ks_unkey(kb), lo, w))), 0.0);
        const double top = block_max_all(R, ub);
        if (!(top > best)) {                  // nothing open can exceed the deviation found
            --lev;
            __syncthreads();
            continue;
        }
        if (threadIdx.x == 0) R.pick = ~0ull;
        __syncthreads();
        if (ub == top) atomicMin(&R.pick, (unsigned long long)b);
        __syncthreads();
        const int pb = (int)R.pick;
        const unsigned c0 = R.below[lev][pb];
        const int cnt = (int)(R.below[lev][pb + 1] - c0);
        const int64_t base = R.base[lev] + c0;
        const uint64_t pa = R.klo[lev] + ((uint64_t)pb << R.shift[lev]);
        uint64_t pe = pa + (((uint64_t)1 << R.shift[lev]) - 1);
        if (pe > R.khi[lev] || pe < pa) pe = R.khi[lev];
        __syncthreads();
        if (threadIdx.x == 0) { R.done[lev][pb >> 5] |= 1u << (pb & 31); R.nvals = 0u; }
        __syncthreads();
        if (cnt <= kKsBlock) {
            ks_each(l, m, [&](double v) {
                const uint64_t k = ks_key(v);
                if (k >= pa && k <= pe) R.vals[atomicAdd(&R.nvals, 1u)] = v;
            });
            __syncthreads();
            best = __builtin_fmax(best, block_max_all(R, ks_ranked(R.vals, cnt, base, dn, lo, w, threadIdx.x & ~63, kKsCount)));
            continue;
        }
        ks_key_range(R, l, m, pa, pe);
        if (R.k0 == R.k1) {
            const double F = ks_F(ks_unkey(R.k0), lo, w);
            best = __builtin_fmax(best, __builtin_fmax(ks_up(base + cnt - 1, dn, F), ks_down(base, dn, F)));
            continue;
        }
        ++lev;                                // at most 10 bits fewer each time: lev < kKsLevels
        ks_build(R, lev, l, m, base);
    }
    return best;
}

// The deviations at the splitters of the huge buckets, and the values between
// them where they may be exceeded, to the bucket's range of the list; each range
// of these is a record (values, places below, place in the list) for ks_solve.
// Every block forms the bounds for itself; a thread has the values between two
// splitters and those at the upper one.
__global__ __launch_bounds__(kKsCount) void ks_split(int64_t n, int64_t ld, const double* __restrict__ x, double lo,
                                                     double w, double scale, int per, void* ws, KsPlan p) {
    const KsView v = ks_view(ws, p, blockIdx.y);
    const int nh = (int)*v.nhuge();
    if (nh == 0) return;
    __shared__ double spl[kKsCount];
    __shared__ unsigned place[kKsSplit + kKsHuge], shu[kKsCount / 64], huge[kKsHuge];
    __shared__ double shd[kKsCount / 64];
    const double* xc = x + (int64_t)blockIdx.y * ld;
    const double dn = (double)n, ib = 1.0 / p.buckets;
    const int t = threadIdx.x, S = (int)v.huge_split()[nh];
    spl[t] = t < S ? v.splitter()[t] : __builtin_inf();
    if (t < nh) huge[t] = v.huge_bucket()[t];
    __syncthreads();
    const bool mine = t < S + nh;
    int h = 0;
    for (int k = 1; k < nh; ++k)
        if (t >= (int)v.huge_split()[k] + k) h = k;
    const int i = t - h, first = (int)v.huge_split()[h], end = (int)v.huge_split()[h + 1], b = (int)huge[h];
    const unsigned open = mine ? v.between()[t] : 0u, at = mine && i < end ? v.at_split()[i] : 0u;
    unsigned total;
    const unsigned r0 = block_scan(open + at, shu, total) - v.huge_values()[h] + v.count()[b];
    double d = 0.0;
    if (at) {
        const double F = ks_F(spl[i], lo, w);
        d = __builtin_fmax(ks_up((int64_t)r0 + open + at - 1, dn, F), ks_down((int64_t)r0 + open, dn, F));
    }
    d = wave_max(__builtin_fmax(d, 0.0));
    if ((t & 63) == 0) shd[t >> 6] = d;
    __syncthreads();
    double best = 0.0;
    for (int k = 0; k < kKsCount / 64; ++k) best = __builtin_fmax(best, shd[k]);
    // bounds of the values between, from the splitters' F and the bucket's edges
    bool take = false;
    if (open) {
        const double fl = i > first ? ks_F(spl[i - 1], lo, w) : ks_bucket_lo(b, ib);
        const double fh = i < end ? ks_F(spl[i], lo, w) : ks_bucket_hi(b, p.buckets, ib);
        take = ks_up((int64_t)r0 + open - 1, dn, fl) > best || ks_down((int64_t)r0, dn, fh) > best;
    }
    // a bucket's range of the list has room for all of its values: they lie in it
    // as those between the splitters do, r0 - count[b] from its start
    unsigned recs;
    const unsigned rec = block_scan(take ? 1u : 0u, shu, recs), to = v.slot()[b] + r0 - v.count()[b];
    if (mine) place[t] = take ? to : kKsNone;
    if (blockIdx.x == 0) {
        if (take) {
            unsigned* out = v.part(0) + 3 * rec;
            out[0] = open;
            out[1] = r0;
            out[2] = to;
        }
        if (t == 0) {
            *v.nsub() = recs;
            if (best > 0.0) atomicMax(v.dmax(), (unsigned long long)__double_as_longlong(best));
        }
    }
    if (recs == 0) return;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * per + t;
    constexpr int kAhead = 4;
    for (int k0 = 0; k0 < per / kKsCount; k0 += kAhead) {
        double u[kAhead];
        int pl[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) u[k] = i0 + (k0 + k) * kKsCount < n ? xc[i0 + (k0 + k) * kKsCount] : 0.0;
        ks_place(spl, u, pl);
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const unsigned bu = ks_bucket(u[k], lo, scale, p.buckets);
            int hu = -1;
            for (int g = 0; g < nh; ++g) hu = huge[g] == bu ? g : hu;
            if (i0 + (k0 + k) * kKsCount >= n || hu < 0 || (pl[k] < S && spl[pl[k]] == u[k])) continue;
            const unsigned at0 = place[pl[k] + hu];
            if (at0 != kKsNone) v.list()[at0 + atomicAdd(&v.taken()[pl[k] + hu], 1u)] = u[k];
        }
    }
}

// The largest deviation in the ranges of one component, range(k, m, r0) giving
// the m values of the k-th and their first rank (m = 0: none to take): a wave a
// range, dealt to the blocks in turn (a block of 16 waves on 16 candidates left
// half the CUs idle: 20 us against 12 for 3 x 2^20 values), and the block its
// ranges that are too large for one; each wave's maximum, in every lane.
template <class Range>
__device__ __forceinline__ double ks_solve_block(KsRefine& R, int count, Range&& range, double dn, double lo, double w,
                                                 int block, int blocks) {
    constexpr int kWaves = kKsCount / 64;
    double d = 0.0;
    const int wave = threadIdx.x >> 6;
    // with a range for each wave none waits for one that takes long
    const int own = count < blocks * kWaves ? kKsWave : kKsBlock;
    if (threadIdx.x == 0) { R.nmid = 0u; R.nbig = 0u; }
    __syncthreads();
    for (int k = wave * blocks + block; k < count; k += blocks * kWaves) {
        int m;
        int64_t r0;
        const double* l = range(k, m, r0);
        if (m > own) {                            // at most 17,407 / 64 of a block, or 1024
            if ((threadIdx.x & 63) == 0)
                R.later[m > kKsBlock ? kKsCount - 1 - atomicAdd(&R.nbig, 1u) : atomicAdd(&R.nmid, 1u)] = k;
        } else if (m > 0) {
            d = __builtin_fmax(d, ks_ranked(l, m, r0, dn, lo, w, 0, 64));
        }
    }
    __syncthreads();
    // a few of up to kKsBlock values: by all waves, one after the other (256 to 512
    // values take a wave 4 to 8 times as long); more of them: a wave each
    const int nmid = (int)R.nmid, nbig = (int)R.nbig;
    const bool each = nmid > 4;
    for (int k = each ? wave : 0; k < nmid; k += each ? kWaves : 1) {
        int m;
        int64_t r0;
        const double* l = range(R.later[k], m, r0);
        d = __builtin_fmax(d, ks_ranked(l, m, r0, dn, lo, w, each ? 0 : 64 * wave, each ? 64 : kKsCount));
    }
    for (int k = 0; k < nbig; ++k) {
        int m;
        int64_t r0;
        const double* l = range(R.later[kKsCount - 1 - k], m, r0);
        d = __builtin_fmax(d, ks_refine(R, l, m, r0, dn, lo, w));
    }
    return wave_max(d);
}

__device__ double kolmogorov_sf(double lam);

__global__ __launch_bounds__(kKsCount) void ks_solve(int64_t n, double lo, double w, void* ws, KsPlan p,
                                                     double* __restrict__ out) {
    __shared__ KsRefine R;
    const KsView v = ks_view(ws, p, blockIdx.y);
    const int ncand = (int)*v.ncand();
    const int64_t most = ks_huge_min(n);
    const auto range = [&](int k, int& m, int64_t& r0) -> const double* {
        if (k < ncand) {
            const unsigned b = v.cand()[k];
            r0 = v.count()[b];
            m = (int)(v.count()[b + 1] - v.count()[b]);
            if (m > most) m = 0;                      // ks_split's
            return v.list() + v.slot()[b];
        }
        const unsigned* r = v.part(0) + 3 * (k - ncand);
        m = (int)r[0];
        r0 = r[1];
        return v.list() + r[2];
    };
    double d = ks_solve_block(R, ncand + (int)*v.nsub(), range, (double)n, lo, w, blockIdx.x, gridDim.x);
    // non-negative doubles order as their bits; one atomic a block (one a wave
    // made 1024 wait for one word)
    __syncthreads();
    if ((threadIdx.x & 63) == 0) R.red[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 0; k < kKsCount / 64; ++k) d = __builtin_fmax(d, R.red[k]);
    if (d > 0.0) atomicMax(v.dmax(), (unsigned long long)__double_as_longlong(d));
    // the last block has D
    __threadfence();
    if (atomicAdd(v.done(), 1u) != gridDim.x - 1) return;
    __threadfence();
    d = __longlong_as_double((long long)atomicMax(v.dmax(), 0ull));
    out[2 * blockIdx.y] = d;
    out[2 * blockIdx.y + 1] = kolmogorov_sf(sqrt((double)n) * d);
}

// The whole test of a sample that one block counts (at most kKsPerBlock
// values, 1024 buckets), in one launch: the tables in LDS, the candidates'
// values in the workspace (3 x 4,099 values: five launches 23 us, this 11 us).
__global__ __launch_bounds__(kKsCount) void ks_one(int64_t n, int64_t ld, const double* __restrict__ x, double lo,
                                                   double w, double scale, void* ws, KsPlan p,
                                                   double* __restrict__ out) {
    __shared__ KsRefine R;
    __shared__ unsigned count[kKsCount + 1], slot[kKsCount], cand[kKsCount], shu[kKsCount / 64];
    __shared__ double shd[kKsCount / 64];
    constexpr int kKeep = kKsPerBlock / kKsCount;
    const KsView v = ks_view(ws, p, blockIdx.x);
    const double* xc = x + (int64_t)blockIdx.x * ld;
    double* list = v.list();
    double val[kKeep];
#pragma unroll
    for (int k = 0; k < kKeep; ++k) {
        const int i = k * kKsCount + threadIdx.x;
        val[k] = i < n ? xc[i] : 0.0;
    }
    count[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kKeep; ++k)
        if (k * kKsCount + (int)threadIdx.x < n) atomicAdd(&count[ks_bucket(val[k], lo, scale, kKsCount)], 1u);
    __syncthreads();
    const int ncand = ks_scan_block<1>(n, count, slot, R.below[0], cand, kKsCount, shu, shd);      // R.below[0]: the next place
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kKeep; ++k)
        if (k * kKsCount + (int)threadIdx.x < n) {
            const int b = ks_bucket(val[k], lo, scale, kKsCount);
            if (slot[b] != kKsNone) list[atomicAdd(&R.below[0][b], 1u)] = val[k];
        }
    __syncthreads();
    const auto range = [&](int k, int& m, int64_t& r0) -> const double* {
        const unsigned b = cand[k];
        r0 = count[b];
        m = (int)(count[b + 1] - count[b]);
        return list + slot[b];
    };
    double d = ks_solve_block(R, ncand, range, (double)n, lo, w, 0, 1);
    if ((threadIdx.x & 63) == 0) shd[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 0; k < kKsCount / 64; ++k) d = __builtin_fmax(d, shd[k]);
    out[2 * blockIdx.x] = d;
    out[2 * blockIdx.x + 1] = kolmogorov_sf(sqrt((double)n) * d);
}

// the deviations of a sorted copy, for samples the buckets do not serve
__global__ __launch_bounds__(kBlock) void ks_kernel(int64_t n, const double* __restrict__ xs, double lo, double hi,
                                                    double* __restrict__ part) {
    __shared__ double sh[kBlock];
    const double w = hi - lo;
    const double dn = (double)n;
    double d = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)kPart * kBlock) {
        const double F = ks_F(xs[i], lo, w);
        d = __builtin_fmax(d, __builtin_fmax(ks_up(i, dn, F), ks_down(i, dn, F)));
    }
    d = block_max(d, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = d;
}

// P(K > lam): alternating series for lam >= 1, theta-function form below.  The
// terms fall so fast that the sum is complete once one does not change it
// (after at most five; all 100 took 18 us).
__device__ double kolmogorov_sf(double lam) {
    if (!(lam > 0.0)) return 1.0;
    const double pi = 3.14159265358979323846;
    double s = 0.0;
    if (lam >= 1.0) {
        for (int k = 1; k <= 100; ++k) {
            const double t = s + ((k & 1) ? 2.0 : -2.0) * exp(-2.0 * (double)k * (double)k * lam * lam);
            if (t == s) break;
            s = t;
        }
        return s < 0.0 ? 0.0 : (s > 1.0 ? 1.0 : s);
    }
    for (int k = 1; k <= 100; ++k) {
        const double m = (double)(2 * k - 1);
        const double t = s + exp(-(m * m) * (pi * pi) / (8.0 * lam * lam));
        if (t == s) break;
        s = t;
    }
    const double p = 1.0 - sqrt(2.0 * pi) / lam * s;
    return p < 0.0 ? 0.0 : (p > 1.0 ? 1.0 : p);
}

// D and the p-value from the partial maxima
__global__ __launch_bounds__(64) void ks_final_kernel(int64_t n, const double* __restrict__ part,
                                                      double* __restrict__ out) {
    double d = 0.0;
    for (int b = threadIdx.x; b < kPart; b += 64) d = __builtin_fmax(d, part[b]);
    d = wave_max(d);
    if (threadIdx.x != 0) return;
    out[0] = d;
    out[1] = kolmogorov_sf(sqrt((double)n) * d);
}

__global__ void fill_nan(double* p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = __builtin_nan("");
}

int launched() { return hipGetLastError() == hipSuccess ? PN_OK : PN_EHIP; }

bool bad_common(int64_t n, int64_t ld, int32_t ncomp) {
    return n < 0 || ld < n || ld > PN_MAX_N || ncomp < 1 || ncomp > kMaxComp;
}

size_t radix_temp_bytes(int64_t n) {
    size_t bytes = 0;
    if (n <= 0) return 0;
    if (rocprim::radix_sort_keys(nullptr, bytes, (const double*)nullptr, (double*)nullptr, (size_t)n) != hipSuccess)
        return 0;
    return bytes;
}

}  // namespace
}  // namespace pn

using namespace pn;

extern "C" {

int pn_histogram(int64_t n, int64_t ld, const double* x, int32_t ncomp, int32_t nbins, double lo, double hi,
                 int64_t* counts, void* stream) {
    if (bad_common(n, ld, ncomp) || nbins < 1 || nbins > 4096 || !(lo < hi) || !std::isfinite(lo) ||
        !std::isfinite(hi) || !counts || (n > 0 && !x))
        return PN_EINVAL;
    const int rc = device_ready();
    if (rc != PN_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    const unsigned blocks = hist_blocks(n);
    if (n == 0 || blocks > 1)
        hipLaunchKernelGGL(zero_i64, dim3(64), dim3(kBlock), 0, s, counts, (int64_t)ncomp * nbins);
    if (n > 0) {
        const double step = (hi - lo) / nbins;
        const int copies = hist_copies(nbins);
        hipLaunchKernelGGL(hist_kernel, dim3(blocks, ncomp), dim3(kHistBlock), nbins * copies * sizeof(unsigned), s, n,
                           ld, x, (int)nbins, copies, lo, hi, step, 1.0 / step, hist_near(lo, hi, step),
                           counts);
    }
    return launched();
}

int pn_histogram2d(int64_t n, int64_t ld, const double* x, const double* y, int32_t ncomp, int32_t nbins,
                   double lo, double hi, int64_t* counts, void* stream) {
    if (bad_common(n, ld, ncomp) || nbins < 1 || nbins > 128 || !(lo < hi) || !std::isfinite(lo) ||
        !std::isfinite(hi) || !counts || (n > 0 && (!x || !y)))
        return PN_EINVAL;
    const int rc = device_ready();
    if (rc != PN_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    const unsigned blocks = hist_blocks(n);
    if (n == 0 || blocks > 1)
        hipLaunchKernelGGL(zero_i64, dim3(64), dim3(kBlock), 0, s, counts, (int64_t)ncomp * nbins * nbins);
    if (n > 0) {
        const double step = (hi - lo) / nbins;
        hipLaunchKernelGGL(hist2d_kernel, dim3(blocks, ncomp), dim3(kHistBlock),
                           (size_t)nbins * nbins * sizeof(unsigned), s, n, ld, x, y, (int)nbins, lo, hi, step,
                           1.0 / step, hist_near(lo, hi, step), counts);
    }
    return launched();
}

size_t pn_stats_workspace_bytes(int64_t n, int32_t ncomp, int32_t ngrid) {
    if (n < 0 || n > PN_MAX_N || ncomp < 1 || ncomp > kMaxComp || ngrid < 0) return 0;
    const size_t pearson = ((size_t)ncomp * kPart * 3 + (size_t)ncomp * 2) * sizeof(double);
    const size_t kde = (size_t)ncomp * kPart * (size_t)ngrid * sizeof(double);
    return pearson > kde ? pearson : kde;
}

int pn_pearson(int64_t n, int64_t ld, const double* x, const double* y, int32_t ncomp, double* out,
               void* workspace, size_t ws_bytes, void* stream) {
    if (bad_common(n, ld, ncomp) || !out || (n > 0 && (!x || !y))) return PN_EINVAL;
    if (!workspace || ws_bytes < pn_stats_workspace_bytes(n, ncomp, 0)) return PN_EINVAL;
    const int rc = device_ready();
    if (rc != PN_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) {
        hipLaunchKernelGGL(fill_nan, dim3(1), dim3(kBlock), 0, s, out, (int)(ncomp * 5));
        return launched();
    }
    if (n <= kPearOne) {
        hipLaunchKernelGGL(pearson_one_kernel, dim3(ncomp), dim3(kPearOneBlock), 0, s, n, ld, x, y, out);
        return launched();
    }
    const int64_t chunks = (n + kPearChunk - 1) / kPearChunk;
    const int parts = chunks < kPearParts ? (int)chunks : kPearParts;
    PearPart* part = (PearPart*)workspace;
    hipLaunchKernelGGL(pearson_part_kernel, dim3(parts, ncomp), dim3(kPearBlock), 0, s, n, ld, x, y, part);
    hipLaunchKernelGGL(pearson_final_kernel, dim3(ncomp), dim3(kPearParts), 0, s, n, parts, part, out);
    return launched();
}

int pn_kde(int64_t n, int64_t ld, const double* x, int32_t ncomp, const double* sigma, int64_t sigma_stride,
           int32_t ngrid, double lo, double hi, double* out, void* workspace, size_t ws_bytes, void* stream) {
    if (bad_common(n, ld, ncomp) || ngrid < 2 || ngrid > 4096 || !(lo < hi) || !std::isfinite(lo) ||
        !std::isfinite(hi) || !out || !sigma || sigma_stride < 1 || (n > 0 && !x))
        return PN_EINVAL;
    if (!workspace || ws_bytes < pn_stats_workspace_bytes(n, ncomp, ngrid)) return PN_EINVAL;
    const int rc = device_ready();
    if (rc != PN_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) {
        hipLaunchKernelGGL(fill_nan, dim3((ncomp * ngrid + kBlock - 1) / kBlock), dim3(kBlock), 0, s, out,
                           (int)(ncomp * ngrid));
        return launched();
    }
    const double nfac = std::pow((double)n, -0.2);
    const double gstep = (hi - lo) / (ngrid - 1);
    const double sqrt2pi = std::sqrt(2.0 * 3.14159265358979323846);
    double* part = (double*)workspace;
    const int tiles = (ngrid + kKdeTile - 1) / kKdeTile;
    const int parts = kde_parts(n, ncomp, tiles);
    hipLaunchKernelGGL(kde_kernel, dim3(parts, ncomp, tiles), dim3(kBlock), 0, s, n, ld, x, sigma, sigma_stride, nfac,
                       (int)ngrid, lo, hi - lo, gstep, part);
    hipLaunchKernelGGL(kde_final_kernel, dim3((ngrid + 15) / 16, ncomp), dim3(kBlock), 0, s, n, sigma, sigma_stride,
                       nfac, sqrt2pi, (int)ngrid, parts, hi - lo, gstep, part, out);
    return launched();
}

// The sorted path's workspace: sorted copy, sort scratch (256-byte aligned),
// partial maxima; 0 where the sort's own scratch size is not known.
static size_t ks_sort_bytes(int64_t n) {
    const size_t tmp = radix_temp_bytes(n);
    if (n > 0 && tmp == 0) return 0;
    return ((size_t)n * sizeof(double) + 255) / 256 * 256 + (tmp + 255) / 256 * 256 + kPart * sizeof(double);
}

size_t pn_ks_workspace_bytes(int64_t n) {
    if (n < 0 || n > PN_MAX_N) return 0;
    const size_t sort = ks_sort_bytes(n);
    if (sort == 0 || n == 0 || n > kKsBucketMax) return sort;
    // three components (the scalar products) side by side
    const size_t buckets = 3 * (size_t)ks_plan(n).bytes;
    return buckets > sort ? buckets : sort;
}

int pn_ks_uniform(int64_t n, int64_t ld, const double* x, int32_t ncomp, double lo, double hi, double* out,
                  void* workspace, size_t ws_bytes, void* stream) {
    if (bad_common(n, ld, ncomp) || !(lo < hi) || !std::isfinite(lo) || !std::isfinite(hi) || !out ||
        (n > 0 && !x))
        return PN_EINVAL;
    const int rc = device_ready();
    if (rc != PN_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) {
        hipLaunchKernelGGL(fill_nan, dim3(1), dim3(kBlock), 0, s, out, (int)(ncomp * 2));
        return launched();
    }
    const size_t need = ks_sort_bytes(n);
    if (need == 0 || !workspace || ws_bytes < need) return PN_EINVAL;
    const double w = hi - lo;
    if (n <= kKsBucketMax && w > 1e-290 && w < 1e290) {
        const KsPlan p = ks_plan(n);
        const int side = (int)(ws_bytes / (size_t)p.bytes < (size_t)ncomp ? ws_bytes / (size_t)p.bytes : (size_t)ncomp);
        if (side > 0 && ((uintptr_t)workspace & 15) == 0) {
            const double scale = p.buckets / w;
            for (int c = 0; c < ncomp; c += side) {
                const int g = ncomp - c < side ? ncomp - c : side;
                const double* xc = x + (int64_t)c * ld;
                if (p.blocks == 1) {
                    hipLaunchKernelGGL(ks_one, dim3(g), dim3(kKsCount), 0, s, n, ld, xc, lo, w, scale, workspace, p,
                                       out + 2 * c);
                    continue;
                }
                hipLaunchKernelGGL(ks_count, dim3(p.blocks, g), dim3(kKsCount), p.buckets * sizeof(unsigned), s, n, ld,
                                   xc, lo, scale, workspace, p);
                hipLaunchKernelGGL(ks_sum, dim3(p.buckets / kBlock, g), dim3(kBlock), 0, s, workspace, p);
                hipLaunchKernelGGL(ks_scan, dim3(g), dim3(kKsCount), 0, s, n, ld, xc, lo, scale, workspace, p);
                hipLaunchKernelGGL(ks_collect, dim3(p.blocks, g), dim3(kKsCount), p.buckets * sizeof(unsigned), s, n,
                                   ld, xc, lo, scale, workspace, p);
                const int per = n <= 262144 ? kKsPerBlock / 4 : kKsPerBlock;
                hipLaunchKernelGGL(ks_split, dim3((unsigned)((n + per - 1) / per), g), dim3(kKsCount), 0, s, n, ld, xc, lo,
                                   w, scale, per, workspace, p);
                hipLaunchKernelGGL(ks_solve, dim3(64, g), dim3(kKsCount), 0, s, n, lo, w, workspace, p, out + 2 * c);
            }
            return launched();
        }
    }
    char* wp = (char*)workspace;
    double* sorted = (double*)wp;
    size_t off = ((size_t)n * sizeof(double) + 255) / 256 * 256;
    void* tmp = wp + off;
    size_t tmp_bytes = radix_temp_bytes(n);
    off += (tmp_bytes + 255) / 256 * 256;
    double* part = (double*)(wp + off);
    for (int c = 0; c < ncomp; ++c) {
        if (rocprim::radix_sort_keys(tmp, tmp_bytes, x + (int64_t)c * ld, sorted, (size_t)n, 0, 64, s) != hipSuccess)
            return PN_EHIP;
        hipLaunchKernelGGL(ks_kernel, dim3(kPart), dim3(kBlock), 0, s, n, sorted, lo, hi, part);
        hipLaunchKernelGGL(ks_final_kernel, dim3(1), dim3(64), 0, s, n, part, out + 2 * c);
    }
    return launched();
}

}  // extern "C"
