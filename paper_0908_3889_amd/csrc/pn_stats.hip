// pn_stats.hip -- the statistics of Sec. V over per-inspiral values on the
// GPU: equal-width and bivariate histograms, the Pearson coefficient, the
// Gaussian kernel density estimator with Silverman's bandwidth, and the
// Kolmogorov-Smirnov statistic against the uniform law.
//
// Every reduction runs over a fixed grid of kPart partial results combined
// in a fixed order, so results do not depend on the device's size or on
// scheduling.  Histogram counts use integer atomics (order-free).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include <rocprim/device/device_radix_sort.hpp>

#include "pn.h"

namespace pn {

int device_ready();   // pn_lib.hip: PN_OK when a gfx950 device is current

namespace {

constexpr int kBlock = 256;
constexpr int kPart = 512;          // partial results per component
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

// the bin of lo <= v <= hi: an estimate from the quotient, corrected against
// the edges themselves
__device__ __forceinline__ int bin_of(double v, int nbins, double lo, double hi, double step) {
    int b = (int)((v - lo) / step);
    b = b < 0 ? 0 : (b > nbins - 1 ? nbins - 1 : b);
    while (b > 0 && v < edge(b, nbins, lo, hi, step)) --b;
    while (b < nbins - 1 && v >= edge(b + 1, nbins, lo, hi, step)) ++b;
    return b;
}

__global__ void zero_i64(int64_t* p, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__global__ __launch_bounds__(kBlock) void hist_kernel(int64_t n, int64_t ld, const double* __restrict__ x, int nbins,
                                                      double lo, double hi, double step, int64_t* __restrict__ counts) {
    extern __shared__ unsigned int sh[];
    const int c = blockIdx.y;
    for (int b = threadIdx.x; b < nbins; b += kBlock) sh[b] = 0u;
    __syncthreads();
    const double* xc = x + (int64_t)c * ld;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        const double v = xc[i];
        if (v >= lo && v <= hi) atomicAdd(&sh[bin_of(v, nbins, lo, hi, step)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nbins; b += kBlock)
        if (sh[b]) atomicAdd((unsigned long long*)&counts[(int64_t)c * nbins + b], (unsigned long long)sh[b]);
}

__global__ __launch_bounds__(kBlock) void hist2d_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                        const double* __restrict__ y, int nbins, double lo, double hi,
                                                        double step, int64_t* __restrict__ counts) {
    extern __shared__ unsigned int sh[];
    const int c = blockIdx.y;
    const int nb2 = nbins * nbins;
    for (int b = threadIdx.x; b < nb2; b += kBlock) sh[b] = 0u;
    __syncthreads();
    const double* xc = x + (int64_t)c * ld;
    const double* yc = y + (int64_t)c * ld;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        const double u = xc[i], v = yc[i];
        if (u >= lo && u <= hi && v >= lo && v <= hi)
            atomicAdd(&sh[bin_of(u, nbins, lo, hi, step) * nbins + bin_of(v, nbins, lo, hi, step)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb2; b += kBlock)
        if (sh[b]) atomicAdd((unsigned long long*)&counts[(int64_t)c * nb2 + b], (unsigned long long)sh[b]);
}

// ---------------------------------------------------------------------------
// fixed-order block reductions
// ---------------------------------------------------------------------------

template <int K>
__device__ __forceinline__ void block_sum(double (&v)[K], double (*sh)[kBlock]) {
#pragma unroll
    for (int k = 0; k < K; ++k) sh[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
#pragma unroll
            for (int k = 0; k < K; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + s];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = sh[k][0];
    __syncthreads();
}

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
// Pearson: pass 1 sums, pass 2 centred sums (workspace: part[c][kPart][3],
// then mean[c][2])
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void sums_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                      const double* __restrict__ y, double* __restrict__ part) {
    __shared__ double sh[2][kBlock];
    const int c = blockIdx.y;
    const double* xc = x + (int64_t)c * ld;
    const double* yc = y + (int64_t)c * ld;
    double v[2] = {0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)kPart * kBlock) {
        v[0] += xc[i];
        v[1] += yc[i];
    }
    block_sum<2>(v, sh);
    if (threadIdx.x == 0) {
        part[((int64_t)c * kPart + blockIdx.x) * 3 + 0] = v[0];
        part[((int64_t)c * kPart + blockIdx.x) * 3 + 1] = v[1];
    }
}

__global__ __launch_bounds__(kBlock) void means_kernel(int64_t n, const double* __restrict__ part,
                                                       double* __restrict__ mean) {
    __shared__ double sh[2][kBlock];
    const int c = blockIdx.x;
    double v[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < kPart; b += kBlock) {
        v[0] += part[((int64_t)c * kPart + b) * 3 + 0];
        v[1] += part[((int64_t)c * kPart + b) * 3 + 1];
    }
    block_sum<2>(v, sh);
    if (threadIdx.x == 0) {
        mean[c * 2 + 0] = v[0] / (double)n;
        mean[c * 2 + 1] = v[1] / (double)n;
    }
}

__global__ __launch_bounds__(kBlock) void centred_kernel(int64_t n, int64_t ld, const double* __restrict__ x,
                                                         const double* __restrict__ y, const double* __restrict__ mean,
                                                         double* __restrict__ part) {
    __shared__ double sh[3][kBlock];
    const int c = blockIdx.y;
    const double* xc = x + (int64_t)c * ld;
    const double* yc = y + (int64_t)c * ld;
    const double mx = mean[c * 2], my = mean[c * 2 + 1];
    double v[3] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)kPart * kBlock) {
        const double dx = xc[i] - mx, dy = yc[i] - my;
        v[0] += dx * dx;
        v[1] += dy * dy;
        v[2] += dx * dy;
    }
    block_sum<3>(v, sh);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) part[((int64_t)c * kPart + blockIdx.x) * 3 + k] = v[k];
    }
}

__global__ __launch_bounds__(kBlock) void pearson_final_kernel(int64_t n, const double* __restrict__ part,
                                                               const double* __restrict__ mean, double* __restrict__ out) {
    __shared__ double sh[3][kBlock];
    const int c = blockIdx.x;
    double v[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < kPart; b += kBlock) {
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] += part[((int64_t)c * kPart + b) * 3 + k];
    }
    block_sum<3>(v, sh);
    if (threadIdx.x == 0) {
        const double nm1 = (double)(n - 1);
        out[c * 5 + 0] = mean[c * 2];
        out[c * 5 + 1] = mean[c * 2 + 1];
        out[c * 5 + 2] = sqrt(v[0] / nm1);
        out[c * 5 + 3] = sqrt(v[1] / nm1);
        out[c * 5 + 4] = v[2] / sqrt(v[0] * v[1]);
    }
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
// the third multiplies the finished sums.  That leaves one exponential per
// (point, segment) instead of one per (point, grid point).  Bound by the FP64
// units: about 26 vector instructions (104 cycles) per 64 of those factors and
// 64 cycles for their matrix instruction, which share them.
//
// The first factor is carried as 2^320 times its value: an anchor up to 45 h
// from a point still has a normal number there, so that a grid point 8 d
// closer is exact down to the smallest density a double holds.  The products
// stay in range for d <= 5/8 (the third factor is then at least exp(-413))
// and (hi - lo)/h . d <= 37 (the second is at most exp(296) inside [lo, hi]);
// v d is clamped to +-75, which only points whose first factor is 0
// everywhere exceed.  Other grids (a step coarse against the bandwidth, or a
// bandwidth that is 0 or not a number) take one exponential per (point, grid
// point).  On 2^20 x 3 points and 201
// grid points that path takes 0.76 ms, the products 0.074 ms.
// ---------------------------------------------------------------------------

__device__ __forceinline__ double kde_h(const double* sigma, int64_t stride, int c, double nfac) {
    return (1.06 * sigma[(int64_t)c * stride]) * nfac;
}

constexpr int kKdeTile = 256;       // grid points of a block
constexpr int kKdeRow = 18;         // LDS row of a point: 16 powers, v, padding (16-byte multiples)

__device__ __forceinline__ bool kde_products(double ih, double gstep, double span) {
    const double d = gstep * ih;
    return d <= 0.625 && (span * ih) * d <= 37.0;
}

// 2^(t + kKdeScale) for t <= 0 (0 below t = -1395, NaN for NaN): the polynomial
// interpolates 2^f on [-1/2, 1/2] at its Chebyshev nodes, formed in 50-digit
// arithmetic (largest error 3.2e-18).
constexpr int kKdeScale = 320;

__device__ __forceinline__ double exp2_scaled(double t) {
    t = t < -1500.0 ? -1500.0 : t;
    const double k = __builtin_rint(t);
    const double f = t - k;
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
    return __builtin_amdgcn_ldexp(p, (int)k + kKdeScale);
}

typedef double double4_t __attribute__((ext_vector_type(4)));

// Chunks of 64 points are dealt to the waves of all blocks in turn.
__device__ __forceinline__ void kde_block_products(int64_t n, const double* __restrict__ xc, double ih, double d,
                                                   double gmid, double* sh, int ngrid, int g0,
                                                   double* __restrict__ out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double (*row)[kKdeRow] = (double (*)[kKdeRow])sh + wave * 64;
    const double m = 16.0 * (double)((lane & 15) - 8);
    const int64_t chunks = (n + 63) / 64;
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    for (int64_t ch = (int64_t)blockIdx.x * (kBlock / 64) + wave; ch < chunks;
         ch += (int64_t)gridDim.x * (kBlock / 64)) {
        const int64_t i = ch * 64 + lane;
        // beyond the end: a point at infinity, whose first factor is 0
        const double x = i < n ? xc[i] : __builtin_inf();
        const double v = (gmid - x) * ih;
        double a = v * d;
        a = __builtin_fmin(__builtin_fmax(a, -75.0), 75.0);
        const double p1 = exp(-a), q1 = exp(a);
        const double p2 = p1 * p1, p3 = p2 * p1, p4 = p2 * p2, q2 = q1 * q1, q3 = q2 * q1, q4 = q2 * q2;
        double2* r = (double2*)row[lane];
        r[0] = make_double2(q4 * q4, q4 * q3);
        r[1] = make_double2(q3 * q3, q4 * q1);
        r[2] = make_double2(q4, q3);
        r[3] = make_double2(q2, q1);
        r[4] = make_double2(1.0, p1);
        r[5] = make_double2(p2, p3);
        r[6] = make_double2(p4, p4 * p1);
        r[7] = make_double2(p3 * p3, p4 * p3);
        row[lane][16] = v;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
            const double* rq = row[4 * q + (lane >> 4)];
            const double u = __builtin_fma(m, d, rq[16]);
            const double e = exp2_scaled((u * u) * -0.72134752044448170368);     // -(log2 e)/2
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(e, rq[lane & 15], acc, 0, 0, 0);
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
// blocks of a CU that fit its LDS), no more than one chunk of 64 points a
// wave needs; from the sizes alone, so that results do not depend on the device.
int kde_parts(int64_t n, int ncomp, int tiles) {
    const int64_t fill = 1024 / ((int64_t)ncomp * tiles);
    const int64_t need = ((n + 63) / 64 + kBlock / 64 - 1) / (kBlock / 64);
    int64_t p = need < fill ? need : fill;
    p = p < 16 ? (need < 16 ? need : 16) : p;
    return (int)(p > kPart ? kPart : p);
}

// ---------------------------------------------------------------------------
// Kolmogorov-Smirnov against U[lo, hi] on a sorted copy
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void ks_kernel(int64_t n, const double* __restrict__ xs, double lo, double hi,
                                                    double* __restrict__ part) {
    __shared__ double sh[kBlock];
    const double w = hi - lo;
    const double dn = (double)n;
    double d = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)kPart * kBlock) {
        const double F = (xs[i] - lo) / w;
        const double up = (double)(i + 1) / dn - F;
        const double dw = F - (double)i / dn;
        d = __builtin_fmax(d, __builtin_fmax(up, dw));
    }
    d = block_max(d, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = d;
}

// P(K > lam): alternating series for lam >= 1, theta-function form below
__device__ double kolmogorov_sf(double lam) {
    if (!(lam > 0.0)) return 1.0;
    const double pi = 3.14159265358979323846;
    double s = 0.0;
    if (lam >= 1.0) {
        for (int k = 1; k <= 100; ++k)
            s += ((k & 1) ? 2.0 : -2.0) * exp(-2.0 * (double)k * (double)k * lam * lam);
        return s < 0.0 ? 0.0 : (s > 1.0 ? 1.0 : s);
    }
    for (int k = 1; k <= 100; ++k) {
        const double m = (double)(2 * k - 1);
        s += exp(-(m * m) * (pi * pi) / (8.0 * lam * lam));
    }
    const double p = 1.0 - sqrt(2.0 * pi) / lam * s;
    return p < 0.0 ? 0.0 : (p > 1.0 ? 1.0 : p);
}

__global__ void ks_final_kernel(int64_t n, const double* __restrict__ part, double* __restrict__ out) {
    if (threadIdx.x != 0) return;
    double d = 0.0;
    for (int b = 0; b < kPart; ++b) d = __builtin_fmax(d, part[b]);
    out[0] = n > 0 ? d : __builtin_nan("");
    out[1] = n > 0 ? kolmogorov_sf(sqrt((double)n) * d) : __builtin_nan("");
}

__global__ void fill_nan(double* p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = __builtin_nan("");
}

int launched() { return hipGetLastError() == hipSuccess ? PN_OK : PN_EHIP; }

bool bad_common(int64_t n, int64_t ld, int32_t ncomp) {
    return n < 0 || ld < n || ld > PN_MAX_N || ncomp < 1 || ncomp > kMaxComp;
}

unsigned blocks_for(int64_t n) {
    const int64_t b = (n + kBlock - 1) / kBlock;
    return (unsigned)(b < 1 ? 1 : (b > 1024 ? 1024 : b));
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
    hipLaunchKernelGGL(zero_i64, dim3(64), dim3(kBlock), 0, s, counts, (int64_t)ncomp * nbins);
    if (n > 0) {
        const double step = (hi - lo) / nbins;
        hipLaunchKernelGGL(hist_kernel, dim3(blocks_for(n), ncomp), dim3(kBlock), nbins * sizeof(unsigned), s, n, ld, x,
                           (int)nbins, lo, hi, step, counts);
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
    hipLaunchKernelGGL(zero_i64, dim3(64), dim3(kBlock), 0, s, counts, (int64_t)ncomp * nbins * nbins);
    if (n > 0) {
        const double step = (hi - lo) / nbins;
        hipLaunchKernelGGL(hist2d_kernel, dim3(blocks_for(n), ncomp), dim3(kBlock),
                           (size_t)nbins * nbins * sizeof(unsigned), s, n, ld, x, y, (int)nbins, lo, hi, step, counts);
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
    double* part = (double*)workspace;
    double* mean = part + (size_t)ncomp * kPart * 3;
    hipLaunchKernelGGL(sums_kernel, dim3(kPart, ncomp), dim3(kBlock), 0, s, n, ld, x, y, part);
    hipLaunchKernelGGL(means_kernel, dim3(ncomp), dim3(kBlock), 0, s, n, part, mean);
    hipLaunchKernelGGL(centred_kernel, dim3(kPart, ncomp), dim3(kBlock), 0, s, n, ld, x, y, mean, part);
    hipLaunchKernelGGL(pearson_final_kernel, dim3(ncomp), dim3(kBlock), 0, s, n, part, mean, out);
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

size_t pn_ks_workspace_bytes(int64_t n) {
    if (n < 0 || n > PN_MAX_N) return 0;
    const size_t tmp = radix_temp_bytes(n);
    if (n > 0 && tmp == 0) return 0;
    // sorted copy, sort scratch (256-byte aligned), partial maxima
    return ((size_t)n * sizeof(double) + 255) / 256 * 256 + (tmp + 255) / 256 * 256 + kPart * sizeof(double);
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
    const size_t need = pn_ks_workspace_bytes(n);
    if (need == 0 || !workspace || ws_bytes < need) return PN_EINVAL;
    char* w = (char*)workspace;
    double* sorted = (double*)w;
    size_t off = ((size_t)n * sizeof(double) + 255) / 256 * 256;
    void* tmp = w + off;
    size_t tmp_bytes = radix_temp_bytes(n);
    off += (tmp_bytes + 255) / 256 * 256;
    double* part = (double*)(w + off);
    for (int c = 0; c < ncomp; ++c) {
        if (rocprim::radix_sort_keys(tmp, tmp_bytes, x + (int64_t)c * ld, sorted, (size_t)n, 0, 64, s) != hipSuccess)
            return PN_EHIP;
        hipLaunchKernelGGL(ks_kernel, dim3(kPart), dim3(kBlock), 0, s, n, sorted, lo, hi, part);
        hipLaunchKernelGGL(ks_final_kernel, dim3(1), dim3(64), 0, s, n, part, out + 2 * c);
    }
    return launched();
}

}  // extern "C"
