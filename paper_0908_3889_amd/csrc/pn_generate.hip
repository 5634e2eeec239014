// pn_generate.hip -- initial data drawn on the GPU from the counter-based
// Philox4x64-10 generator (Salmon, Moraes, Dror & Shaw, SC11): masses,
// isotropic spins (Marsaglia's method) and initial frequencies, one lane per
// inspiral, each inspiral from its own counter range.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "pn.h"

namespace pn {

int device_ready();   // pn_lib.hip: PN_OK when a gfx950 device is current

namespace {

constexpr int kBlock = 256;
constexpr int kMaxAttempts = 64;

constexpr uint64_t kM0 = 0xD2E7470EE14C6C93ull, kM1 = 0xCA5A826395121157ull;
constexpr uint64_t kW0 = 0x9E3779B97F4A7C15ull, kW1 = 0xBB67AE8584CAA73Bull;

struct U4 {
    uint64_t x[4];
};

// a ^ b ^ c, one instruction per half
__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
    const unsigned lo = __builtin_amdgcn_bitop3_b32((unsigned)a, (unsigned)b, (unsigned)c, 0x96);
    const unsigned hi = __builtin_amdgcn_bitop3_b32((unsigned)(a >> 32), (unsigned)(b >> 32), (unsigned)(c >> 32), 0x96);
    return ((uint64_t)hi << 32) | lo;
}

// ten rounds of (x0, x1, x2, x3) -> (hi(M1 x2) ^ x1 ^ k0, lo(M1 x2),
// hi(M0 x0) ^ x3 ^ k1, lo(M0 x0)), the key advanced between rounds
__device__ __forceinline__ U4 philox(uint64_t c0, uint64_t c1, uint64_t k0, uint64_t k1) {
    uint64_t x0 = c0, x1 = c1, x2 = 0, x3 = 0;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) { k0 += kW0; k1 += kW1; }
        // both halves of a product from one set of multiply-adds (four; the
        // upper half and the product taken separately cost seven)
        const unsigned __int128 p0 = (unsigned __int128)kM0 * x0, p1 = (unsigned __int128)kM1 * x2;
        x0 = xor3((uint64_t)(p1 >> 64), x1, k0);
        x1 = (uint64_t)p1;
        x2 = xor3((uint64_t)(p0 >> 64), x3, k1);
        x3 = (uint64_t)p0;
    }
    return U4{{x0, x1, x2, x3}};
}

__device__ __forceinline__ double uniform(uint64_t w) { return (double)(w >> 11) * 0x1p-53; }

// 2 u - 1 of the uniform u = (w >> 11) 2^-53, from the two words of w >> 11:
// every partial sum is a multiple of 2^-52 of magnitude at most 1, so nothing
// is rounded
__device__ __forceinline__ double symmetric(uint64_t w) {
    const unsigned hi = (unsigned)(w >> 43), lo = (unsigned)(w >> 11);
    return __builtin_fma((double)hi, 0x1p-20, __builtin_fma((double)lo, 0x1p-52, -1.0));
}

// products and sums rounded one by one, as the definition writes them
__device__ __forceinline__ double affine(double lo, double hi, double u) {
#pragma clang fp contract(off)
    return lo + (hi - lo) * u;
}

// The two attempts of one block; true if one of them is accepted.
__device__ __forceinline__ bool sphere_block(uint64_t i, uint64_t block, uint64_t k0, double* s) {
#pragma clang fp contract(off)
    const U4 w = philox(i, block, k0, 0);
    const double a1 = symmetric(w.x[0]), a2 = symmetric(w.x[1]);
    const double b1 = symmetric(w.x[2]), b2 = symmetric(w.x[3]);
    const double qa = a1 * a1 + a2 * a2;
    const double qb = b1 * b1 + b2 * b2;
    const bool first = qa < 1.0;
    const double q = first ? qa : qb;
    const double r = 2.0 * sqrt(1.0 - (q < 1.0 ? q : 0.0));
    s[0] = (first ? a1 : b1) * r;
    s[1] = (first ? a2 : b2) * r;
    s[2] = 1.0 - 2.0 * q;
    return q < 1.0;
}

// The blocks of sphere `sphere` after its first, until an attempt is accepted.
__device__ __forceinline__ void sphere_rest(uint64_t i, int sphere, uint64_t k0, double* s) {
    const uint64_t first = 1 + (uint64_t)sphere * (kMaxAttempts / 2);
#pragma unroll 1
    for (int k = 1; k < kMaxAttempts / 2; ++k)
        if (sphere_block(i, first + (uint64_t)k, k0, s)) return;
    s[0] = 0.0; s[1] = 0.0; s[2] = 1.0;
}

// Every inspiral takes its first block of both spheres (4.6 % of the spheres
// have no accepted attempt there); the block collects the spheres that failed
// and its first lanes take their further blocks.  A wave that went on until
// its last lane was accepted drew 2.1 blocks a sphere.  Bound by the integer
// instructions of the Philox rounds (about 230 a block drawn) over the 96
// bytes written: 2^22 inspirals 150 us before, 106 us this way (the writes
// alone 65 us).
__global__ __launch_bounds__(kBlock) void generate_kernel(int64_t n, int64_t ld, int64_t first, pn_gen_spec sp,
                                                          double* __restrict__ m, double* __restrict__ S,
                                                          double* __restrict__ L, double* __restrict__ w0) {
#pragma clang fp contract(off)
    __shared__ double again[2][3][kBlock];
    __shared__ unsigned short queue[2 * kBlock];
    __shared__ unsigned count;
    const int tid = threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.x * kBlock;
    const int64_t j = j0 + tid;
    const uint64_t i = (uint64_t)(first + j);
    const uint64_t key = sp.seed;
    if (tid == 0) count = 0u;
    __syncthreads();
    double s[2][3];
    bool ok[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        ok[b] = sphere_block(i, 1 + (uint64_t)b * (kMaxAttempts / 2), key, s[b]) || j >= n;
        if (!ok[b]) queue[atomicAdd(&count, 1u)] = (unsigned short)(2 * tid + b);
    }
    __syncthreads();
    const int left = (int)count;
    for (int q = tid; q < left; q += kBlock) {
        const int t = queue[q] >> 1, b = queue[q] & 1;
        double v[3];
        sphere_rest((uint64_t)(first + j0 + t), b, key, v);
#pragma unroll
        for (int c = 0; c < 3; ++c) again[b][c][t] = v[c];
    }
    __syncthreads();
    if (j >= n) return;
#pragma unroll
    for (int b = 0; b < 2; ++b)
        if (!ok[b]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) s[b][c] = again[b][c][tid];
        }
    const U4 b = philox(i, 0, key, 0);
    const double q = affine(sp.q_lo, sp.q_hi, uniform(b.x[0]));
    const double c1 = affine(sp.chi1_lo, sp.chi1_hi, uniform(b.x[1]));
    const double c2 = affine(sp.chi2_lo, sp.chi2_hi, uniform(b.x[2]));
    const double om = affine(sp.omega0_lo, sp.omega0_hi, uniform(b.x[3]));
    const double m1 = q / (1.0 + q);
    const double m2 = 1.0 / (1.0 + q);
    const double a1 = c1 * (m1 * m1);
    const double a2 = c2 * (m2 * m2);
    m[j] = m1;
    m[ld + j] = m2;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        S[c * ld + j] = a1 * s[0][c];
        S[(3 + c) * ld + j] = a2 * s[1][c];
        L[c * ld + j] = c == 2 ? 1.0 : 0.0;
    }
    w0[j] = om;
}

bool bad_range(double lo, double hi) { return !(std::isfinite(lo) && std::isfinite(hi) && lo <= hi); }

}  // namespace
}  // namespace pn

using namespace pn;

extern "C" int pn_generate(int64_t n, int64_t ld, int64_t first, const pn_gen_spec* spec, double* m, double* S0,
                           double* L0, double* omega0, void* stream) {
    if (n < 0 || ld < n || ld > PN_MAX_N || first < 0 || first > INT64_MAX - n || !spec) return PN_EINVAL;
    const pn_gen_spec& s = *spec;
    if (bad_range(s.q_lo, s.q_hi) || !(s.q_lo > 0.0) || bad_range(s.chi1_lo, s.chi1_hi) ||
        bad_range(s.chi2_lo, s.chi2_hi) || s.chi1_lo < 0.0 || s.chi1_hi > 1.0 || s.chi2_lo < 0.0 ||
        s.chi2_hi > 1.0 || bad_range(s.omega0_lo, s.omega0_hi) || !(s.omega0_lo > 0.0))
        return PN_EINVAL;
    if (n > 0 && (!m || !S0 || !L0 || !omega0)) return PN_EINVAL;
    if (n == 0) return PN_OK;
    const int rc = device_ready();
    if (rc != PN_OK) return rc;
    hipLaunchKernelGGL(generate_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       (hipStream_t)stream, n, ld, first, s, m, S0, L0, omega0);
    return hipGetLastError() == hipSuccess ? PN_OK : PN_EHIP;
}
