// Poisson noise of a transient frame (Algorithm 1 step 2.4, after the blur
// of step 2.3), gfx950:
//     T = Poisson(tau * sigma_n) / sigma_n,  sigma_n = Var(tau) / 10^(nr / 10),
// Var the population variance of the whole frame.
//
// k_noise_moments / k_noise_scale   frame mean and variance: per-thread
//     Welford updates, merged pairwise (Chan et al.) in fixed trees within
//     each block and then across the blocks, all fp64, so the result is
//     reproducible.
// k_poisson   a workgroup sorts a tile of elements by what they need (nothing,
//     inversion, rejection) and draws each kind densely.  Uniform t of element i
//     is word t mod 4 of Philox4x64-10 (Salmon, Moraes, Dror and Shaw, SC
//     2011) at counter (i, t / 4, 0, 0), key (seed, 0x4e4c4f53), scaled from
//     its top 53 bits.  lambda < 10: inversion by sequential search;
//     otherwise Hormann's transformed rejection with squeeze (PTRS).  exp,
//     log and log k! use fixed recipes of IEEE basic operations (compiled
//     without contraction), so the integer decisions are those of any
//     implementation performing the same operations in the same order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "nlos_internal.h"

namespace nlos {

namespace {

struct Moments {
    double n, mean, m2;
};

// x / k from y, the correctly rounded 1 / k: the quotient of the product, then
// one correction by its remainder, which fma gives exactly -- correctly rounded
// (Markstein), so the same double as the division, in three operations with y
// off the chain of x.  (Quotients below the normal range may differ in their
// last bit; where that can happen here they are far below the sums they join.)
__device__ __forceinline__ double div_by(double x, double k, double y)
{
    const double q = x * y;
    const double r = fma(-q, k, x);
    return r == r ? fma(r, y, q) : q;   // (an infinite x stays one)
}


// The same for a known divisor (an infinite x gives no number, as it does in
// every sum this joins).
__device__ __forceinline__ double div_known(double x, double k, double y)
{
    const double q = x * y;
    return fma(fma(-q, k, x), y, q);
}
// Correctly rounded reciprocals of the first steps of a running count that is
// the same for every lane (scalar reads).
struct Reciprocals {
    double y[64];
    constexpr Reciprocals() : y()
    {
        for (int k = 1; k < 64; ++k) y[k] = 1.0 / (double)k;
    }
};
__device__ const Reciprocals kRecip{};

__device__ __forceinline__ double recip(int k) { return k < 64 ? kRecip.y[k] : 1.0 / (double)k; }

__device__ __forceinline__ Moments merge(Moments a, Moments b)
{
    if (b.n == 0.0) return a;
    if (a.n == 0.0) return b;
    Moments r;
    r.n = a.n + b.n;
    const double d = b.mean - a.mean;
    r.mean = a.mean + d * (b.n / r.n);
    r.m2 = (a.m2 + b.m2) + d * d * (a.n * (b.n / r.n));
    return r;
}

__device__ Moments block_merge(Moments m)
{
    __shared__ double sn[kNoiseBlock], smean[kNoiseBlock], sm2[kNoiseBlock];
    sn[threadIdx.x] = m.n;
    smean[threadIdx.x] = m.mean;
    sm2[threadIdx.x] = m.m2;
    __syncthreads();
    for (int w = kNoiseBlock / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
            const Moments a{sn[threadIdx.x], smean[threadIdx.x], sm2[threadIdx.x]};
            const Moments b{sn[threadIdx.x + w], smean[threadIdx.x + w], sm2[threadIdx.x + w]};
            const Moments r = merge(a, b);
            sn[threadIdx.x] = r.n;
            smean[threadIdx.x] = r.mean;
            sm2[threadIdx.x] = r.m2;
        }
        __syncthreads();
    }
    return Moments{sn[0], smean[0], sm2[0]};
}

}  // namespace

__global__ void __launch_bounds__(kNoiseBlock) k_noise_moments(const float* tau, int64_t n, double* part)
{
    Moments m{0.0, 0.0, 0.0};
    const int64_t stride = (int64_t)gridDim.x * kNoiseBlock;
    // (eight reads in flight before the chain of updates; past the end they
    // reread the last element and are not used)
    int k = 0;
    for (int64_t i = (int64_t)blockIdx.x * kNoiseBlock + threadIdx.x; i < n; i += 8 * stride) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = tau[min(i + e * stride, n - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (i + e * stride >= n) break;
            ++k;
            const double x = (double)v[e];
            m.n = (double)k;
            const double d = x - m.mean;
            m.mean = m.mean + div_by(d, m.n, recip(__builtin_amdgcn_readfirstlane(k)));
            m.m2 = m.m2 + d * (x - m.mean);
        }
    }
    m = block_merge(m);
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x] = m.n;
        part[3 * blockIdx.x + 1] = m.mean;
        part[3 * blockIdx.x + 2] = m.m2;
    }
}

// One workgroup: thread t merges blocks t, t + 256, ... in order, then the
// per-thread moments are merged pairwise in a fixed tree -> mean, population
// variance, sigma_n.
__global__ void __launch_bounds__(kNoiseBlock) k_noise_scale(const double* part, int nb, double nr_db, double* out)
{
    Moments m{0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nb; b += kNoiseBlock)
        m = merge(m, Moments{part[3 * b], part[3 * b + 1], part[3 * b + 2]});
    m = block_merge(m);
    if (threadIdx.x == 0) {
        const double var = m.n > 0.0 ? m.m2 / m.n : 0.0;
        out[0] = m.mean;
        out[1] = var;
        out[2] = var / pow(10.0, nr_db / 10.0);
    }
}

// ---------------------------------------------------------------------------
namespace {

// 64 x 64 -> 128 bits by four 32-bit multiply-adds.
__device__ __forceinline__ void mul128(uint64_t m, uint64_t x, uint64_t& lo, uint64_t& hi)
{
    const uint32_t ml = (uint32_t)m, mh = (uint32_t)(m >> 32), xl = (uint32_t)x, xh = (uint32_t)(x >> 32);
    const uint64_t a = (uint64_t)ml * xl;
    const uint64_t b = (uint64_t)mh * xl + (a >> 32);
    const uint64_t c = (uint64_t)ml * xh + (uint32_t)b;
    hi = (uint64_t)mh * xh + (b >> 32) + (c >> 32);
    lo = (c << 32) | (uint32_t)a;
}

// The four words of block `blk` of element i.
__device__ __forceinline__ void philox4x64_10(uint64_t c[4], int64_t i, uint64_t blk, uint64_t seed)
{
    uint64_t k0 = seed, k1 = 0x4e4c4f53ull;
    c[0] = (uint64_t)i;
    c[1] = blk;
    c[2] = c[3] = 0ull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B97F4A7C15ull;
            k1 += 0xBB67AE8584CAA73Bull;
        }
        uint64_t a0, h0, a1, h1;
        mul128(0xD2E7470EE14C6C93ull, c[0], a0, h0);
        mul128(0xCA5A826395121157ull, c[2], a1, h1);
        c[0] = h1 ^ c[1] ^ k0;
        c[1] = a1;
        c[2] = h0 ^ c[3] ^ k1;
        c[3] = a0;
    }
}

__device__ __forceinline__ double uniform_of(uint64_t word)
{
    return (double)(word >> 11) * (1.0 / 9007199254740992.0);
}

constexpr double kLn2Hi = 6.93147180369123816490e-01;
constexpr double kLn2Lo = 1.90821492927058770002e-10;
constexpr double kLog2e = 1.44269504088896338700e+00;
constexpr double kPi = 3.14159265358979323846;

// e^x = 2^n e^r, |r| <= ln2 / 2, Taylor terms to r^13; 0 below -708.
__device__ double rexp(double x)
{
    if (x < -708.0) return 0.0;
    const double n = floor(x * kLog2e + 0.5);
    const double r = (x - n * kLn2Hi) - n * kLn2Lo;
    double s = 1.0, t = 1.0;
#pragma unroll
    for (int k = 1; k <= 13; ++k) {
        t = div_known(t * r, (double)k, 1.0 / (double)k);
        s = s + t;
    }
    return ldexp(s, (int)n);
}

// log x = e ln2 + 2 atanh((m - 1) / (m + 1)), m in [1/sqrt2, sqrt2), series to s^29.
__device__ double rlog(double x)
{
    int e;
    double m = frexp(x, &e);
    if (m < 0.70710678118654752440) {
        m = m * 2.0;
        e = e - 1;
    }
    const double s = (m - 1.0) / (m + 1.0), s2 = s * s;
    double t = s, acc = 0.0;
#pragma unroll
    for (int k = 1; k <= 29; k += 2) {
        acc = acc + div_known(t, (double)k, 1.0 / (double)k);
        t = t * s2;
    }
    return 2.0 * acc + ((double)e * kLn2Hi + (double)e * kLn2Lo);
}

// log k!: the product below 20, Stirling's series above.
__device__ double rlogfact(double k)
{
    if (k < 20.0) {
        double f = 1.0;
        for (double i = 2.0; i <= k; i = i + 1.0) f = f * i;
        return rlog(f);
    }
    const double ik = 1.0 / k, ik2 = ik * ik;
    const double series = ik * (1.0 / 12.0 - ik2 * (1.0 / 360.0 - ik2 * (1.0 / 1260.0 - ik2 * (1.0 / 1680.0))));
    return (k * rlog(k) - k) + 0.5 * rlog(2.0 * kPi * k) + series;
}

// lambda < 10: inversion by sequential search.  The step k is the same for
// every lane of the wavefront, so its reciprocal is a scalar read.
__device__ __forceinline__ int64_t poisson_inversion(double lam, double u)
{
    double p = rexp(-lam), F = p;
    int k = 0, got = 0;
    bool go = u > F;
    while (__any(go) && k < 1000) {
        ++k;
        p = div_known(p * lam, (double)k, recip(k));
        F = F + p;
        if (go) {
            got = k;
            go = u > F;
        }
    }
    return got;
}

// lambda >= 10: Hormann's transformed rejection.  The proposal of uniforms U,
// V; `sure`: accepted by the squeeze, whatever the exact test says.
struct Ptrs {
    double a, b, vr;
};

__device__ __forceinline__ Ptrs ptrs_of(double lam)
{
    Ptrs q;
    q.b = 0.931 + 2.53 * sqrt(lam);
    q.a = -0.059 + 0.02483 * q.b;
    q.vr = 0.9277 - 3.6224 / (q.b - 2.0);
    return q;
}

__device__ __forceinline__ double ptrs_propose(const Ptrs& q, double lam, double U, double V, double* us, bool* sure)
{
    *us = 0.5 - fabs(U);
    *sure = *us >= 0.07 && V <= q.vr;
    return floor((2.0 * q.a / *us + q.b) * U + lam + 0.43);
}

// From the first proposal on, with the exact test; c: the element's block 0.
__device__ int64_t ptrs_count(double lam, uint64_t seed, int64_t i, uint64_t c[4])
{
    const Ptrs q = ptrs_of(lam);
    const double invalpha = 1.1239 + 1.1328 / (q.b - 3.4);
    const double loglam = rlog(lam), logalpha = rlog(invalpha);
    for (int it = 0; it < 100000; ++it) {
        const bool second = it & 1;   // (a block holds the uniforms of two proposals)
        if (it > 0 && !second) philox4x64_10(c, i, (uint64_t)(it >> 1), seed);
        const double U = uniform_of(second ? c[2] : c[0]) - 0.5;
        const double V = uniform_of(second ? c[3] : c[1]);
        double us;
        bool sure;
        const double kd = ptrs_propose(q, lam, U, V, &us, &sure);
        if (sure) return (int64_t)kd;
        if (kd < 0.0 || (us < 0.013 && V > us)) continue;
        const double lhs = (rlog(V) + logalpha) - rlog(q.a / (us * us) + q.b);
        const double rhs = (-lam + kd * loglam) - rlogfact(kd);
        if (lhs <= rhs) return (int64_t)kd;
    }
    return -1;
}

}  // namespace

// A tile of at most kNoiseTile elements per workgroup.  Lanes of one wavefront
// need very different work (a frame's zeros none, inversion or rejection, and a
// seventh of the rejections the logarithms of the exact test), and a wavefront
// pays for its most expensive lane: so the tile's elements are listed by kind
// (inversions from the front of the list, rejections from its back) and each
// list is worked off by full wavefronts; the proposals that the squeeze does
// not settle are listed once more.  Bound: VALU (the generator's 72 quarter-rate
// multiply-adds, then the fp64 recipes).  4.2 M elements, 60% zeros, 39% below
// 10, 1% above: 167 us with an element per thread and IEEE divisions by the
// recipes' constants, 50 so (59 without the lists' pieces taken in turn and
// with each proposal's generator run again for the exact test; tiles of 512,
// 1024 and 4096 elements are 1.4, 1.04 and 1.1 times slower).
__global__ void __launch_bounds__(kNoiseBlock)
    k_poisson(const float* tau, int64_t n, int tile, int64_t first, const double* sigma_n, uint64_t seed, float* out)
{
    __shared__ float st[kNoiseTile];
    __shared__ uint16_t list[kNoiseTile], rest[kNoiseTile];
    __shared__ int count[4];   // inversions, rejections, unsettled proposals, pieces taken
    const double sn = *sigma_n;
    const bool ok = sn > 0.0 && isfinite(sn);
    const int64_t base = (int64_t)blockIdx.x * tile;
    const int m = (int)min((int64_t)tile, n - base), tid = (int)threadIdx.x, lane = tid & 63;
    if (tid < 4) count[tid] = 0;
    __syncthreads();
    for (int e0 = 0; e0 < m; e0 += kNoiseBlock) {
        const int e = e0 + tid;
        const float t = e < m ? tau[base + e] : 0.f;
        const double lam = ok && t > 0.f ? (double)t * sn : 0.0;
        const bool inv = lam > 0.0 && lam < 10.0, rej = lam > 0.0 && !inv;
        if (e < m) {
            st[e] = t;
            if (!inv && !rej) out[base + e] = 0.f;
        }
        const uint64_t mi = __ballot(inv), mr = __ballot(rej), below = (1ull << lane) - 1ull;
        int bi = 0, br = 0;
        if (lane == 0) {
            if (mi) bi = atomicAdd(&count[0], (int)__popcll(mi));
            if (mr) br = atomicAdd(&count[1], (int)__popcll(mr));
        }
        bi = __builtin_amdgcn_readfirstlane(bi);
        br = __builtin_amdgcn_readfirstlane(br);
        if (inv) list[bi + (int)__popcll(mi & below)] = (uint16_t)e;
        if (rej) list[m - 1 - (br + (int)__popcll(mr & below))] = (uint16_t)e;
    }
    __syncthreads();
    // Pieces of 64, rejections first: a wavefront takes the next one, so that
    // the long chain of a piece of rejections runs beside the inversions.  A
    // tile with few rejections settles them at once; with many, the unsettled
    // ones are listed and settled by full wavefronts.
    const int n_inv = count[0], n_rej = count[1];
    const int p_rej = (n_rej + 63) / 64, p_all = p_rej + (n_inv + 63) / 64;
    const bool at_once = n_rej <= kNoiseTile / 4;
    for (;;) {
        int pc = 0;
        if (lane == 0) pc = atomicAdd(&count[3], 1);
        pc = __builtin_amdgcn_readfirstlane(pc);
        if (pc >= p_all) break;
        const bool rej = pc < p_rej;
        const int j = (rej ? pc : pc - p_rej) * 64 + lane;
        if (j >= (rej ? n_rej : n_inv)) continue;
        const int e = rej ? list[m - 1 - j] : list[j];
        const double lam = (double)st[e] * sn;
        uint64_t c[4];
        philox4x64_10(c, first + base + e, 0ull, seed);
        int64_t got;
        if (!rej) {
            got = poisson_inversion(lam, uniform_of(c[0]));
        } else {
            double us;
            bool sure;
            const double kd = ptrs_propose(ptrs_of(lam), lam, uniform_of(c[0]) - 0.5, uniform_of(c[1]), &us, &sure);
            got = (int64_t)kd;
            if (!sure) {
                if (!at_once) {
                    rest[atomicAdd(&count[2], 1)] = (uint16_t)e;
                    continue;
                }
                got = ptrs_count(lam, seed, first + base + e, c);
            }
        }
        out[base + e] = (float)((double)got / sn);
    }
    if (at_once) return;   // uniform
    __syncthreads();
    const int n_rest = count[2];
    for (int j = tid; j < n_rest; j += kNoiseBlock) {
        const int e = rest[j];
        uint64_t c[4];
        philox4x64_10(c, first + base + e, 0ull, seed);
        out[base + e] = (float)((double)ptrs_count((double)st[e] * sn, seed, first + base + e, c) / sn);
    }
}

hipError_t launch_noise_scale(const float* tau, int64_t n, double nr_db, double* out, double* part, int nb,
                              hipStream_t st)
{
    hipLaunchKernelGGL(k_noise_moments, dim3((unsigned)nb), dim3(kNoiseBlock), 0, st, tau, n, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_noise_scale, dim3(1), dim3(kNoiseBlock), 0, st, part, nb, nr_db, out);
    return hipGetLastError();
}

hipError_t launch_poisson(const float* tau, int64_t n, const double* sigma_n, uint64_t seed, float* out,
                          hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    // element i's uniforms belong to i, whichever launch draws it
    const int tile = noise_tile(n);
    for (int64_t first = 0; first < n;) {
        const int64_t m = noise_launch(n - first, tile);
        hipLaunchKernelGGL(k_poisson, dim3((unsigned)((m + tile - 1) / tile)), dim3(kNoiseBlock), 0, st, tau + first, m,
                           tile, first, sigma_n, seed, out + first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        first += m;
    }
    return hipSuccess;
}

}  // namespace nlos
