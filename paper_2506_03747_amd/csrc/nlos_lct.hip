// The paper's FFT ("light-cone") forward route, gfx950: Section 2 rewrites
// Eq. (1) with u = z^2, v = (t c / 2)^2 as a 3-D convolution of the
// resampled volume with a cone (Eq. (3)-(5)), which Algorithm 1 steps 1.1-2.3
// evaluate with 3-D FFTs.  A cross-check of the direct operator, for a
// confocal N x N scan co-registered with the depth map, no stand-off, no
// cosine terms (Eq. (1) as printed), M = T a power of two.
//
// The volume holds at most one sample per pixel and the cone one layer (two
// at a tie) per lateral offset, so the convolution is a sum of N^4 shifted
// samples, 1 / 500 of the multiplications that a dense product needs; the
// transforms spend their time streaming zeros.  Two evaluations:
//
//   by samples (lct_by_samples; every size but thin, wide volumes)
//   k_lct_samples each pixel's coarse v-sample and weight, and their sums.
//   k_lct_list    the cone's layer of each lateral offset |dx|, |dy|; present
//                 pixels with their weights in fixed point, compacted.
//   k_lct_sum     a workgroup per row piece of scan points: every pixel's
//                 weight into the points' LDS rows, then the time resampling,
//                 the jitter and the write-out.
//
//   by transforms (N^2 > kLctThin M, or rows past the LDS)
//   k_lct_clear / k_lct_volume   R_z V on the (2N, 2N, 2M) zero-padded grid:
//       pixel (x, y) at depth layer j = floor(D / dz) (dz = c dt / 2) adds
//       albedo / (J M), J = j + 1, at coarse v-sample (J^2 - 1) / M (the
//       1 / sqrt(i) fold to i = J^2 of M^2 samples, then pairwise means).
//   k_lct_psf    cone: lateral offset n = -N .. N-1 cells at x = n / N,
//       layers z = k / M; 1 at the layer(s) nearest (4 slope)^2 (x^2 + y^2)
//       when below M, slope = w / (M c dt).
//   FFT, product, inverse FFT (hipFFT, fp64: the v^(-3/2) resampling below
//       amplifies the first bins ~1e8-fold over the last, and fp32 transform
//       noise would swamp them).
//   k_lct_out    time bin j: mean of the convolution over its fine v-span
//       [j^2, (j+1)^2), divided by (J dz)^3 (Eq. (3)).
//   k_lct_jitter Gaussian jitter (Section 2 / step 2.3), fp32 output.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <algorithm>
#include <cstdint>
#include <map>
#include <mutex>
#include <utility>

#include "nlos_internal.h"

namespace nlos {

__global__ void k_lct_clear(double2* a, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) a[i] = make_double2(0.0, 0.0);
}

// The sample of pixel p: coarse v-sample c and weight albedo / (J M); false
// where the pixel is absent or past the window.
__device__ __forceinline__ bool lct_sample(const LctArgs& a, int64_t p, int* c, double* w)
{
    const int M = a.M;
    const double D = (double)a.depth[p];
    const double A = a.albedo ? (double)a.albedo[p] : 0.5;
    const bool present = (!a.mask || a.mask[p] != 0) && A > 0.0 && isfinite(D) && D > 0.0;
    if (!present) return false;
    const double jd = floor(D / a.dz);
    if (!(jd >= 0.0 && jd < (double)M)) return false;
    const int64_t J = (int64_t)jd + 1;
    *c = (int)((J * J - 1) / M);
    *w = (1.0 / (double)J) / (double)M * A;
    return true;
}

// Lateral offset (nx, ny) cells: its distance from the cone's axis in layers
// over M, the layer floor and the smallest distance to a layer of 0 .. 2M - 1
// (the candidates next to zs M: the true nearest layers are among them).
__device__ __forceinline__ double lct_cone_best(const LctArgs& a, int nx, int ny, double* zs, double* kf)
{
    const int N = a.N, M = a.M;
    const double x = (double)nx / (double)N, y = (double)ny / (double)N;
    *zs = a.cone * (x * x + y * y);
    *kf = floor(*zs * (double)M);
    double best = fabs(*zs - (double)(2 * M - 1) / (double)M);
    for (int d = -1; d <= 2; ++d) {
        const double kk = *kf + d;
        if (kk < 0.0 || kk > (double)(2 * M - 1)) continue;
        best = fmin(best, fabs(*zs - kk / (double)M));
    }
    return best;
}

__global__ void k_lct_volume(const LctArgs a, double2* vol)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int N = a.N, M = a.M;
    if (p >= (int64_t)N * N) return;
    int c;
    double w;
    if (!lct_sample(a, p, &c, &w)) return;
    const int x = (int)(p / N), y = (int)(p % N);
    vol[((int64_t)x * 2 * N + y) * 2 * M + c] = make_double2(w, 0.0);
}

// One thread per element of the (2N, 2N, 2M) grid (coalesced stores); each
// finds its column's nearest layer(s) to (4 slope)^2 (x^2 + y^2): the
// candidates next to zs M (the true nearest layers are among them), every
// one at the minimal distance marked (ties), layers >= M dropped.  Past the
// grid the minimum falls on the last layer, which is dropped.
__global__ void k_lct_psf(const LctArgs a, double2* psf, int64_t n3)
{
    const int N = a.N, M = a.M;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n3; p += stride) {
        const int k = (int)(p % (2 * M));
        const int64_t col = p / (2 * M);
        const int ix = (int)(col / (2 * N)), iy = (int)(col % (2 * N));
        double v = 0.0;
        if (k < M) {
            const int nx = ix < N ? ix : ix - 2 * N, ny = iy < N ? iy : iy - 2 * N;
            double zs, kf;
            const double best = lct_cone_best(a, nx, ny, &zs, &kf);
            if (fabs(zs - (double)k / (double)M) == best) v = 1.0;
        }
        psf[p] = make_double2(v, 0.0);
    }
}

__global__ void k_lct_mul(double2* vol, const double2* psf, int64_t n, double scale)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double2 u = vol[i], v = psf[i];
        vol[i] = make_double2((u.x * v.x - u.y * v.y) * scale, (u.x * v.y + u.y * v.x) * scale);
    }
}

__global__ void k_lct_out(const LctArgs a, const double2* conv, double* pre)
{
    const int N = a.N, M = a.M;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= (int64_t)N * N * M) return;
    const int j = (int)(p % M);
    const int64_t xy = p / M;
    const int x = (int)(xy / N), y = (int)(xy % N);
    const double2* col = conv + ((int64_t)x * 2 * N + y) * 2 * M;
    const int64_t lo = (int64_t)j * j, hi = (int64_t)(j + 1) * (j + 1);
    double s = 0.0;
    for (int64_t c = lo / M; c <= (hi - 1) / M && c < M; ++c) {
        const int64_t ov = min(hi, (c + 1) * M) - max(lo, c * M);
        if (ov > 0) s += (double)ov / (double)(2 * j + 1) * col[c].x;
    }
    const double v = ((double)(j + 1) * a.dz) * ((double)(j + 1) * a.dz);
    pre[p] = s / pow(v, 1.5);
}

__global__ void k_lct_jitter(const LctArgs a, const double* pre, float* out)
{
    const int M = a.M;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= (int64_t)a.N * a.N * M) return;
    const int t = (int)(p % M);
    const double* row = pre + (p - t);
    double acc = 0.0;
    for (int i = -a.R; i <= a.R; ++i) {
        const int src = t - i;
        if (src >= 0 && src < M) acc += a.taps[i + a.R] * row[src];
    }
    out[p] = (float)acc;
}

// ---------------------------------------------------------------------------
// By samples.
//
// Table entry of lateral offset (|dx|, |dy|), 0 .. N - 1 each (the cone
// depends on the offset's squares only): the layer nearest its distance, M
// when that is past the window, and kLctTie when the next layer is as near.
constexpr uint32_t kLctTie = 0x8000u;

// The samples and the sum of each workgroup's 256 weights.
__global__ void __launch_bounds__(256) k_lct_samples(const LctArgs a, LctSample* smp, double* part, LctList* list)
{
    __shared__ double red[4];
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p == 0) {
        list->n = 0;
        list->ties = 0;
    }
    int c = 0;
    double w = 0.0;
    if (p < (int64_t)a.N * a.N) {
        if (!lct_sample(a, p, &c, &w)) w = 0.0;
        smp[p] = LctSample{w, (uint32_t)c, 0u};
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) w += __shfl_xor(w, d);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// The sum of all weights, by every workgroup for itself and in the same order
// everywhere; the cone's table; present pixels, appended in any order (every
// later sum is of integers), one counter add per wavefront.
__global__ void __launch_bounds__(256) k_lct_list(const LctArgs a, const LctSample* smp, const double* part,
                                                  uint16_t* tab, double* gain, LctPixel* pix, LctList* list)
{
    __shared__ double red[4];
    const int N = a.N, M = a.M, lane = (int)threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool in = p < (int64_t)N * N;
    const LctSample q = in ? smp[p] : LctSample{0.0, 0u, 0u};
    double total = 0.0;
    for (unsigned i = threadIdx.x; i < gridDim.x; i += 256) total += part[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) total += __shfl_xor(total, d);
    if (lane == 0) red[threadIdx.x >> 6] = total;
    for (int64_t j = p; j < M; j += (int64_t)gridDim.x * 256) {
        // time bin j: over the 2 j + 1 fine samples of its span and (J dz)^3
        const double t = (double)(j + 1) * a.dz;
        gain[j] = 1.0 / ((double)(2 * j + 1) * (t * t * t));
    }
    bool tie = false;
    if (in) {
        double zs, kf;
        const double best = lct_cone_best(a, (int)(p / N), (int)(p % N), &zs, &kf);
        // (a nearest layer of 0 .. M - 1 is kf or kf + 1; past the grid kf >= M)
        const bool lo = kf < (double)M && fabs(zs - kf / (double)M) == best;
        const bool hi = kf + 1.0 < (double)M && fabs(zs - (kf + 1.0) / (double)M) == best;
        tie = lo && hi;
        uint32_t v = (uint32_t)M;
        if (hi) v = (uint32_t)kf + 1u;
        if (lo) v = (uint32_t)kf | (hi ? kLctTie : 0u);
        tab[p] = (uint16_t)v;
    }
    if (__any(tie) && lane == 0) list->ties = 1;
    __syncthreads();
    // (enlarged by more than its rounding: no sum of increments passes 2^62 + N^2 / 2)
    total = (((red[0] + red[1]) + red[2]) + red[3]) * (1.0 + 0x1p-24);
    if (p == 0) list->unit = isfinite(total) ? total * 0x1p-62 : __longlong_as_double(0x7ff8000000000000ll);
    const bool on = q.w > 0.0;
    const unsigned long long m = __ballot(on);
    if (m == 0ull) return;
    int base = 0;
    if (lane == 0) base = atomicAdd(&list->n, (int)__popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    if (on) {
        const double x = isfinite(total) ? rint(q.w * (0x1p62 / total)) : 0.0;
        pix[base + __popcll(m & ((1ull << lane) - 1ull))] =
            LctPixel{(unsigned long long)x, q.c, (uint32_t)(p / N) << 16 | (uint32_t)(p % N)};
    }
}

// A workgroup owns NP scan points (x', y'0 .. y'0 + NP - 1): one row of M
// 64-bit sums each in LDS.  A lane takes a pixel and adds its weight at bin
// c + layer(|x' - x|, |y' - y|) of each row: per pair a table address, a
// 16-bit table read (2 N^2 bytes, mostly from the L1; a copy in LDS measured
// no faster and took the second workgroup's room), add, compare, ds_add_u64.
// Weights are fixed point, w s rounded to an integer, so that a row's sums do
// not depend on the order.  s is 2^62 over the sum of all weights: no bin can
// wrap, a sample is within 2^-63 of that sum, and one bright pixel among dim
// ones costs them no bits (2^62 / (N^2 max w) did: beside one 10^10 times
// brighter a pixel kept 16 at N = 64).  Root mean square error of the rows
// against that of fp64 transforms (models of both on a smooth surface, albedo
// 0.05 to 1): before the resampling 0.30 of it at N = 64, 0.57 at 128, 0.92 at
// 384, 1.65 at 512 (0.8, 1.6, 2.6 and 4.7 with the former scale), 0.12 to 0.73
// with three pixels 10^4 times brighter (31 to 10^4); after it, relative to the
// output, 1 to 3 10^-16 against 10^-9 to 8 10^-12, as it amplifies the transforms'
// noise in the first bins.
// Bound: the LDS adds (bank conflicts included) and VALU, about 15 cycles per
// wavefront and pair; then the write-out's fp64 resampling and jitter.  128^2
// points and pixels, 1024 bins: 13.2 ms by transforms; 367 us with 1024
// threads, a table read and add at a time; 220 us with the reads of all rows
// before the adds and the jitter from a sliding window; 168 us (back to back) with four
// workgroups of 512 threads per CU, so that one's write-out runs under
// another's adds; 163 with the weights made integers once per pixel instead of
// once per workgroup.
template <int NP, bool TIES>
__device__ __forceinline__ void lct_add(const LctPixel* __restrict__ pix, int n, const uint16_t* __restrict__ tab,
                                        int N, int M, int x1, int y1,
                                        unsigned long long* rows, int pitch, int tid, int nthr)
{
    if (tid >= n) return;
    LctPixel q = pix[tid];
    for (int i = tid; i < n; i += nthr) {
        const int x = (int)(q.xy >> 16), y = (int)(q.xy & 0xffffu);
        const uint32_t c = q.c;
        const unsigned long long inc = q.inc;
        q = pix[min(i + nthr, n - 1)];   // the next one lands while this one is added
        const int row = abs(x1 - x) * N;
        // every row's table entry before any add, so that one wait serves all
        // (a row past the grid repeats the last one; it is not written out)
        uint32_t v[NP];
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            v[r] = tab[row + abs(min(y1 + r, N - 1) - y)];
        }
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            const uint32_t k = (TIES ? v[r] & ~kLctTie : v[r]) + c;
            unsigned long long* dst = rows + (size_t)r * pitch + k;
            if (k < (uint32_t)M) __hip_atomic_fetch_add(dst, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (TIES && (v[r] & kLctTie) && k + 1u < (uint32_t)M)
                __hip_atomic_fetch_add(dst + 1, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

template <int NP>
__global__ void __launch_bounds__(1024) k_lct_sum(const LctArgs a, const uint16_t* __restrict__ tab,
                                                  const LctPixel* __restrict__ pix, const double* __restrict__ gain,
                                                  const LctList* __restrict__ list, float* __restrict__ out)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = a.N, M = a.M, R = a.R, nthr = (int)blockDim.x, tid = (int)threadIdx.x;
    const int pitch = lct_pitch(a);   // R zeros around each row, for the jitter
    unsigned long long* rows = reinterpret_cast<unsigned long long*>(smem);
    const int nt = (N + NP - 1) / NP;
    const int x1 = (int)blockIdx.x / nt, y1 = (int)(blockIdx.x % nt) * NP;
    const int n = list->n;
    const double unit = list->unit;
    for (int i = tid; i < NP * pitch; i += nthr) rows[i] = 0ull;
    const bool ties = list->ties != 0;
    __syncthreads();
    if (ties)
        lct_add<NP, true>(pix, n, tab, N, M, x1, y1, rows + R, pitch, tid, nthr);
    else
        lct_add<NP, false>(pix, n, tab, N, M, x1, y1, rows + R, pitch, tid, nthr);
    __syncthreads();
    // time bin j: the mean over its fine v-span [j^2, (j + 1)^2) (at most three
    // coarse samples), over (J dz)^3; in place, through registers
    // (an infinite weight leaves no number anywhere, as the transforms do)
    const int lm = 31 - __clz(M);
    double pre[kLctPer];
#pragma unroll
    for (int e = 0; e < kLctPer; ++e) {
        const int i = tid + e * nthr;
        pre[e] = 0.0;
        if (i >= NP * M) continue;
        const int r = i >> lm, j = i & (M - 1);
        const unsigned long long* col = rows + (size_t)r * pitch + R;
        const int lo = j * j, hi = lo + 2 * j + 1;   // (at most 2^28)
        const int c0 = lo >> lm, c1 = (hi - 1) >> lm;
        double sum = 0.0;
        for (int c = c0; c <= c1; ++c) sum += (double)(min(hi, (c + 1) << lm) - max(lo, c << lm)) * (double)col[c];
        pre[e] = sum * unit * gain[j];
    }
    __syncthreads();
    double* rowd = reinterpret_cast<double*>(rows);
#pragma unroll
    for (int e = 0; e < kLctPer; ++e) {
        const int i = tid + e * nthr;
        if (i < NP * M) rowd[(size_t)(i >> lm) * pitch + R + (i & (M - 1))] = pre[e];
    }
    __syncthreads();
    // jitter: a lane makes kLctV consecutive outputs from a sliding window, one
    // LDS read per tap for all of them (lanes kLctV doubles apart: every bank
    // in turn, as kLctV is odd)
    const int nseg = (M + kLctV - 1) / kLctV;
    for (int i = tid; i < NP * nseg; i += nthr) {
        const int r = i / nseg, t0 = (i - r * nseg) * kLctV;
        if (y1 + r >= N) break;
        const int last = pitch - 1;
        const double* h = rowd + (size_t)r * pitch;
        // output t0 + m, tap k: row word t0 + m + 2 R - k
        double w[kLctV], acc[kLctV];
#pragma unroll
        for (int m = 0; m < kLctV; ++m) {
            w[m] = h[min(t0 + m + 2 * R, last)];
            acc[m] = a.taps[0] * w[m];
        }
        for (int k = 1; k <= 2 * R; ++k) {
#pragma unroll
            for (int m = kLctV - 1; m > 0; --m) w[m] = w[m - 1];
            w[0] = h[t0 + 2 * R - k];
#pragma unroll
            for (int m = 0; m < kLctV; ++m) acc[m] += a.taps[k] * w[m];
        }
        float* o = out + ((size_t)x1 * N + (y1 + r)) * M + t0;
#pragma unroll
        for (int m = 0; m < kLctV; ++m)
            if (t0 + m < M) o[m] = (float)acc[m];
    }
}

// Scan points per workgroup, threads and LDS of k_lct_sum.  4096 bins in all
// leave room for four workgroups per CU (8192 and two: 1.13 times the time at
// 128^2, 1024 bins); fewer points while that leaves CUs idle.  A thread
// resamples at most kLctPer bins, so the longest rows take 1024 threads.
struct LctShape {
    int np, threads;
    size_t lds;
};

static LctShape lct_shape(const LctArgs& a)
{
    LctShape s{8, 512, 0};
    while (s.np > 1 && ((int64_t)s.np * a.M > 4096 || (int64_t)a.N * ((a.N + s.np - 1) / s.np) < 512)) s.np /= 2;
    if (s.np * a.M > s.threads * kLctPer) s.threads = 1024;
    s.lds = (size_t)s.np * lct_pitch(a) * 8;
    return s;
}

// The sum by samples costs N^4 adds (0.41 to 0.75 ps each), the transforms about
// 100 ps for each of their 8 N^2 M grid points; thin, wide volumes are the only
// ones where the transforms cost less.
bool lct_by_samples(const LctArgs& a)
{
    return a.M <= kLctMaxRow && (int64_t)a.N * a.N <= kLctThin * a.M;
}

LctLayout lct_samples_layout(const LctArgs& a)
{
    const size_t n2 = (size_t)a.N * a.N;
    LctLayout l;
    l.pix = (n2 * 2 + 255) & ~(size_t)255;
    l.gain = l.pix + ((n2 * sizeof(LctPixel) + 255) & ~(size_t)255);
    l.list = l.gain + (((size_t)a.M * 8 + 255) & ~(size_t)255);
    l.smp = l.list + 256;
    l.part = l.smp + ((n2 * sizeof(LctSample) + 255) & ~(size_t)255);
    l.bytes = l.part + (((n2 + 255) / 256 * 8 + 255) & ~(size_t)255);
    return l;
}

template <int NP>
static hipError_t launch_lct_sum(const LctArgs& a, const LctShape& sh, const uint16_t* tab, const LctPixel* pix,
                                 const double* gain, const LctList* list, float* out, hipStream_t st)
{
    const hipError_t e = hipFuncSetAttribute((const void*)k_lct_sum<NP>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)(a.N * ((a.N + NP - 1) / NP));
    hipLaunchKernelGGL(k_lct_sum<NP>, dim3(blocks), dim3((unsigned)sh.threads), sh.lds, st, a, tab, pix, gain,
                       list, out);
    return hipGetLastError();
}

hipError_t launch_lct_samples(const LctArgs& a, void* ws, float* out, hipStream_t st)
{
    const LctLayout l = lct_samples_layout(a);
    unsigned char* w = static_cast<unsigned char*>(ws);
    uint16_t* tab = reinterpret_cast<uint16_t*>(w);
    LctPixel* pix = reinterpret_cast<LctPixel*>(w + l.pix);
    double* gain = reinterpret_cast<double*>(w + l.gain);
    LctList* list = reinterpret_cast<LctList*>(w + l.list);
    const LctShape sh = lct_shape(a);
    if (a.M > kLctMaxRow || a.N > 65535 || sh.lds > kLctLds || sh.np * a.M > sh.threads * kLctPer)
        return hipErrorInvalidValue;
    LctSample* smp = reinterpret_cast<LctSample*>(w + l.smp);
    double* part = reinterpret_cast<double*>(w + l.part);
    const unsigned nb = (unsigned)(((int64_t)a.N * a.N + 255) / 256);
    hipLaunchKernelGGL(k_lct_samples, dim3(nb), dim3(256), 0, st, a, smp, part, list);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lct_list, dim3(nb), dim3(256), 0, st, a, smp, part, tab, gain, pix, list);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    switch (sh.np) {
    case 8: return launch_lct_sum<8>(a, sh, tab, pix, gain, list, out, st);
    case 4: return launch_lct_sum<4>(a, sh, tab, pix, gain, list, out, st);
    case 2: return launch_lct_sum<2>(a, sh, tab, pix, gain, list, out, st);
    default: return launch_lct_sum<1>(a, sh, tab, pix, gain, list, out, st);
    }
}

// ---------------------------------------------------------------------------
// FFT plans: one per (N, M), created on first use and kept (the FFT library
// allocates its tables then); execution is serialised per plan because the
// stream and work area are plan state.
namespace {

struct PlanEntry {
    hipfftHandle plan = nullptr;
    size_t work = 0;
    bool ok = false;
};

std::mutex g_plan_mu;
std::map<std::pair<int, int>, PlanEntry> g_plans;

PlanEntry* get_plan(int N, int M)
{
    auto& e = g_plans[std::make_pair(N, M)];
    if (e.ok) return &e;
    if (hipfftCreate(&e.plan) != HIPFFT_SUCCESS) return nullptr;
    if (hipfftSetAutoAllocation(e.plan, 0) != HIPFFT_SUCCESS ||
        hipfftMakePlan3d(e.plan, 2 * N, 2 * N, 2 * M, HIPFFT_Z2Z, &e.work) != HIPFFT_SUCCESS) {
        hipfftDestroy(e.plan);
        e.plan = nullptr;
        return nullptr;
    }
    e.ok = true;
    return &e;
}

}  // namespace

int lct_fft_work_bytes(int N, int M, size_t* bytes)
{
    std::lock_guard<std::mutex> lk(g_plan_mu);
    PlanEntry* e = get_plan(N, M);
    if (!e) return -1;
    *bytes = e->work;
    return 0;
}

static hipError_t grid_launch_check() { return hipGetLastError(); }

hipError_t launch_lct(const LctArgs& a, double2* vol, double2* psf, void* fft_work, float* out, hipStream_t st,
                      int* fft_status)
{
    *fft_status = 0;
    const int N = a.N, M = a.M;
    const int64_t n3 = (int64_t)(2 * N) * (2 * N) * (2 * M);
    const unsigned cb = (unsigned)std::min<int64_t>(8192, (n3 + 255) / 256);
    hipLaunchKernelGGL(k_lct_clear, dim3(cb), dim3(256), 0, st, vol, n3);
    hipError_t e = grid_launch_check();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lct_volume, dim3((unsigned)(((int64_t)N * N + 255) / 256)), dim3(256), 0, st, a, vol);
    if ((e = grid_launch_check()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_lct_psf, dim3(cb), dim3(256), 0, st, a, psf, n3);
    if ((e = grid_launch_check()) != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> lk(g_plan_mu);
        PlanEntry* pe = get_plan(N, M);
        if (!pe || hipfftSetStream(pe->plan, st) != HIPFFT_SUCCESS ||
            hipfftSetWorkArea(pe->plan, fft_work) != HIPFFT_SUCCESS ||
            hipfftExecZ2Z(pe->plan, reinterpret_cast<hipfftDoubleComplex*>(vol),
                          reinterpret_cast<hipfftDoubleComplex*>(vol), HIPFFT_FORWARD) != HIPFFT_SUCCESS ||
            hipfftExecZ2Z(pe->plan, reinterpret_cast<hipfftDoubleComplex*>(psf),
                          reinterpret_cast<hipfftDoubleComplex*>(psf), HIPFFT_FORWARD) != HIPFFT_SUCCESS) {
            *fft_status = -1;
            return hipSuccess;
        }
        hipLaunchKernelGGL(k_lct_mul, dim3(cb), dim3(256), 0, st, vol, psf, n3, 1.0 / (double)n3);
        if ((e = grid_launch_check()) != hipSuccess) return e;
        if (hipfftExecZ2Z(pe->plan, reinterpret_cast<hipfftDoubleComplex*>(vol),
                          reinterpret_cast<hipfftDoubleComplex*>(vol), HIPFFT_BACKWARD) != HIPFFT_SUCCESS) {
            *fft_status = -1;
            return hipSuccess;
        }
    }
    const int64_t no = (int64_t)N * N * M;
    double* pre = reinterpret_cast<double*>(psf);   // the transformed cone is no longer needed
    hipLaunchKernelGGL(k_lct_out, dim3((unsigned)((no + 255) / 256)), dim3(256), 0, st, a, vol, pre);
    if ((e = grid_launch_check()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_lct_jitter, dim3((unsigned)((no + 255) / 256)), dim3(256), 0, st, a, pre, out);
    return grid_launch_check();
}

}  // namespace nlos
