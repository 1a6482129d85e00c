// Smooth time response and its adjoint (confocal), gfx950.
//
// The hard forward bins each pair's arrival; its gradient with respect to
// depth is zero almost everywhere.  The smooth forward gives each pair the
// continuous Gaussian response of the detector jitter (Section 2, temporal
// jitter; sigma = FWHM / (2 sqrt(2 ln 2)) / dt in bins):
//     tau_s[s][k] = sum_p w_sp N(k + 1/2 - u_sp),  |k - floor(u_sp)| <= Rs,
// Rs = ceil(6 sigma), N the normalised Gaussian.  The weight w and arrival u
// are those of the hard forward (Eq. (1) with the cosine and stand-off
// extensions).  Arrivals are computed in fp64: an fp32 distance puts u off by
// ~1e-4 bins at u ~ 1000, which would move the Gaussian samples by ~1e-5.
//
// k_smooth_prep  record summaries and the polynomials' kernels.
// k_smooth_mom   forward for sigma >= 1.2 bins: 5 to 8 moments of the sub-bin
//                offset per pair into LDS rows, then a convolution of each
//                moment row with its kernel, four bins per thread.
// k_smooth       forward otherwise, where the moment rows of one scan point do
//                not fit in LDS, or for few records: a workgroup owns a tile of
//                scan points (LDS rows of 64-bit fixed-point bins), a lane one
//                patch; 2 Rs + 1 LDS adds per pair, Gaussian samples by a
//                three-exponential recurrence.
// k_adj_moments, k_adjoint_mom   adjoint for the same widths: the upstream
//                gradient's correlations with the polynomials' kernels once
//                per scan point, then per pair a polynomial in the sub-bin
//                offset and its derivative.
// k_adjoint      gather otherwise, or for few records or scan points: a lane
//                owns one patch and loops over a range of scan points whose
//                upstream-gradient rows are staged in LDS; per
//                pair G0 = sum g N(x), G1 = sum g (x / sigma^2) N(x) give
//                dL/dw = G0 and dL/du = w G1; per-record partial gradients
//                (fp64) per scan range, summed in a fixed order afterwards
//                (k_adjoint_reduce, one thread per output word).
// k_grad_scatter / k_grad_gather   record gradients -> depth and albedo maps
//                through the central-difference normals and true areas.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "nlos_device.h"
#include "nlos_internal.h"

namespace nlos {

namespace {

typedef unsigned long long u64s;

__device__ __forceinline__ int smooth_active(const SmoothArgs& a)
{
    int n = a.n_cap;
    if (a.n_active) {
        n = *a.n_active;
        n = n < 0 ? 0 : (n > a.n_cap ? a.n_cap : n);
    }
    return n;
}

// A wave-uniform value, kept in scalar registers.
__device__ __forceinline__ float uniform_f(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ double uniform_d(double v)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Weight, arrival and their patch derivatives of one confocal pair.
struct PairS {
    float w;        // weight
    float w_a;      // w / a
    float dw_dz;    // dw / dpz
    float dwn;      // dw / dn = dwn * (dx, dy, pz)
    float du_dz;    // du / dpz (bins per metre)
    double u;       // arrival (bins), fp64
};

__device__ __forceinline__ PairS pair_smooth(float4 A, float4 B, float wx, float wy, double o, float gg,
                                             double inv, bool cosines, bool derivs)
{
    PairS r;
    const float dx = A.x - wx, dy = A.y - wy, pz = A.z;
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, pz * pz));
    const float ri2 = __builtin_amdgcn_rcpf(r2);   // weights only: 1 ulp is ample
    const float ri4 = ri2 * ri2;
    // fp64 arrival from the same fp32 coordinates: (2 r + o) * inv, with
    // 2 r = 2 rf + (r^2 - rf^2) / rf, rf an fp32 square root: one Newton step,
    // the residual exact in fp64 (relative error ~1e-14, far below what the
    // Gaussian samples can see; r^2 > 0 since pz > 0)
    const double ex = (double)A.x - (double)wx, ey = (double)A.y - (double)wy, ez = (double)pz;
    const double r2d = (ex * ex + ey * ey) + ez * ez;
    const float rf = __builtin_amdgcn_sqrtf((float)r2d);
    const double rfd = (double)rf;
    const double rr = fma((double)__builtin_amdgcn_rcpf(rf), fma(-rfd, rfd, r2d), rfd + rfd);
    r.u = (rr + o) * inv;
    if (cosines) {
        // w = a gg pz^2 c^2 / r^8, c = -n.(p - w) clamped at 0
        const float c = fmaxf(-(B.x * dx + B.y * dy + B.z * pz), 0.f);
        const float k = gg * pz * pz * ri4 * ri4;
        r.w_a = k * c * c;
        r.w = A.w * r.w_a;
        if (derivs) {
            r.dw_dz = A.w * k * (2.f * c * c * __builtin_amdgcn_rcpf(pz) - 2.f * c * B.z) - r.w * 8.f * pz * ri2;
            r.dwn = -2.f * A.w * k * c;
        }
    } else {
        r.w_a = gg * ri4;
        r.w = A.w * r.w_a;
        if (derivs) {
            r.dw_dz = -r.w * 4.f * pz * ri2;
            r.dwn = 0.f;
        }
    }
    if (derivs) r.du_dz = (float)inv * 2.f * pz * __builtin_amdgcn_rsqf(r2);   // (gradients: 1 ulp is ample)
    return r;
}

}  // namespace

// ---------------------------------------------------------------------------
// Smooth forward.  RS > 0: the support radius is RS (= a.Rs), known at
// compile time, so a pair whose whole support lies inside the window takes a
// straight-line tap sequence with no bounds tests and the tap offsets folded
// into the LDS instructions; RS = 0, or a support that crosses the window's
// ends, takes the general loop.
template <int TX, int TY, bool COS, int RS>
__global__ void __launch_bounds__(kBlock) k_smooth(const SmoothArgs a)
{
    constexpr int NH = TX * TY;
    extern __shared__ __align__(16) unsigned char smem[];
    u64s* hist = reinterpret_cast<u64s*>(smem);
    double* so = reinterpret_cast<double*>(smem + (size_t)NH * a.stride * 8);
    float* sg = reinterpret_cast<float*>(so + NH);
    float* red = sg + NH;
    const int n_act = smooth_active(a);
    const int split = (int)(blockIdx.x % a.n_split);
    const int tile = (int)(blockIdx.x / a.n_split);
    const int tx0 = (tile / a.tiles_y) * TX, ty0 = (tile % a.tiles_y) * TY;
    const int chunk = (n_act + a.n_split - 1) / a.n_split;
    const int pb = min(n_act, split * chunk), pe = min(n_act, pb + chunk);

    for (int i = threadIdx.x; i < NH * a.stride; i += blockDim.x) hist[i] = 0ull;
    if (threadIdx.x < NH) {
        const int j = threadIdx.x;
        const int ix = min(tx0 + j / TY, a.rx.n - 1), iy = min(ty0 + j % TY, a.ry.n - 1);
        double off, g;
        device_leg(canon(a.rx, ix), canon(a.ry, iy), a.cx, a.cy, a.s, &off, &g);
        so[j] = off + off;
        sg[j] = (float)(g * g);
    }
    float wx[TX], wy[TY];
#pragma unroll
    for (int c = 0; c < TX; ++c) wx[c] = canon(a.rx, min(tx0 + c, a.rx.n - 1));
#pragma unroll
    for (int r = 0; r < TY; ++r) wy[r] = canon(a.ry, min(ty0 + r, a.ry.n - 1));
    // weight bound over the record summaries: a_max / r_min^4 (every cosine
    // factor and stand-off weight is at most 1) -> fixed-point scale
    float wb = 0.f;
    {
        const float x0 = fminf(wx[0], wx[TX - 1]), x1 = fmaxf(wx[0], wx[TX - 1]);
        const float y0 = fminf(wy[0], wy[TY - 1]), y1 = fmaxf(wy[0], wy[TY - 1]);
        for (int i = threadIdx.x; i < a.n_stats; i += blockDim.x) {
            const StatF c = load_stat(a.stats, i);
            if (c.count <= 0) continue;
            const float ddx = fmaxf(fmaxf(x0 - c.x1, c.x0 - x1), 0.f);
            const float ddy = fmaxf(fmaxf(y0 - c.y1, c.y0 - y1), 0.f);
            const float r2 = fmaf(ddx, ddx, fmaf(ddy, ddy, c.z0 * c.z0));
            wb = fmaxf(wb, c.amax / (r2 * r2));
        }
    }
    wb = wave_max_f(wb);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = wb;
    __syncthreads();
    float W = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) W = fmaxf(W, red[w]);
    const float s = W > 0.f ? 2147483648.0f / (W * a.norm) : 1.0f;   // increments <= 2^31
    const float sn = s * a.norm;
    const int T = a.T, Rs = a.Rs;
    const float inv_s2 = a.inv_s2, c1 = a.c1;

    for (int base = pb; base < pe; base += blockDim.x) {
        const int p = base + (int)threadIdx.x;
        if (p >= pe) continue;
        const float4 A = a.patches[2 * (size_t)p];
        const float4 B = a.patches[2 * (size_t)p + 1];
#pragma unroll
        for (int c = 0; c < TX; ++c) {
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                const int j = c * TY + r;
                if (tx0 + c >= a.rx.n || ty0 + r >= a.ry.n) continue;
                const PairS q = pair_smooth(A, B, wx[c], wy[r], so[j], sg[j], a.inv, COS, false);
                const double k0d = floor(q.u);
                if (q.w <= 0.f || k0d + Rs < 0.0 || k0d - Rs > (double)(T - 1)) continue;
                const int k0 = (int)k0d;
                const float f = (float)(q.u - k0d);
                const float x0 = 0.5f - f;
                const float amp = q.w * sn;
                u64s* row = hist + (size_t)j * a.stride;
                // centre and upward: e_{m+1} = e_m q_m, q_{m+1} = q_m c1
                float e = __expf(-0.5f * x0 * x0 * inv_s2);
                const float e0 = e;
                float qm = __expf(-(1.0f - f) * inv_s2);
                if (RS > 0 && k0 >= RS && k0 + RS < T) {
                    u64s* ctr = row + k0;
#pragma unroll
                    for (int m = 0; m <= RS; ++m) {
                        __hip_atomic_fetch_add(ctr + m, (u64s)(uint32_t)fmaf(amp, e, 0.5f), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                        e *= qm;
                        qm *= c1;
                    }
                    e = e0;
                    float dm = __expf(-f * inv_s2);
#pragma unroll
                    for (int m = 1; m <= RS; ++m) {
                        e *= dm;
                        dm *= c1;
                        __hip_atomic_fetch_add(ctr - m, (u64s)(uint32_t)fmaf(amp, e, 0.5f), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    continue;
                }
                for (int m = 0; m <= Rs; ++m) {
                    const int k = k0 + m;
                    if (k >= T) break;
                    if (k >= 0) {
                        const uint32_t inc = (uint32_t)fmaf(amp, e, 0.5f);
                        if (inc) __hip_atomic_fetch_add(row + k, (u64s)inc, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    e *= qm;
                    qm *= c1;
                }
                // downward: e_{m-1} = e_m d_m, d_{m-1} = d_m c1
                e = e0;
                float dm = __expf(-f * inv_s2);
                for (int m = -1; m >= -Rs; --m) {
                    e *= dm;
                    dm *= c1;
                    const int k = k0 + m;
                    if (k < 0) break;
                    if (k < T) {
                        const uint32_t inc = (uint32_t)fmaf(amp, e, 0.5f);
                        if (inc) __hip_atomic_fetch_add(row + k, (u64s)inc, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
        }
    }
    __syncthreads();
    const float inv_s = 1.0f / s;
    for (int i = threadIdx.x; i < NH * T; i += blockDim.x) {
        const int j = i / T, t = i - j * T;
        const int ix = tx0 + j / TY, iy = ty0 + j % TY;
        if (ix >= a.rx.n || iy >= a.ry.n) continue;
        const u64s x = hist[(size_t)j * a.stride + t];
        const float v = fmaf((float)(uint32_t)(x >> 32), 4294967296.0f, (float)(uint32_t)x) * inv_s;
        float* o = a.out + ((size_t)ix * a.ry.n + iy) * (size_t)T + t;
        if (a.atomic_out)
            unsafeAtomicAdd(o, v);
        else
            *o = v;
    }
}

// ---------------------------------------------------------------------------
// Moments of the sub-bin offset.  With t = f - 1/2 the pair's offset from the
// centre of its bin k0 = floor(u), its contribution w N(d + 1/2 - f) =
// w N(d - t) to bin k0 + d is, for every d, a polynomial in -t up to an error
// that MomentFit bounds:
//     N(d - t) = sum_{m < n} (-t)^m K_m(d),
// the polynomial through the n Chebyshev nodes of [-1/2, 1/2].  A pair
// therefore adds w (-t)^m to moment row m at bin k0 (n LDS adds instead of
// 2 Rs + 1), and the flush convolves moment row m with K_m.  Interpolation
// spreads the error evenly over the bin where a Taylor series about its
// centre piles it up at the edges: at sigma = 2.65 bins and n = 6, 2.5e-8
// (relative L2 over the support, worst t) against 8e-7.
// K_m(-d) = (-1)^m K_m(d), as the nodes are symmetric.

// K_m(d), |d| <= Rs, fp32 of the fp64 value.
__device__ __forceinline__ float moment_tap(const MomentFit& f, int m, int d)
{
    const int ad = d < 0 ? -d : d;
    if (ad > f.Rs || ((m & 1) && d == 0)) return 0.f;
    double k = 0.0;
    for (int j = 0; j < f.n; ++j) {
        const double x = ((double)ad + f.node[j]) / f.sigma;
        k += f.coef[m * kMaxMoments + j] * exp(-0.5 * x * x);
    }
    k *= f.norm;
    return (float)((d < 0 && (m & 1)) ? -k : k);
}

// The first n_stats workgroups make the record summaries of the forward (none
// for the adjoint); the others the kernels' table, the same for every
// workgroup of the launches behind (scalar reads there):
//   forward  [m][taps_fwd(Rs)]   word e = K_m(Rs - e), zeros past 2 Rs
//   adjoint  [m][taps_adj(Rs)]   word 0 = K_m(0), word 3 + d = K_m(d), zeros
//                                elsewhere
__global__ void __launch_bounds__(kStatBlock)
    k_smooth_prep(const SmoothArgs a, const MomentFit f, int adjoint)
{
    if ((int)blockIdx.x < a.n_stats) {
        chunk_stats_body(a.patches, smooth_active(a), a.stats, (int)blockIdx.x);
        return;
    }
    const int pitch = adjoint ? taps_adj(f.Rs) : taps_fwd(f.Rs);
    const int nb = (int)gridDim.x - a.n_stats;
    for (int i = ((int)blockIdx.x - a.n_stats) * kStatBlock + (int)threadIdx.x; i < f.n * pitch; i += nb * kStatBlock) {
        const int m = i / pitch, e = i % pitch;
        a.mtaps[i] = adjoint ? (e == 0 || e > 3 ? moment_tap(f, m, e == 0 ? 0 : e - 3) : 0.f)
                             : moment_tap(f, m, f.Rs - e);   // (0 past the support)
    }
}

typedef const __attribute__((address_space(4))) float* kconst;

// Distance terms of one pair from its squared distance in fp64 (r2d) and fp32
// (r2f): the bin k0 = floor(u), mt = 1/2 - (u - k0) and the reciprocals the
// weight takes.  u = 2 r inv + o inv with 2 r = 2 rf + (r^2 - rf^2) / rf, rf an
// fp32 root: one Newton step, its residual exact in fp64 (relative error
// ~1e-14; an fp32 arrival would put u off by ~1e-4 bins at u ~ 1000).  The
// step, below 1e-4 bins, goes to mt alone: where it would carry u over a bin
// edge, mt leaves [-1/2, 1/2] by that much, which the polynomials take as is.
struct Arrival {
    int k0;
    float mt;
    float ri2;    // 1 / r^2
    float rinv;   // 1 / r
};

__device__ __forceinline__ Arrival arrival(double r2d, float r2f, double inv2, double oi, float invf)
{
    Arrival q;
    const float rf = __builtin_amdgcn_sqrtf(r2f);
    q.ri2 = __builtin_amdgcn_rcpf(r2f);   // (weights: 1 ulp is ample)
    q.rinv = rf * q.ri2;
    const double rfd = (double)rf;
    const double base = fma(rfd, inv2, oi);
    const float step = (float)fma(-rfd, rfd, r2d) * (q.rinv * invf);
    q.k0 = (int)base;   // base >= 0; a saturated conversion fails the range test
    q.mt = (0.5f - (float)__builtin_amdgcn_fract(base)) - step;
    return q;
}

// Nearest integer of a float within the int32 range (one instruction).
__device__ __forceinline__ int round_i(float v)
{
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// Squared distance past which every arrival of a scan point with offset o lies
// at least two bins past bin T - 1 + Rs, the last one that reaches the window
// (enlarged by 1e-5: the fp32 squares round).
__device__ __forceinline__ float cull_r2(const SmoothArgs& a, double o)
{
    const double r = 0.5 * ((double)(a.T + a.Rs + 2) / a.inv - o);
    return r > 0.0 ? (float)(r * r * 1.00001) : 0.f;
}

// Smooth forward by moments.  A workgroup owns NP scan points of one wall row
// (x0 .. x0 + NP - 1, y), NM moment rows each, and streams all records (or its
// share of them), a patch per lane.  Terms of y are per patch, shared by the
// NP points.  A wavefront whose patches all arrive past the window (a record
// wavefront is a small square of the surface) goes on at once; the record
// order deals a 16 x 16-pixel block's four wavefronts to the four SIMDs, so
// what is skipped thins all of them alike.
// Bound: the LDS adds -- a 64-lane ds_add_u64 takes 7.5 cycles on consecutive
// bins, 10.9 on random ones and 8.6 more per lane that shares a bin; here 13
// on average, NM of them per pair -- with VALU (about 50 instructions per pair
// that reaches the window) close behind.  128^2 points and patches, 1024 bins:
// radius 16 (NM = 6) 0.80 -> 0.65 ms; 48 x 40 points, 3840 patches, 1501 bins,
// radius 31: 185 us by taps, 69 by moments.
template <bool COS, int NM, int NP, int WG>
__global__ void __launch_bounds__(kBlock, 4 * WG) k_smooth_mom(const SmoothArgs a)
{
    constexpr int NR = NP * NM, PITCH = smooth_mom_pitch(NP, NM, WG);
    extern __shared__ __align__(16) unsigned char smem[];
    u64s* hist = reinterpret_cast<u64s*>(smem);   // row (point c, moment m) = c NM + m; bin k0 at k0 + Rs
    double* so = reinterpret_cast<double*>(smem + (size_t)NR * PITCH * 8);
    float* sg = reinterpret_cast<float*>(so + NP);
    float* red = sg + NP;
    const int n_act = smooth_active(a);
    const int split = (int)(blockIdx.x % a.n_split);
    const int tile = (int)(blockIdx.x / a.n_split);
    const int tx0 = (tile / a.tiles_y) * NP, ty0 = tile % a.tiles_y;
    const int chunk = (n_act + a.n_split - 1) / a.n_split;
    const int pb = min(n_act, split * chunk), pe = min(n_act, pb + chunk);
    const int T = a.T, Rs = a.Rs;

    static_assert(PITCH % 2 == 0, "rows are cleared 16 bytes at a time");
    for (int i = threadIdx.x; i < NR * PITCH / 2; i += kBlock) reinterpret_cast<uint4*>(hist)[i] = uint4{0, 0, 0, 0};
    if (threadIdx.x < NP) {
        const int c = threadIdx.x;
        double off, g;
        device_leg(canon(a.rx, min(tx0 + c, a.rx.n - 1)), canon(a.ry, ty0), a.cx, a.cy, a.s, &off, &g);
        so[c] = off + off;
        sg[c] = (float)(g * g);
    }
    float wx[NP];
#pragma unroll
    for (int c = 0; c < NP; ++c) wx[c] = uniform_f(canon(a.rx, min(tx0 + c, a.rx.n - 1)));
    const float wy = uniform_f(canon(a.ry, ty0));
    const float x0 = fminf(wx[0], wx[NP - 1]), x1 = fmaxf(wx[0], wx[NP - 1]);
    // weight bound over the record summaries: a_max / r_min^4 -> scale
    float wb = 0.f;
    for (int i = threadIdx.x; i < a.n_stats; i += kBlock) {
        const StatF c = load_stat(a.stats, i);
        if (c.count <= 0) continue;
        const float ddx = fmaxf(fmaxf(x0 - c.x1, c.x0 - x1), 0.f);
        const float ddy = fmaxf(fmaxf(wy - c.y1, c.y0 - wy), 0.f);
        const float r2 = fmaf(ddx, ddx, fmaf(ddy, ddy, c.z0 * c.z0));
        wb = fmaxf(wb, c.amax / (r2 * r2));
    }
    wb = wave_max_f(wb);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = wb;
    __syncthreads();
    float W = 0.f;
    for (int w = 0; w < kBlock / 64; ++w) W = fmaxf(W, red[w]);
    const float s = W > 0.f ? 1073741824.0f / W : 1.0f;   // |increments| <= 2^30
    double oi[NP];
    float gs[NP];
    float cut = 0.f;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
        const double o = uniform_d(so[c]);
        oi[c] = uniform_d(o * a.inv);
        gs[c] = uniform_f(sg[c] * s);
        cut = fmaxf(cut, cull_r2(a, o));
    }
    cut = uniform_f(cut);
    const double inv2 = 2.0 * a.inv, wyd = (double)wy;
    const float invf = (float)a.inv;
    const int n_pts = NP > 1 ? min(NP, a.rx.n - tx0) : 1;   // (fewer at the wall's end)

    for (int base = pb; base < pe; base += kBlock) {
        const int p = base + (int)threadIdx.x;
        if (p >= pe) continue;
        const float4 A = a.patches[2 * (size_t)p];
        const float4 B = a.patches[2 * (size_t)p + 1];
        const float dy = A.y - wy;
        const float dxm = fmaxf(fmaxf(x0 - A.x, A.x - x1), 0.f);
        if (__all(fmaf(dxm, dxm, fmaf(dy, dy, A.z * A.z)) >= cut)) continue;
        const double px = (double)A.x, ey = (double)A.y - wyd, ez = (double)A.z;
        const double yz2 = fma(ey, ey, ez * ez);
        // w = a g pz^2 c^2 / r^8, c = -n.(p - w) clamped at 0 (a g / r^4 without cosines)
        const float cyz = fmaf(-B.y, dy, -B.z * A.z);
        const float aw = COS ? A.w * (A.z * A.z) : A.w;
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            if (c >= n_pts) break;   // uniform
            const double ex = px - (double)wx[c];
            const double r2d = fma(ex, ex, yz2);
            const Arrival q = arrival(r2d, (float)r2d, inv2, oi[c], invf);
            const float ri4 = q.ri2 * q.ri2;
            const float cn = COS ? fmaxf(fmaf(-B.x, A.x - wx[c], cyz), 0.f) : 1.f;
            const float h = COS ? cn * ri4 : 1.f;
            float v = (aw * gs[c]) * (COS ? h * h : ri4);
            // the support [k0 - Rs, k0 + Rs] meets the bins [0, T)
            if (v <= 0.f || (uint32_t)q.k0 + (uint32_t)Rs > (uint32_t)(T - 1 + 2 * Rs)) continue;
            u64s* r0 = hist + (c * NM) * PITCH + (q.k0 + Rs);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                // even moments are non-negative (w > 0, (-t)^m >= 0): no sign extension
                const int iv = round_i(v);
                const u64s inc = (m & 1) ? (u64s)(long long)iv : (u64s)(uint32_t)iv;
                __hip_atomic_fetch_add(r0 + m * PITCH, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                v *= q.mt;
            }
        }
    }
    __syncthreads();
    // moment rows -> float, in place (row r starts at the same byte; values
    // pass through registers so that no thread overwrites what another
    // reads), and zeros behind each row: the last windows reach past it
    constexpr int kPer = (NR * PITCH + kBlock - 1) / kBlock;
    float vals[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = min((int)threadIdx.x + k * kBlock, NR * PITCH - 1);
        // (the low word as a signed one: of a small negative sum it is near
        // 2^32 and would round there)
        const int2 x = reinterpret_cast<const int2*>(hist)[i];
        vals[k] = fmaf((float)(x.y - (x.x >> 31)), 4294967296.0f, (float)x.x);
    }
    __syncthreads();
    float* F = reinterpret_cast<float*>(smem);     // row r at float offset 2 r PITCH
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = (int)threadIdx.x + k * kBlock;
        if (i < NR * PITCH) F[i + (i / PITCH) * PITCH] = vals[k];
    }
    static_assert(PITCH >= 8, "room for the zeros");
    for (int i = threadIdx.x; i < NR * 8; i += kBlock) F[(i / 8) * 2 * PITCH + PITCH + i % 8] = 0.f;
    __syncthreads();
    // Each thread takes V = 4 consecutive bins of one scan point.  Bin k0 + v
    // is sum_m sum_e F_m[k0 + v + e] K_m(Rs - e): per moment a sliding window
    // of two 16-byte LDS reads (one new per four taps; rows start and k0 are
    // multiples of four floats), taps as scalars.  The sums run over m downwards,
    // then e; the largest row's, last, four taps at a time, so that few additions
    // round at the size of the result.
    // Rows with fewer groups of bins than threads leave wavefronts over: the taps
    // are then dealt to up to four sets of wavefronts, whose sums meet in LDS
    // (the rows are no longer read) and are added in the order of the taps (four
    // to six of sixteen wavefronts at work: the two cases above 0.69 ms and 84 us).
    const float inv_sc = 1.0f / s;
    constexpr int V = 4;
    const int nseg = (T + V - 1) / V, npp = taps_fwd(Rs), n_out = NP * nseg;
    kconst kt = (kconst)a.mtaps;
    const bool vec_out = !a.atomic_out && (T & 3) == 0 && ((uintptr_t)a.out & 15) == 0;
    // taps e0 .. e1 - 1 of output group o (multiples of four)
    const auto convolve = [&](int c, int k0, int e0, int e1, float (&acc)[V]) {
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = 0.f;
#pragma unroll
        for (int m = NM - 1; m >= 0; --m) {
            const float4* f4 = reinterpret_cast<const float4*>(F + (size_t)(c * NM + m) * 2 * PITCH + k0);
            kconst tm = kt + m * npp;
            float4 lo = f4[e0 / 4];
#pragma unroll 4
            for (int e = e0; e < e1; e += 4) {
                const float4 hi = f4[e / 4 + 1];
                const float w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                float part[V];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float t = tm[e + i];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        if (m > 0)
                            acc[v] = fmaf(w[v + i], t, acc[v]);
                        else
                            part[v] = i == 0 ? w[v] * t : fmaf(w[v + i], t, part[v]);
                    }
                }
                if (m == 0) {
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] += part[v];
                }
                lo = hi;
            }
        }
    };
    const auto store = [&](int c, int k0, const float (&acc)[V]) {
        float* dst = a.out + ((size_t)(tx0 + c) * a.ry.n + ty0) * (size_t)T + k0;
        if (vec_out && k0 + V <= T) {
            *reinterpret_cast<float4*>(dst) = make_float4(acc[0] * inv_sc, acc[1] * inv_sc, acc[2] * inv_sc, acc[3] * inv_sc);
            return;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (k0 + v >= T) break;
            if (a.atomic_out)
                unsafeAtomicAdd(dst + v, acc[v] * inv_sc);
            else
                dst[v] = acc[v] * inv_sc;
        }
    };
    float acc[V];
    const int span = (n_out + 63) / 64;                       // wavefronts per set
    const int sets = min(4, (kBlock / 64) / span);            // (0: more groups than threads)
    if (sets <= 1) {
        for (int o = threadIdx.x; o < n_out; o += kBlock) {
            const int c = o / nseg, k0 = (o - c * nseg) * V;
            if (tx0 + c >= a.rx.n) continue;
            convolve(c, k0, 0, npp, acc);
            store(c, k0, acc);
        }
        return;
    }
    const int set = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) / span);
    const int o = (int)threadIdx.x - set * span * 64;
    const int c = o / nseg, k0 = (o - c * nseg) * V;
    const bool on = set < sets && o < n_out && tx0 + c < a.rx.n;
    const int per = (npp / 4 + sets - 1) / sets * 4;
    if (on) convolve(c, k0, min(npp, set * per), min(npp, (set + 1) * per), acc);
    __syncthreads();
    float4* part = reinterpret_cast<float4*>(smem);           // [sets - 1][n_out]
    if (on && set > 0) part[(set - 1) * n_out + o] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    __syncthreads();
    if (!on || set > 0) return;
    for (int i = 0; i + 1 < sets; ++i) {
        const float4 q = part[i * n_out + o];
        acc[0] += q.x;
        acc[1] += q.y;
        acc[2] += q.z;
        acc[3] += q.w;
    }
    store(c, k0, acc);
}

// ---------------------------------------------------------------------------
// Adjoint gather.  RS as in k_smooth: a support inside the window takes a
// straight-line tap sequence (G1 = x0 G0 + sum g N(x) m there).
template <bool COS, int RS>
__global__ void __launch_bounds__(kBlock) k_adjoint(const SmoothArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = a.T, Rs = a.Rs, NR = a.rows;
    float* rowbuf = reinterpret_cast<float*>(smem);                        // [NR][T]
    double* so = reinterpret_cast<double*>(smem + (((size_t)NR * T * 4 + 15) & ~(size_t)15));
    float* swx = reinterpret_cast<float*>(so + NR);
    float* swy = swx + NR;
    float* sg = swy + NR;
    const int n_act = smooth_active(a);
    const int p = (int)blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
    const int split = (int)blockIdx.y;
    const int S = a.rx.n * a.ry.n;
    const int per = (S + a.n_split - 1) / a.n_split;
    const int s0 = min(S, split * per), s1 = min(S, s0 + per);
    const bool live = p < n_act;
    float4 A = make_float4(0.f, 0.f, 1.f, 0.f), B = make_float4(0.f, 0.f, -1.f, 0.f);
    if (live) {
        A = a.patches[2 * (size_t)p];
        B = a.patches[2 * (size_t)p + 1];
    }
    double gz = 0.0, ga = 0.0, gnx = 0.0, gny = 0.0, gnz = 0.0;
    const float inv_s2 = a.inv_s2, c1 = a.c1;

    for (int j0 = s0; j0 < s1; j0 += NR) {
        const int nr = min(NR, s1 - j0);
        __syncthreads();
        // stage rows [j0, j0 + nr) of the upstream gradient (float4 when aligned)
        if ((T & 3) == 0) {
            const float4* src = reinterpret_cast<const float4*>(a.grad_out + (size_t)j0 * T);
            float4* dst = reinterpret_cast<float4*>(rowbuf);
            for (int i = threadIdx.x; i < nr * (T >> 2); i += blockDim.x) dst[i] = src[i];
        } else {
            const float* src = a.grad_out + (size_t)j0 * T;
            for (int i = threadIdx.x; i < nr * T; i += blockDim.x) rowbuf[i] = src[i];
        }
        if (threadIdx.x < nr) {
            const int h = j0 + threadIdx.x;
            const float wx = canon(a.rx, h / a.ry.n), wy = canon(a.ry, h % a.ry.n);
            double off, g;
            device_leg(wx, wy, a.cx, a.cy, a.s, &off, &g);
            so[threadIdx.x] = off + off;
            swx[threadIdx.x] = wx;
            swy[threadIdx.x] = wy;
            sg[threadIdx.x] = (float)(g * g);
        }
        __syncthreads();
        if (!live) continue;
        for (int jj = 0; jj < nr; ++jj) {
            const PairS q = pair_smooth(A, B, swx[jj], swy[jj], so[jj], sg[jj], a.inv, COS, true);
            const double k0d = floor(q.u);
            if (k0d + Rs < 0.0 || k0d - Rs > (double)(T - 1)) continue;
            const int k0 = (int)k0d;
            const float f = (float)(q.u - k0d);
            const float* g = rowbuf + (size_t)jj * T;
            // G0 = sum g N(x), G1 = sum g x N(x), x = m + 1/2 - f (N without
            // its normalisation; applied below)
            float G0 = 0.f, G1 = 0.f;
            const float x0 = 0.5f - f;
            float e = __expf(-0.5f * x0 * x0 * inv_s2);
            const float e0 = e;
            float qm = __expf(-(1.0f - f) * inv_s2);
            if (RS > 0 && k0 >= RS && k0 + RS < T) {
                const float* gc = g + k0;
                float G1m = 0.f;
#pragma unroll
                for (int m = 0; m <= RS; ++m) {
                    const float gv = gc[m] * e;
                    G0 += gv;
                    G1m = fmaf(gv, (float)m, G1m);
                    e *= qm;
                    qm *= c1;
                }
                e = e0;
                float dm = __expf(-f * inv_s2);
#pragma unroll
                for (int m = 1; m <= RS; ++m) {
                    e *= dm;
                    dm *= c1;
                    const float gv = gc[-m] * e;
                    G0 += gv;
                    G1m = fmaf(gv, -(float)m, G1m);
                }
                G1 = fmaf(x0, G0, G1m);
            } else {
                for (int m = 0; m <= Rs; ++m) {
                    const int k = k0 + m;
                    if (k >= T) break;
                    if (k >= 0) {
                        const float gv = g[k] * e;
                        G0 += gv;
                        G1 = fmaf(gv, x0 + (float)m, G1);
                    }
                    e *= qm;
                    qm *= c1;
                }
                e = e0;
                float dm = __expf(-f * inv_s2);
                for (int m = -1; m >= -Rs; --m) {
                    e *= dm;
                    dm *= c1;
                    const int k = k0 + m;
                    if (k < 0) break;
                    if (k < T) {
                        const float gv = g[k] * e;
                        G0 += gv;
                        G1 = fmaf(gv, x0 + (float)m, G1);
                    }
                }
            }
            G0 *= a.norm;
            G1 *= a.norm * inv_s2;
            // dL/dw = G0, dL/du = w G1
            const float dz = fmaf(G0, q.dw_dz, q.w * G1 * q.du_dz);
            gz += (double)dz;
            ga += (double)(G0 * q.w_a);
            if (COS) {
                const float gn = G0 * q.dwn;
                gnx += (double)(gn * (A.x - swx[jj]));
                gny += (double)(gn * (A.y - swy[jj]));
                gnz += (double)(gn * A.z);
            }
        }
    }
    if (live) {
        double* o = a.partial + ((size_t)split * a.n_cap + p) * kAdjStride;
        o[0] = gz;
        o[1] = ga;
        o[2] = gnx;
        o[3] = gny;
        o[4] = gnz;
    }
}

// ---------------------------------------------------------------------------
// Adjoint by moments.  For a pair with bin k0 and offset t (as in
// k_smooth_mom), G0 = sum_k g[k] N(x) over the support is the polynomial
//     P(-t) = sum_{m < n} (-t)^m C_m[k0],
// and G1 = sum_k g[k] (x / sigma^2) N(x) = -sum_k g[k] N'(x) is -P'(-t), of
// the correlations C_m[k0] = sum_{|d|<=Rs} g[k0 + d] K_m(d).  k_adj_moments
// computes C_0 .. C_{n-1} once per scan point (bins k0 = -H .. T4 + H - 1, H
// and T4 the radius and T rounded up to 4; a bin's n values side by side, NS
// apart with NS odd so that neighbouring bins start on different banks);
// k_adjoint_mom then needs n LDS reads and one Horner pass for P and P'.

// A thread produces V = 4 consecutive bins k0 .. k0 + 3 of one scan point from
// sliding windows of its upstream gradient on either side (zero outside
// 0 .. T - 1; one new 16-byte read per side and four taps).  The kernels have
// the parity of their order, so
//     C_m[k0] = K_m(0) g[k0] + sum_{d=1..Rs} K_m(d) (g[k0 + d] + (-1)^m g[k0 - d]):
// a bin's mirrored sums serve every even row and its mirrored differences
// every odd row.  The kernels are scalar reads (written by an earlier launch).
// The 4 NS values of a thread go through LDS (its own wavefront's piece), so
// that the stores are contiguous over the wavefront.  ALIGNED: T a multiple of
// 4 and the gradient 16-byte aligned; else the same 16-byte reads at addresses
// that are multiples of 4, and single ones at the ends of a row (all reads
// single: 48 x 40 points, 1501 bins, radius 31, 55 us; so, 38).
// Bound: HBM, NS words written per bin and point (128^2 points, 1056 bins of 7
// words: 484 MB in 107 us), and past a radius of about 24 the 8 to 11
// operations per tap and bin.
template <int NM, bool ALIGNED>
__global__ void __launch_bounds__(256) k_adj_moments(const SmoothArgs a)
{
    constexpr int V = 4, NS = adj_row_words(NM);
    __shared__ __align__(16) float tr[4][64 * V * NS];
    const int T = a.T, L = a.mlen, Q = L / V, H = adj_halo(a.Rs);
    const int64_t n_thr = (int64_t)a.sn * Q;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    if (t < n_thr) {
        const int s = (int)(t / Q), k0 = (int)(t % Q) * V - H;
        const float* g = a.grad_out + (size_t)s * T;
        const auto read4 = [&](int k) {
            if constexpr (ALIGNED) {   // wholly inside the row or wholly in the padding
                return (k >= 0 && k < T) ? *reinterpret_cast<const float4*>(g + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
                // one 16-byte read at the nearest four bins of the row that
                // exist; the lanes at its ends read theirs singly instead
                struct __attribute__((packed, aligned(4))) Four {
                    float x, y, z, w;
                };
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (T >= 4) {
                    const Four f = *reinterpret_cast<const Four*>(g + min(max(k, 0), T - 4));
                    v = make_float4(f.x, f.y, f.z, f.w);
                }
                if (k < 0 || k + 4 > T) {
                    const auto one = [&](int i) { return (i >= 0 && i < T) ? g[i] : 0.f; };
                    v = make_float4(one(k), one(k + 1), one(k + 2), one(k + 3));
                }
                return v;
            }
        };
        kconst kc = (kconst)a.mtaps;
        const int np = taps_adj(a.Rs);
        float4 mid = read4(k0);
        float acc[V][NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const float k = kc[m * np];
            acc[0][m] = (m & 1) ? 0.f : mid.x * k;
            acc[1][m] = (m & 1) ? 0.f : mid.y * k;
            acc[2][m] = (m & 1) ? 0.f : mid.z * k;
            acc[3][m] = (m & 1) ? 0.f : mid.w * k;
        }
        float4 r0 = mid, l0 = mid;
        // distances d = b - 3 .. b, `last` of them within the support
        const auto block = [&](int b, int last) {
            const float4 r1 = read4(k0 + b), l1 = read4(k0 - b);
            const float r[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};   // g[k0 + b - 4 + i]
            const float l[8] = {l1.x, l1.y, l1.z, l1.w, l0.x, l0.y, l0.z, l0.w};   // g[k0 - b + i]
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // d = b - 3 + i
                if (i >= last) break;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const float hi = r[v + 1 + i], lo = l[v + 3 - i];
                    const float sum = hi + lo, dif = hi - lo;
#pragma unroll
                    for (int m = 0; m < NM; ++m) acc[v][m] = fmaf((m & 1) ? dif : sum, kc[m * np + b + i], acc[v][m]);
                }
            }
            r0 = r1;
            l0 = l1;
        };
        int b = 4;
#pragma unroll 2
        for (; b <= a.Rs; b += 4) block(b, 4);
        // (the rest by count, not by zero taps: nothing past the support is used)
        if (b - 3 <= a.Rs) block(b, a.Rs - b + 4);
        float* mine = tr[wave] + lane * V * NS;
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int m = 0; m < NS; ++m) mine[v * NS + m] = m < NM ? acc[v][m] : 0.f;
    }
    // (a wavefront's LDS operations run in order; its piece is no one else's)
    __builtin_amdgcn_wave_barrier();
    const int64_t t0 = t - lane;   // the wavefront's first thread: its output is contiguous
    if (t0 >= n_thr) return;
    const int n4 = (int)(n_thr - t0 < 64 ? n_thr - t0 : 64) * NS;
    float4* dst = reinterpret_cast<float4*>(a.moments + t0 * V * NS);
    const float4* src = reinterpret_cast<const float4*>(tr[wave]);
#pragma unroll
    for (int i = 0; i < NS; ++i)
        if (i * 64 + lane < n4) dst[i * 64 + lane] = src[i * 64 + lane];
}

// Gather: PPT patches per thread, a range of scan points per workgroup whose
// correlation rows are staged in LDS a few points at a time.  The patch's
// albedo weight a is left out of the pair sums (all are linear in it) and
// joins them at the end.  Wavefronts whose patches all arrive past the window
// skip the pair.  Bound: VALU (about 80 instructions per pair that reaches the
// window) and the staging, which reads every row once per block of PPT x 1024
// patches.  128^2 points and patches, 1024 bins, radius 16: 0.67 -> 0.49 ms;
// 48 x 40 points, 3840 patches, 1501 bins, radius 31: 522 us by taps, 95 with
// the correlations.
// PIECE: the launch takes sn scan points from s0 on and adds to the partials of
// the pieces before (an instance of its own: the offset and the sum in one kernel
// for all cost the whole scans of these sizes 0.5 and 6%).
template <bool COS, int NM, bool DB, bool PIECE>
__global__ void __launch_bounds__(kBlock) k_adjoint_mom(const SmoothArgs a)
{
    constexpr int NS = adj_row_words(NM), PPT = kAdjPatches, NB = DB ? 2 : 1;
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = a.T, L = a.mlen, NR = a.rows, Rs = a.Rs, H = adj_halo(a.Rs);
    // NB buffers of NR scan points' rows [NR][L][NS], then per buffer the
    // points' offsets in bins (fp64), positions, gains and cull distances
    const size_t buf_bytes = (size_t)NR * NS * L * 4;
    double* so = reinterpret_cast<double*>(smem + NB * buf_bytes);
    float* swx = reinterpret_cast<float*>(so + NB * NR);
    float* swy = swx + NB * NR;
    float* sg = swy + NB * NR;
    float* sc = sg + NB * NR;
    const int n_act = smooth_active(a);
    // Every workgroup gets patches and scan points from all over the scene,
    // as near the borders more pairs arrive past the window: the blocks with
    // records take the pieces of 256 (a 16 x 16-pixel block, one wavefront
    // each on the four SIMDs) in turn, and the splits the stages of NR points.
    const int nbx = (n_act + PPT * kBlock - 1) / (PPT * kBlock);
    if ((int)blockIdx.x >= nbx) return;   // (nothing reads this block's partials)
    const int split = (int)blockIdx.y;
    const int S = PIECE ? a.sn : a.rx.n * a.ry.n;
    const auto patch = [&](int i) {
        return (((int)threadIdx.x / 256 + 4 * i) * nbx + (int)blockIdx.x) * 256 + (int)threadIdx.x % 256;
    };
    double px[PPT], py[PPT];
    float4 B[PPT];       // normal; w: depth
    float tp[PPT];       // 2 / pz
    bool live[PPT];
    double gz[PPT], ga[PPT], gnx[PPT], gny[PPT], gn[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int p = patch(i);
        live[i] = p < n_act;
        float4 A = make_float4(0.f, 0.f, 1.f, 0.f);
        B[i] = make_float4(0.f, 0.f, -1.f, 0.f);
        if (live[i]) {
            A = a.patches[2 * (size_t)p];
            B[i] = a.patches[2 * (size_t)p + 1];
        }
        B[i].w = A.z;
        px[i] = (double)A.x;
        py[i] = (double)A.y;
        tp[i] = 2.f / A.z;
        gz[i] = ga[i] = gnx[i] = gny[i] = gn[i] = 0.0;
    }
    // the constants of scan points [j, j + nr) into buffer b
    auto stage_consts = [&](int b, int j, int nr) {
        if ((int)threadIdx.x < nr) {
            const int h = (PIECE ? a.s0 : 0) + j + (int)threadIdx.x;
            const float wx = canon(a.rx, h / a.ry.n), wy = canon(a.ry, h % a.ry.n);
            double off, g;
            device_leg(wx, wy, a.cx, a.cy, a.s, &off, &g);
            so[b * NR + threadIdx.x] = (off + off) * a.inv;
            sc[b * NR + threadIdx.x] = cull_r2(a, off + off);
            swx[b * NR + threadIdx.x] = wx;
            swy[b * NR + threadIdx.x] = wy;
            sg[b * NR + threadIdx.x] = (float)(g * g);
        }
    };
    // DB: the rows of scan points [j, j + nr) into buffer b by global->LDS
    // loads, 16 bytes per lane at the wavefront's LDS base + 16 lane; they
    // land while the other buffer is in use.  Wavefront w moves the pieces of
    // 64 float4 numbered w, w + 16, ... (L is a multiple of 4: whole pieces
    // of the contiguous rows, the last one masked past the end)
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    auto stage_rows_db = [&](int b, int j, int nr) {
        const float4* s4 = reinterpret_cast<const float4*>(a.moments + (size_t)j * NS * L);
        float* dst = reinterpret_cast<float*>(smem + b * buf_bytes);
        const int n4 = nr * NS * (L >> 2);
        for (int pc = wave; pc * 64 < n4; pc += kBlock / 64) {
            const int i = pc * 64 + lane;
            if (i < n4)
                __builtin_amdgcn_global_load_lds((const void*)(s4 + i),
                                                 (__attribute__((address_space(3))) void*)(dst + (size_t)pc * 256), 16,
                                                 0, 0);
        }
    };
    const double inv2 = 2.0 * a.inv;
    const float invf = (float)a.inv, inv2f = (float)inv2;
    const int n_all = (S + NR - 1) / NR;   // stages of all splits: this one's are split, split + n_split, ...
    const int nst = split < n_all ? (n_all - split + a.n_split - 1) / a.n_split : 0;
    if (DB && nst > 0) {
        const int j = split * NR;
        stage_rows_db(0, j, min(NR, S - j));
        stage_consts(0, j, min(NR, S - j));
    }
    for (int st = 0; st < nst; ++st) {
        const int j0 = (split + st * a.n_split) * NR;
        const int nr = min(NR, S - j0);
        const int b = DB ? (st & 1) : 0;
        if (DB) {
            // this wavefront's loads into buffer b have landed; past the
            // barrier every wavefront's have, and buffer b ^ 1 (the stage
            // before) is no longer read: the next stage goes there
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (st + 1 < nst) {
                const int j = j0 + a.n_split * NR;
                stage_rows_db(b ^ 1, j, min(NR, S - j));
                stage_consts(b ^ 1, j, min(NR, S - j));
            }
        } else {
            __syncthreads();
            // stage the correlation rows of scan points [j0, j0 + nr): contiguous,
            // four loads in flight per thread before their LDS stores (a load
            // past the end rereads the last element; its store is skipped)
            const float4* s4 = reinterpret_cast<const float4*>(a.moments + (size_t)j0 * NS * L);
            float4* d4 = reinterpret_cast<float4*>(smem);
            const int n4 = nr * NS * (L >> 2);
            for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * kBlock) {
                const int last = n4 - 1;
                const float4 v0 = s4[min(i0, last)];
                const float4 v1 = s4[min(i0 + kBlock, last)];
                const float4 v2 = s4[min(i0 + 2 * kBlock, last)];
                const float4 v3 = s4[min(i0 + 3 * kBlock, last)];
                __builtin_amdgcn_sched_barrier(0);
                d4[i0] = v0;
                if (i0 + kBlock < n4) d4[i0 + kBlock] = v1;
                if (i0 + 2 * kBlock < n4) d4[i0 + 2 * kBlock] = v2;
                if (i0 + 3 * kBlock < n4) d4[i0 + 3 * kBlock] = v3;
            }
            stage_consts(0, j0, nr);
            __syncthreads();
        }
        const float* rowbuf = reinterpret_cast<const float*>(smem + b * buf_bytes);
        for (int jj = 0; jj < nr; ++jj) {
            // the scan point's constants, read once for the patches below
            const double wxj = (double)uniform_f(swx[b * NR + jj]), wyj = (double)uniform_f(swy[b * NR + jj]);
            const float gj = uniform_f(sg[b * NR + jj]), cut = uniform_f(sc[b * NR + jj]);
            const double oij = uniform_d(so[b * NR + jj]);
            const float* row = rowbuf + (size_t)jj * L * NS;
#pragma unroll
            for (int i = 0; i < PPT; ++i) {
                if (!live[i]) continue;
                const double ex = px[i] - wxj, ey = py[i] - wyj, ez = (double)B[i].w;
                const double r2d = fma(ex, ex, fma(ey, ey, ez * ez));
                const float r2f = (float)r2d;
                if (__all(r2f >= cut)) continue;
                const Arrival q = arrival(r2d, r2f, inv2, oij, invf);
                if ((uint32_t)q.k0 + (uint32_t)Rs > (uint32_t)(T - 1 + 2 * Rs)) continue;
                const float* c = row + __mul24(q.k0 + H, NS);   // (24 bits hold T + 2 H)
                float D = c[NM - 1];   // P'(-t), one term behind P(-t)
                float P = fmaf(D, q.mt, c[NM - 2]);
#pragma unroll
                for (int m = NM - 3; m >= 0; --m) {
                    D = fmaf(D, q.mt, P);
                    P = fmaf(P, q.mt, c[m]);
                }
                // dL/dw = G0 = P, dL/du = w G1 = -w P'; w = a wa
                const float pz = B[i].w, ri4 = q.ri2 * q.ri2;
                const float du = (inv2f * pz) * q.rinv;
                if (COS) {
                    // wa = g pz^2 c^2 / r^8: d wa / dpz = wa (2 / pz - 8 pz / r^2) - 2 kc n_z,
                    // d wa / dn = -2 kc (p - w), kc = g pz^2 c / r^8
                    const float dx = (float)ex, dy = (float)ey;
                    const float cn = fmaxf(-(B[i].x * dx + B[i].y * dy + B[i].z * pz), 0.f);
                    const float kc = (gj * pz * pz) * (ri4 * ri4) * cn;
                    const float wa = kc * cn;
                    const float h = fmaf(-8.f * pz, q.ri2, tp[i]);
                    gz[i] += (double)(wa * fmaf(P, h, -D * du));
                    ga[i] += (double)(P * wa);
                    const float g = P * kc;
                    gn[i] += (double)g;
                    gnx[i] += (double)(g * dx);
                    gny[i] += (double)(g * dy);
                } else {
                    const float wa = gj * ri4;   // d wa / dpz = -4 wa pz / r^2
                    gz[i] += (double)(wa * fmaf(P, -4.f * pz * q.ri2, -D * du));
                    ga[i] += (double)(P * wa);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int p = patch(i);
        if (!live[i]) continue;
        const double aw = (double)a.patches[2 * (size_t)p].w;
        double* o = a.partial + ((size_t)split * a.n_cap + p) * kAdjStride;
        const auto put = [&](int k, double v) {
            if constexpr (PIECE)
                o[k] = a.s0 > 0 ? o[k] + v : v;
            else
                o[k] = v;
        };
        put(0, aw * (gz[i] - 2.0 * (double)B[i].z * gn[i]));
        put(1, ga[i]);
        put(2, -2.0 * aw * gnx[i]);
        put(3, -2.0 * aw * gny[i]);
        put(4, -2.0 * aw * (double)B[i].w * gn[i]);
    }
}

// Sum the per-split partials in split order -> grad_rec [n_cap][8] floats
// {0, 0, dL/dpz, dL/da, dL/dn_x, dL/dn_y, dL/dn_z, 0}; zeros past n_active.
__global__ void __launch_bounds__(256) k_adjoint_reduce(const SmoothArgs a, float* grad_rec)
{
    // one thread per output word of a record: words 2 .. 6 sum their field's
    // partials over the splits in split order (32 splits' values read before
    // any is added, so that their latencies overlap), words 0, 1 and 7 are 0
    const int n_act = smooth_active(a);
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t p = t >> 3;
    const int k = (int)(t & 7) - 2;
    if (p >= a.n_cap) return;
    double g = 0.0;
    if (p < n_act && k >= 0 && k < kAdjStride) {
        constexpr int kB = 32;
        const size_t step = (size_t)a.n_cap * kAdjStride;
        const double* q = a.partial + (size_t)p * kAdjStride + k;
        int sp = 0;
        for (; sp + kB <= a.n_split; sp += kB) {
            double v[kB];
#pragma unroll
            for (int i = 0; i < kB; ++i) v[i] = q[(size_t)(sp + i) * step];
#pragma unroll
            for (int i = 0; i < kB; ++i) g += v[i];
        }
        for (; sp < a.n_split; ++sp) g += q[(size_t)sp * step];
    }
    grad_rec[t] = (float)g;
}

// ---------------------------------------------------------------------------
// Record gradients -> maps.
__device__ __forceinline__ float deriv_f(const float* d, int n, int i, int64_t stride, float h)
{
    if (n < 2) return 0.f;
    if (i == 0) return (d[stride] - d[0]) / h;
    if (i == n - 1) return (d[0] - d[-stride]) / h;
    return (d[stride] - d[-stride]) / (2.f * h);
}

__global__ void k_grad_zero(const GradMapArgs g, int64_t npx)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < npx; i += stride) {
        g.scratch[i] = 0.f;
        g.scratch[npx + i] = 0.f;
        g.scratch[2 * npx + i] = 0.f;
        if (g.grad_albedo) g.grad_albedo[i] = 0.f;
    }
}

// Per record: dL/dpz as is; dL/dD_x, dL/dD_y through n = (D_x, D_y, -1)/len
// and a = rho dx dy len (cosines); dL/drho = dL/da * area.  Written to the
// record's own pixel, so no two records collide.
__global__ void __launch_bounds__(256) k_grad_scatter(const GradMapArgs g, int64_t npx)
{
    int n = g.n_cap;
    if (g.n_active) {
        n = *g.n_active;
        n = n < 0 ? 0 : (n > g.n_cap ? g.n_cap : n);
    }
    const int p = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (p >= n) return;
    const int idx = __float_as_int(g.patches[2 * (size_t)p + 1].w);
    const int ix = idx / g.ay.n, iy = idx % g.ay.n;
    const float* D = g.depth + idx;
    const float gx = deriv_f(D, g.ax.n, ix, g.ay.n, g.hx);
    const float gy = deriv_f(D, g.ay.n, iy, 1, g.hy);
    const float len = sqrtf(1.f + gx * gx + gy * gy);
    const float rho = g.albedo ? g.albedo[idx] : 0.5f;
    const float* q = g.grad_rec + (size_t)p * 8;
    const float dpz = q[2], da = q[3], dnx = q[4], dny = q[5], dnz = q[6];
    const float area = g.hx * g.hy * (g.cosines ? len : 1.f);
    if (g.grad_albedo) g.grad_albedo[idx] = da * area;
    g.scratch[idx] = dpz;
    if (g.cosines) {
        const float il = 1.f / len;
        const float il3 = il * il * il;
        const float dot = dnx * gx + dny * gy - dnz;
        const float darea = da * rho * g.hx * g.hy * il;
        g.scratch[npx + idx] = dnx * il - dot * gx * il3 + darea * gx;
        g.scratch[2 * npx + idx] = dny * il - dot * gy * il3 + darea * gy;
    }
}

// Coefficient of D[i] in the derivative at sample i' (|i - i'| <= 1) of an
// axis of n samples with spacing h (central inside, one-sided at borders).
__device__ __forceinline__ float stencil(int n, int ip, int i, float h)
{
    if (n < 2) return 0.f;
    if (ip == 0) return (i == 1 ? 1.f : (i == 0 ? -1.f : 0.f)) / h;
    if (ip == n - 1) return (i == n - 1 ? 1.f : (i == n - 2 ? -1.f : 0.f)) / h;
    return (i == ip + 1 ? 1.f : (i == ip - 1 ? -1.f : 0.f)) / (2.f * h);
}

__global__ void __launch_bounds__(256) k_grad_gather(const GradMapArgs g, int64_t npx)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= npx) return;
    const int nx = g.ax.n, ny = g.ay.n;
    const int ix = (int)(idx / ny), iy = (int)(idx % ny);
    float v = g.scratch[idx];
    const float* sx = g.scratch + npx;
    const float* sy = g.scratch + 2 * npx;
    for (int d = -1; d <= 1; ++d) {
        const int jx = ix + d;
        if (jx >= 0 && jx < nx) v = fmaf(sx[(int64_t)jx * ny + iy], stencil(nx, jx, ix, g.hx), v);
        const int jy = iy + d;
        if (jy >= 0 && jy < ny) v = fmaf(sy[(int64_t)ix * ny + jy], stencil(ny, jy, iy, g.hy), v);
    }
    g.grad_depth[idx] = v;
}

// ---------------------------------------------------------------------------
// Launchers.
template <int TX, int TY, int RS>
static hipError_t launch_smooth_rs(const SmoothArgs& a, int64_t n_blocks, size_t lds, hipStream_t st)
{
    const void* k = a.cosines ? (const void*)k_smooth<TX, TY, true, RS> : (const void*)k_smooth<TX, TY, false, RS>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (a.cosines)
        hipLaunchKernelGGL((k_smooth<TX, TY, true, RS>), dim3((unsigned)n_blocks), dim3(kBlock), lds, st, a);
    else
        hipLaunchKernelGGL((k_smooth<TX, TY, false, RS>), dim3((unsigned)n_blocks), dim3(kBlock), lds, st, a);
    return hipGetLastError();
}

// Support radii with a straight-line tap sequence: ceil(6 sigma) for the
// jitter widths of the paper's configurations (FWHM / bin = 70/16, 50/8,
// 30/4 ps give 12, 16, 20); any other radius runs the general loop.
template <int TX, int TY>
static hipError_t launch_smooth_shape(const SmoothArgs& a, int64_t n_blocks, size_t lds, hipStream_t st)
{
    if (a.Rs == 12) return launch_smooth_rs<TX, TY, 12>(a, n_blocks, lds, st);
    if (a.Rs == 16) return launch_smooth_rs<TX, TY, 16>(a, n_blocks, lds, st);
    if (a.Rs == 20) return launch_smooth_rs<TX, TY, 20>(a, n_blocks, lds, st);
    return launch_smooth_rs<TX, TY, 0>(a, n_blocks, lds, st);
}

hipError_t launch_smooth(const SmoothArgs& a, int tx, int ty, int64_t n_blocks, size_t lds, hipStream_t st)
{
    if (n_blocks <= 0) return hipSuccess;
    if (n_blocks > 0x7fffffff) return hipErrorInvalidValue;
    if (tx == 4 && ty == 4) return launch_smooth_shape<4, 4>(a, n_blocks, lds, st);
    if (tx == 4 && ty == 2) return launch_smooth_shape<4, 2>(a, n_blocks, lds, st);
    if (tx == 2 && ty == 2) return launch_smooth_shape<2, 2>(a, n_blocks, lds, st);
    if (tx == 2 && ty == 1) return launch_smooth_shape<2, 1>(a, n_blocks, lds, st);
    if (tx == 1 && ty == 1) return launch_smooth_shape<1, 1>(a, n_blocks, lds, st);
    return hipErrorInvalidValue;
}

hipError_t launch_smooth_prep(const SmoothArgs& a, const MomentFit& f, bool adjoint, hipStream_t st)
{
    const int words = f.n * (adjoint ? taps_adj(f.Rs) : taps_fwd(f.Rs));
    int nb = (words + kStatBlock - 1) / kStatBlock;
    if (nb > 16) nb = 16;
    hipLaunchKernelGGL(k_smooth_prep, dim3((unsigned)(a.n_stats + nb)), dim3(kStatBlock), 0, st, a, f, adjoint ? 1 : 0);
    return hipGetLastError();
}

template <int NM, int NP, int WG>
static hipError_t launch_smooth_mom(const SmoothArgs& a, int64_t n_blocks, hipStream_t st)
{
    if (a.T + 2 * a.Rs > smooth_mom_pitch(NP, NM, WG)) return hipErrorInvalidValue;
    constexpr size_t lds = smooth_mom_lds(NP, NM, WG);
    const void* k = a.cosines ? (const void*)k_smooth_mom<true, NM, NP, WG> : (const void*)k_smooth_mom<false, NM, NP, WG>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (a.cosines)
        hipLaunchKernelGGL((k_smooth_mom<true, NM, NP, WG>), dim3((unsigned)n_blocks), dim3(kBlock), lds, st, a);
    else
        hipLaunchKernelGGL((k_smooth_mom<false, NM, NP, WG>), dim3((unsigned)n_blocks), dim3(kBlock), lds, st, a);
    return hipGetLastError();
}

template <int NM>
static hipError_t launch_smooth_mom_np(const SmoothArgs& a, int points, int wg, int64_t n_blocks, hipStream_t st)
{
    if (wg == 2) {
        if (points == 3) return launch_smooth_mom<NM, 3, 2>(a, n_blocks, st);
        if (points == 2) return launch_smooth_mom<NM, 2, 2>(a, n_blocks, st);
        if (points == 1) return launch_smooth_mom<NM, 1, 2>(a, n_blocks, st);
    }
    if (wg == 1 && points == 1) return launch_smooth_mom<NM, 1, 1>(a, n_blocks, st);
    return hipErrorInvalidValue;
}

hipError_t launch_smooth_moments(const SmoothArgs& a, int moments, int points, int wg, int64_t n_blocks, hipStream_t st)
{
    if (n_blocks <= 0) return hipSuccess;
    if (n_blocks > 0x7fffffff) return hipErrorInvalidValue;
    switch (moments) {
    case 5: return launch_smooth_mom_np<5>(a, points, wg, n_blocks, st);
    case 6: return launch_smooth_mom_np<6>(a, points, wg, n_blocks, st);
    case 7: return launch_smooth_mom_np<7>(a, points, wg, n_blocks, st);
    case 8: return launch_smooth_mom_np<8>(a, points, wg, n_blocks, st);
    }
    return hipErrorInvalidValue;
}

template <int RS>
static hipError_t launch_adjoint_rs(const SmoothArgs& a, const dim3& grid, size_t lds, hipStream_t st)
{
    const void* k = a.cosines ? (const void*)k_adjoint<true, RS> : (const void*)k_adjoint<false, RS>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (a.cosines)
        hipLaunchKernelGGL((k_adjoint<true, RS>), grid, dim3(kBlock), lds, st, a);
    else
        hipLaunchKernelGGL((k_adjoint<false, RS>), grid, dim3(kBlock), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_adjoint(const SmoothArgs& a, int64_t patch_blocks, size_t lds, hipStream_t st)
{
    if (patch_blocks > 0) {
        if (patch_blocks > 0x7fffffff || a.n_split > 65535) return hipErrorInvalidValue;
        const dim3 grid((unsigned)patch_blocks, (unsigned)a.n_split);
        if (a.Rs == 12) return launch_adjoint_rs<12>(a, grid, lds, st);
        if (a.Rs == 16) return launch_adjoint_rs<16>(a, grid, lds, st);
        if (a.Rs == 20) return launch_adjoint_rs<20>(a, grid, lds, st);
        return launch_adjoint_rs<0>(a, grid, lds, st);
    }
    return hipSuccess;
}

template <int NM, bool DB, bool PIECE>
static hipError_t launch_adjoint_gather(const SmoothArgs& a, const dim3& grid, size_t lds, hipStream_t st)
{
    const void* k =
        a.cosines ? (const void*)k_adjoint_mom<true, NM, DB, PIECE> : (const void*)k_adjoint_mom<false, NM, DB, PIECE>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (a.cosines)
        hipLaunchKernelGGL((k_adjoint_mom<true, NM, DB, PIECE>), grid, dim3(kBlock), lds, st, a);
    else
        hipLaunchKernelGGL((k_adjoint_mom<false, NM, DB, PIECE>), grid, dim3(kBlock), lds, st, a);
    return hipGetLastError();
}

template <int NM>
static hipError_t launch_adjoint_mom(SmoothArgs a, int64_t patch_blocks, size_t lds, bool dbuf, int64_t piece,
                                     hipStream_t st)
{
    if (lds < adj_mom_lds(dbuf ? 2 : 1, a.rows, NM, a.mlen)) return hipErrorInvalidValue;
    const int64_t S = (int64_t)a.rx.n * a.ry.n;
    for (int64_t s0 = 0; s0 < S; s0 += piece) {
        a.s0 = (int32_t)s0;
        a.sn = (int32_t)(S - s0 < piece ? S - s0 : piece);
        // one thread per (scan point, 4 bins of a correlation row)
        const int64_t blocks = ((int64_t)a.sn * (a.mlen / 4) + 255) / 256;
        if (blocks * 256 > UINT32_MAX) return hipErrorInvalidValue;
        if ((a.T & 3) == 0 && ((uintptr_t)a.grad_out & 15) == 0)   // (then so is every piece's)
            hipLaunchKernelGGL((k_adj_moments<NM, true>), dim3((unsigned)blocks), dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_adj_moments<NM, false>), dim3((unsigned)blocks), dim3(256), 0, st, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const dim3 grid((unsigned)patch_blocks, (unsigned)a.n_split);
        if (piece >= S)
            e = dbuf ? launch_adjoint_gather<NM, true, false>(a, grid, lds, st)
                     : launch_adjoint_gather<NM, false, false>(a, grid, lds, st);
        else
            e = dbuf ? launch_adjoint_gather<NM, true, true>(a, grid, lds, st)
                     : launch_adjoint_gather<NM, false, true>(a, grid, lds, st);
        if (e != hipSuccess) return e;
        a.grad_out += (size_t)a.sn * a.T;
    }
    return hipSuccess;
}

hipError_t launch_adjoint_moments(const SmoothArgs& a, const MomentFit& f, int64_t patch_blocks, size_t lds, bool dbuf,
                                  int64_t piece, hipStream_t st)
{
    if (patch_blocks <= 0) return hipSuccess;
    if (patch_blocks > 0x7fffffff || a.n_split > 65535 || a.rows < 1 || a.mlen != adj_row_bins(a.T, a.Rs) || piece < 1)
        return hipErrorInvalidValue;
    const hipError_t e = launch_smooth_prep(a, f, true, st);
    if (e != hipSuccess) return e;
    switch (f.n) {
    case 6: return launch_adjoint_mom<6>(a, patch_blocks, lds, dbuf, piece, st);
    case 7: return launch_adjoint_mom<7>(a, patch_blocks, lds, dbuf, piece, st);
    case 8: return launch_adjoint_mom<8>(a, patch_blocks, lds, dbuf, piece, st);
    case 9: return launch_adjoint_mom<9>(a, patch_blocks, lds, dbuf, piece, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_adjoint_reduce(const SmoothArgs& a, float* grad_rec, hipStream_t st)
{
    if (a.n_cap <= 0) return hipSuccess;
    const int64_t blocks = ((int64_t)a.n_cap * 8 + 255) / 256;   // one thread per output word
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_adjoint_reduce, dim3((unsigned)blocks), dim3(256), 0, st, a, grad_rec);
    return hipGetLastError();
}

hipError_t launch_grad_maps(const GradMapArgs& g, hipStream_t st)
{
    const int64_t npx = (int64_t)g.ax.n * g.ay.n;
    int64_t zb = (npx + 255) / 256;
    if (zb > 8192) zb = 8192;
    hipLaunchKernelGGL(k_grad_zero, dim3((unsigned)zb), dim3(256), 0, st, g, npx);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (g.n_cap > 0) {
        hipLaunchKernelGGL(k_grad_scatter, dim3((unsigned)((g.n_cap + 255) / 256)), dim3(256), 0, st, g, npx);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_grad_gather, dim3((unsigned)((npx + 255) / 256)), dim3(256), 0, st, g, npx);
    return hipGetLastError();
}

}  // namespace nlos
