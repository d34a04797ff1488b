// Pseudo-elliptical NFW deflection on gfx950: the second profile family the
// paper names for its method (Sec. 5), in the frame construction of
// Algorithm 1 (Sec. 2.2.2).  With m = M d (M = Rot(Phi) diag(1-eps, 1+eps)
// Rot(-Phi), d = theta - centre), R^2 = d . m and x = R / r_s,
//     alpha = 4 kappa_s (g(x) / x^2) m,   g(x) = ln(x/2) + F(x),
//     F(x) = atanh(s)/s, s = sqrt(1 - x^2) (x < 1);  atan(r)/r, r = sqrt(x^2 - 1) (x > 1)
// (the textbook arccosh / arccos forms of F written through s and r).  Below
// x = 1/2 the two logarithms of g cancel; there g/x^2 is evaluated as
//     [ln(2/x)/(1 + s) + log1p(-x^2 / (2 (1 + s))) / x^2] / s,
// the same quantity with the cancellation done exactly.  The centre (R = 0)
// contributes 0.  FP32: node offsets from the exact split of the centre, as in
// the isothermal FP32 field; FP64: theta - centre in FP64.
#include "lens_path.hpp"
#include "lens_tiles.hpp"

#include <type_traits>

namespace lens {

enum : int { N64_XC = 0, N64_YC, N64_A, N64_B, N64_C, N64_IRS2, N64_K4, N64_STRIDE = 8 };
enum : int {
    N32_CXH = 0, N32_CXL, N32_CYH, N32_CYL, N32_A, N32_B, N32_C, N32_IRS2, N32_K, N32_STRIDE = 12
};

// Constants of every halo (one thread each) and the status: invalid for a
// non-finite or out-of-domain parameter (0 <= eps < 1, r_s > 0, kappa_s >= 0)
// or a centre beyond 2^22 nodes of the grid origin.
__global__ __launch_bounds__(256) void k_nfw_prep(NfwPtrs h, GridDesc g, double* __restrict__ t64,
                                                  float* __restrict__ t32, int* __restrict__ st,
                                                  int* __restrict__ status)
{
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    bool bad = false;
    for (int p = threadIdx.x; p < h.n; p += 256) {
        const double xc = h.x[p], yc = h.y[p], eps = h.eps[p], phi = h.phi[p], rs = h.r_s[p], ks = h.kappa_s[p];
        const bool ok = isfinite(xc) && isfinite(yc) && isfinite(phi) && eps >= 0.0 && eps < 1.0 && rs > 0.0 &&
                        isfinite(rs) && ks >= 0.0 && isfinite(ks);
        double s2, c2;
        sincos(2.0 * phi, &s2, &c2);
        const double A = 1.0 - eps * c2, B = -eps * s2, C = 1.0 + eps * c2;
        double* u = t64 + (size_t)p * N64_STRIDE;
        u[N64_XC] = xc;
        u[N64_YC] = yc;
        u[N64_A] = A;
        u[N64_B] = B;
        u[N64_C] = C;
        u[N64_IRS2] = 1.0 / (rs * rs);
        u[N64_K4] = 4.0 * ks;
        u[N64_STRIDE - 1] = 0.0;
        const double cxn = (xc - g.x0) / g.h, cyn = (yc - g.y0) / g.h;
        const bool near = fabs(cxn) < 4194304.0 && fabs(cyn) < 4194304.0;
        const double cxh = near ? rint(cxn) : 0.0, cyh = near ? rint(cyn) : 0.0;
        const double h2 = g.h * g.h;
        float* v = t32 + (size_t)p * N32_STRIDE;
        v[N32_CXH] = (float)cxh;
        v[N32_CXL] = (float)(cxn - cxh);
        v[N32_CYH] = (float)cyh;
        v[N32_CYL] = (float)(cyn - cyh);
        v[N32_A] = (float)(A * h2);
        v[N32_B] = (float)(B * h2);
        v[N32_C] = (float)(C * h2);
        v[N32_IRS2] = (float)(1.0 / (rs * rs));
        v[N32_K] = (float)(4.0 * ks / g.h);
        for (int k = N32_K + 1; k < N32_STRIDE; k++) v[k] = 0.0f;
        bad |= !(ok && near);
    }
    if (bad) atomicOr(&s_bad, 1);
    __syncthreads();
    if (threadIdx.x == 0) {
        *st = s_bad ? kStatusInvalid : kStatusOk;
        if (status) *status = *st;
    }
}

// g(x) / x^2 for x^2 > 0 (see the file comment), by ranges of z = 1 - x^2 = s^2:
//   z > 3/4 (x < 1/2): ln(2/x) = -ln(x^2/4)/2, and log1p(-u)/x^2, u = x^2/(2 (1 + s))
//     <= 0.067, as -(1 + u/2 + u^2/3 + ...)/(2 (1 + s)): nothing is divided by x^2;
//   |z| <= 0.2 (around x = 1): F = 1 + z/3 + z^2/5 + ..., one series for both signs;
//   else F = atanh(s)/s or atan(r)/r.
// Terms are kept until the first one left out is below half the unit roundoff.
// Roots and reciprocals are the hardware's in FP32 (1 ulp) and the refined
// estimates in FP64 (about 1 ulp), quotients corrected by one residual; the
// logarithm is the hardware's in FP32, and there atanh(s) = ln(1 + s) - ln(x),
// whose terms do not cancel for s >= 0.44.  x^2 may be as small as a product can
// be (a node next to the centre, a large r_s): the hardware logarithm takes no
// denormal, so ln4 scales a small argument first, and an x^2 that underflowed to
// zero is taken as the smallest value whose quarter is not zero.
template <typename V>
struct NfwMath;

template <>
struct NfwMath<float> {
    static constexpr int kU = 6, kZ = 10;  // 0.067^6 / 7 = 1.3e-8, 0.2^10 / 21 = 5e-9
    __device__ __forceinline__ static float ln(float v) { return 0.69314718056f * __builtin_amdgcn_logf(v); }
    __device__ __forceinline__ static float root(float v) { return __builtin_amdgcn_sqrtf(v); }
    __device__ __forceinline__ static float rcp(float v) { return __builtin_amdgcn_rcpf(v); }
    __device__ __forceinline__ static float atn(float v) { return atanf(v); }
    __device__ __forceinline__ static float ath(float s, float x2) { return fmaf(-0.5f, ln(x2), ln(1.0f + s)); }
    // ln(x2 / 4) for x2 below 1
    __device__ __forceinline__ static float ln4(float x2)
    {
        const bool lo = x2 < 0x1p-100f;
        return 0.69314718056f * (__builtin_amdgcn_logf(x2 * (lo ? 0x1p60f : 0.25f)) - (lo ? 62.0f : 0.0f));
    }
    static constexpr float tiny = 0x1p-149f;
};

template <>
struct NfwMath<double> {
    static constexpr int kU = 13, kZ = 22;  // 0.067^13 / 14 = 4e-17, 0.2^22 / 45 = 1e-17
    __device__ __forceinline__ static double ln(double v) { return log(v); }
    __device__ __forceinline__ static double root(double v) { return sqrt_est64(v); }
    __device__ __forceinline__ static double rcp(double v) { return rcp_est64(v); }
    __device__ __forceinline__ static double atn(double v) { return atan(v); }
    __device__ __forceinline__ static double ath(double s, double) { return atanh(s); }
    __device__ __forceinline__ static double ln4(double x2) { return log(0.25 * x2); }
    static constexpr double tiny = 0x1p-1072;
};

template <typename V>
__device__ __forceinline__ V nfw_quot(V n, V d)
{
    const V r = NfwMath<V>::rcp(d), q = n * r;
    return fma(fma(-q, d, n), r, q);
}

template <typename V>
__device__ __forceinline__ V nfw_gx2(V x2)
{
    using M = NfwMath<V>;
    x2 = fmax(x2, M::tiny);
    const V z = V(1) - x2;
    if (z > V(0.75)) {
        const V s = M::root(z), iq = M::rcp(V(1) + s), hq = V(0.5) * iq, u = x2 * hq;
        V p = V(1) / V(M::kU);
#pragma unroll
        for (int k = M::kU - 1; k >= 1; k--) p = fma(p, u, V(1) / V(k));
        return nfw_quot(fma(V(-0.5) * M::ln4(x2), iq, -hq * p), s);
    }
    V F;
    if (fabs(z) <= V(0.2)) {
        F = V(1) / V(2 * M::kZ - 1);
#pragma unroll
        for (int k = M::kZ - 2; k >= 0; k--) F = fma(F, z, V(1) / V(2 * k + 1));
    } else if (z > V(0)) {
        const V s = M::root(z);
        F = nfw_quot(M::ath(s, x2), s);
    } else {
        const V r = M::root(-z);
        F = nfw_quot(M::atn(r), r);
    }
    return nfw_quot(fma(V(0.5), M::ln(V(0.25) * x2), F), x2);
}

// One copy of the FP64 profile for the tiled kernel's near nodes: inlined eight
// times it takes 256 registers (one wave per SIMD).
__device__ __noinline__ double nfw_gx2_call(double x2) { return nfw_gx2(x2); }

// FP32 field: NPL consecutive nodes of row blockIdx.y per thread.
template <int NPL>
__global__ __launch_bounds__(256) void k_nfw32(const float* __restrict__ t32, int np, int nx,
                                               float* __restrict__ ax, float* __restrict__ ay,
                                               const int* __restrict__ st)
{
    const int j = blockIdx.y;
    const int i0 = (blockIdx.x * 256 + threadIdx.x) * NPL;
    if ((int)(blockIdx.x * 256 * NPL) >= nx) return;
    const bool bad = *st != kStatusOk;
    float sx[NPL], sy[NPL];
#pragma unroll
    for (int k = 0; k < NPL; k++) sx[k] = sy[k] = 0.0f;
    const float fj = (float)j;
    if (!bad)  // uniform over the launch
        pots_wg<N32_STRIDE, N32_CYH, N32_CYL, N32_B, N32_C>(t32, np, fj, [&](const float* c, float4 rc) {
            const float A = c[N32_A], B = c[N32_B], irs2 = c[N32_IRS2], K = c[N32_K];
            const float nyv = rc.x, bny = rc.y, cny = rc.z;  // the row part
#pragma unroll
            for (int k = 0; k < NPL; k++) {
                const float nxv = ((float)(i0 + k) - c[N32_CXH]) - c[N32_CXL];
                const float m1 = fmaf(A, nxv, bny), m2 = fmaf(B, nxv, cny);
                const float R2 = fmaf(nxv, m1, nyv * m2);
                if (R2 > 0.0f) {
                    const float kg = K * nfw_gx2(R2 * irs2);
                    sx[k] = fmaf(kg, m1, sx[k]);
                    sy[k] = fmaf(kg, m2, sy[k]);
                }
            }
        });
    const size_t row = (size_t)j * nx;
#pragma unroll
    for (int k = 0; k < NPL; k++)
        if (i0 + k < nx) {
            ax[row + i0 + k] = bad ? __builtin_nanf("") : sx[k];
            ay[row + i0 + k] = bad ? __builtin_nanf("") : sy[k];
        }
}

// FP64 field: one node per thread.
__global__ __launch_bounds__(256) void k_nfw64(const double* __restrict__ t64, int np, GridDesc g,
                                               double* __restrict__ ax, double* __restrict__ ay,
                                               const int* __restrict__ st)
{
    const int j = blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= g.nx) return;
    const bool bad = *st != kStatusOk;
    const double t1 = node_coord(g.x0, i, g.h), t2 = node_coord(g.y0, j, g.h);
    double s1 = 0.0, s2 = 0.0;
    for (int p = 0; p < np && !bad; p++) {
        const double* c = t64 + (size_t)p * N64_STRIDE;
        const double d1 = t1 - c[N64_XC], d2 = t2 - c[N64_YC];
        const double m1 = c[N64_A] * d1 + c[N64_B] * d2, m2 = c[N64_B] * d1 + c[N64_C] * d2;
        const double R2 = d1 * m1 + d2 * m2;
        if (R2 > 0.0) {
            const double kg = c[N64_K4] * nfw_gx2(R2 * c[N64_IRS2]);
            s1 += kg * m1;
            s2 += kg * m2;
        }
    }
    const size_t n = (size_t)j * g.nx + i;
    ax[n] = bad ? __builtin_nan("") : s1;
    ay[n] = bad ? __builtin_nan("") : s2;
}

// ---------------------------------------------------------------- tiled field

// The NFW halos as a tile's summand (lens_tiles.hpp): the profile is analytic
// away from the centre like the isothermal one (x = 1 is a removable point), so
// the same criterion with core 0 holds.  The profile's logarithms and roots bound
// it, by vector issue: 4096^2 x 702 in FP32 21.6 ms by the direct sum, 0.35 by tiles.
struct NfwProfile {
    const double* t64;
    const float* t32;

    __device__ __forceinline__ bool far(int p, float xc, float yc, float hw, float c) const
    {
        const float* r = t32 + (size_t)p * N32_STRIDE;
        return tile_far((xc - r[N32_CXH]) - r[N32_CXL], (yc - r[N32_CYH]) - r[N32_CYL], r[N32_A], r[N32_B], r[N32_C],
                        0.0f, hw, c);
    }

    // FP64 offsets and sums; the profile in FP64 (FULL) or, for an FP32 field, FP32.
    template <bool FULL>
    __device__ __forceinline__ void far_at(const unsigned short* list, int k0, int k1, double c1, double c2, double e1,
                                           double e2, double& s1, double& s2) const
    {
        double r1 = 0.0, r2 = 0.0;  // two partial sums, taken in turn
        for_list(list + k0, k1 - k0, [&](int p) {
            const double* c = t64 + (size_t)p * N64_STRIDE;
            const double d1 = (c1 - c[N64_XC]) + e1, d2 = (c2 - c[N64_YC]) + e2;
            const double m1 = fma(c[N64_A], d1, c[N64_B] * d2), m2 = fma(c[N64_B], d1, c[N64_C] * d2);
            const double x2 = fma(d1, m1, d2 * m2) * c[N64_IRS2];
            const double kg = c[N64_K4] * (FULL ? nfw_gx2_call(x2) : (double)nfw_gx2((float)x2));
            const double q1 = fma(kg, m1, r1), q2 = fma(kg, m2, r2);
            r1 = s1;
            r2 = s2;
            s1 = q1;
            s2 = q2;
        });
        s1 += r1;
        s2 += r2;
    }

    template <int NK>
    __device__ __forceinline__ void near32(int p, const float* fi, float fj, float* sx, float* sy) const
    {
        const float* c = t32 + (size_t)p * N32_STRIDE;
        const float A = c[N32_A], B = c[N32_B], irs2 = c[N32_IRS2], K = c[N32_K];
        const float nyv = (fj - c[N32_CYH]) - c[N32_CYL], bny = B * nyv, cny = c[N32_C] * nyv;
#pragma unroll 1
        for (int k = 0; k < NK; k += 4) {
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const float nxv = ((k ? fi[NK - 4 + q] : fi[q]) - c[N32_CXH]) - c[N32_CXL];
                const float m1 = fmaf(A, nxv, bny), m2 = fmaf(B, nxv, cny);
                const float R2 = fmaf(nxv, m1, nyv * m2);
                const float kg = R2 > 0.0f ? K * nfw_gx2(R2 * irs2) : 0.0f;
                if (k) {
                    sx[NK - 4 + q] = fmaf(kg, m1, sx[NK - 4 + q]);
                    sy[NK - 4 + q] = fmaf(kg, m2, sy[NK - 4 + q]);
                } else {
                    sx[q] = fmaf(kg, m1, sx[q]);
                    sy[q] = fmaf(kg, m2, sy[q]);
                }
            }
        }
    }

    template <int NK>
    __device__ __forceinline__ void near64(int p, const double* t1, double t2, double* sx, double* sy) const
    {
        const double* c = t64 + (size_t)p * N64_STRIDE;
        const double d2 = t2 - c[N64_YC];
#pragma unroll
        for (int k = 0; k < NK; k++) {
            const double d1 = t1[k] - c[N64_XC];
            const double m1 = c[N64_A] * d1 + c[N64_B] * d2, m2 = c[N64_B] * d1 + c[N64_C] * d2;
            const double R2 = d1 * m1 + d2 * m2;
            const double kg = R2 > 0.0 ? c[N64_K4] * nfw_gx2_call(R2 * c[N64_IRS2]) : 0.0;
            sx[k] += kg * m1;
            sy[k] += kg * m2;
        }
    }
};

template <int T, int NW>
__global__ __launch_bounds__(64 * NW) void k_nfw_tiled32(const double* __restrict__ t64, const float* __restrict__ t32,
                                                     int np, GridDesc g, int ntx, float* __restrict__ ax,
                                                     float* __restrict__ ay, const int* __restrict__ st)
{
    __shared__ typename Tile32<T, NW>::Lds lds;
    int ti, tj;
    tile_at((int)blockIdx.x, ntx, ti, tj);
    tile32_body<T, NW>(lds, NfwProfile{t64, t32}, np, g, ti * T, tj * T, ax, ay, *st != kStatusOk, (float*)nullptr, 0);
}

template <int T>
__global__ __launch_bounds__(256) void k_nfw_tiled64(const double* __restrict__ t64, const float* __restrict__ t32,
                                                     int np, GridDesc g, int ntx, double* __restrict__ ax,
                                                     double* __restrict__ ay, const int* __restrict__ st)
{
    __shared__ typename Tile64<T>::Lds lds;
    int ti, tj;
    tile_at((int)blockIdx.x, ntx, ti, tj);
    tile64_body<T>(lds, NfwProfile{t64, t32}, np, g, ti * T, tj * T,
                   FieldSink64{ax, ay, nullptr, g.nx, g.ny, *st != kStatusOk});
}

// ---------------------------------------------------------------- launcher

constexpr TileCost kNfwCost32 = {540.0, 480.0, 64.0, 60.0, 3.6};
constexpr TileCost kNfwCost64 = {1650.0, 1650.0, 256.0, 200.0, 5.1};

size_t nfw_scratch(int np) { return (size_t)(np > 0 ? np : 1) * (N64_STRIDE * 8 + N32_STRIDE * 4) + 256; }

hipError_t launch_nfw(const NfwPtrs& h, const GridDesc& g, bool fp32, void* ax, void* ay, int* status,
                      void* scratch, const KernelEvents* ev, hipStream_t s)
{
    const int np = h.n > 0 ? h.n : 1;
    double* t64 = (double*)scratch;
    float* t32 = (float*)(t64 + (size_t)np * N64_STRIDE);
    int* st = (int*)(t32 + (size_t)np * N32_STRIDE);
    k_nfw_prep<<<1, 256, 0, s>>>(h, g, t64, t32, st, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const double nodes = (double)g.nx * g.ny;
    // Tiled from 2^23 (FP32) or 2^24 (FP64) terms on, where its chain of 35 or 150 us
    // is repaid (tiled against direct: FP32 512 x 500 x 100 38 / 61 us, 2048^2 x 302
    // 85 / 1400, and the direct kernel before this function's rewriting 2490; FP64
    // 300^2 x 60 159 / 155, 512 x 500 x 100 191 / 204, 2048^2 x 302 836 / 6890), but in
    // FP64 not thin grids (65536 x 2 x 140 149 / 445, 90000 x 6 x 60 244 / 265, 60000 x 12
    // x 60 318 / 201; in FP32 the tiles are the faster even at two rows).
    const int side = tile_side_for(nodes, nodes, h.n, fp32 ? kNfwCost32 : kNfwCost64);
    if (h.n >= 4 && h.n <= kTileMaxP && nodes * h.n >= (fp32 ? 8388608.0 : 16777216.0) &&
        (fp32 || !tiles_too_thin(g, side, 256))) {
        const int ntx = (g.nx + side - 1) / side;
        const dim3 grid((unsigned)(ntx * ((g.ny + side - 1) / side)));
        auto go = [&](auto t) {
            constexpr int T = decltype(t)::value;
            // eight waves for the largest tile: its chain bounds a launch of few such tiles
            // (4096^2 x 702: 425 us with four)
            constexpr int NW = T == 128 ? 8 : 4;
            if (fp32)
                return launch_ev(ev, k_nfw_tiled32<T, NW>, grid, dim3(64 * NW), s, (const double*)t64, (const float*)t32, h.n, g,
                                 ntx, (float*)ax, (float*)ay, (const int*)st);
            return launch_ev(ev, k_nfw_tiled64<T>, grid, dim3(256), s, (const double*)t64, (const float*)t32, h.n, g, ntx,
                             (double*)ax, (double*)ay, (const int*)st);
        };
        switch (side) {
        case 32: return go(std::integral_constant<int, 32>());
        case 64: return go(std::integral_constant<int, 64>());
        default: return go(std::integral_constant<int, 128>());
        }
    }
    if (fp32) {
        const dim3 grid((unsigned)((g.nx + 511) / 512), (unsigned)g.ny);
        return launch_ev(ev, k_nfw32<2>, grid, dim3(256), s, (const float*)t32, h.n, g.nx, (float*)ax, (float*)ay,
                         (const int*)st);
    }
    const dim3 grid((unsigned)((g.nx + 255) / 256), (unsigned)g.ny);
    return launch_ev(ev, k_nfw64, grid, dim3(256), s, (const double*)t64, h.n, g, (double*)ax, (double*)ay,
                     (const int*)st);
}

}  // namespace lens
