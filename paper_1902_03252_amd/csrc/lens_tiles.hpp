// Deflection field by tiles: near potentials summed directly at every node, the
// far ones through one polynomial per tile.
//
// A potential's deflection is analytic away from a^2 + R^2 = 0 (a the core
// radius, R the pseudo-elliptical radius), so over a tile of T x T nodes that
// lies far enough from its centre it is a polynomial to working precision.
// For every tile, the potentials are split by a geometric criterion; the sum of
// the far ones is evaluated at N x N Chebyshev points only and interpolated to
// the T x T nodes, the near ones (a handful) are evaluated at every node as in
// the direct field.  Work per node: about (near + far N^2 / T^2 + 1) profile
// evaluations instead of P.
//
// Criterion.  Along a line in x (the same in y with A and C exchanged) R^2 =
// A X^2 + E', X the complex abscissa from the point of least R, so the nearest
// singularity of the deflection is at X = -X_c +- i sqrt((E' + a^2)/A) from
// the tile's centre line, at distance sqrt((a^2 + R^2)/A) from the centre of
// the interval.  With q^2 = min over the tile's vertical centre line of a^2 +
// R^2 (a quadratic, minimised exactly), every singularity lies outside the
// ellipse with foci at the interval's ends and semi-major axis c half widths
// when q^2 >= A (c hw)^2: the sum of a point's distances to the two ends is at
// least twice its distance to the centre.  Then interpolation in N Chebyshev
// points converges as rho^-N, rho = c + sqrt(c^2 - 1).  Largest tensor
// interpolation error found over the family (eps up to 0.95, any position
// angle and direction, core and cut radii from 0 to infinity, the potential
// exactly at the criterion), in units of w_p = K (1 + eps)/sqrt(1 - eps):
//     N = 8:  c = 3: 5.2e-7    c = 3.5: 1.3e-7
//     N = 16: c = 4: 1.9e-15   c = 4.5: 3e-16     c = 5: 5e-17
// (circular singular profiles are the worst; the NFW profile's are alike).
#pragma once

#include "lens_path.hpp"

namespace lens {

constexpr int kTileMaxP = 2048;  // potentials of a tiled field (LDS lists)
// Fewest isothermal potentials that an FP64 field takes far terms for.  The
// interpolation has a rounding of its own, the direct sum one per potential:
// against long double (24 models each, tiled over direct, rms and maximum) 4
// potentials 1.02-1.03 and 1.18-1.22, 8 0.95-1.01 and 1.02-1.05, 12 0.90-0.97 and
// 0.97-0.99, 120 0.62.  (An FP32 field's far part is in FP64 and the smaller
// error at any count.)
constexpr int kTileMinP64 = 12;

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// DCT row a of N Chebyshev samples f(cos(pi (2k + 1) / 2N)): coefficient a is
// sum_k kDct[a][k] f_k.  Filled at compile time from a cosine series.
constexpr double cos_const(double x)
{
    // range reduction to [0, pi/4] on the quarter circle, then the Taylor series
    // to order 22 (below 1e-17 there)
    const double pi = 3.14159265358979323846264338327950288;
    while (x > pi) x -= 2.0 * pi;
    if (x < 0.0) x = -x;
    const bool neg = x > 0.5 * pi;
    if (neg) x = pi - x;
    const bool sn = x > 0.25 * pi;
    if (sn) x = 0.5 * pi - x;
    double term = sn ? x : 1.0, sum = term;
    for (int k = sn ? 2 : 1; k < 24; k += 2) {
        term *= -x * x / (double(k) * double(k + 1));
        sum += term;
    }
    return neg ? -sum : sum;
}

template <int N>
struct Dct {
    double d[N * N];  // [a][k]
    double xi[N];     // Chebyshev points
    constexpr Dct() : d(), xi()
    {
        const double pi = 3.14159265358979323846264338327950288;
        for (int k = 0; k < N; k++) xi[k] = cos_const(pi * (2 * k + 1) / (2.0 * N));
        for (int a = 0; a < N; a++)
            for (int k = 0; k < N; k++) {
                // cos(a (2k+1) pi / 2N) with the angle reduced exactly in units of pi / 2N
                const int m = (a * (2 * k + 1)) % (4 * N);
                const int r = m > 2 * N ? 4 * N - m : m;
                d[a * N + k] = (a ? 2.0 : 1.0) / N * cos_const(pi * r / (2.0 * N));
            }
    }
};
// per translation unit: static device copies
static __device__ const Dct<8> kDct8;
static __device__ const Dct<16> kDct16;

// Criterion constants (c of the file comment).
constexpr float kFarC32 = 3.0f;
constexpr float kFarC64 = 4.5f;

// Orders a wave's LDS writes before its following LDS reads.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Whether a potential (node-unit FP32 table row: centre, M h^2, a^2) is far from
// the tile whose centre is (xc, yc) and half width hw (node units).  A NaN
// (a degenerate row) leaves the potential near.  The quadratic is a difference of
// large terms when eps is near 1 and the centre far away along the long axis: its
// rounding (a unit roundoff of each coefficient, two of the offset, counted twice
// in the square, and four of the operations, on the sum of the terms' sizes; 8 u,
// taken as 10) is subtracted, so that a potential it could decide stays near.  (a^2,
// which only adds, has its rounding in lim's factor; the bound stays finite, so that
// terms beyond FP32 are far.)
__device__ __forceinline__ bool tile_far(float dx, float dy, float A, float B, float C, float a2, float hw, float c)
{
    const float t = fminf(fmaxf(-B * dx * __builtin_amdgcn_rcpf(C), dy - hw), dy + hw);
    const float u = fminf(fmaxf(-B * dy * __builtin_amdgcn_rcpf(A), dx - hw), dx + hw);
    constexpr float r = 6e-7f, big = 3e38f;
    const float v1 = A * dx * dx, v2 = 2.0f * B * dx * t, v3 = C * t * t;
    const float h1 = A * u * u, h2 = 2.0f * B * dy * u, h3 = C * dy * dy;
    const float qv = ((v1 + v2) + (v3 + a2)) - fminf(r * ((v1 + fabsf(v2)) + v3), big);
    const float qh = ((h1 + h2) + (h3 + a2)) - fminf(r * ((h1 + fabsf(h2)) + h3), big);
    const float lim = c * c * hw * hw * 1.0001f;
    return qv >= A * lim && qh >= C * lim && A > 0.0f && C > 0.0f;
}

// Near/far lists of one tile of at most kTileMaxP potentials: near ones first (in
// order), then the far ones (in order).  Called by all NTH threads of the workgroup (two
// barriers); isfar(p) is evaluated once per potential.
struct TileLists {
    unsigned long long near[kTileMaxP / 64];
    unsigned short list[kTileMaxP];
    int n_near;
};

template <int NTH = 256, class F>
__device__ __forceinline__ void tile_lists(TileLists& L, int np, F&& isfar)
{
    const int tid = threadIdx.x;
    const int words = (np + 63) >> 6;
    for (int p0 = 0; p0 < np; p0 += NTH) {  // uniform trip count
        const int p = p0 + tid;
        const bool nr = p < np && !isfar(p);
        const unsigned long long m = __ballot(nr);
        if (lane_id() == 0 && (p >> 6) < words) L.near[p >> 6] = m;
    }
    __syncthreads();
    int total = 0;
    for (int w = 0; w < words; w++) total += __popcll(L.near[w]);
    for (int p = tid; p < np; p += NTH) {
        const int w = p >> 6;
        int before = 0;
        for (int k = 0; k < w; k++) before += __popcll(L.near[k]);
        const unsigned long long m = L.near[w];
        before += __popcll(m & ((1ull << (p & 63)) - 1ull));
        if ((m >> (p & 63)) & 1ull)
            L.list[before] = (unsigned short)p;
        else
            L.list[total + p - before] = (unsigned short)p;
    }
    if (tid == 0) L.n_near = total;
    __syncthreads();
}

// Runs f(p) for the list entries [0, n) with a wave-uniform p; all 64 lanes call
// it.  64 entries are loaded at a time, one per lane.
template <class F>
__device__ __forceinline__ void for_list(const unsigned short* list, int n, F&& f)
{
    for (int b = 0; b < n; b += 64) {
        const int cnt = min(64, n - b);
        const int mine = lane_id() < cnt ? (int)list[b + lane_id()] : 0;
        for (int k = 0; k < cnt; k++) f(__builtin_amdgcn_readlane(mine, k));
    }
}

// FP64 constants of one potential in wave-uniform registers (the first ten
// values of its table row; the cut radius is 0 for an uncut profile only).
struct Far64 {
    double xc, yc, A, B, C, a2, s2, ra, rs, K;
};
static_assert(T64_K == 9 && T64_RS == 8, "ten leading values");

__device__ __forceinline__ Far64 load_far(const double* __restrict__ t)
{
    return {t[T64_XC], t[T64_YC], t[T64_A],  t[T64_B],  t[T64_C],
            t[T64_A2], t[T64_S2], t[T64_RA], t[T64_RS], t[T64_K]};
}

// FP64 deflection of a far potential at the point c + e (FULL: the arithmetic of
// add_alpha64; c + e and not one coordinate, so that the offset from the
// potential is rounded relative to itself) or at the point c (!FULL).  !FULL: the
// hardware root and reciprocal estimates unrefined (relative error 2^-24, the FP32 unit roundoff),
// for the far part of an FP32 field: three such factors and no other rounding
// above 2^-52 leave it within about 4 u w_p.
template <bool FULL, bool CUT>
__device__ __forceinline__ void add_far(const Far64& p, double c1, double c2, double e1, double e2, double& s1,
                                        double& s2)
{
    double d1 = c1 - p.xc, d2 = c2 - p.yc;
    if constexpr (FULL) {
        d1 += e1;
        d2 += e2;
    }
    const double m1 = fma(p.A, d1, p.B * d2);
    const double m2 = fma(p.B, d1, p.C * d2);
    const double R2 = fma(d1, m1, d2 * m2);
    const double a2 = p.a2 + R2, b2 = p.s2 + R2;
    double qa, f;
    if constexpr (FULL)
        qa = sqrt_est64(a2) + p.ra;
    else
        qa = fma(a2, __builtin_amdgcn_rsq(a2), p.ra);
    if constexpr (!CUT) {
        f = FULL ? rcp_est64(qa) : __builtin_amdgcn_rcp(qa);
    } else if constexpr (FULL) {
        const double qs = sqrt_est64(b2) + p.rs;
        f = (qs - qa) * rcp_est64(qa * qs);
    } else {
        const double qs = fma(b2, __builtin_amdgcn_rsq(b2), p.rs);
        f = (qs - qa) * __builtin_amdgcn_rcp(qa * qs);
    }
    const double kf = p.K * f;
    s1 = fma(kf, m1, s1);
    s2 = fma(kf, m2, s2);
}

// Sum of the far potentials list[k0..k1) at c + e, two at a time: their
// constants' scalar loads are in flight together, their evaluations (one serial
// chain each) interleave when both are of one kind, and they go to two partial
// sums.
template <bool FULL>
__device__ __forceinline__ void far_sum(const double* __restrict__ tab64, const unsigned short* list, int k0, int k1,
                                        double c1, double c2, double e1, double e2, double& s1, double& s2)
{
    double r1 = 0.0, r2 = 0.0;
    for (int b = k0; b < k1; b += 64) {
        const int cnt = min(64, k1 - b);
        const int mine = lane_id() < cnt ? (int)list[b + lane_id()] : 0;
        auto row = [&](int k) { return load_far(tab64 + (size_t)__builtin_amdgcn_readlane(mine, k) * T64_STRIDE); };
        auto cut = [](const Far64& p) { return __double_as_longlong(p.rs) != 0; };
        auto one = [&](const Far64& p, double& x, double& y) {
            if (cut(p))
                add_far<FULL, true>(p, c1, c2, e1, e2, x, y);
            else
                add_far<FULL, false>(p, c1, c2, e1, e2, x, y);
        };
        int k = 0;
        for (; k + 2 <= cnt; k += 2) {
            const Far64 p = row(k), q = row(k + 1);
            if (cut(p) && cut(q)) {
                add_far<FULL, true>(p, c1, c2, e1, e2, s1, s2);
                add_far<FULL, true>(q, c1, c2, e1, e2, r1, r2);
            } else if (!cut(p) && !cut(q)) {
                add_far<FULL, false>(p, c1, c2, e1, e2, s1, s2);
                add_far<FULL, false>(q, c1, c2, e1, e2, r1, r2);
            } else {
                one(p, s1, s2);
                one(q, r1, r2);
            }
        }
        if (k < cnt) one(row(k), s1, s2);
    }
    s1 += r1;
    s2 += r2;
}

// Minimum over groups of 8 consecutive lanes (every lane gets it).
template <typename V>
__device__ __forceinline__ V min8(V v)
{
    v = fmin(v, dpp_mov<0xB1>(v));   // lane ^ 1
    v = fmin(v, dpp_mov<0x4E>(v));   // lane ^ 2
    return fmin(v, dpp_mov<0x141>(v));  // the other half of the 8 lanes
}

// Exchanges x's odd rows of N lanes (N = 16, 32) with y's even ones.
template <int N>
__device__ __forceinline__ void row_swap(unsigned& x, unsigned& y)
{
    if constexpr (N == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    }
}
template <int N>
__device__ __forceinline__ void row_swap(float& x, float& y)
{
    unsigned a = __float_as_uint(x), b = __float_as_uint(y);
    row_swap<N>(a, b);
    x = __uint_as_float(a);
    y = __uint_as_float(b);
}
template <int N>
__device__ __forceinline__ void row_swap(double& x, double& y)
{
    unsigned a = (unsigned)__double2loint(x), b = (unsigned)__double2loint(y);
    unsigned c = (unsigned)__double2hiint(x), d = (unsigned)__double2hiint(y);
    row_swap<N>(a, b);
    row_swap<N>(c, d);
    x = __hiloint2double((int)c, (int)a);
    y = __hiloint2double((int)d, (int)b);
}

// A unit: the 32 x 2 NK nodes that a wave holds, NK = 8 or 4 per lane.  Lane l holds
// row l % 16 (l % 8 for NK = 4) and value k column
//   NK = 8: 16 (k / 4) + 4 (l / 16) + k % 4,   NK = 4: 16 (l / 8 % 2) + 4 (l / 16) + k.
template <int NK>
__device__ __forceinline__ int unit_row()
{
    return lane_id() & (2 * NK - 1);
}
template <int NK>
__device__ __forceinline__ int unit_col(int k)
{
    const int lane = lane_id(), b = NK == 8 ? k >> 2 : (lane >> 3) & 1;
    return 16 * b + 4 * (lane >> 4) + (k & 3);
}

// Range record of one block of 32 x 8 nodes (kRec values): the deflection
// range over the block's nodes (min ax, max ax, min ay, max ay), over its first
// row, over its first column, and the first node's deflection; nodes outside
// the grid do not count.  A triangle tile's range is the union of its blocks',
// the first columns of the blocks to their right, the first rows of the blocks
// above and the first node of the block diagonally above (tile_range_rec).
//
// Writes the records of a unit (two for NK = 8, one for NK = 4).  The maxima are
// kept as minima of the negatives, and the four of a lane end in the four 16-lane
// groups of one register (two row exchanges), so one butterfly serves all: group q
// of 16 lanes holds min ax, min ay, -max ax, -max ay for q = 0 .. 3.  All 64 lanes
// call it.
template <int NK, typename V>
__device__ __forceinline__ void write_records(const V* sx, const V* sy, int i0, int j0, int nx, int ny, int nbx,
                                              V* __restrict__ rec)
{
    const int lane = lane_id(), q = lane >> 4, row = unit_row<NK>();
    const V inf = V(INFINITY);
    V a = inf, b = inf, c = inf, d = inf;
    const bool rin = j0 + row < ny;
    if (i0 + 32 <= nx && j0 + 2 * NK <= ny) {  // the usual case: no node outside
        a = sx[0];
        b = sx[0];
        c = sy[0];
        d = sy[0];
#pragma unroll
        for (int k = 1; k < NK; k++) {
            a = fmin(a, sx[k]);
            b = fmax(b, sx[k]);
            c = fmin(c, sy[k]);
            d = fmax(d, sy[k]);
        }
        b = -b;
        d = -d;
    } else {
#pragma unroll
        for (int k = 0; k < NK; k++)
            if (rin && i0 + unit_col<NK>(k) < nx) {
                a = fmin(a, sx[k]);
                b = fmin(b, -sx[k]);
                c = fmin(c, sy[k]);
                d = fmin(d, -sy[k]);
            }
    }
    if constexpr (NK == 4) {  // the row's other block of 16 columns
        a = fmin(a, dpp_mov<0x128>(a));  // lane ^ 8
        b = fmin(b, dpp_mov<0x128>(b));
        c = fmin(c, dpp_mov<0x128>(c));
        d = fmin(d, dpp_mov<0x128>(d));
    }
    row_swap<32>(a, b);
    row_swap<32>(c, d);
    a = fmin(a, b);  // lanes 0..31: a, 32..63: b
    c = fmin(c, d);
    row_swap<16>(a, c);
    const V r = fmin(a, c);  // the row's four values by q
    // first column: group 0 holds it as s[0]
    V x = sx[0], y = sy[0];
    row_swap<16>(x, y);
    V f = x;  // groups 0 and 1: ax and ay of the first column
    y = x;
    row_swap<32>(f, y);  // and groups 2 and 3
    f = rin ? (q >= 2 ? -f : f) : inf;
    if constexpr (NK == 4) f = (lane & 8) ? inf : f;
    const V all = min8(r), col = min8(f);
    if ((lane & 7) == 0 && (NK == 8 || (lane & 8) == 0) && rin && i0 < nx) {
        V* o = rec + ((size_t)((j0 + row) >> 3) * nbx + (i0 >> 5)) * kRec;
        const int slot = 2 * (q & 1) + (q >> 1);
        o[slot] = q >= 2 ? -all : all;
        o[4 + slot] = q >= 2 ? -r : r;
        o[8 + slot] = q >= 2 ? -col : col;
        if (q == 0) {
            o[12] = sx[0];
            o[13] = sy[0];
        }
    }
}

// Stores a wave's unit to a field plane, a lane's four nodes in 16 bytes a time also
// where a row does not start at a multiple of 16 (global stores ask for the element's
// alignment alone): node by node, each instruction would touch every line of the
// unit for a quarter of it.  4095^2 nodes, 4 potentials in FP32 89 -> 41 us, 12 in
// FP64 113 -> 77; the direct sums take 46 and 260.
template <int NK, typename V>
__device__ __forceinline__ void store_unit(const V* s, V* __restrict__ out, int i0, int j0, int nx, int ny)
{
    const int j = j0 + unit_row<NK>();
    if (j >= ny) return;
#pragma unroll
    for (int b = 0; b < NK / 4; b++) {
        const int i = i0 + unit_col<NK>(4 * b);
        V* o = out + (size_t)j * nx + i;
        if (i + 3 < nx) {
            constexpr int W = 16 / (int)sizeof(V);
            typedef V vecw __attribute__((ext_vector_type(W), aligned(sizeof(V))));
#pragma unroll
            for (int r = 0; r < 4; r += W) {
                vecw v;
#pragma unroll
                for (int q = 0; q < W; q++) v[q] = s[4 * b + r + q];
                *reinterpret_cast<vecw*>(o + r) = v;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (i + r < nx) o[r] = s[4 * b + r];
        }
    }
}

// ---------------------------------------------------------------- profiles

// The isothermal family of the tables (tab64, tab32) as a tile's summand.
struct IsoProfile {
    const double* tab64;
    const float* tab32;

    __device__ __forceinline__ bool far(int p, float xc, float yc, float hw, float c) const
    {
        const float* r = tab32 + (size_t)p * T32_STRIDE;
        // (a cut radius whose square overflows keeps the FP32 table's form)
        return tab64[(size_t)p * T64_STRIDE + T64_S2] <= 1e300 &&
               tile_far((xc - r[T32_CXH]) - r[T32_CXL], (yc - r[T32_CYH]) - r[T32_CYL], r[T32_A], r[T32_B], r[T32_C],
                        r[T32_A2], hw, c);
    }

    // Sum of list[k0..k1) at c + e: for an FP32 field, or in full FP64.
    template <bool FULL>
    __device__ __forceinline__ void far_at(const unsigned short* list, int k0, int k1, double c1, double c2, double e1,
                                           double e2, double& s1, double& s2) const
    {
        far_sum<FULL>(tab64, list, k0, k1, c1, c2, e1, e2, s1, s2);
    }

    // Adds potential p at NK nodes of one row (per lane): node-unit columns fi, row fj.
    template <int NK>
    __device__ __forceinline__ void near32(int p, const float* fi, float fj, float* sx, float* sy) const
    {
        const float* c = tab32 + (size_t)p * T32_STRIDE;
        const float nyv = (fj - c[T32_CYH]) - c[T32_CYL];
        const float4 rc =
            make_float4(c[T32_BP] * nyv, c[T32_CQ] * nyv, fmaf(c[T32_DQ] * nyv, nyv, c[T32_A2]), c[T32_RSK]);
        field32_pot<NK, 1>(c, &rc, fi, sx, sy);
    }
    template <int NK>
    __device__ __forceinline__ void near64(int p, const double* t1, double t2, double* sx, double* sy) const
    {
        const Far64 c = load_far(tab64 + (size_t)p * T64_STRIDE);
        if (__double_as_longlong(c.rs) == 0)
            near64_nodes<NK, false>(c, t1, t2, sx, sy);
        else
            near64_nodes<NK, true>(c, t1, t2, sx, sy);
    }
    // add_alpha64 at a node: offset (d1, d2) from the centre, B d2 and C d2.
    template <bool CUT>
    __device__ __forceinline__ static void node64(const Far64& c, double d1, double d2, double bd2, double cd2,
                                                  double& sx, double& sy)
    {
        const double m1 = fma(c.A, d1, bd2), m2 = fma(c.B, d1, cd2);
        const double R2 = fma(d1, m1, d2 * m2);
        const double qa = sqrt_est64(fmax(fabs(c.a2 + R2), 1e-300)) + c.ra;
        double f;
        if constexpr (CUT) {
            const double qs = sqrt_est64(c.s2 + R2) + c.rs;
            f = (qs - qa) * rcp_est64(qa * qs);
        } else {
            f = rcp_est64(qa);
        }
        const double kf = c.K * f;
        sx = fma(kf, m1, sx);
        sy = fma(kf, m2, sy);
    }
    // NK nodes of a row, the profile kind decided once, four nodes' chains
    // interleaved at a time (all eight would cost the occupancy its registers).
    template <int NK, bool CUT>
    __device__ __forceinline__ static void near64_nodes(const Far64& c, const double* t1, double t2, double* sx,
                                                        double* sy)
    {
        const double d2 = t2 - c.yc, bd2 = c.B * d2, cd2 = c.C * d2;
#pragma unroll
        for (int q = 0; q < NK; q += 4) {
#pragma unroll
            for (int k = q; k < q + 4; k++) node64<CUT>(c, t1[k] - c.xc, d2, bd2, cd2, sx[k], sy[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// ---------------------------------------------------------------- FP32 tiles

// One tile of T x T nodes per workgroup of NW waves.
template <int T, int NW = 4>
struct Tile32 {
    struct Lds {
        TileLists lists;
        double part[NW][2][64];
        double coef[2][64];
        float cheb[8][T];
        float g[16][T];
        float c00[2];
    };
};

// Tile (ti, tj) of workgroup `tile`, ntx tiles a row, each row's tiles turned by one
// more column.  Workgroups go to the CUs in turn, so a CU's tiles lie a few whole
// rows apart: in one column without the turn, and a column through a lens's centre
// then ends last (4096^2 x 200 FP32, four tiles a CU: they ended 37 to 87 us into
// the launch, 60 on average; with the turn the kernel takes 79 instead of 89, in
// another model 74 instead of 96).
__device__ __forceinline__ void tile_at(int tile, int ntx, int& ti, int& tj)
{
    tj = tile / ntx;
    ti = (tile - tj * ntx + tj) % ntx;
}

// The FP32 field of the tile at node (i0, j0) by a workgroup of NW waves.
//   1. lists (FP32 criterion, one potential per thread);
//   2. far sum at the 8 x 8 Chebyshev points, lane = point, the waves sharing
//      the far list, in FP64 with unrefined estimates (add_far<false>);
//   3. Chebyshev coefficients (two 8-point transforms per component, FP64),
//      then per node row the 8 coefficients in x (FP64, stored as FP32); the
//      constant term is kept apart, so that what is interpolated is the
//      variation over the tile and its rounding is relative to that;
//   4. per unit of 32 x 16 (T = 32: 32 x 8) nodes: interpolation in x as a matrix product
//      (v_mfma_f32_16x16x4f32, x nodes by rows, inner index the coefficient),
//      near potentials per node, the constant term last.
// Bound by vector issue (256 chains of 512^2 x 50, T = 32: vector instructions in
// 76 % of the cycles, of them a third of the time FP64, the far sums) once there
// are tiles enough, by one tile's chain before that.  Against the direct FP32 sum
// (kernel times): 4096^2 x 200 1402 -> 79 us, 1024^2 x 50 34.3 -> 14.0, the
// 96-sample batch 4800 -> 750, the 256 chains 1230 -> 503.
template <int T, int NW = 4, class P>
__device__ __forceinline__ void tile32_body(typename Tile32<T, NW>::Lds& L, const P& prof, int np, const GridDesc& g,
                                            int i0, int j0, float* __restrict__ ax, float* __restrict__ ay,
                                            bool bad, float* __restrict__ rec, int nbx)
{
    constexpr int NTH = 64 * NW;
    const int tid = threadIdx.x;
    constexpr float hw = 0.5f * (T - 1);
    const int lane = lane_id(), wt = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float xc = (float)i0 + hw, yc = (float)j0 + hw;
    tile_lists<NTH>(L.lists, np, [&](int p) { return prof.far(p, xc, yc, hw, kFarC32); });
    const int nn = __builtin_amdgcn_readfirstlane(L.lists.n_near), nf = np - nn;
    {
        const double c1 = g.x0 + (double)xc * g.h, c2 = g.y0 + (double)yc * g.h, half = (double)hw * g.h;
        double s1 = 0.0, s2 = 0.0;
        prof.template far_at<false>(L.lists.list + nn, wt * nf / NW, (wt + 1) * nf / NW,
                                    c1 + kDct8.xi[lane & 7] * half, c2 + kDct8.xi[lane >> 3] * half, 0.0, 0.0, s1, s2);
        L.part[wt][0][lane] = s1;
        L.part[wt][1][lane] = s2;
    }
    __syncthreads();
    for (int c = wt; c < 2; c += NW) {  // component c: one wave each
        double v = L.part[0][c][lane];
        for (int w = 1; w < NW; w++) v += L.part[w][c][lane];
        L.coef[c][lane] = v;
        wave_lds_sync();
        const int a = lane & 7, k = lane >> 3;
        double u = 0.0;  // transform in x: point index lane & 7
        for (int m = 0; m < 8; m++) u = fma(kDct8.d[8 * a + m], L.coef[c][8 * k + m], u);
        wave_lds_sync();
        L.coef[c][lane] = u;  // [k][a]
        wave_lds_sync();
        double w = 0.0;  // transform in y: coefficient b = k
        for (int m = 0; m < 8; m++) w = fma(kDct8.d[8 * k + m], L.coef[c][8 * m + a], w);
        wave_lds_sync();
        if (lane == 0) {
            L.c00[c] = (float)w;
            w -= (double)(float)w;  // the constant's rounding stays in the interpolated part
        }
        L.coef[c][lane] = w;  // [b][a]
    }
    __syncthreads();
    {
        const int row = tid % T;
        double tb[8];
        const double y = ((double)row - hw) * (1.0 / (double)hw);
        tb[0] = 1.0;
        tb[1] = y;
#pragma unroll
        for (int b = 2; b < 8; b++) tb[b] = fma(2.0 * y, tb[b - 1], -tb[b - 2]);
        if (tid < T)
#pragma unroll
            for (int b = 0; b < 8; b++) L.cheb[b][row] = (float)tb[b];
        for (int q = tid / T; q < 16; q += NTH / T) {  // (component, a)
            const double* co = L.coef[q >> 3] + (q & 7);
            double v = 0.0;
#pragma unroll
            for (int b = 7; b >= 0; b--) v = fma(co[8 * b], tb[b], v);
            L.g[q][row] = (float)v;
        }
    }
    __syncthreads();
    // units of 32 x 16 nodes, or of 32 x 8 where the tile has only two of those for
    // four waves
    constexpr int NK = T == 32 || NW == 8 ? 4 : 8;
    constexpr int UX = T / 32, UNITS = UX * (T / (2 * NK));
    const int li = lane & 15, lk = lane >> 4;
    // (an invalid model's field is NaN)
    const float cx = bad ? __builtin_nanf("") : L.c00[0], cy = bad ? __builtin_nanf("") : L.c00[1];
    for (int u = wt; u < UNITS; u += NW) {
        const int cu = (u % UX) * 32, ru = (u / UX) * 2 * NK;
        if (i0 + cu >= g.nx || j0 + ru >= g.ny) continue;
        float sx[NK], sy[NK], fi[NK];
        if constexpr (NK == 8) {
            floatx4 acc[2][2];  // [component][column block]
#pragma unroll
            for (int c = 0; c < 2; c++)
#pragma unroll
                for (int b = 0; b < 2; b++) {
                    acc[c][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int k = 1; k >= 0; k--)
                        acc[c][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.cheb[4 * k + lk][cu + 16 * b + li],
                                                                         L.g[8 * c + 4 * k + lk][ru + li], acc[c][b],
                                                                         0, 0, 0);
                }
#pragma unroll
            for (int k = 0; k < 8; k++) {
                sx[k] = acc[0][k >> 2][k & 3];
                sy[k] = acc[1][k >> 2][k & 3];
            }
        } else {
            // the product's 16 rows are 8 node rows of x, then of y: a lane gets one
            // component of both column blocks and trades one with lane ^ 8
            floatx4 acc[2];  // [column block]
#pragma unroll
            for (int b = 0; b < 2; b++) {
                acc[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 1; k >= 0; k--)
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.cheb[4 * k + lk][cu + 16 * b + li],
                                                                  L.g[(li & 8) + 4 * k + lk][ru + (li & 7)], acc[b],
                                                                  0, 0, 0);
            }
            const bool second = (li & 8) != 0;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const float other = dpp_mov<0x128>(second ? acc[0][k] : acc[1][k]);
                sx[k] = second ? other : acc[0][k];
                sy[k] = second ? acc[1][k] : other;
            }
        }
#pragma unroll
        for (int k = 0; k < NK; k++) fi[k] = (float)(i0 + cu + unit_col<NK>(k));
        const float fj = (float)(j0 + ru + unit_row<NK>());
        for_list(L.lists.list, nn, [&](int p) { prof.template near32<NK>(p, fi, fj, sx, sy); });
#pragma unroll
        for (int k = 0; k < NK; k++) {
            sx[k] += cx;
            sy[k] += cy;
        }
        if (rec) write_records<NK>(sx, sy, i0 + cu, j0 + ru, g.nx, g.ny, nbx, rec);
        store_unit<NK>(sx, ax, i0 + cu, j0 + ru, g.nx, g.ny);
        store_unit<NK>(sy, ay, i0 + cu, j0 + ru, g.nx, g.ny);
    }
}

// ---------------------------------------------------------------- FP64 tiles

// The same in FP64 with 16 x 16 Chebyshev points (one per thread of the
// workgroup) and v_mfma_f64_16x16x4f64.  The row coefficients (16 per row and
// component) are formed by the lanes that feed them to the matrix product, once
// per group of 16 rows, so they need no LDS.  Bound by FP64 issue (48 % of the
// cycles at 1000 x 777 x 75, where 800 tiles leave a third of the CUs' time idle;
// 62 % at 2047 x 1531 x 120).  Against the direct FP64 sum: 1000 x 777 x 75
// 106 -> 51 us, the call of 2047 x 1531 x 120 484 -> 110 (85 in the kernel).
template <int T>
struct Tile64 {
    struct Lds {
        TileLists lists;
        double f[2][256], u[2][256];
        double cheb[16][T];
    };
};

// Where a tile's units go: to the field planes, with the range
// records where asked for.
struct FieldSink64 {
    double *ax, *ay, *rec;
    int nx, ny;
    bool bad;  // the whole field is NaN

    template <int NK>
    __device__ __forceinline__ bool wants(int, int) const  // wave-uniform
    {
        return true;
    }
    template <int NK>
    __device__ __forceinline__ void put(double* sx, double* sy, int i0, int j0) const
    {
        if (bad)
#pragma unroll
            for (int k = 0; k < NK; k++) sx[k] = sy[k] = __builtin_nan("");
        if (rec) write_records<NK>(sx, sy, i0, j0, nx, ny, (nx + 31) >> 5, rec);
        store_unit<NK>(sx, ax, i0, j0, nx, ny);
        store_unit<NK>(sy, ay, i0, j0, nx, ny);
    }
};

template <int T, class P, class Sink>
__device__ __forceinline__ void tile64_body(typename Tile64<T>::Lds& L, const P& prof, int np, const GridDesc& g,
                                            int i0, int j0, const Sink& sink)
{
    constexpr float hw = 0.5f * (T - 1);
    const int tid = threadIdx.x, lane = lane_id(), wt = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float xc = (float)i0 + hw, yc = (float)j0 + hw;
    tile_lists(L.lists, np, [&](int p) { return prof.far(p, xc, yc, hw, kFarC64); });
    const int nn = __builtin_amdgcn_readfirstlane(L.lists.n_near), nf = np - nn;
    const int lo = tid & 15, hi = tid >> 4;
    // The polynomial is in (t - c)/half, t the nodes' rounded FP64 coordinates
    // (node_coord) and c the tile centre's: nodes then keep their own position
    // to a rounding relative to the tile, as theta - theta_c does in the direct sum.
    const double c1 = g.x0 + (double)xc * g.h, c2 = g.y0 + (double)yc * g.h;
    const double half = (double)hw * g.h, ihalf = 1.0 / half;
    {
        double s1 = 0.0, s2 = 0.0;
        prof.template far_at<true>(L.lists.list + nn, 0, nf, c1, c2, kDct16.xi[lo] * half, kDct16.xi[hi] * half, s1, s2);
        L.f[0][tid] = s1;
        L.f[1][tid] = s2;
    }
    if (tid < T) {
        const double x = (node_coord(g.x0, i0 + tid, g.h) - c1) * ihalf;
        double a = 1.0, b = x;
        for (int m = 0; m < 16; m++) {
            L.cheb[m][tid] = a;
            const double n = fma(2.0 * x, b, -a);
            a = b;
            b = n;
        }
    }
    __syncthreads();
    // the value at a middle point is taken off before the transforms and added
    // last, at the nodes: the transforms' and the interpolation's rounding is then
    // relative to the variation over the tile
    const double r0 = L.f[0][16 * 8 + 8], r1 = L.f[1][16 * 8 + 8];
    {
        double u0 = 0.0, u1 = 0.0;  // transform in x: point row hi, coefficient lo
#pragma unroll
        for (int m = 0; m < 16; m++) {
            const double d = kDct16.d[16 * lo + m];
            u0 = fma(d, L.f[0][16 * hi + m] - r0, u0);
            u1 = fma(d, L.f[1][16 * hi + m] - r1, u1);
        }
        L.u[0][tid] = u0;
        L.u[1][tid] = u1;
    }
    __syncthreads();
    {
        double w0 = 0.0, w1 = 0.0;  // transform in y: coefficient hi in y, lo in x
#pragma unroll
        for (int m = 0; m < 16; m++) {
            const double d = kDct16.d[16 * hi + m];
            w0 = fma(d, L.u[0][16 * m + lo], w0);
            w1 = fma(d, L.u[1][16 * m + lo], w1);
        }
        L.f[0][tid] = w0;
        L.f[1][tid] = w1;
    }
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4;
    // output value r of lane l of the matrix product is row l / 16 + 4 r: the x
    // nodes are assigned so that a lane holds four consecutive ones
    const int xi = 4 * (li & 3) + (li >> 2);
    constexpr int NK = T == 32 ? 4 : 8, RU = 2 * NK;  // units of 32 x RU nodes, as Tile32
    constexpr int NC = NK == 8 ? 2 : 1;  // components per lane of the product (NK = 4: one, by li / 8)
    const int row = unit_row<NK>();
    for (int ru = RU * wt; ru < T; ru += 4 * RU) {
        if (j0 + ru >= g.ny) break;
        const double t2 = node_coord(g.y0, j0 + ru + row, g.h);
        double B[NC][4];  // coefficient 4 s + lk of row ru + row
        {
            const double y = (t2 - c2) * ihalf;
            double tb[16];
            tb[0] = 1.0;
            tb[1] = y;
#pragma unroll
            for (int b = 2; b < 16; b++) tb[b] = fma(2.0 * y, tb[b - 1], -tb[b - 2]);
#pragma unroll
            for (int c = 0; c < NC; c++) {
                const double* f = L.f[NK == 8 ? c : li >> 3];
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    double v = 0.0;
#pragma unroll
                    for (int b = 15; b >= 0; b--) v = fma(f[16 * b + 4 * s + lk], tb[b], v);
                    B[c][s] = v;
                }
            }
        }
        for (int cu = 0; cu < T; cu += 32) {
            if (i0 + cu >= g.nx) break;
            if (!sink.template wants<NK>(i0 + cu, j0 + ru)) continue;
            doublex4 acc[NC][2];
#pragma unroll
            for (int b = 0; b < 2; b++) {
#pragma unroll
                for (int c = 0; c < NC; c++) acc[c][b] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 3; s >= 0; s--) {
                    const double A = L.cheb[4 * s + lk][cu + 16 * b + xi];
#pragma unroll
                    for (int c = 0; c < NC; c++)
                        acc[c][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(A, B[c][s], acc[c][b], 0, 0, 0);
                }
            }
            double sx[NK], sy[NK], t1[NK];
            if constexpr (NK == 8) {
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    sx[k] = acc[0][k >> 2][k & 3];
                    sy[k] = acc[1][k >> 2][k & 3];
                }
            } else {
                const bool second = (li & 8) != 0;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const double other = dpp_mov<0x128>(second ? acc[0][0][k] : acc[0][1][k]);
                    sx[k] = second ? other : acc[0][0][k];
                    sy[k] = second ? acc[0][1][k] : other;
                }
            }
#pragma unroll
            for (int k = 0; k < NK; k++) t1[k] = node_coord(g.x0, i0 + cu + unit_col<NK>(k), g.h);
            for_list(L.lists.list, nn, [&](int p) { prof.template near64<NK>(p, t1, t2, sx, sy); });
#pragma unroll
            for (int k = 0; k < NK; k++) {
                sx[k] += r0;
                sy[k] += r1;
            }
            sink.template put<NK>(sx, sy, i0 + cu, j0 + ru);
        }
    }
}

}  // namespace lens
