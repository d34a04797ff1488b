// The paper's mixed-precision gradient for SIE lenses on gfx950 (Sec. 3.2,
// Sec. 3.3, Appendix A.3): grad Psi in single precision at every pixel, in
// double precision inside blocks of pixels centred on the halos (pc x pc for
// the cluster-scale halos, pg x pg for the galaxy-scale ones), then in double
// precision again wherever the source-plane criteria of Sec. 3.3, evaluated on
// that field, ask for it.
//
// Launch sequence (one call, the caller's stream):
//   k_mix_prep     constants of every potential and the corner of its block (one
//                  workgroup), SIE check
//   k_mix_field32  FP32 field at every node (SIE form alpha = K m / R with
//                  R = sqrt(d . M d): one reciprocal square root per
//                  potential), written as double; mask cleared
//   k_mix_blocks   FP64 gradient of the halos' blocks, marked 1
//   k_mix_scan     criteria on the field so far, pixels marked 2; counts
//   k_mix_stats    counts and status to the caller's stats
//   k_mix_pixels   FP64 gradient of the pixels marked 2 one by one, or
//   k_mix_dp       by tiles
// The FP32 field decides which pixels the criteria take, so it is summed over
// the potentials at every pixel; the FP64 gradient of the criteria pixels (a
// fifth of the benchmark image) goes through the tiled field: 0.4 ms against 4.2
// for the sum over 702 halos at each of 8.8 M pixels.
#include "lens_path.hpp"
#include "lens_tiles.hpp"

#include <algorithm>
#include <type_traits>

namespace lens {

// ---------------------------------------------------------------- constants

// The block of halo p: `size` x `size` pixels (pc for the first n_cluster halos, pg
// for the others) spanning node indices [k - size/2, k - size/2 + size) on each axis,
// k = (x_c - x0)/h rounded half away from zero.  corner[p] = k - size/2.
__global__ __launch_bounds__(256) void k_mix_prep(PotPtrs pot, GridDesc g, int n_cluster, int pc, int pg,
                                                  double* __restrict__ tab64, float* __restrict__ tab32,
                                                  double* __restrict__ bterm, int2* __restrict__ corner,
                                                  MixState* __restrict__ st)
{
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    bool bad = false;
    for (int p = threadIdx.x; p < pot.n; p += 256) {
        double row[T64_STRIDE], terms[3];
        prep_one(pot, g, p, p, tab64, tab32, bterm, row, terms);
        // the criteria and blocks are derived for the SIE (Sec. 3.2): no core, no cut
        const bool out = terms[2] != 0.0 || pot.r_core[p] != 0.0 || !isinf(pot.r_cut[p]) || pot.r_cut[p] < 0.0;
        bad |= out;
        const int half = (p < n_cluster ? pc : pg) / 2;
        // (a valid centre is within 2^22 nodes)
        corner[p] = out ? make_int2(0, 0)
                        : make_int2((int)llround((pot.x[p] - g.x0) / g.h) - half,
                                    (int)llround((pot.y[p] - g.y0) / g.h) - half);
    }
    if (bad) atomicOr(&s_bad, 1);
    __syncthreads();
    if (threadIdx.x == 0) st->status = s_bad ? kStatusInvalid : kStatusOk;
}

// ---------------------------------------------------------------- FP32 field

// Reciprocal root (the hardware instruction, 1 ulp) issued at raised wave
// priority.  On gfx950 two waves of a SIMD issue a simple FP32 operation each in
// the same four cycles, but a transcendental takes the SIMD alone for eight;
// spread through the waves' streams they leave the simple operations unpaired
// (probe at 8 waves per SIMD, this loop's mix: 4.19 cycles per instruction).  A
// wave that reaches one goes first, the others' simple operations then pair up:
// 3.19 cycles.  The closing s_setprio is also the wait state between a
// transcendental and the first use of its result.  With few waves per SIMD there
// is nothing to pair and the fixed order costs latency (300 x 211 x 30: 12 us
// against 9), so the single-node layout uses the plain instruction.
__device__ __forceinline__ float rsq_pri(float x)
{
    float r;
    asm("s_setprio 3\n\tv_rsq_f32 %0, %1\n\ts_setprio 0" : "=v"(r) : "v"(x));
    return r;
}

// FP32 SIE contribution of table row c for NPL columns in each of NR rows (sx,
// sy: [NR][NPL]): node-unit offsets from the exact centre split (as in the
// general FP32 field), m = M d, R^2 = d . m clamped below at 1e-30 (the centre,
// where m = 0, contributes 0), alpha += (K/h) m / R.  Without CLAMP the caller
// knows that R^2 stays above 1e-30 (the result is then the same bit for bit).
template <int NPL, int NR, bool CLAMP>
__device__ __forceinline__ void sie32_pot(const float* __restrict__ c, const float4* rc, const float* fi, float* sx,
                                          float* sy)
{
    const float cxh = c[T32_CXH], cxl = c[T32_CXL];
    const float A = c[T32_A], B = c[T32_B], K = c[T32_K];
#pragma unroll
    for (int k = 0; k < NPL; k++) {
        const float nxv = (fi[k] - cxh) - cxl;
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const float m1 = fmaf(A, nxv, rc[r].y);
            const float m2 = fmaf(B, nxv, rc[r].z);
            float R2 = fmaf(nxv, m1, rc[r].x * m2);
            if constexpr (CLAMP) R2 = fmaxf(R2, 1e-30f);
            const float kr = K * (NPL * NR > 1 ? rsq_pri(R2) : __builtin_amdgcn_rsqf(R2));
            sx[r * NPL + k] = fmaf(kr, m1, sx[r * NPL + k]);
            sy[r * NPL + k] = fmaf(kr, m2, sy[r * NPL + k]);
        }
    }
}

// Workgroup = 256 * NPL columns of NR consecutive rows; each thread NPL
// consecutive columns of every row, so the column offset is formed once for the
// NR rows.  The row parts (n_y, B n_y, C n_y) of up to 256 potentials at a time
// are formed by one thread each, in LDS, with a bit per potential that needs the
// clamp: its centre within a node of the block, or M so flat that R^2 is not
// safely above 1e-30 half a node away (a potential stored with M = 0 among
// them).  Bound by vector issue: 7 simple operations, 2 / NR for the column
// offset and the reciprocal root per pixel and potential.  Writes the FP32 field
// as double and clears the mask.
template <int NPL, int NR>
__global__ __launch_bounds__(256) void k_mix_field32(const float* __restrict__ tab32, int np, int nx, int ny,
                                                     double* __restrict__ ax, double* __restrict__ ay,
                                                     unsigned char* __restrict__ mask,
                                                     const MixState* __restrict__ st)
{
    const int j0 = blockIdx.y * NR;
    const int ib = blockIdx.x * 256 * NPL, i0 = ib + threadIdx.x * NPL;
    float fi[NPL], sx[NR * NPL], sy[NR * NPL];
#pragma unroll
    for (int k = 0; k < NPL; k++) fi[k] = (float)(i0 + k);
#pragma unroll
    for (int q = 0; q < NR * NPL; q++) sx[q] = sy[q] = 0.0f;
    const bool bad = st->status != kStatusOk;
    if constexpr (NPL * NR == 1) {
        // few waves: the plain loop over the potentials, whose loads the compiler groups
        // (643 x 569 x 284: 53 us against 76 in runs by the clamp)
        if (!bad)
            pots_wg<T32_STRIDE, T32_CYH, T32_CYL, T32_B, T32_C>(
                tab32, np, (float)j0, [&](const float* c, float4 rc) { sie32_pot<1, 1, true>(c, &rc, fi, sx, sy); });
    } else {
        __shared__ float4 srow[NR * 256];
        __shared__ unsigned long long sclamp[4];
        for (int p0 = 0; p0 < np && !bad; p0 += 256) {  // uniform over the launch
            const int pc = min(256, np - p0);
            if (p0 > 0) __syncthreads();  // the previous chunk has been read
            bool clamp = false;
            if ((int)threadIdx.x < pc) {
                const float* c = tab32 + (size_t)(p0 + threadIdx.x) * T32_STRIDE;
                const float A = c[T32_A], B = c[T32_B], C = c[T32_C];
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    const float nyv = ((float)(j0 + r) - c[T32_CYH]) - c[T32_CYL];
                    srow[r * 256 + threadIdx.x] = make_float4(nyv, B * nyv, C * nyv, 0.0f);
                }
                const float cx = c[T32_CXH], cy = c[T32_CYH], det = A * C - B * B, tr = A + C;
                const bool inside = cx >= (float)(ib - 2) && cx <= (float)(ib + 256 * NPL + 1) && cy >= (float)(j0 - 2) &&
                                    cy <= (float)(j0 + NR + 1);
                // smallest eigenvalue of M h^2 >= det / tr; R^2 >= that / 4 outside
                clamp = inside || !(det > 1e-4f * tr * tr) || !(det > 1e-27f * tr);
            }
            const unsigned long long b = __ballot(clamp);
            if (lane_id() == 0) sclamp[threadIdx.x >> 6] = b;
            __syncthreads();
            for (int w = 0; w * 64 < pc; w++) {
                const unsigned long long lw = sclamp[w];
                const unsigned long long cl =
                    ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(lw >> 32)) << 32) |
                    (unsigned)__builtin_amdgcn_readfirstlane((int)lw);
                const int n = min(64, pc - 64 * w);
                auto add = [&](int q, auto clamped) {
                    const int p = 64 * w + q;
                    float4 rc[NR];
#pragma unroll
                    for (int r = 0; r < NR; r++) rc[r] = srow[r * 256 + p];
                    sie32_pot<NPL, NR, decltype(clamped)::value>(tab32 + (size_t)(p0 + p) * T32_STRIDE, rc, fi, sx, sy);
                };
                for (int q = 0; q < n; q++) {  // a run without the clamp, then one with it
                    const unsigned long long rest = cl >> q;
                    const int stop = rest ? min(n, q + __builtin_ctzll(rest)) : n;
                    for (; q < stop; q++) add(q, std::false_type());
                    if (q < n) add(q, std::true_type());
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < NR; r++) {
        if (j0 + r >= ny) break;
        const size_t row = (size_t)(j0 + r) * nx;
#pragma unroll
        for (int k = 0; k < NPL; k++) {
            if (i0 + k < nx) {
                ax[row + i0 + k] = bad ? __builtin_nan("") : (double)sx[r * NPL + k];
                ay[row + i0 + k] = bad ? __builtin_nan("") : (double)sy[r * NPL + k];
                mask[row + i0 + k] = 0;
            }
        }
    }
}

// ---------------------------------------------------------------- DP blocks and criteria

// 1/sqrt(x) in FP64 for a positive normal x: the hardware estimate (relative
// error below 2^-24 on gfx950, measured) refined by one Newton-Raphson step
// y <- y (3/2 - x y^2 / 2), which squares the error: ~2^-47 relative.  FULL: with
// the next term of the series, y (1 + e/2 + 3 e^2/8), e = 1 - x y^2: ~1 ulp, as the
// tiles' terms.
template <bool FULL>
__device__ __forceinline__ double rsq64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    if constexpr (FULL) {
        const double e = fma(-(x * y), y, 1.0);
        return fma(y * e, fma(0.375, e, 0.5), y);
    }
    return fma(y, fma(-0.5 * x * y, y, 0.5), y);
}

// FP64 SIE contribution of table row t at (t1, t2): alpha += K m / R, m = M d,
// R^2 = d . m, clamped below at 1e-300 (the centre, where m = 0, contributes 0).
template <bool FULL>
__device__ __forceinline__ void sie64_add(const double* __restrict__ t, double t1, double t2, double& s1,
                                          double& s2)
{
    const double d1 = t1 - t[T64_XC], d2 = t2 - t[T64_YC];
    const double m1 = fma(t[T64_A], d1, t[T64_B] * d2);
    const double m2 = fma(t[T64_B], d1, t[T64_C] * d2);
    const double R2 = fmax(fma(d1, m1, d2 * m2), 1e-300);
    const double kr = t[T64_K] * rsq64<FULL>(R2);
    s1 = fma(kr, m1, s1);
    s2 = fma(kr, m2, s2);
}

// FP64 gradient of pixel (i, j) by the sum over all halos, eight at a time: their
// scalar loads, from beyond the scalar cache for some hundred halos, are in flight
// together (6730^2 x 702 blocks 398 us, four at a time 409, one 451).
template <bool FULL>
__device__ __forceinline__ void pixel64(const double* __restrict__ tab64, int np, const GridDesc& g, int i, int j,
                                        double* __restrict__ ax, double* __restrict__ ay)
{
    const double t1 = node_coord(g.x0, i, g.h), t2 = node_coord(g.y0, j, g.h);
    double s1 = 0.0, s2 = 0.0;
#pragma unroll 8
    for (int m = 0; m < np; m++) sie64_add<FULL>(tab64 + (size_t)m * T64_STRIDE, t1, t2, s1, s2);
    const size_t o = (size_t)j * g.nx + i;
    ax[o] = s1;
    ay[o] = s2;
}

// The FP64 blocks of the halos, side size0 for the first n0 and size1 for the others,
// clipped to the grid: per0 (per1) workgroups mark a halo's pixels in the mask and
// write their FP64 gradient, 256 pixels at a time.  A pixel of several blocks belongs to
// the first of those halos: the blocks that come before and touch the 256 pixels' rows
// are listed in LDS, 256 halos at a time, and the pixels that are left are packed into
// whole waves.  One launch for both kinds, so that the few pixels left to the second
// do not add a chain of their own.  Bound by FP64 issue (6730^2 x 702: 398 us; 426
// without the lists, which repeated shared pixels: 100 x 64 x 702 504 us a call, now 277;
// 300 x 211 x 100 with blocks of 400 375, now 72; 600 x 500 x 702 749, now 481).
__global__ __launch_bounds__(256) void k_mix_blocks(int np, GridDesc g, int n0, int size0, int per0, int size1, int per1,
                                                    const int2* __restrict__ corner, const double* __restrict__ tab64,
                                                    double* __restrict__ ax, double* __restrict__ ay,
                                                    unsigned char* __restrict__ mask, const MixState* __restrict__ st)
{
    __shared__ int4 touch[256];  // blocks [x, z) x [y, w)
    __shared__ unsigned short left[256];
    __shared__ int s_n[4];
    if (st->status != kStatusOk) return;
    const int lane = lane_id(), wave = threadIdx.x >> 6, b0 = n0 * per0;
    const bool first = (int)blockIdx.x < b0;
    const int rest = first ? (int)blockIdx.x : (int)blockIdx.x - b0, per = first ? per0 : per1;
    const int p = (first ? 0 : n0) + rest / per, size = first ? size0 : size1;
    const unsigned chunk = (unsigned)(rest % per);  // of `per` workgroups of the halo
    const int2 c = corner[p];
    const int i0 = max(c.x, 0), j0 = max(c.y, 0), i1 = min(c.x + size, g.nx), j1 = min(c.y + size, g.ny);
    if (i0 >= i1 || j0 >= j1) return;
    const unsigned w = (unsigned)(i1 - i0), n = w * (unsigned)(j1 - j0);
    // entries of the workgroup's lists: `in` of every thread in order
    auto pack = [&](bool in, int& total) {
        const unsigned long long m = __ballot(in);
        if (lane == 0) s_n[wave] = __popcll(m);
        __syncthreads();
        int at = __popcll(m & ((1ull << lane) - 1ull));
        for (int k = 0; k < wave; k++) at += s_n[k];
        total = s_n[0] + s_n[1] + s_n[2] + s_n[3];
        return at;
    };
    for (unsigned q0 = chunk * 256; q0 < n; q0 += (unsigned)per * 256) {
        const unsigned q = q0 + threadIdx.x;
        const int j = j0 + (int)(q / w), i = i0 + (int)(q % w);
        const int ja = j0 + (int)(q0 / w), jb = j0 + (int)((min(q0 + 256u, n) - 1) / w);  // rows of the 256
        bool mine = q < n;
        for (int b = 0; b < p && __syncthreads_or(mine); b += 256) {
            const int h = b + (int)threadIdx.x;
            int4 t = make_int4(0, 0, 0, 0);
            bool in = false;
            if (h < p) {
                const int2 d = corner[h];
                const int sz = h < n0 ? size0 : size1;
                t = make_int4(d.x, d.y, d.x + sz, d.y + sz);
                in = t.x < i1 && t.z > i0 && t.y <= jb && t.w > ja;
            }
            int cnt;
            const int at = pack(in, cnt);
            if (in) touch[at] = t;
            __syncthreads();
            for (int k = 0; k < cnt && mine; k++)
                mine = !(i >= touch[k].x && i < touch[k].z && j >= touch[k].y && j < touch[k].w);
        }
        int cnt;
        const int at = pack(mine, cnt);
        if (mine) left[at] = (unsigned short)threadIdx.x;
        __syncthreads();
        if ((int)threadIdx.x < cnt) {
            const unsigned r = q0 + left[threadIdx.x];
            const int jr = j0 + (int)(r / w), ir = i0 + (int)(r % w);
            pixel64<false>(tab64, np, g, ir, jr, ax, ay);
            mask[(size_t)jr * g.nx + ir] = 1;
        }
        __syncthreads();  // the lists are read
    }
}

// Criteria of Sec. 3.3 on the field so far, one workgroup per 256 columns of
// kScanRows rows, thread = column, the previous row's values kept in registers
// and the left neighbour taken from the lane beside it (every value read once,
// plus a row above the block and a column beside each wave):
//     d1 = ax(i,j) - ax(i-1,j), d2 = ay(i,j) - ay(i,j-1),
//     d3 = ax(i,j) - ax(i,j-1), d4 = ay(i,j) - ay(i-1,j),
//     |dx - d1| < t12, |dx - d2| < t12, |d3| > t34 or |d4| > t34,
// a difference whose neighbour is outside the image not being evaluated.
// Pixels outside the blocks where one holds are marked 2.  counts[workgroup]
// receives its block pixels and its criteria pixels (no atomics: thousands of
// workgroups on one counter would queue for it).
constexpr int kScanRows = 16;
__global__ __launch_bounds__(256) void k_mix_scan(const double* __restrict__ ax, const double* __restrict__ ay,
                                                  GridDesc g, double t12, double t34, unsigned char* __restrict__ mask,
                                                  uint2* __restrict__ counts, const MixState* __restrict__ st)
{
    __shared__ unsigned s_cnt[4][2];
    unsigned nb = 0, nc = 0;
    if (st->status == kStatusOk) {  // uniform over the launch
        const int i = blockIdx.x * 256 + threadIdx.x, j0 = blockIdx.y * kScanRows;
        const int ic = min(i, g.nx - 1), il = max(ic - 1, 0);
        const bool in = i < g.nx, edge = lane_id() == 0;
        double px = 0.0, py = 0.0;
        if (j0 > 0) {
            px = ax[(size_t)(j0 - 1) * g.nx + ic];
            py = ay[(size_t)(j0 - 1) * g.nx + ic];
        }
        const int j1 = min(j0 + kScanRows, g.ny);
        for (int j = j0; j < j1; j++) {
            const size_t row = (size_t)j * g.nx;
            const double x = ax[row + ic], y = ay[row + ic];
            const unsigned char m = mask[row + ic];
            double lx = __shfl_up(x, 1, 64), ly = __shfl_up(y, 1, 64);
            if (edge) {
                lx = ax[row + il];
                ly = ay[row + il];
            }
            bool need = false;
            if (i > 0) need = fabs(g.h - (x - lx)) < t12 || fabs(y - ly) > t34;
            if (j > 0) need = need || fabs(g.h - (y - py)) < t12 || fabs(x - px) > t34;
            need = need && in && m == 0;
            if (need) mask[row + ic] = 2;
            nc += need ? 1u : 0u;
            nb += in && m == 1 ? 1u : 0u;
            px = x;
            py = y;
        }
    }
    for (int k = 32; k >= 1; k >>= 1) {
        nb += __shfl_xor(nb, k, 64);
        nc += __shfl_xor(nc, k, 64);
    }
    if (lane_id() == 0) {
        s_cnt[threadIdx.x >> 6][0] = nb;
        s_cnt[threadIdx.x >> 6][1] = nc;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        counts[blockIdx.y * gridDim.x + blockIdx.x] =
            make_uint2(s_cnt[0][0] + s_cnt[1][0] + s_cnt[2][0] + s_cnt[3][0],
                       s_cnt[0][1] + s_cnt[1][1] + s_cnt[2][1] + s_cnt[3][1]);
}

// Units of a tile that hold criteria pixels, those pixels stored.
struct CriteriaSink {
    double *ax, *ay;
    const unsigned char* mask;
    int nx, ny;

    template <int NK>
    __device__ __forceinline__ bool wants(int i0, int j0) const
    {
        const int j = j0 + unit_row<NK>();
        bool any = false;
        if (j < ny)
#pragma unroll
            for (int k = 0; k < NK; k++) {
                const int i = i0 + unit_col<NK>(k);
                any = any || (i < nx && mask[(size_t)j * nx + i] == 2);
            }
        return __ballot(any) != 0;
    }
    template <int NK>
    __device__ __forceinline__ void put(const double* sx, const double* sy, int i0, int j0) const
    {
        const int j = j0 + unit_row<NK>();
        if (j >= ny) return;
#pragma unroll
        for (int k = 0; k < NK; k++) {
            const int i = i0 + unit_col<NK>(k);
            const size_t o = (size_t)j * nx + i;
            if (i < nx && mask[o] == 2) {
                ax[o] = sx[k];
                ay[o] = sy[k];
            }
        }
    }
};

// FP64 gradient of the criteria pixels one by one, where the image has no more than
// `few` of them: a workgroup takes every so-many-th run of 256 pixels and collects their
// criteria pixels in LDS first, so that whole waves work on them.  As many workgroups
// as give each two waves of them take part, for balance, and enough to read the mask.
constexpr int kRun = 256;
__global__ __launch_bounds__(256) void k_mix_pixels(const double* __restrict__ tab64, int np, GridDesc g, unsigned few,
                                                    const unsigned char* __restrict__ mask, double* __restrict__ ax,
                                                    double* __restrict__ ay, const MixState* __restrict__ st)
{
    __shared__ struct {
        unsigned list[kRun + 256];
        unsigned n;
    } L;
    if (st->status != kStatusOk || st->n_crit == 0 || st->n_crit > few) return;
    const unsigned nn = (unsigned)g.nx * (unsigned)g.ny, runs = (nn + kRun - 1) / kRun, t = threadIdx.x;
    const unsigned step = min(gridDim.x, max(2048u, st->n_crit / 128));
    if (blockIdx.x >= step) return;
    if (t == 0) L.n = 0;
    __syncthreads();
    for (unsigned r = blockIdx.x; r < runs; r += step) {
#pragma unroll
        for (int k = 0; k < kRun / 256; k++) {
            const unsigned q = r * kRun + k * 256 + t;
            const bool in = q < nn && mask[q] == 2;
            const unsigned long long m = __ballot(in);
            if (m == 0) continue;
            unsigned at = 0;
            if (lane_id() == 0) at = atomicAdd(&L.n, (unsigned)__popcll(m));
            at = (unsigned)__builtin_amdgcn_readfirstlane((int)at) +
                 __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            if (in) L.list[at] = q;
        }
        __syncthreads();
        const unsigned n = L.n;
        const bool last = r + step >= runs;
        const unsigned done = last ? n : n & ~255u;
        for (unsigned e = t; e < done; e += 256) {
            const unsigned q = L.list[e], j = q / (unsigned)g.nx;
            pixel64<true>(tab64, np, g, (int)(q - j * (unsigned)g.nx), (int)j, ax, ay);
        }
        __syncthreads();
        if (done) {  // uniform: the rest, fewer than 256, to the front
            const unsigned keep = t < n - done ? L.list[done + t] : 0u;
            __syncthreads();
            if (t < n - done) L.list[t] = keep;
            if (t == 0) L.n = n - done;
            __syncthreads();
        }
    }
}

// The same by the tiled FP64 field (lens_tiles.hpp) on the tiles that hold any, where
// there are more (6730^2 x 702, 8.8M pixels: 440 us against 4117 pixel by pixel).
template <int T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mix_dp(
    const double* __restrict__ tab64, const float* __restrict__ tab32, int np, GridDesc g, int ntx, unsigned few,
    const unsigned char* __restrict__ mask, double* __restrict__ ax, double* __restrict__ ay,
    const MixState* __restrict__ st)
{
    __shared__ typename Tile64<T>::Lds lds;
    if (st->status != kStatusOk || st->n_crit <= few) return;
    const int tj = blockIdx.x / ntx, ti = blockIdx.x - tj * ntx;
    const int i = ti * T + (int)(threadIdx.x % T);
    bool any = false;
    for (int j = tj * T + (int)(threadIdx.x / T); j < min(g.ny, tj * T + T); j += 256 / T)
        any = any || (i < g.nx && mask[(size_t)j * g.nx + i] == 2);
    if (!__syncthreads_or(any)) return;
    tile64_body<T>(lds, IsoProfile{tab64, tab32}, np, g, ti * T, tj * T, CriteriaSink{ax, ay, mask, g.nx, g.ny});
}

// Totals and status.
__global__ __launch_bounds__(1024) void k_mix_stats(MixState* __restrict__ st, const uint2* __restrict__ counts,
                                                    int n, long long* __restrict__ stats)
{
    __shared__ unsigned long long s_n[2];
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long nb = 0, nc = 0;
    for (int k = threadIdx.x; k < n; k += 1024) {
        nb += counts[k].x;
        nc += counts[k].y;
    }
    if (nb) atomicAdd(&s_n[0], nb);
    if (nc) atomicAdd(&s_n[1], nc);
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool ok = st->status == kStatusOk;
        stats[0] = ok ? (long long)s_n[0] : 0;
        stats[1] = ok ? (long long)s_n[1] : 0;
        stats[2] = ok ? (long long)(s_n[0] + s_n[1]) : 0;
        stats[3] = st->status;
        st->n_crit = ok ? (unsigned)s_n[1] : 0u;
    }
}

// ---------------------------------------------------------------- launcher

static dim3 scan_grid(const GridDesc& g)
{
    return dim3((unsigned)((g.nx + 255) / 256), (unsigned)((g.ny + kScanRows - 1) / kScanRows));
}

size_t mixed_counts(const GridDesc& g) { return (size_t)scan_grid(g).x * scan_grid(g).y; }

hipError_t launch_mixed(const PotPtrs& pot, const GridDesc& g, const MixedLaunch& ml, hipStream_t s)
{
    const long long n_nodes = (long long)g.nx * g.ny;
    k_mix_prep<<<1, 256, 0, s>>>(pot, g, ml.n_cluster, ml.pc, ml.pg, ml.tab64, ml.tab32, ml.bterm, ml.corner, ml.st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // FP32 field layout: two columns of four rows per thread once there are
    // workgroups enough (6730^2 x 702: 5.93 ms against 6.97 for 1 x 4, 6.35 for 2 x 2,
    // 6.07 for 4 x 4, and 8.12 for the former 4 x 1 with the clamp everywhere), one
    // column below (1200 x 900 x 200: 76 us against 86), single nodes for small images
    // (643 x 569 x 284: 53 us against 76 for 1 x 4; 900 x 1000 x 500 178, 141 for 1 x 4).
    auto field = [&](auto kern, int c, int r) {
        return launch_ev(ml.ev, kern, dim3((unsigned)((g.nx + 256 * c - 1) / (256 * c)), (unsigned)((g.ny + r - 1) / r)),
                         dim3(256), s, (const float*)ml.tab32, pot.n, g.nx, g.ny, ml.ax, ml.ay, ml.mask,
                         (const MixState*)ml.st);
    };
    e = n_nodes >= (4ll << 20)   ? field(k_mix_field32<2, 4>, 2, 4)
        : n_nodes >= (1ll << 19) ? field(k_mix_field32<1, 4>, 1, 4)
                                 : field(k_mix_field32<1, 1>, 1, 1);
    if (e != hipSuccess) return e;
    // blocks: 256 pixels per workgroup, a few workgroups per CU in all at least
    auto per = [&](int n, int size) {
        if (n <= 0 || size <= 0) return 0;
        const long long px = (long long)std::min(size, g.nx) * std::min(size, g.ny);
        return (int)std::min(std::max(1ll, 16384ll / n), (px + 255) / 256);
    };
    const int n0 = ml.n_cluster, n1 = pot.n - n0, per0 = per(n0, ml.pc), per1 = per(n1, ml.pg);
    if (per0 || per1) {
        k_mix_blocks<<<(unsigned)(n0 * per0 + n1 * per1), 256, 0, s>>>(pot.n, g, n0, ml.pc, per0, ml.pg, per1, ml.corner,
                                                                      ml.tab64, ml.ax, ml.ay, ml.mask, ml.st);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const dim3 sg = scan_grid(g);
    k_mix_scan<<<sg, 256, 0, s>>>(ml.ax, ml.ay, g, ml.t12, ml.t34, ml.mask, ml.counts, ml.st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_mix_stats<<<1, 1024, 0, s>>>(ml.st, ml.counts, (int)mixed_counts(g), ml.stats);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // Criteria pixels one by one where that is cheaper (their number is known on the
    // device only, hence both launches, of which one does the work): kPixel cycles per 64
    // of them and halo, against the tiles' cost and kTile cycles per 64 of them for the
    // masked loads and stores (whole calls, us, by tiles / one by one: 3000^2 x 3 with
    // 7.8 M of them 257 / 113, 1500^2 x 15 with 1.9 M 98 / 69, 1200 x 900 x 200 with 4000
    // 258 / 203 and with 0.67 M 270 / 330).  More halos than a tile's lists hold: one by
    // one (2000^2 x 2060 12200 / 7580).
    double cost;
    const int side = tile_side_for((double)n_nodes, (double)n_nodes, pot.n, kTileCost64, &cost);
    constexpr double kPixel = 125.0, kTile = 2500.0;
    const double each = (kPixel * pot.n - kTile) / (64.0 * 1024.0);
    const bool all = pot.n > kTileMaxP || each * (double)n_nodes <= cost;
    const unsigned few = all ? ~0u : (unsigned)(cost / each);
    k_mix_pixels<<<(unsigned)std::min<long long>((n_nodes + kRun - 1) / kRun, 8192), 256, 0, s>>>(
        ml.tab64, pot.n, g, few, ml.mask, ml.ax, ml.ay, ml.st);
    if ((e = hipGetLastError()) != hipSuccess || all) return e;
    auto dp = [&](auto t) {
        constexpr int T = decltype(t)::value;
        const int ntx = (g.nx + T - 1) / T;
        k_mix_dp<T><<<(unsigned)(ntx * ((g.ny + T - 1) / T)), 256, 0, s>>>(ml.tab64, ml.tab32, pot.n, g, ntx, few, ml.mask,
                                                                          ml.ax, ml.ay, ml.st);
        return hipGetLastError();
    };
    return side == 32   ? dp(std::integral_constant<int, 32>())
           : side == 64 ? dp(std::integral_constant<int, 64>())
                        : dp(std::integral_constant<int, 128>());
}

}  // namespace lens
