// Batched image-plane chi^2 on gfx950: n lens models (a sampler's proposals)
// with their own potentials and grids, sharing one set of observed systems,
// evaluated by a fixed number of batch-wide launches:
//   k_bhead   constants of every potential, source positions of every
//             (sample, observed image), FP64
//   k_bsys    one wave per sample: error bound, barycentres, system rows,
//             counters
//   k_bmap    work-item -> sample maps of the field and triangle stages
//   k_btiled  FP32 or FP64 deflection, one workgroup per (sample, tile), heaviest
//             samples first; by a direct sum for the samples that batch_side says
//   k_btri    one workgroup per (sample, 32 tiles of a row), heaviest samples first
//   k_bfbpos  FP64 image positions of every hit (a workgroup per sample) and
//             the FP64 re-test of every undecided FP32 test
//   k_btail   one workgroup per sample: sort, matching, chi^2
// The per-sample work follows exactly the single-evaluation path (same device
// functions, Rexroth et al. 2019, Sec. 2.2.1-2.2.2 and Algorithm 1).
#include "lens_path.hpp"
#include "lens_tiles.hpp"

#include <type_traits>

namespace lens {

static_assert(kBatchMax == kTailStage, "the batch tail stages one sample's hits in LDS");

// ============================================================== head

__global__ __launch_bounds__(256) void k_bhead(BatchPlan bp, PotPtrs pot, ObsPtrs obs, double* __restrict__ tab64,
                                               float* __restrict__ tab32, double* __restrict__ bterm,
                                               double* __restrict__ beta_x, double* __restrict__ beta_y)
{
    const int t = threadIdx.x;
    const int p0 = bp.pot_off[0], np_all = bp.pot_off[bp.n] - p0;
    // constants: potential p (chunk-local index q) uses its sample's grid
    for (int q = blockIdx.x * 256 + t; q < np_all; q += gridDim.x * 256) {
        int lo = 0, hi = bp.n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (bp.pot_off[mid] - p0 <= q) lo = mid; else hi = mid - 1;
        }
        prep_one(pot, bp.grid[lo], p0 + q, q, tab64, tab32, bterm);
    }
    // source positions: one wave per (sample, observed image)
    const long long nwaves = (long long)gridDim.x * 4;
    const long long nitems = (long long)bp.n * obs.n_img;
    for (long long it = (long long)blockIdx.x * 4 + (t >> 6); it < nitems; it += nwaves) {
        const int s = (int)(it / obs.n_img), j = (int)(it % obs.n_img);
        const double t1 = obs.x[j], t2 = obs.y[j];
        double s1 = 0.0, s2 = 0.0;
        for (int p = bp.pot_off[s] + lane_id(); p < bp.pot_off[s + 1]; p += 64) {
            double row[T64_STRIDE], K, a1, a2;
            row64(pot, p, row, K, a1, a2);
            add_alpha64(row, t1, t2, s1, s2);
        }
        const double a1 = wave_sum(s1), a2 = wave_sum(s2);
        const double r = obs.dls[system_of(obs.sys_off, obs.n_sys, j)];
        if (lane_id() == 0) {
            beta_x[it] = src_map(t1, r, a1);
            beta_y[it] = src_map(t2, r, a2);
        }
    }
}

// One wave per sample: fixed-order bound reductions over its potentials, then
// its system rows (as the single-evaluation head), counters and status.
__global__ __launch_bounds__(256) void k_bsys(BatchPlan bp, ObsPtrs obs, const double* __restrict__ bterm,
                                              const double* __restrict__ beta_x, const double* __restrict__ beta_y,
                                              double* __restrict__ sysrow, BatchState bs)
{
    const int s = (int)((blockIdx.x * 256 + threadIdx.x) >> 6);
    if (s >= bp.n) return;
    const int lane = lane_id();
    const int p0 = bp.pot_off[0];
    const int pa = bp.pot_off[s] - p0, pb = bp.pot_off[s + 1] - p0;
    double w = 0.0, jt = 0.0, bad = 0.0;
    for (int q = pa + lane; q < pb; q += 64) {
        w += bterm[3 * q + 0];
        jt += bterm[3 * q + 1];
        bad += bterm[3 * q + 2];
    }
    const double W = wave_sum(w), J = wave_sum(jt), B = wave_sum(bad);
    const double e_alpha = kU32 * (64.0 + (pb - pa)) * W + J + 1e-9;
    const GridDesc g = bp.grid[s];
    const double xlo = g.x0, xhi = g.x0 + (g.nx - 1) * g.h, ylo = g.y0, yhi = g.y0 + (g.ny - 1) * g.h;
    bool ok = B == 0.0 && obs.sys_off[0] == 0 && obs.sys_off[obs.n_sys] == obs.n_img;
    for (int i = lane; i < obs.n_sys; i += 64) {
        const int j0 = obs.sys_off[i], j1 = obs.sys_off[i + 1];
        bool oki = j0 <= j1 && j0 >= 0 && j1 <= obs.n_img;
        double bx = 0.0, by = 0.0;
        if (oki) {
            for (int j = j0; j < j1; j++) {
                bx += beta_x[(size_t)s * obs.n_img + j];
                by += beta_y[(size_t)s * obs.n_img + j];
                oki = oki && obs.sigma[j] > 0.0 && isfinite(obs.sigma[j]) && isfinite(obs.x[j]) &&
                      isfinite(obs.y[j]);
            }
            if (j1 > j0) {
                bx /= (j1 - j0);
                by /= (j1 - j0);
            }
        }
        const double r = obs.dls[i];
        oki = oki && isfinite(r) && r >= 0.0;
        const double bxn = (bx - g.x0) / g.h, byn = (by - g.y0) / g.h;
        oki = oki && fabs(bxn) < 4194304.0 && fabs(byn) < 4194304.0;
        const double theta = fmax(fmax(fabs(xlo - bx), fabs(xhi - bx)), fmax(fabs(ylo - by), fabs(yhi - by)));
        const double eb = r * e_alpha + 4.0 * kU32 * theta + 2.0 * kU32 * r * (W + e_alpha) +
                          g.h * kNodeSplitErr + 1e-9;
        double* row = sysrow + ((size_t)s * obs.n_sys + i) * SYS_STRIDE;
        row[SYS_BX] = bx;
        row[SYS_BY] = by;
        row[SYS_BXH] = rint(bxn);
        row[SYS_BXL] = bxn - rint(bxn);
        row[SYS_BYH] = rint(byn);
        row[SYS_BYL] = byn - rint(byn);
        row[SYS_R] = r;
        row[SYS_EB] = eb * (1.0 + 1e-6);
        ok = ok && oki;
    }
    ok = __ballot(!ok) == 0;
    if (lane == 0) {
        bs.status[s] = ok ? kStatusOk : kStatusInvalid;
        bs.n_hits[s] = 0;
        bs.n_fb[s] = 0;
        if (s == 0) *bs.n_flags = 0;
    }
}

// Work-item -> position-in-plan maps (one workgroup per sample).
__global__ __launch_bounds__(256) void k_bmap(BatchPlan bp, int* __restrict__ fmap, int* __restrict__ tmap)
{
    const int k = blockIdx.x;
    for (long long i = bp.fitem_off[k] + threadIdx.x; i < bp.fitem_off[k + 1]; i += 256) fmap[i] = k;
    for (long long i = bp.titem_off[k] + threadIdx.x; i < bp.titem_off[k + 1]; i += 256) tmap[i] = k;
}

// ============================================================== field

// One workgroup per (sample, tile); the map gives the sample (heaviest samples
// first).  The tiled field of the single evaluation (lens_tiles.hpp) with each
// sample's own tile side, or, where that is 0 (batch_side), the direct sum.
template <int T>
__device__ __forceinline__ void btile(void* lds, const IsoProfile& prof, int np, const GridDesc& g, int tile, float* fx,
                                      float* fy, float* rec)
{
    const int ntx = (g.nx + T - 1) / T, tj = tile / ntx, ti = tile - tj * ntx;
    tile32_body<T>(*reinterpret_cast<typename Tile32<T>::Lds*>(lds), prof, np, g, ti * T, tj * T, fx, fy, false, rec,
                   (g.nx + 31) >> 5);
}
template <int T>
__device__ __forceinline__ void btile(void* lds, const IsoProfile& prof, int np, const GridDesc& g, int tile, double* fx,
                                      double* fy, double* rec)
{
    const int ntx = (g.nx + T - 1) / T, tj = tile / ntx, ti = tile - tj * ntx;
    tile64_body<T>(*reinterpret_cast<typename Tile64<T>::Lds*>(lds), prof, np, g, ti * T, tj * T,
                   FieldSink64{fx, fy, rec, g.nx, g.ny, false});
}

// The direct sum of the single evaluation in two forms.  Few potentials: the field is
// memory traffic, and a wave takes 64 columns x 8 rows with no barrier (bdirect_few).
// Otherwise (bdirect) one workgroup per unit of 64 columns x 8 rows (128 x 4 and 256 x 2
// where the grid has no more rows): lane = column, two rows per wave.  The table rows
// of 64 potentials at a time are staged in LDS: with thousands of potentials on few
// nodes there are too few waves to hide a scalar load from beyond its cache per
// potential.
constexpr int kUnitY = 8;  // rows of a range record

// LDS of a unit; v: range records by 32 columns and wave: range, first row, first column.
template <typename V>
struct DirectLds;
template <>
struct DirectLds<float> {
    float v[2][4][12];
    float4 rows[4][2][64];  // per wave: row parts of field32_pot
    float c[64][T32_STRIDE];
};
template <>
struct DirectLds<double> {
    double v[2][4][12];
    double c[64][10];
};

// Sums of the wave's rows j and j + 1 at column i; all threads call it, a wave whose
// rows lie outside the grid with act = false.
__device__ __forceinline__ void direct_rows(DirectLds<float>& L, const IsoProfile& prof, int np, const GridDesc&, int i,
                                            int j, bool act, float* sx, float* sy)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const float fi = (float)i;
    for (int b = 0; b < np; b += 64) {
        const int cnt = min(64, np - b);
        if (b) __syncthreads();  // the previous 64 potentials have been read
        for (int q = threadIdx.x; q < cnt * T32_STRIDE; q += 256) (&L.c[0][0])[q] = prof.tab32[(size_t)b * T32_STRIDE + q];
        __syncthreads();
        if (!act) continue;
        if (lane < cnt) {
            const float* c = L.c[lane];
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const float nyv = ((float)(j + r) - c[T32_CYH]) - c[T32_CYL];
                L.rows[wave][r][lane] =
                    make_float4(c[T32_BP] * nyv, c[T32_CQ] * nyv, fmaf(c[T32_DQ] * nyv, nyv, c[T32_A2]), c[T32_RSK]);
            }
        }
        wave_lds_sync();
#pragma unroll 2
        for (int k = 0; k < cnt; k++) {
            const float4 rc[2] = {L.rows[wave][0][k], L.rows[wave][1][k]};
            field32_pot<1, 2>(L.c[k], rc, &fi, sx, sy);
        }
    }
}
__device__ __forceinline__ void direct_rows(DirectLds<double>& L, const IsoProfile& prof, int np, const GridDesc& g,
                                            int i, int j, bool act, double* sx, double* sy)
{
    const int lane = lane_id();
    const double t1 = node_coord(g.x0, i, g.h), t2[2] = {node_coord(g.y0, j, g.h), node_coord(g.y0, j + 1, g.h)};
    auto add = [&](int k, auto has) {
        const Far64 c = load_far(L.c[k]);
        const double d1 = t1 - c.xc;
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const double d2 = t2[r] - c.yc;
            IsoProfile::node64<decltype(has)::value>(c, d1, d2, c.B * d2, c.C * d2, sx[r], sy[r]);
        }
    };
    for (int b = 0; b < np; b += 64) {
        const int cnt = min(64, np - b);
        if (b) __syncthreads();
        for (int q = threadIdx.x; q < cnt * 10; q += 256)
            (&L.c[0][0])[q] = prof.tab64[(size_t)(b + q / 10) * T64_STRIDE + q % 10];
        __syncthreads();
        if (!act) continue;
        const unsigned long long cut = __ballot(lane < cnt && __double_as_longlong(L.c[lane][T64_RS]) != 0);
        for (int k = 0; k < cnt;) {  // two of a kind at a time: their chains interleave
            const unsigned kinds = (unsigned)(cut >> k) & 3u;
            const bool two = k + 1 < cnt;
            if (two && kinds == 3u) {
                add(k, std::true_type());
                add(k + 1, std::true_type());
                k += 2;
            } else if (two && kinds == 0u) {
                add(k, std::false_type());
                add(k + 1, std::false_type());
                k += 2;
            } else {
                if (kinds & 1u)
                    add(k, std::true_type());
                else
                    add(k, std::false_type());
                k++;
            }
        }
    }
}

// Minimum over 32 columns of eight values per lane, in lane l the one of index
// l / 16 % 2 + 2 (l / 8 % 2) + 4 (l / 4 % 2): half of the values change lanes at each of
// the first three steps, so that there are 9 exchanges, not 40.
template <typename V>
__device__ __forceinline__ V min32x8(V* v)
{
    const int lane = lane_id();
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        row_swap<16>(v[k], v[k + 1]);
        v[k] = fmin(v[k], v[k + 1]);
    }
    const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
#pragma unroll
    for (int k = 0; k < 8; k += 4) {
        const V other = dpp_mov<0x128>(b3 ? v[k] : v[k + 2]);  // lane ^ 8
        v[k] = fmin(b3 ? v[k + 2] : v[k], other);
    }
    const V other = dpp_mov<0x141>(b2 ? v[0] : v[4]);  // the other half of 8 lanes
    V r = fmin(b2 ? v[4] : v[0], other);
    r = fmin(r, dpp_mov<0xB1>(r));
    return fmin(r, dpp_mov<0x4E>(r));
}

// Range records (write_records) of the unit at row j0 with nr rows, nwx waves to a
// pair of rows: over the wave's rows and 32 columns, then over the waves of the
// columns; the maxima as minima of the negatives.
template <typename V>
__device__ __forceinline__ void unit_records(DirectLds<V>& L, const V* sx, const V* sy, int nr, int i, int j0, int nwx,
                                             int nx, int nbx, V* __restrict__ rec)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6, half = lane >> 5, k0 = lane & 31;
    const int row0 = 2 * (wave / nwx);  // of the unit
    const V inf = V(INFINITY);
    V v[8], c[4];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = inf;
    if (i < nx) {
#pragma unroll
        for (int r = 0; r < 2; r++)
            if (row0 + r < nr) {
                v[0] = fmin(v[0], sx[r]);
                v[1] = fmin(v[1], -sx[r]);
                v[2] = fmin(v[2], sy[r]);
                v[3] = fmin(v[3], -sy[r]);
            }
        if (row0 == 0) {
            v[4] = sx[0];
            v[5] = -sx[0];
            v[6] = sy[0];
            v[7] = -sy[0];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; k++) c[k] = v[k];
    const V m = min32x8(v);
    if ((lane & 3) == 0) L.v[half][wave][((lane >> 4) & 1) + ((lane >> 2) & 2) + (lane & 4)] = m;
    if (k0 == 0)  // the first column's rows
#pragma unroll
        for (int k = 0; k < 4; k++) L.v[half][wave][8 + k] = c[k];
    __syncthreads();
    if (row0 == 0 && i - k0 < nx) {
        V* o = rec + ((size_t)(j0 >> 3) * nbx + (i >> 5)) * kRec;
        if (k0 < 12) {
            V q = L.v[half][wave][k0];
            for (int w = wave + nwx; w < 4; w += nwx) q = fmin(q, L.v[half][w][k0]);
            o[k0] = (k0 & 1) ? -q : q;
        }
        if (k0 == 0) {
            o[12] = sx[0];
            o[13] = sy[0];
        }
    }
}

// Rows R0 .. R0 + 3 of a column of the unit at row j0: potential p's part.
template <int R0>
__device__ __forceinline__ void add_rows(const IsoProfile& prof, int p, const GridDesc&, int i, int j0, float* sx,
                                         float* sy)
{
    const float* c = prof.tab32 + (size_t)p * T32_STRIDE;
    const float fi = (float)i;
    float4 rc[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const float nyv = ((float)(j0 + R0 + r) - c[T32_CYH]) - c[T32_CYL];
        rc[r] = make_float4(c[T32_BP] * nyv, c[T32_CQ] * nyv, fmaf(c[T32_DQ] * nyv, nyv, c[T32_A2]), c[T32_RSK]);
    }
    field32_pot<1, 4>(c, rc, &fi, sx + R0, sy + R0);
}
template <int R0>
__device__ __forceinline__ void add_rows(const IsoProfile& prof, int p, const GridDesc& g, int i, int j0, double* sx,
                                         double* sy)
{
    const Far64 c = load_far(prof.tab64 + (size_t)p * T64_STRIDE);
    const double d1 = node_coord(g.x0, i, g.h) - c.xc;
    auto rows = [&](auto has) {
#pragma unroll
        for (int r = R0; r < R0 + 4; r++) {
            const double d2 = node_coord(g.y0, j0 + r, g.h) - c.yc;
            IsoProfile::node64<decltype(has)::value>(c, d1, d2, c.B * d2, c.C * d2, sx[r], sy[r]);
        }
    };
    if (__double_as_longlong(c.rs) == 0)
        rows(std::false_type());
    else
        rows(std::true_type());
}

constexpr int kFewP = 12;  // potentials below which a wave takes a unit by itself

template <typename V>
__device__ __forceinline__ void bdirect_few(const IsoProfile& prof, int np, const GridDesc& g, int item,
                                            V* __restrict__ fx, V* __restrict__ fy, V* __restrict__ rec)
{
    const int nux = (g.nx + 63) / 64, unit = 4 * item + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int uj = unit / nux, lane = lane_id(), i = (unit - uj * nux) * 64 + lane, j0 = uj * kUnitY;
    if (j0 >= g.ny) return;  // the last workgroup's spare waves
    const int nr = min(kUnitY, g.ny - j0);
    V sx[kUnitY] = {}, sy[kUnitY] = {};
    for (int p = 0; p < np; p++) {
        add_rows<0>(prof, p, g, i, j0, sx, sy);
        if (nr > 4) add_rows<4>(prof, p, g, i, j0, sx, sy);
    }
    // records as unit_records, of one wave
    V v[8], c[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const V* s = k < 2 ? sx : sy;
        c[k] = (k & 1) ? -s[0] : s[0];
        v[4 + k] = i < g.nx ? c[k] : V(INFINITY);
#pragma unroll
        for (int r = 1; r < kUnitY; r++)
            if (r < nr) c[k] = fmin(c[k], (k & 1) ? -s[r] : s[r]);
        v[k] = i < g.nx ? c[k] : V(INFINITY);
    }
    const V m = min32x8(v);
    if ((i & ~31) < g.nx) {
        V* o = rec + ((size_t)uj * ((g.nx + 31) >> 5) + (i >> 5)) * kRec;
        if ((lane & 3) == 0) {
            const int k = ((lane >> 4) & 1) + ((lane >> 2) & 2) + (lane & 4);
            o[k] = (k & 1) ? -m : m;
        }
        if ((lane & 31) == 0) {
#pragma unroll
            for (int k = 0; k < 4; k++) o[8 + k] = (k & 1) ? -c[k] : c[k];
            o[12] = sx[0];
            o[13] = sy[0];
        }
    }
    if (i >= g.nx) return;
#pragma unroll
    for (int r = 0; r < kUnitY; r++)
        if (r < nr) {
            fx[(size_t)(j0 + r) * g.nx + i] = sx[r];
            fy[(size_t)(j0 + r) * g.nx + i] = sy[r];
        }
}

// Waves of a unit along x: the grid's few rows (2, 4) leave them columns.
__host__ __device__ inline int unit_waves_x(const GridDesc& g) { return g.ny <= 2 ? 4 : g.ny <= 4 ? 2 : 1; }

template <typename V>
__device__ __forceinline__ void bdirect(DirectLds<V>& L, const IsoProfile& prof, int np, const GridDesc& g, int unit,
                                        V* __restrict__ fx, V* __restrict__ fy, V* __restrict__ rec)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nwx = unit_waves_x(g);
    const int ux = 64 * nwx, nux = (g.nx + ux - 1) / ux, uj = unit / nux, wy = wave / nwx;
    const int ib = (unit - uj * nux) * ux + 64 * (wave - wy * nwx), i = ib + lane_id();
    const int j0 = uj * kUnitY, j = j0 + 2 * wy;
    V sx[2] = {}, sy[2] = {};
    direct_rows(L, prof, np, g, i, j, j < g.ny && ib < g.nx, sx, sy);
    unit_records(L, sx, sy, min(kUnitY, g.ny - j0), i, j0, nwx, g.nx, (g.nx + 31) >> 5, rec);
    if (i >= g.nx) return;
#pragma unroll
    for (int r = 0; r < 2; r++)
        if (j + r < g.ny) {
            fx[(size_t)(j + r) * g.nx + i] = sx[r];
            fy[(size_t)(j + r) * g.nx + i] = sy[r];
        }
}

template <typename V>
__device__ __forceinline__ void bfield(void* lds, const BatchPlan& bp, const int* __restrict__ fmap,
                                       const double* __restrict__ tab64, const float* __restrict__ tab32,
                                       V* __restrict__ fx, V* __restrict__ fy, V* __restrict__ rec)
{
    const int k = fmap[blockIdx.x];
    const int s = bp.perm[k];
    const GridDesc g = bp.grid[s];
    const int item = (int)(blockIdx.x - bp.fitem_off[k]);
    const int q0 = bp.pot_off[s] - bp.pot_off[0], np = bp.pot_off[s + 1] - bp.pot_off[s];
    const IsoProfile prof{tab64 + (size_t)q0 * T64_STRIDE, tab32 + (size_t)q0 * T32_STRIDE};
    V* ox = fx + bp.node_off[s];
    V* oy = fy + bp.node_off[s];
    V* r = rec + bp.rr_off[s];
    switch (bp.side[s]) {  // uniform over the workgroup
    case 0:
        if (np < kFewP)
            bdirect_few(prof, np, g, item, ox, oy, r);
        else
            bdirect(*static_cast<DirectLds<V>*>(lds), prof, np, g, item, ox, oy, r);
        break;
    case 32: btile<32>(lds, prof, np, g, item, ox, oy, r); break;
    case 64: btile<64>(lds, prof, np, g, item, ox, oy, r); break;
    default: btile<128>(lds, prof, np, g, item, ox, oy, r); break;
    }
}

// (six waves: no accumulation registers; five took 537 us of the 256 chains, six 503)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_btiled32(BatchPlan bp, const int* __restrict__ fmap,
                                                  const double* __restrict__ tab64, const float* __restrict__ tab32,
                                                  float* __restrict__ fx, float* __restrict__ fy,
                                                  float* __restrict__ rec)
{
    __shared__ __align__(16) unsigned char lds[sizeof(Tile32<128>::Lds)];
    static_assert(sizeof lds >= sizeof(DirectLds<float>));
    bfield<float>(lds, bp, fmap, tab64, tab32, fx, fy, rec);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_btiled64(
    BatchPlan bp, const int* __restrict__ fmap, const double* __restrict__ tab64, const float* __restrict__ tab32,
    double* __restrict__ fx, double* __restrict__ fy, double* __restrict__ rec)
{
    __shared__ __align__(16) unsigned char lds[sizeof(Tile64<128>::Lds)];
    static_assert(sizeof lds >= sizeof(DirectLds<double>));
    bfield<double>(lds, bp, fmap, tab64, tab32, fx, fy, rec);
}

// ============================================================== triangles

__device__ __forceinline__ float lane_val(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_val(double v, int l) { return bcast(v, l); }

// A system's cut of cells by their boxes: cell (i, j) of the grid with
// deflections in [lo, hi] holds the barycentre in neither triangle if
//   fma(-r, hi_x, i h) > above[0]  or  fma(-r, lo_x, (i + 1) h) < below[0],
// or the same in y.  The bounds hold the barycentre's offset from the grid's first
// node, E_B, and room for this form's own rounding: 16 u (u = 2^-24 or 2^-53) of
// the grid's and the barycentre's extent, where it is at most 6 u of them, and for
// the deflection's part 4 E_B (E_B holds 2 u r W, the part is below 3 u r W); FP64:
// 1e-9, as for the tiles, and 1e-8 E_B, which holds both (E_B >= 2^-22 of the farthest corner
// and 2^-23 r W).  A negative r is not cut.
template <typename V>
struct CellCut {
    V r, above[2], below[2];
};
template <typename V>
__device__ __forceinline__ CellCut<V> cell_cut(const GridDesc& g, const SysVals& y)
{
    CellCut<V> c;
    V o[2], w[2];
    if constexpr (sizeof(V) == 4) {
        const float h = (float)g.h;
        c.r = y.r32;
        o[0] = (-y.bxh - y.bxl) * h;
        o[1] = (-y.byh - y.byl) * h;
        w[0] = 5.0f * y.e + 1e-6f * (fabsf(o[0]) + (float)g.nx * h);
        w[1] = 5.0f * y.e + 1e-6f * (fabsf(o[1]) + (float)g.ny * h);
    } else {
        c.r = y.r;
        o[0] = g.x0 - y.bx;
        o[1] = g.y0 - y.by;
        w[0] = w[1] = 1e-9 + 1e-8 * (double)y.e;
    }
#pragma unroll
    for (int d = 0; d < 2; d++) {
        c.above[d] = c.r < V(0) ? V(INFINITY) : w[d] - o[d];
        c.below[d] = c.r < V(0) ? V(-INFINITY) : -w[d] - o[d];
    }
    return c;
}

// One workgroup per (sample, tile row, kTriTiles consecutive tile columns) work
// item, heaviest samples first.  Culling: lane l bounds tile l % 32's source-plane
// vertices from the range records and tests two systems' barycentres per ballot
// against that box, the waves taking turns in a chunk of 64 systems; LDS holds one
// word per system, bit t = tile t passes.  Each tile with a passing system is then
// cut into strips of 64 cells, one per lane, the strips dealt to the four waves
// and the next strip's nodes loaded meanwhile.  A cell is first tested by the box
// of its deflections alone (CellCut: 4 FMAs and 4 compares per system); the few
// near cells load their nodes again and take the triangle tests.
// Bound by latency and instruction issue together (54 % of the cycles issue a
// vector instruction, 60 % of the waves' time is spent waiting, for records and
// fields that the field stage left in HBM), hence four waves to a tile, no LDS
// tile, and few registers (6 waves per SIMD).  32 x 8 tiles, one wave per (row, 64
// columns) with the tiles in LDS before: 96 samples 334 -> 192 us, 256 chains of
// 512^2 668 -> 210 us.  Items of 8 and 16 tiles took 297 and 226 us (222, 207),
// of 64 191 us (247): workgroups without a passing tile against balance.
// Hits go to the sample's own list (system << 32 | triangle id), undecided tests
// to the batch list (sample << 44 | system << 31 | triangle id).
static_assert(kTriTiles == 32, "two systems of 32 tiles per ballot, one word per system");
template <class S, typename V>
__global__ __launch_bounds__(256) void k_btri(BatchPlan bp, const int* __restrict__ tmap, int nsys,
                                              const double* __restrict__ sysrow, const V* __restrict__ fx,
                                              const V* __restrict__ fy, const V* __restrict__ rr, BatchState bs,
                                              int mode, double tau, int hcap, unsigned long long* __restrict__ hits,
                                              unsigned long long* __restrict__ flags, long long flag_cap,
                                              unsigned* __restrict__ part)
{
    constexpr int RW = 64 / S::TX;               // cell rows of a strip
    constexpr int NS = S::TX * S::TY / 256;      // strips per wave and tile
    constexpr int SB = 64 / kTriTiles;           // systems per ballot
    __shared__ unsigned long long spass[kTriTiles], sany[4];
    __shared__ unsigned sp[4][2];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = lane_id();
    unsigned npair = 0, nbbox = 0;  // passing (tile, system) pairs (wave-uniform); bbox passes per lane
    const int k = tmap[blockIdx.x];
    const int s = bp.perm[k];
    const GridDesc g = bp.grid[s];
    const int tiles_x = (g.nx - 2) / S::TX + 1;
    const int blocks_x = (tiles_x + kTriTiles - 1) / kTriTiles;
    const int local = (int)(blockIdx.x - bp.titem_off[k]);
    const int band = local / blocks_x, c0 = (local - band * blocks_x) * kTriTiles;
    const double* rows = sysrow + (size_t)s * nsys * SYS_STRIDE;
    const V* sfx = fx + bp.node_off[s];
    const V* sfy = fy + bp.node_off[s];
    const float tau32 = (float)(tau * g.h * g.h);
    const int cj0 = band * S::TY, ncy = min(S::TY, g.ny - 1 - cj0);  // of every tile of the row
    // the lane's cell of the wave's strip n of tile t
    auto cell = [&](int t, int n, int& gi, int& gj) -> bool {
        const int ci0 = (c0 + t) * S::TX, li = lane % S::TX, lj = RW * (wave + 4 * n) + lane / S::TX;
        const bool in = lj < ncy && ci0 + li < g.nx - 1;
        gi = in ? ci0 + li : ci0;
        gj = in ? cj0 + lj : cj0;
        return in;
    };
    const V h = (V)g.h;
    for (int sb = 0; sb < nsys; sb += 64) {
        if (sb) __syncthreads();  // spass is read
        CellCut<V> cut;
        {
            const int sys = min(sb + lane, nsys - 1);
            cut = cell_cut<V>(g, sys_vals<V>(rows + (size_t)sys * SYS_STRIDE));
        }
        // the range and box values are needed here only: an opaque lane keeps the
        // compiler from holding them in registers over the strips below
        int cl = lane;
        asm volatile("" : "+v"(cl));
        const int col = c0 + (cl & (kTriTiles - 1));
        const bool act = col < tiles_x;
        const Tile T = tile_of<S>(g, tiles_x, band * tiles_x + (act ? col : 0));
        double rng[4] = {0.0, 0.0, 0.0, 0.0};
        if (act) tile_range_rec<S, V>(rr + bp.rr_off[s], (g.nx + 31) >> 5, (g.ny + 7) >> 3, T, rng);
        unsigned long long any = 0;
        for (int c = wave; c < kTriTiles && sb + c * SB < nsys; c += 4) {
            const int sys = sb + c * SB + cl / kTriTiles;
            bool in = false;
            if (act && sys < nsys) {
                const double* row = rows + (size_t)sys * SYS_STRIDE;
                in = tile_box_contains(g, T, rng, row[SYS_R], sizeof(V) == 4 ? row[SYS_EB] : 1e-9, row[SYS_BX],
                                       row[SYS_BY]);
            }
            const unsigned long long m = __ballot(in);
            npair += (unsigned)__popcll(m);
            any |= m;
            if (lane == 0) spass[c] = m;
        }
        if (lane == 0) sany[wave] = any;
        __syncthreads();
        const unsigned long long all = sany[0] | sany[1] | sany[2] | sany[3];
        // tiles that a system passes
        unsigned tiles = (unsigned)__builtin_amdgcn_readfirstlane((int)(all | (all >> 32)));
        if (tiles == 0) continue;
        // bit t: tile t passes system sb + lane
        const unsigned mine = sb + lane < nsys ? ((const unsigned*)spass)[lane] : 0;
        int t = __ffs((int)tiles) - 1, n = 0, gi, gj;
        bool in = cell(t, n, gi, gj);
        V a[8];
        load_cell(sfx, sfy, g, gi, gj, a);
        while (tiles) {
            const int tc = t, ci = gi, cj = gj;
            const bool cin = in;
            const V lx = fmin(fmin(a[0], a[1]), fmin(a[2], a[3])), hx = fmax(fmax(a[0], a[1]), fmax(a[2], a[3]));
            const V ly = fmin(fmin(a[4], a[5]), fmin(a[6], a[7])), hy = fmax(fmax(a[4], a[5]), fmax(a[6], a[7]));
            if (++n == NS) {
                n = 0;
                tiles &= tiles - 1;
                t = tiles ? __ffs((int)tiles) - 1 : t;
            }
            if (tiles) {
                in = cell(t, n, gi, gj);
                load_cell(sfx, sfy, g, gi, gj, a);
            }
            if (__ballot(cin) == 0) continue;  // outside the grid
            const V x0 = (V)ci * h, x1 = (V)(ci + 1) * h, y0 = (V)cj * h, y1 = (V)(cj + 1) * h;
            unsigned long long m = __ballot(((mine >> tc) & 1) != 0);
            while (m) {
                const int l = __ffsll((long long)m) - 1;
                m &= m - 1;
                const V r = lane_val(cut.r, l);
                const bool near = cin && !(fma(-r, hx, x0) > lane_val(cut.above[0], l)) &&
                                  !(fma(-r, lx, x1) < lane_val(cut.below[0], l)) &&
                                  !(fma(-r, hy, y0) > lane_val(cut.above[1], l)) &&
                                  !(fma(-r, ly, y1) < lane_val(cut.below[1], l));
                if (__ballot(near) == 0) continue;
                // few cells come here: their nodes (in the caches) and the system's row again
                // rather than in registers all along
                V av[8];
                load_cell(sfx, sfy, g, ci, cj, av);
                const SysVals y = sys_vals<V>(rows + (size_t)(sb + l) * SYS_STRIDE);
                const unsigned bits = near ? test_cell(g, ci, cj, av, y, mode, tau32, nbbox) : 0u;
                if (__ballot(bits != 0) == 0) continue;  // the common case: no hit, nothing undecided
                const unsigned long long sys = (unsigned)(sb + l);
                const unsigned tid0 = (unsigned)(2 * (cj * (g.nx - 1) + ci));
                const unsigned long long hb = sys << 32, fb = ((unsigned long long)s << 44) | (sys << 31);
                wave_append((bits & 3u) == kHit, hb | tid0, &bs.n_hits[s], hits + (size_t)s * hcap, hcap);
                wave_append((bits >> 2) == kHit, hb | (tid0 + 1), &bs.n_hits[s], hits + (size_t)s * hcap, hcap);
                wave_append((bits & 3u) == kFlag, fb | tid0, bs.n_flags, flags, flag_cap);
                wave_append((bits >> 2) == kFlag, fb | (tid0 + 1), bs.n_flags, flags, flag_cap);
            }
        }
    }
    write_part_sum(part, blockIdx.x, npair, nbbox, sp);
}

// ============================================================== positions and fallback

// Workgroups [0, kBfbSub n): the FP64 position of every certain hit, one wave
// per hit, kBfbSub workgroups per sample.  The kBfbFlagBlocks workgroups
// beyond: persistent waves over the batch's undecided tests, each decided
// exactly on FP64 vertices and, if a hit, appended with its position to its
// sample's fallback list.  Each item is a chain of dependent steps (the three
// vertices over the potentials, the wave reductions, the position), so the
// launch spreads the items over many waves.
constexpr int kBfbSub = 4;
constexpr int kBfbFlagBlocks = 2048;
__global__ __launch_bounds__(256) void k_bfbpos(BatchPlan bp, int nsys, const double* __restrict__ tab64,
                                                const double* __restrict__ sysrow, BatchState bs, int hcap,
                                                const unsigned long long* __restrict__ hits,
                                                const unsigned long long* __restrict__ flags, long long flag_cap,
                                                unsigned long long* __restrict__ fb, double* __restrict__ pos,
                                                double* __restrict__ fb_pos)
{
    const int p0 = bp.pot_off[0];
    const int wave = threadIdx.x >> 6;
    if ((int)blockIdx.x < bp.n * kBfbSub) {
        const int s = blockIdx.x / kBfbSub, sub = blockIdx.x - s * kBfbSub;
        if (bs.status[s] != kStatusOk) return;
        const int nh = (int)min((unsigned long long)hcap, bs.n_hits[s]);
        const GridDesc g = bp.grid[s];
        const double* tab = tab64 + (size_t)(bp.pot_off[s] - p0) * T64_STRIDE;
        const int np = bp.pot_off[s + 1] - bp.pot_off[s];
        for (int q = sub * 4 + wave; q < nh; q += 4 * kBfbSub) {
            const unsigned long long key = hits[(size_t)s * hcap + q];
            const int sys = (int)(key >> 32), tid = (int)(key & 0xffffffffu);
            const double* row = sysrow + ((size_t)s * nsys + sys) * SYS_STRIDE;
            double vx[3], vy[3], tx[3], ty[3];
            vertices64(tab, np, g, tid, row[SYS_R], vx, vy, tx, ty);
            if (lane_id() == 0)
                image_position(vx, vy, tx, ty, row[SYS_BX], row[SYS_BY], pos[2 * ((size_t)s * hcap + q)],
                               pos[2 * ((size_t)s * hcap + q) + 1]);
        }
        return;
    }
    const long long nwaves = (long long)(gridDim.x - bp.n * kBfbSub) * 4;
    const long long w0 = (long long)(blockIdx.x - bp.n * kBfbSub) * 4 + wave;
    const long long nf = (long long)min((unsigned long long)flag_cap, *bs.n_flags);
    for (long long it = w0; it < nf; it += nwaves) {
        const unsigned long long key = flags[it];
        const int s = (int)(key >> 44), sys = (int)((key >> 31) & 0x1fff), tid = (int)(key & 0x7fffffffu);
        if (bs.status[s] != kStatusOk) continue;
        const GridDesc g = bp.grid[s];
        const double* tab = tab64 + (size_t)(bp.pot_off[s] - p0) * T64_STRIDE;
        const int np = bp.pot_off[s + 1] - bp.pot_off[s];
        const double* row = sysrow + ((size_t)s * nsys + sys) * SYS_STRIDE;
        double vx[3], vy[3], tx[3], ty[3];
        vertices64(tab, np, g, tid, row[SYS_R], vx, vy, tx, ty);
        if (lane_id() == 0 && contains_exact(vx, vy, row[SYS_BX], row[SYS_BY])) {
            const unsigned long long slot = atomicAdd(&bs.n_fb[s], 1ull);
            if ((long long)slot < hcap) {
                const size_t o = (size_t)s * hcap + slot;
                fb[o] = ((unsigned long long)sys << 32) | (unsigned)tid;
                image_position(vx, vy, tx, ty, row[SYS_BX], row[SYS_BY], fb_pos[2 * o], fb_pos[2 * o + 1]);
            }
        }
    }
}

// ============================================================== tail

// One workgroup of 256 threads per sample: merge the sample's certain and
// fallback hits, rank-sort them by (system, triangle id), pair each observed
// image with the nearest predicted image of its system (ties to the lower
// triangle id), chi2_i in image order (+inf without a predicted image) and
// chi^2 in a fixed order (Sec. 2.2.1).  Needs hcap <= 1024 and at most 1024
// images and systems (checked on the host).
__global__ __launch_bounds__(256) void k_btail(ObsPtrs obs, BatchState bs, int hcap,
                                               long long flag_cap, const unsigned long long* __restrict__ hits,
                                               const unsigned long long* __restrict__ fb,
                                               const double* __restrict__ pos, const double* __restrict__ fb_pos,
                                               double* __restrict__ chi2, double* __restrict__ chi2_sys,
                                               int* __restrict__ n_pred, int* __restrict__ status,
                                               unsigned long long* __restrict__ agg,
                                               const unsigned* __restrict__ part, long long n_parts,
                                               int* __restrict__ out_nh, int* __restrict__ out_hits,
                                               double* __restrict__ out_xy)
{
    constexpr int NT = 256, CAP = 2 * kTailStage;
    {  // chunk statistics (tile passes, bbox passes), one slice of the tiles per workgroup
        const long long per = (n_parts + gridDim.x - 1) / gridDim.x;
        const long long q0 = (long long)blockIdx.x * per, q1 = min(n_parts, q0 + per);
        unsigned long long a = 0, b = 0;
        for (long long q = q0 + threadIdx.x; q < q1; q += NT) {
            a += part[2 * q];
            b += part[2 * q + 1];
        }
        for (int m = 32; m >= 1; m >>= 1) {
            a += __shfl_xor(a, m, 64);
            b += __shfl_xor(b, m, 64);
        }
        if (lane_id() == 0 && (a | b) != 0) {
            atomicAdd(&agg[4], a);
            atomicAdd(&agg[5], b);
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&agg[3], *bs.n_flags);  // undecided tests
    }
    __shared__ unsigned long long key[CAP];
    __shared__ double upx[CAP], upy[CAP];
    __shared__ double scon[kTailStage];
    __shared__ int sfirst[kTailStage], send[kTailStage];
    const int t = threadIdx.x, s = blockIdx.x;
    const int nimg = obs.n_img, nsys = obs.n_sys;
    const unsigned long long nc = bs.n_hits[s], nfb = bs.n_fb[s];
    int st = bs.status[s];
    const bool over = nc > (unsigned long long)hcap || nfb > (unsigned long long)hcap ||
                      *bs.n_flags > (unsigned long long)flag_cap;
    if (st == kStatusOk && over) st = kStatusCapacity;
    double* cs_out = chi2_sys + (size_t)s * nsys;
    int* np_out = n_pred + (size_t)s * nsys;
    if (t == 0) {
        status[s] = st;
        atomicAdd(&agg[0], nc + nfb);
        atomicAdd(&agg[1], nfb);
        if (st != kStatusOk) atomicAdd(&agg[2], 1ull);
    }
    if (st != kStatusOk) {
        for (int i = t; i < nsys; i += NT) {
            cs_out[i] = __builtin_nan("");
            np_out[i] = 0;
        }
        if (t == 0) {
            chi2[s] = __builtin_nan("");
            if (out_nh) out_nh[s] = 0;
        }
        return;
    }
    const int n = (int)(nc + nfb), ncert = (int)nc;
    for (int q = t; q < n; q += NT) {
        const bool c = q < ncert;
        const size_t o = (size_t)s * hcap + (c ? q : q - ncert);
        const unsigned long long h = c ? hits[o] : fb[o];
        key[q] = ((h >> 32) << 44) | ((h & 0x7fffffffull) << 12) | (unsigned long long)q;
        upx[q] = c ? pos[2 * o] : fb_pos[2 * o];
        upy[q] = c ? pos[2 * o + 1] : fb_pos[2 * o + 1];
    }
    for (int i = t; i < nsys; i += NT) {
        sfirst[i] = 0;
        send[i] = 0;
    }
    __syncthreads();
    {
        constexpr int PER = CAP / NT;
        unsigned long long mine[PER];
        int rank[PER];
#pragma unroll
        for (int u = 0; u < PER; u++) {
            const int q = t + NT * u;
            rank[u] = 0;
            mine[u] = q < n ? key[q] : 0;
            if (q < n)
                for (int r = 0; r < n; r++) rank[u] += key[r] < mine[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; u++)
            if (t + NT * u < n) key[rank[u]] = mine[u];
        __syncthreads();
    }
    for (int q = t; q < n; q += NT) {
        const int sy = (int)(key[q] >> 44);
        if (q == 0 || (int)(key[q - 1] >> 44) != sy) sfirst[sy] = q;
        if (q == n - 1 || (int)(key[q + 1] >> 44) != sy) send[sy] = q + 1;
        if (out_hits) {  // the sorted hits and their positions, as the single evaluation writes them
            const size_t o = (size_t)s * hcap + q;
            const int idx = (int)(key[q] & 0xfff);
            out_hits[2 * o] = sy;
            out_hits[2 * o + 1] = (int)((key[q] >> 12) & 0x7fffffffull);
            out_xy[2 * o] = upx[idx];
            out_xy[2 * o + 1] = upy[idx];
        }
    }
    if (out_nh && t == 0) out_nh[s] = n;
    __syncthreads();
    for (int j = t; j < nimg; j += NT) {
        const int i = system_of(obs.sys_off, nsys, j);
        int best = -1;
        double bd = 0.0;
        const double ox = obs.x[j], oy = obs.y[j];
        for (int q = sfirst[i]; q < send[i]; q++) {
            const int idx = (int)(key[q] & 0xfff);
            const double dx = ox - upx[idx], dy = oy - upy[idx];
            const double d2 = dx * dx + dy * dy;
            if (best < 0 || d2 < bd) {
                best = q;
                bd = d2;
            }
        }
        const double sg = obs.sigma[j];
        scon[j] = best >= 0 ? bd / (sg * sg) : 0.0;
    }
    __syncthreads();
    for (int i = t; i < nsys; i += NT) {
        double c = 0.0;
        for (int j = obs.sys_off[i]; j < obs.sys_off[i + 1]; j++) c += scon[j];
        c = send[i] > sfirst[i] ? c : INFINITY;
        cs_out[i] = c;
        np_out[i] = send[i] - sfirst[i];
        upx[i] = c;
    }
    __syncthreads();
    if (t < 64) {
        double v = 0.0;
        for (int i = t; i < nsys; i += 64) v += upx[i];
        v = wave_sum(v);
        if (t == 0) chi2[s] = v;
    }
}

// ============================================================== launchers

static inline unsigned bcdiv(long long a, long long b) { return (unsigned)((a + b - 1) / b); }

hipError_t launch_bhead(const BatchPlan& bp, const PotPtrs& pot, const ObsPtrs& obs, double* tab64, float* tab32,
                        double* bterm, double* bx, double* by, int np_chunk, hipStream_t s)
{
    long long nb = bcdiv((long long)bp.n * obs.n_img, 4);
    const long long nb2 = bcdiv(np_chunk, 256);
    if (nb < nb2) nb = nb2;
    if (nb < 1) nb = 1;
    if (nb > 4096) nb = 4096;
    k_bhead<<<(unsigned)nb, 256, 0, s>>>(bp, pot, obs, tab64, tab32, bterm, bx, by);
    return hipGetLastError();
}

hipError_t launch_bsys(const BatchPlan& bp, const ObsPtrs& obs, const double* bterm, const double* bx,
                       const double* by, double* sysrow, const BatchState& bs, hipStream_t s)
{
    k_bsys<<<bcdiv(bp.n, 4), 256, 0, s>>>(bp, obs, bterm, bx, by, sysrow, bs);
    return hipGetLastError();
}

hipError_t launch_bmap(const BatchPlan& bp, int* fmap, int* tmap, hipStream_t s)
{
    k_bmap<<<bp.n, 256, 0, s>>>(bp, fmap, tmap);
    return hipGetLastError();
}

// Tile side of a sample's field in a launch of `total` nodes, 0 for the direct sum:
// where a single evaluation would never be tiled, whatever its size (tiled_side).
// Whole calls with such samples tiled (all their potentials near) / by the direct sum:
// FP64 64 of 512^2 x 3 283 / 169 us, 8 of 120^2 x 2100 1422 / 655 (mixed 1006 / 398),
// 2 of 100000 x 2 x 100 312 / 106.
int batch_side(const GridDesc& g, int np, double total, bool fp32)
{
    if (np < (fp32 ? 4 : kTileMinP64) || np > kTileMaxP) return 0;
    const int side = tile_side_for((double)g.nx * g.ny, total, np, fp32 ? kTileCost32 : kTileCost64);
    return tiles_too_thin(g, side, fp32 ? kThinNodes32 : kThinNodes64) ? 0 : side;
}

// Work items of a sample's field (workgroups).
long long batch_items(const GridDesc& g, int side, int np)
{
    if (side) return (long long)((g.nx + side - 1) / side) * ((g.ny + side - 1) / side);
    const int ux = np < kFewP ? 64 : 64 * unit_waves_x(g);
    const long long units = (long long)((g.nx + ux - 1) / ux) * ((g.ny + kUnitY - 1) / kUnitY);
    return np < kFewP ? (units + 3) / 4 : units;
}

hipError_t launch_bfield(bool fp32, const BatchPlan& bp, const int* fmap, long long n_items, const double* tab64,
                         const float* tab32, void* fx, void* fy, void* rec, const KernelEvents* ev, hipStream_t s)
{
    const dim3 grid((unsigned)n_items), block(256);
    if (fp32) return launch_ev(ev, k_btiled32, grid, block, s, bp, fmap, tab64, tab32, (float*)fx, (float*)fy, (float*)rec);
    return launch_ev(ev, k_btiled64, grid, block, s, bp, fmap, tab64, tab32, (double*)fx, (double*)fy, (double*)rec);
}

template <class F>
static hipError_t with_bshape(int shape, F f)
{
    switch (shape) {
    case 2: return f(TileShape<64, 16>());
    case 3: return f(TileShape<64, 8>());
    case 4: return f(TileShape<32, 16>());
    default: return f(TileShape<32, 8>());
    }
}

hipError_t launch_btri(const BatchPlan& bp, const int* tmap, long long n_items, int nsys, const double* sysrow,
                       const void* fx, const void* fy, const void* rr, bool fp32, const BatchState& bs, int mode,
                       double tau, int hcap, unsigned long long* hits, unsigned long long* flags, long long flag_cap,
                       unsigned* part, int shape, hipStream_t s)
{
    const unsigned nb = (unsigned)n_items;
    return with_bshape(shape, [&](auto sh) {
        using S = decltype(sh);
        if (fp32)
            k_btri<S, float><<<nb, 256, 0, s>>>(bp, tmap, nsys, sysrow, (const float*)fx, (const float*)fy,
                                                (const float*)rr, bs, mode, tau, hcap, hits, flags, flag_cap, part);
        else
            k_btri<S, double><<<nb, 256, 0, s>>>(bp, tmap, nsys, sysrow, (const double*)fx,
                                                 (const double*)fy, (const double*)rr, bs, mode, tau, hcap, hits,
                                                 flags, flag_cap, part);
        return hipGetLastError();
    });
}

hipError_t launch_bfbpos(const BatchPlan& bp, int nsys, const double* tab64, const double* sysrow,
                         const BatchState& bs, int hcap, const unsigned long long* hits,
                         const unsigned long long* flags, long long flag_cap, unsigned long long* fb, double* pos,
                         double* fb_pos, hipStream_t s)
{
    k_bfbpos<<<bp.n * kBfbSub + kBfbFlagBlocks, 256, 0, s>>>(bp, nsys, tab64, sysrow, bs, hcap, hits, flags,
                                                             flag_cap, fb, pos, fb_pos);
    return hipGetLastError();
}

hipError_t launch_btail(const BatchPlan& bp, const ObsPtrs& obs, const BatchState& bs, int hcap, long long flag_cap,
                        const unsigned long long* hits, const unsigned long long* fb, const double* pos,
                        const double* fb_pos, double* chi2, double* chi2_sys, int* n_pred, int* status,
                        unsigned long long* agg, const unsigned* part, long long n_parts, int* out_nh,
                        int* out_hits, double* out_xy, hipStream_t s)
{
    k_btail<<<bp.n, 256, 0, s>>>(obs, bs, hcap, flag_cap, hits, fb, pos, fb_pos, chi2, chi2_sys, n_pred, status,
                                 agg, part, n_parts, out_nh, out_hits, out_xy);
    return hipGetLastError();
}

__global__ void k_zero_u64(unsigned long long* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ void k_bstats(const unsigned long long* agg, long long n_tests, long long* stats)
{
    if (threadIdx.x == 0) {
        stats[0] = (long long)agg[0];  // hits
        stats[1] = (long long)agg[3];  // undecided FP32 tests
        stats[2] = (long long)agg[4];  // (tile, system) pairs
        stats[3] = (long long)agg[5];  // bounding-box passes
        stats[4] = agg[2] ? 1 : 0;     // any sample not OK
        stats[5] = (long long)agg[1];  // fallback hits
        stats[6] = n_tests;
        stats[7] = (long long)agg[2];  // samples not OK
    }
}

hipError_t launch_bstats(const unsigned long long* agg, long long n_tests, long long* stats, hipStream_t s)
{
    k_bstats<<<1, 64, 0, s>>>(agg, n_tests, stats);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, int n, hipStream_t s)
{
    k_zero_u64<<<bcdiv(n, 256), 256, 0, s>>>(p, n);
    return hipGetLastError();
}

}  // namespace lens
