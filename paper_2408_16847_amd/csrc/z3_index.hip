// Sky-cell index: latitude bands x longitude cells, points sorted by cell.
//
// The paper finds the neighbours of each pivot with an octree (cBalls, "log N steps"
// per pivot).  On the GPU the catalogue is instead bucketed once into a regular grid:
// band k holds colatitudes [k H, (k+1) H), and inside band k the points are split into
// ncell_k equal longitude cells (one cell per point of the band on average).  Points are
// stored in cell order, so any longitude window of a band is a contiguous index range
// (two ranges when it wraps through phi = 0), which the multipole kernel streams with
// coalesced loads.  The order inside a cell is the original catalogue order, which makes
// the index and every later sum deterministic.
#include <algorithm>
#include <cmath>
#include <new>

#include "z3_internal.h"

#ifndef Z3_BAND_HEIGHT_FACTOR
#define Z3_BAND_HEIGHT_FACTOR 1.4
#endif

namespace z3 {

// ---- small device helpers ------------------------------------------------------------

__device__ __forceinline__ void atomic_min_pos_double(double *addr, double v)
{
    // non-negative doubles order like their bit patterns
    atomicMin(reinterpret_cast<unsigned long long *>(addr), (unsigned long long)__double_as_longlong(v));
}

__device__ __forceinline__ void atomic_max_pos_double(double *addr, double v)
{
    atomicMax(reinterpret_cast<unsigned long long *>(addr), (unsigned long long)__double_as_longlong(v));
}

__device__ __forceinline__ double colatitude(double x, double y, double z)
{
    return atan2(sqrt(x * x + y * y), z);
}

__device__ __forceinline__ double longitude(double x, double y)
{
    double phi = atan2(y, x);
    if (phi < 0.0) phi += kTwoPi;
    return phi;
}

// ---- kernels ---------------------------------------------------------------------------

// Colatitude range of the positions and their largest deviation | |r|^2 - 1 | from unit
// length (non-finite -> +inf), and which 64ths of the longitude circle hold points (a bit each),
// one pass over the coordinates: a grid-stride extremum per thread, a block reduction, one
// atomic per block and quantity.
__global__ __launch_bounds__(256) void k_sky_range(const double *xyz, int64_t n, double *range /* [3], sectors */)
{
    __shared__ double smin[256], smax[256], sdev[256];
    __shared__ unsigned long long ssec;
    double lo = 4.0, hi = 0.0, dev = 0.0;
    unsigned long long sec = 0;
    if (threadIdx.x == 0) ssec = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
        const double th = colatitude(x, y, z);
        lo = fmin(lo, th);
        hi = fmax(hi, th);
        double d = fabs((x * x + y * y + z * z) - 1.0);
        if (!(d <= 1e300)) d = INFINITY;
        dev = fmax(dev, d);
        sec |= 1ull << (min(max((int)(longitude(x, y) * (64.0 / kTwoPi)), 0), 63));
    }
    smin[threadIdx.x] = lo;
    smax[threadIdx.x] = hi;
    sdev[threadIdx.x] = dev;
    __syncthreads();
    atomicOr(&ssec, sec);
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + o]);
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + o]);
            sdev[threadIdx.x] = fmax(sdev[threadIdx.x], sdev[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomic_min_pos_double(&range[0], smin[0]);
        atomic_max_pos_double(&range[1], smax[0]);
        if (sdev[0] > 0.0) atomic_max_pos_double(&range[2], sdev[0]);
        atomicOr(reinterpret_cast<unsigned long long *>(range + 3), ssec);
    }
}

// Start of a build: the edge table (by value, so that it needs no copy from the host) and the
// empty range of k_sky_range.
__global__ void k_index_begin(EdgeTab e, EdgeTab *edges, double *range)
{
    const double *src = reinterpret_cast<const double *>(&e);
    double *dst = reinterpret_cast<double *>(edges);
    for (int i = threadIdx.x; i < (int)(sizeof(EdgeTab) / sizeof(double)); i += blockDim.x) dst[i] = src[i];
    if (threadIdx.x == 0) { range[0] = kPi; range[1] = 0.0; range[2] = 0.0; range[3] = 0.0; }
}

// No points in any band or cell; the bands' colatitude ranges start empty, [lo0, 0].
__global__ void k_clear_counts(int *band_count, double *band_th, int nbands, double lo0, int *cell_count, int64_t cells)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cells || i < nbands;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i < cells) cell_count[i] = 0;
        if (i < nbands) {
            band_count[i] = 0;
            band_th[2 * i] = lo0;
            band_th[2 * i + 1] = 0.0;
        }
    }
}

// Adds one point per valid lane to its band's count and colatitude range, in LDS or in memory.
// Points in a map's order share a band with most of their wave, which then sends one update for
// them all; a catalogue in no spatial order has up to 64 bands in a wave, and beyond a small
// group each lane sends its own.  The range's atomics are left out where the range read already
// covers the point (a stale read only sends an atomic too many).
__device__ __forceinline__ void add_to_bands(bool valid, int k, double th, double lo0, int *count, double *th_lo,
                                             double *th_hi, int stride)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t todo = __ballot(valid);
    while (todo) {
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const int kl = __shfl(k, leader, kWave);
        const bool mine = (todo >> lane & 1) && k == kl;
        const uint64_t grp = __ballot(mine);
        if (__popcll(grp) < 16) break;
        double lo = mine ? th : lo0, hi = mine ? th : 0.0;
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o, kWave));
            hi = fmax(hi, __shfl_xor(hi, o, kWave));
        }
        if (lane == leader) {
            atomicAdd(&count[kl], (int)__popcll(grp));
            atomic_min_pos_double(&th_lo[(int64_t)kl * stride], lo);
            atomic_max_pos_double(&th_hi[(int64_t)kl * stride], hi);
        }
        todo &= ~grp;
    }
    if (todo >> lane & 1) {
        atomicAdd(&count[k], 1);
        const volatile double *lo = th_lo + (int64_t)k * stride, *hi = th_hi + (int64_t)k * stride;
        if (!(*lo <= th)) atomic_min_pos_double(&th_lo[(int64_t)k * stride], th);
        if (!(*hi >= th)) atomic_max_pos_double(&th_hi[(int64_t)k * stride], th);
    }
}

// A point's band and longitude, on the sky or on a plane (strip of y, cell coordinate of x).
struct BandRule {
    double inv_h, x0, y0, sx, lo0;  // plane: origin and scale; lo0: an empty band's lower bound
    int nbands;
};

template <bool PLANE>
__device__ __forceinline__ int band_of(const double *xyz, int64_t n, int64_t i, const BandRule &r, double &th, double &phi)
{
    const double x = xyz[i], y = xyz[n + i];
    if constexpr (PLANE) {
        th = y - r.y0;  // >= 0: y0 is the smallest y
        phi = (x - r.x0) * r.sx;
    } else {
        th = colatitude(x, y, xyz[2 * n + i]);
        phi = longitude(x, y);
    }
    const int k = (int)(th * r.inv_h);
    return k < 0 ? 0 : (k >= r.nbands ? r.nbands - 1 : k);
}

// Band of every point, with per-band counts and colatitude ranges.
template <bool PLANE>
__global__ void k_band_of_point(const double *xyz, int64_t n, BandRule r, int *band, double *phi_out, int *band_count,
                                double *band_th /* [nbands][2] */)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;
    int k = -1;
    double th = 0.0;
    if (valid) {
        double phi;
        band[i] = k = band_of<PLANE>(xyz, n, i, r, th, phi);
        phi_out[i] = phi;
    }
    add_to_bands(valid, k, th, r.lo0, band_count, band_th, band_th + 1, 2);
}

// The same for up to kLdsBands bands: a block of 1024 threads takes a contiguous run of `run`
// points, counts in LDS and sends its totals once.  Points in random order otherwise update a
// few hundred addresses from every lane (150,000 points of a cap: 355 us with one wave-wide
// reduction per band of a wave, 201 us with an atomic per lane).
constexpr int kLdsBands = 2048;
constexpr int kLdsBandThreads = 1024;

template <bool PLANE>
__global__ __launch_bounds__(kLdsBandThreads) void k_band_of_point_lds(const double *xyz, int64_t n, int64_t run, BandRule r,
                                                                       int *band, double *phi_out, int *band_count,
                                                                       double *band_th)
{
    __shared__ int count[kLdsBands];
    __shared__ double lo[kLdsBands], hi[kLdsBands];
    for (int k = threadIdx.x; k < r.nbands; k += kLdsBandThreads) {
        count[k] = 0;
        lo[k] = r.lo0;
        hi[k] = 0.0;
    }
    __syncthreads();
    const int64_t beg = (int64_t)blockIdx.x * run, end = min(n, beg + run);
    for (int64_t i0 = beg; i0 < end; i0 += kLdsBandThreads) {
        const int64_t i = i0 + threadIdx.x;
        const bool valid = i < end;
        int k = -1;
        double th = 0.0;
        if (valid) {
            double phi;
            band[i] = k = band_of<PLANE>(xyz, n, i, r, th, phi);
            phi_out[i] = phi;
        }
        add_to_bands(valid, k, th, r.lo0, count, lo, hi, 1);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < r.nbands; k += kLdsBandThreads)
        if (count[k]) {
            atomicAdd(&band_count[k], count[k]);
            atomic_min_pos_double(&band_th[2 * k], lo[k]);
            atomic_max_pos_double(&band_th[2 * k + 1], hi[k]);
        }
}

template <bool PLANE>
static z3_status launch_band_of_point(const double *xyz, int64_t n, const BandRule &r, int *band, double *phi, int *count,
                                      double *th, hipStream_t s)
{
    if (n <= 0) return Z3_OK;
    if (r.nbands <= kLdsBands) {
        const int64_t blocks = std::min<int64_t>((n + kLdsBandThreads - 1) / kLdsBandThreads, 512);
        const int64_t run = ((n + blocks - 1) / blocks + kLdsBandThreads - 1) / kLdsBandThreads * kLdsBandThreads;
        hipLaunchKernelGGL(k_band_of_point_lds<PLANE>, dim3((unsigned)((n + run - 1) / run)), dim3(kLdsBandThreads), 0, s, xyz,
                           n, run, r, band, phi, count, th);
    } else {
        hipLaunchKernelGGL(k_band_of_point<PLANE>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, xyz, n, r, band, phi,
                           count, th);
    }
    return check_launch("k_band_of_point");
}

// The band table from the counts and colatitude ranges, and [2]: number of cells, largest
// count.  One block walks the bands 1024 at a time with running offsets.  At most 4 (2^29 - 1)
// + 2^26 cells: their number is exact in 32 unsigned bits, also where it is too large for the table.
constexpr int kTableThreads = 1024;
__global__ __launch_bounds__(kTableThreads) void k_band_table(int nbands, double h, const int *count, const double *band_th,
                                                             Band *bands, uint32_t *stats)
{
    __shared__ int wpts[kTableThreads / kWave], wmax[kTableThreads / kWave];
    __shared__ uint32_t wcells[kTableThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int pt0 = 0, most = 0;  // of the bands before this round
    uint32_t cell0 = 0;
    for (int k0 = 0; k0 < nbands; k0 += kTableThreads) {
        const int k = k0 + (int)threadIdx.x;
        const int npts = k < nbands ? count[k] : 0;
        const int ncell = k < nbands ? max(1, kCellsPerPoint * npts) : 0;
        int p = npts, mx = npts;
        uint32_t c = (uint32_t)ncell;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int tp = __shfl_up(p, o, kWave);
            const uint32_t tc = __shfl_up(c, o, kWave);
            if (lane >= o) { p += tp; c += tc; }
            mx = max(mx, __shfl_xor(mx, o, kWave));
        }
        __syncthreads();  // the previous round's wave sums are read
        if (lane == kWave - 1) { wpts[wave] = p; wcells[wave] = c; wmax[wave] = mx; }
        __syncthreads();
        int pb = pt0 + p - npts;
        uint32_t cb = cell0 + c - (uint32_t)ncell;
        for (int w = 0; w < kTableThreads / kWave; ++w) {
            if (w < wave) { pb += wpts[w]; cb += wcells[w]; }
            pt0 += wpts[w];
            cell0 += wcells[w];
            most = max(most, wmax[w]);
        }
        if (k < nbands) {
            Band b;
            b.npts = npts;
            b.pt_start = pb;
            b.ncell = ncell;
            b.cell_off = (int)cb;
            b.cells_per_rad = (float)((double)ncell / kTwoPi);
            const double lo = npts ? band_th[2 * (int64_t)k] : k * h, hi = npts ? band_th[2 * (int64_t)k + 1] : k * h;
            b.th_lo = lo;
            b.th_hi = hi;
            sincos(0.5 * lo, &b.sh_lo, &b.ch_lo);
            sincos(0.5 * hi, &b.sh_hi, &b.ch_hi);
            const double slo = sin(lo), shi = sin(hi);
            const double smin = fmin(slo, shi);
            const double smax = (lo <= 0.5 * kPi && hi >= 0.5 * kPi) ? 1.0 : fmax(slo, shi);
            b.inv_smin = smin > 0.0 ? (float)(1.0 / smin) : INFINITY;
            b.inv_smax = smax > 0.0 ? (float)(1.0 / smax) : INFINITY;
            b.pad_ = 0;
            bands[k] = b;
        }
    }
    if (threadIdx.x == 0) { stats[0] = cell0; stats[1] = (uint32_t)most; }
}

__global__ void k_cell_of_point(int64_t n, const int *band, const double *phi, const Band *bands,
                                int *cell, int *cell_count)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Band &bd = bands[band[i]];
    int c = (int)floor(phi[i] * ((double)bd.ncell / kTwoPi));
    c = c < 0 ? 0 : (c >= bd.ncell ? bd.ncell - 1 : c);
    int g = bd.cell_off + c;
    cell[i] = g;
    atomicAdd(&cell_count[g], 1);
}

// ---- pivots on a plane -------------------------------------------------------------------
// The plane reuses the sphere's grid: strips of y play the latitude bands and
// (x - x0) * sx in [0, 2 pi) the longitude of the cells.

// Per-block minima and maxima of x and y ([block][4]: min x, max x, min y, max y).
__global__ void k_plane_range(const double *xyz, int64_t n, double *part)
{
    __shared__ double sh[4][256];
    double v[4] = {INFINITY, -INFINITY, INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = xyz[i], y = xyz[n + i];
        v[0] = fmin(v[0], x); v[1] = fmax(v[1], x);
        v[2] = fmin(v[2], y); v[3] = fmax(v[3], y);
    }
    for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sh[0][threadIdx.x] = fmin(sh[0][threadIdx.x], sh[0][threadIdx.x + o]);
            sh[1][threadIdx.x] = fmax(sh[1][threadIdx.x], sh[1][threadIdx.x + o]);
            sh[2][threadIdx.x] = fmin(sh[2][threadIdx.x], sh[2][threadIdx.x + o]);
            sh[3][threadIdx.x] = fmax(sh[3][threadIdx.x], sh[3][threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 4) part[4 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

// [2][n] plane positions -> [3][n] with z = 0 (the records and the d2 test then see
// dz = 0 exactly)
__global__ void k_plane_xyz(const double *xy, int64_t n, double *xyz)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    xyz[i] = xy[i];
    xyz[n + i] = xy[n + i];
    xyz[2 * n + i] = 0.0;
}

// The points of every cell, from its first entry on in the order of the atomics (counting the cell's
// count back down), which is near the original one.  k_sort_cells moves each point past the later
// ones before it: from the last entry on, the points of a crowded cell come in about the reverse
// order and all pass each other (1,000 stacks of 300 points, one of each in turn: index and
// values 6.5 ms so, 2.8 ms this way).
__global__ void k_scatter(int64_t n, const int *cell, const int *cell_start, int *cell_count, int *order)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int c = cell[i];
    int pos = cell_start[c + 1] - atomicSub(&cell_count[c], 1);
    order[pos] = (int)i;
}

// Put the points of every cell in increasing original index (cells hold ~1 point).
__global__ void k_sort_cells(int64_t ncells, const int *cell_start, int *order)
{
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells) return;
    int s = cell_start[c], e = cell_start[c + 1];
    for (int i = s + 1; i < e; ++i) {
        int v = order[i];
        int j = i - 1;
        while (j >= s && order[j] > v) {
            order[j + 1] = order[j];
            --j;
        }
        order[j + 1] = v;
    }
}

// The catalogue in index order, and the doubled-band arrays: index-order point i of band k (first
// point s_k, n_k points) is stored at 2 s_k + (i - s_k) and again n_k positions later.
__global__ void k_gather_points(int64_t n, const int *perm, const double *xyz, const double *w, const int *band,
                                const Band *bands, double *x, double *y, double *z, double *ws, int *bs, int *permdbl,
                                double *wdbl)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int j = perm[i], k = band[j];
    x[i] = xyz[j];
    y[i] = xyz[n + j];
    z[i] = xyz[2 * n + j];
    const double wj = w ? w[j] : 1.0;
    ws[i] = wj;
    bs[i] = k;
    const int64_t np = bands[k].npts, q = (int64_t)bands[k].pt_start + i;
    permdbl[q] = j;
    permdbl[q + np] = j;
    if (w) {
        wdbl[q] = wj;
        wdbl[q + np] = wj;
    }
}

// Values w x in index order and the doubled-band records of every map.
__global__ void k_values(int64_t n, int nmaps, const int *perm, const int *band, const Band *bands, const double *x,
                         const double *y, const double *z, const double *w, const double *xv, double *v, double4 *rec)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t j = perm[i];
    const Band &bd = bands[band[i]];
    const int64_t np = bd.npts, q = (int64_t)bd.pt_start + i;
    const double xi = x[i], yi = y[i], zi = z[i], wi = w[i];
    for (int m = 0; m < nmaps; ++m) {
        const double val = wi * xv[(size_t)m * n + j];
        v[(size_t)m * n + i] = val;
        const double4 r = make_double4(xi, yi, zi, val);
        rec[(size_t)m * 2 * n + q] = r;
        rec[(size_t)m * 2 * n + q + np] = r;
    }
}

// Values of map group g in doubled-band order, kMapGroup maps interleaved per point
// (missing maps of the last group are 0).
__global__ void k_group_values(int64_t n, int nmaps, const int *band, const Band *bands, const double *v,
                               double *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Band &bd = bands[band[i]];
    const int64_t q = 2 * (int64_t)bd.pt_start + (i - bd.pt_start);
    const int ng = (nmaps + kMapGroup - 1) / kMapGroup;
    for (int g = 0; g < ng; ++g) {
        double *o = out + (size_t)g * 2 * n * kMapGroup;
        for (int k = 0; k < kMapGroup; ++k) {
            const int m = g * kMapGroup + k;
            const double val = m < nmaps ? v[(size_t)m * n + i] : 0.0;
            o[(size_t)q * kMapGroup + k] = val;
            o[(size_t)(q + bd.npts) * kMapGroup + k] = val;
        }
    }
}

// Per-record value matrix of the MFMA many-map kernel: row q of the doubled-band order
// holds the ldv map values of its point (maps >= nmaps are 0).  One thread per (point, map).
__global__ void k_value_matrix(int64_t n, int nmaps, int ldv, const int *band, const Band *bands, const double *v,
                               double *out64, float *out32)
{
    const int64_t total = n * ldv;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = t / ldv;
        const int m = (int)(t - i * ldv);
        const Band &bd = bands[band[i]];
        const int64_t q = 2 * (int64_t)bd.pt_start + (i - bd.pt_start);
        const double val = m < nmaps ? v[(size_t)m * n + i] : 0.0;
        out64[q * ldv + m] = val;
        out64[(q + bd.npts) * ldv + m] = val;
        out32[q * ldv + m] = (float)val;
        out32[(q + bd.npts) * ldv + m] = (float)val;
    }
}

// ---- exclusive scan of int counts (n < 2^31 total) -----------------------------------

constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;
constexpr int kScanTile = kScanThreads * kScanPer;

__global__ void k_scan_tiles(const int *in, int64_t n, int *out, int *tile_sums)
{
    __shared__ int sh[kScanThreads];
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int v[kScanPer];
    int sum = 0;
    for (int k = 0; k < kScanPer; ++k) {
        int64_t i = base + k;
        v[k] = i < n ? in[i] : 0;
        sum += v[k];
    }
    sh[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        int t = threadIdx.x >= (unsigned)off ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    int run = sh[threadIdx.x] - sum;  // exclusive prefix of this thread
    for (int k = 0; k < kScanPer; ++k) {
        int64_t i = base + k;
        if (i < n) out[i] = run;
        run += v[k];
    }
    if (threadIdx.x == kScanThreads - 1) tile_sums[blockIdx.x] = sh[threadIdx.x];
}

__global__ void k_scan_add(int *out, int64_t n, const int *tile_offsets)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] += tile_offsets[i / kScanTile];
}

// Scratch ints of exclusive_scan over n counts.
static int64_t scan_ints(int64_t n)
{
    int64_t total = 0;
    for (int64_t tiles = (n + kScanTile - 1) / kScanTile;; tiles = (tiles + kScanTile - 1) / kScanTile) {
        total += 2 * (tiles + 1);
        if (tiles <= 1) return total;
    }
}

// out[i] = sum_{k<i} in[k] for i in [0, n); tmp holds scan_ints(n).
static z3_status exclusive_scan(const int *in, int64_t n, int *out, int *tmp, hipStream_t s)
{
    const int64_t tiles = n > kScanTile ? (n + kScanTile - 1) / kScanTile : 1;
    int *sums = tmp, *offs = tmp + tiles + 1;
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, in, n, out, sums);
    z3_status st = check_launch("k_scan_tiles");
    if (st != Z3_OK || tiles == 1) return st;
    if ((st = exclusive_scan(sums, tiles, offs, offs + tiles + 1, s)) != Z3_OK) return st;
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, n, offs);
    return check_launch("k_scan_add");
}

// The index's arrays go back to the kept blocks; `waited`: no work that uses them is in flight.
static void free_ptrs(z3_index idx, bool waited)
{
    void *blocks[] = {idx->d_edges, idx->d_bands, idx->d_cell_start, idx->d_x, idx->d_y, idx->d_z, idx->d_w,
                      idx->d_perm, idx->d_band, idx->d_wdbl, idx->d_permdbl, idx->d_v, idx->d_rec, idx->d_vgrp,
                      idx->d_vmat64, idx->d_vmat32};
    for (void *p : blocks) return_block(p, waited ? idx->device : -1);
    void *ps[] = {idx->cap_ws, idx->d_phi_bounds, idx->d_phi_tab};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    for (void *p : idx->cap_retired) (void)hipFree(p);
    idx->cap_retired.clear();
}

void free_index(z3_index idx)
{
    (void)hipSetDevice(idx->device);
    free_ptrs(idx, wait_device(idx->device) == Z3_OK);
    delete idx;
}

template <class T>
static z3_status dalloc(T **p, size_t count, const char *what)
{
    *p = nullptr;
    return device_block((void **)p, (count ? count : 1) * sizeof(T), what);
}

static inline unsigned grid_for(int64_t n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

z3_status build_index_impl(int64_t n, const double *xyz, const double *w, int nbins,
                           const double *edges, double cell_size, hipStream_t s, z3_index *out, bool planar)
{
    z3_index idx = new (std::nothrow) z3_index_s();
    if (!idx) return fail(Z3_ERR_OUT_OF_MEMORY, "z3_build_index: host allocation failed");
    (void)hipGetDevice(&idx->device);
    idx->n = n;
    idx->nbins = nbins;
    idx->planar = planar;
    z3_status st = Z3_OK;
    // temporaries: given back on return (every path out of this function synchronises the
    // stream first; where the runtime refuses that, they are set aside)
    struct Temps {
        void *p[10] = {};
        int count = 0;
        void *pin = nullptr;
        int dev = 0;
        bool waited = true;
        ~Temps()
        {
            for (int i = 0; i < count; ++i) return_block(p[i], waited ? dev : -1);
            pinned_give(pin, waited);
        }
    } tmp;
    tmp.dev = idx->device;
    auto bail = [&](z3_status code) {
        tmp.waited = hipStreamSynchronize(s) == hipSuccess;
        if (!tmp.waited) (void)hipGetLastError();  // `code` is what the caller sees
        free_ptrs(idx, tmp.waited);
        delete idx;
        return code;
    };
    auto temp = [&](auto **p, size_t count, const char *what) {
        const z3_status e = dalloc(p, count, what);
        if (e == Z3_OK) tmp.p[tmp.count++] = *p;
        return e;
    };
    // plane: the [2][n] positions become [3][n] with z = 0
    if (planar && n > 0) {
        double *xyz3 = nullptr;
        if ((st = temp(&xyz3, 3 * (size_t)n, "alloc plane positions")) != Z3_OK) return bail(st);
        hipLaunchKernelGGL(k_plane_xyz, dim3(grid_for(n)), dim3(256), 0, s, xyz, n, xyz3);
        if ((st = check_launch("k_plane_xyz")) != Z3_OK) return bail(st);
        xyz = xyz3;
    }
    // plane: bounding box of the points (x0 = min x, y0 = min y, extents lx, ly)
    double lx = 0.0, ly = 0.0, scale = 0.0;
    if (planar && n > 0) {
        const int nblk = (int)std::min<int64_t>((n + 255) / 256, kPinnedBytes / (4 * sizeof(double)));
        double *d_part = nullptr;
        if ((st = temp(&d_part, 4 * (size_t)nblk, "alloc plane range")) != Z3_OK) return bail(st);
        if ((st = pinned_take(&tmp.pin)) != Z3_OK) return bail(st);
        hipLaunchKernelGGL(k_plane_range, dim3(nblk), dim3(256), 0, s, xyz, n, d_part);
        st = check_launch("k_plane_range");
        const double *part = static_cast<const double *>(tmp.pin);
        if (st == Z3_OK)
            st = check_hip(hipMemcpyAsync(tmp.pin, d_part, 4 * (size_t)nblk * sizeof(double), hipMemcpyDeviceToHost, s),
                           "copy plane range");
        if (st == Z3_OK) st = check_hip(hipStreamSynchronize(s), "sync");
        if (st != Z3_OK) return bail(st);
        double v[4] = {INFINITY, -INFINITY, INFINITY, -INFINITY};
        for (int b = 0; b < nblk; ++b) {
            v[0] = std::min(v[0], part[4 * b]); v[1] = std::max(v[1], part[4 * b + 1]);
            v[2] = std::min(v[2], part[4 * b + 2]); v[3] = std::max(v[3], part[4 * b + 3]);
        }
        if (!(std::isfinite(v[0]) && std::isfinite(v[1]) && std::isfinite(v[2]) && std::isfinite(v[3])))
            return bail(fail(Z3_ERR_INVALID_ARG, "z3_build_index_planar: positions are not finite"));
        idx->plane_x0 = v[0];
        idx->plane_y0 = v[2];
        lx = v[1] - v[0];
        ly = v[3] - v[2];
        scale = std::max(std::max(std::fabs(v[0]), std::fabs(v[1])), std::max(std::fabs(v[2]), std::fabs(v[3])));
        // cell coordinate (x - x0) sx stays below 2 pi
        idx->plane_sx = kTwoPi / (lx * (1.0 + 1e-12) + 1e-300 + 1e-15 * scale);
    }
    for (int b = 0; b <= nbins; ++b) {
        double e = edges[b];
        idx->edges.e[b] = e;
        if (planar) {
            // plane: rad_out is the enlarged radius, hav_out / hav_in the enlarged / reduced
            // squared radii of the window search (membership is the exact d2 test); the
            // absolute guard covers the rounding of coordinates of size `scale`
            const double g = 1e-14 * scale, r = sqrt(e);
            idx->edges.rad_out[b] = r * (1.0 + 1e-9) + g;
            idx->edges.hav_out[b] = idx->edges.rad_out[b] * idx->edges.rad_out[b];
            const double rin = std::max(0.0, r * (1.0 - 1e-9) - g);
            idx->edges.hav_in[b] = rin * rin;
            continue;
        }
        // Rounding guards for the window search only (membership is decided by the exact
        // d2 test): the FP64 squared chord of two FP64 unit vectors differs from the
        // exact chord by far less than 1e-9 relative at the separations supported here.
        idx->edges.hav_out[b] = 0.25 * e * (1.0 + 1e-9) + 1e-16;
        idx->edges.hav_in[b] = 0.25 * e * (1.0 - 1e-9) - 1e-16;
        double r = 2.0 * asin(std::min(1.0, sqrt(e) / 2.0));
        idx->edges.rad_out[b] = r * (1.0 + 1e-9) + 1e-12;
    }
    double *d_range = nullptr;
    if ((st = dalloc(&idx->d_edges, 1, "alloc edges")) != Z3_OK) return bail(st);
    if ((st = temp(&d_range, 4, "alloc range")) != Z3_OK) return bail(st);
    if (!tmp.pin && (st = pinned_take(&tmp.pin)) != Z3_OK) return bail(st);
    hipLaunchKernelGGL(k_index_begin, dim3(1), dim3(256), 0, s, idx->edges, idx->d_edges, d_range);
    if ((st = check_launch("k_index_begin")) != Z3_OK) return bail(st);

    // ---- band height; sky positions: colatitude range and unit-length check --------------
    // Sky positions must be unit vectors: the windows are angular while membership is the
    // chord test on the raw vectors, and the windows' guards (1e-9 relative) cover a
    // deviation | |r|^2 - 1 | of up to kMaxNormDev only.
    double h = cell_size;
    double area = 1.0;
    if (planar) {
        // the same 1.4 x mean spacing as on the sphere
        area = lx * ly;
        if (!(area > 0.0)) area = std::max(lx, ly) * std::max(lx, ly) / (double)std::max<int64_t>(n, 1);
        if (!(area > 0.0)) area = 1.0;
        if (h <= 0.0) h = Z3_BAND_HEIGHT_FACTOR * sqrt(area / (double)std::max<int64_t>(n, 1));
    } else {
        const double *rg = static_cast<const double *>(tmp.pin);
        if (n > 0) {
            unsigned g = grid_for(n) < 2048u ? grid_for(n) : 2048u;
            hipLaunchKernelGGL(k_sky_range, dim3(g), dim3(256), 0, s, xyz, n, d_range);
            st = check_launch("k_sky_range");
        }
        if (st == Z3_OK)
            st = check_hip(hipMemcpyAsync(tmp.pin, d_range, 4 * sizeof(double), hipMemcpyDeviceToHost, s), "copy range");
        if (st == Z3_OK) st = check_hip(hipStreamSynchronize(s), "sync");
        if (st != Z3_OK) return bail(st);
        if (!(rg[2] <= kMaxNormDev))
            return bail(fail(Z3_ERR_INVALID_ARG,
                             "z3_build_index: positions are not unit vectors (max | |r|^2 - 1 | = %g, limit %g)", rg[2],
                             kMaxNormDev));
        area = 2.0 * kPi * (cos(std::min(rg[0], rg[1])) - cos(std::max(rg[0], rg[1])));
        if (!(area > 0.0)) area = 1e-12;
        uint64_t sectors;
        __builtin_memcpy(&sectors, rg + 3, sizeof(sectors));
        if (sectors) idx->sky_part = __builtin_popcountll(sectors) / 64.0;
        if (h <= 0.0) {
            // 1.4 x the mean point spacing: about two HEALPix rings per band (ring spacing
            // 2 / (3 Nside) rad at low latitudes, mean spacing ~1.023 / Nside).  Each band
            // costs every pivot one longitude window per bin, whose set-up (window bounds,
            // cell lookups, the mixed path's flush into FP64) outweighs the few candidates
            // that a taller band adds at the window ends; measured on HEALPix maps at Nside
            // 512 and 2048 against 0.6 (one ring per band) to 2.6, 1.3-1.8 is best.
            h = Z3_BAND_HEIGHT_FACTOR * sqrt(area / (double)std::max<int64_t>(n, 1));
        }
    }
    idx->density = (double)n / area;
    int nbands = 1;
    if (planar) {
        const double nb_d = std::floor(ly / h) + 1.0;
        if (!(nb_d <= (double)(1 << 26))) return bail(fail(Z3_ERR_INVALID_ARG, "z3_build_index_planar: cell_size too small"));
        nbands = (int)nb_d;
    } else {
        h = std::min(h, kPi);
        nbands = (int)std::ceil(kPi / h);
        if (nbands < 1) nbands = 1;
        if (nbands > (1 << 26)) return bail(fail(Z3_ERR_INVALID_ARG, "z3_build_index: cell_size too small"));
    }
    idx->band_h = h;
    idx->nbands = nbands;

    // ---- bands -------------------------------------------------------------------------
    int *d_band = nullptr, *d_band_count = nullptr, *d_cell = nullptr, *d_cell_count = nullptr, *d_scan = nullptr;
    uint32_t *d_stats = nullptr;
    double *d_phi = nullptr, *d_band_th = nullptr;
    if ((st = temp(&d_band, n, "alloc band")) != Z3_OK) return bail(st);
    if ((st = temp(&d_phi, n, "alloc phi")) != Z3_OK) return bail(st);
    if ((st = temp(&d_band_count, (size_t)nbands + 2, "alloc band count")) != Z3_OK) return bail(st);
    if ((st = temp(&d_band_th, 2 * (size_t)nbands, "alloc band theta")) != Z3_OK) return bail(st);
    if ((st = dalloc(&idx->d_bands, nbands, "alloc bands")) != Z3_OK) return bail(st);
    d_stats = reinterpret_cast<uint32_t *>(d_band_count + nbands);
    // The table's totals are read back at the end.  They are read before there is any cell array
    // where they may say that the catalogue is refused (a band of more than 2^26 points, 2^31
    // cells), and where the arrays for the most cells there can be are not to be had.
    int64_t cells = (int64_t)kCellsPerPoint * n + nbands;  // a band without points has one
    bool known = 64 * n > (int64_t)UINT32_MAX || cells >= (int64_t)0x7fffffff;
    const double lo0 = planar ? INFINITY : 4.0;
    // (the scan also covers the entry after the last cell, which holds n)
    auto cell_arrays = [&]() {
        z3_status e = Z3_OK;
        if (!d_cell) e = temp(&d_cell, n, "alloc cell");
        if (e == Z3_OK && !d_cell_count) e = temp(&d_cell_count, cells + 1, "alloc cell count");
        if (e == Z3_OK && !d_scan) e = temp(&d_scan, scan_ints(cells + 1), "scan alloc");
        if (e == Z3_OK && !idx->d_cell_start) e = dalloc(&idx->d_cell_start, cells + 1, "alloc cell start");
        return e;
    };
    auto clear_counts = [&](int bands, int64_t ncells) {
        const int64_t len = std::max<int64_t>(ncells, bands);
        hipLaunchKernelGGL(k_clear_counts, dim3(std::min(grid_for(len), 8192u)), dim3(256), 0, s, d_band_count, d_band_th,
                           bands, lo0, d_cell_count, ncells);
        return check_launch("k_clear_counts");
    };
    if (!known) {
        st = cell_arrays();
        if (st != Z3_OK && st != Z3_ERR_OUT_OF_MEMORY) return bail(st);
        known = st != Z3_OK;
    }
    if ((st = clear_counts(nbands, known ? 0 : cells + 1)) != Z3_OK) return bail(st);
    const BandRule rule{1.0 / h, idx->plane_x0, idx->plane_y0, idx->plane_sx, lo0, nbands};
    st = planar ? launch_band_of_point<true>(xyz, n, rule, d_band, d_phi, d_band_count, d_band_th, s)
                : launch_band_of_point<false>(xyz, n, rule, d_band, d_phi, d_band_count, d_band_th, s);
    if (st != Z3_OK) return bail(st);
    hipLaunchKernelGGL(k_band_table, dim3(1), dim3(kTableThreads), 0, s, nbands, h, d_band_count, d_band_th,
                       idx->d_bands, d_stats);
    if ((st = check_launch("k_band_table")) != Z3_OK) return bail(st);
    const uint32_t *stats = static_cast<const uint32_t *>(tmp.pin);
    auto read_stats = [&]() {
        z3_status e = check_hip(hipMemcpyAsync(tmp.pin, d_stats, 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, s), "copy");
        return e == Z3_OK ? check_hip(hipStreamSynchronize(s), "sync") : e;
    };
    if (known) {
        if ((st = read_stats()) != Z3_OK) return bail(st);
        // the multipole kernel addresses a band's doubled records (64 B per point) with 32-bit
        // byte offsets
        if ((int64_t)stats[1] * 64 > (int64_t)UINT32_MAX)
            return bail(fail(Z3_ERR_UNSUPPORTED, "z3_build_index: %u points in one latitude band", stats[1]));
        if (stats[0] >= 0x7fffffffu) return bail(fail(Z3_ERR_OVERFLOW, "z3_build_index: too many points or cells"));
        cells = stats[0];
        if ((st = cell_arrays()) != Z3_OK) return bail(st);
        if ((st = clear_counts(0, cells + 1)) != Z3_OK) return bail(st);
    }

    // ---- cells, sort -----------------------------------------------------------------------
    if ((st = dalloc(&idx->d_perm, n, "alloc perm")) != Z3_OK) return bail(st);
    if ((st = dalloc(&idx->d_x, n, "alloc x")) != Z3_OK) return bail(st);
    if ((st = dalloc(&idx->d_y, n, "alloc y")) != Z3_OK) return bail(st);
    if ((st = dalloc(&idx->d_z, n, "alloc z")) != Z3_OK) return bail(st);
    if ((st = dalloc(&idx->d_w, n, "alloc w")) != Z3_OK) return bail(st);
    idx->unit_w = (w == nullptr);
    if ((st = dalloc(&idx->d_band, n, "alloc band")) != Z3_OK) return bail(st);
    if ((st = dalloc(&idx->d_permdbl, 2 * n, "alloc perm2")) != Z3_OK) return bail(st);
    if (!idx->unit_w && (st = dalloc(&idx->d_wdbl, 2 * n, "alloc w2")) != Z3_OK) return bail(st);
    if (n > 0)
        hipLaunchKernelGGL(k_cell_of_point, dim3(grid_for(n)), dim3(256), 0, s, n, d_band, d_phi, idx->d_bands,
                           d_cell, d_cell_count);
    if ((st = exclusive_scan(d_cell_count, cells + 1, idx->d_cell_start, d_scan, s)) != Z3_OK) return bail(st);
    if (n > 0) {
        hipLaunchKernelGGL(k_scatter, dim3(grid_for(n)), dim3(256), 0, s, n, d_cell, idx->d_cell_start,
                           d_cell_count, idx->d_perm);
        hipLaunchKernelGGL(k_sort_cells, dim3(grid_for(cells)), dim3(256), 0, s, cells, idx->d_cell_start,
                           idx->d_perm);
        hipLaunchKernelGGL(k_gather_points, dim3(grid_for(n)), dim3(256), 0, s, n, idx->d_perm, xyz, w, d_band,
                           idx->d_bands, idx->d_x, idx->d_y, idx->d_z, idx->d_w, idx->d_band, idx->d_permdbl,
                           idx->d_wdbl);
    }
    if ((st = check_launch("k_gather_points")) != Z3_OK) return bail(st);
    if ((st = read_stats()) != Z3_OK) return bail(st);
    idx->ncells = stats[0];
    *out = idx;
    return Z3_OK;
}

// Rebuild every per-map array from new values x [nmaps][n] (catalogue order) into the
// buffers already attached: kernels only, on `s`.
static z3_status fill_values(z3_index idx, int nmaps, const double *x, hipStream_t s)
{
    z3_status st;
    if (idx->n == 0) return Z3_OK;
    hipLaunchKernelGGL(k_values, dim3(grid_for(idx->n)), dim3(256), 0, s, idx->n, nmaps, idx->d_perm, idx->d_band,
                       idx->d_bands, idx->d_x, idx->d_y, idx->d_z, idx->d_w, x, idx->d_v, idx->d_rec);
    if ((st = check_launch("k_values")) != Z3_OK) return st;
    if (nmaps > 1) {
        hipLaunchKernelGGL(k_group_values, dim3(grid_for(idx->n)), dim3(256), 0, s, idx->n, nmaps, idx->d_band,
                           idx->d_bands, idx->d_v, idx->d_vgrp);
        const int ldv = batch_ldv(nmaps);
        const int64_t nt = idx->n * ldv;
        const int64_t g = (nt + 255) / 256 < (1 << 20) ? (nt + 255) / 256 : (1 << 20);
        hipLaunchKernelGGL(k_value_matrix, dim3((unsigned)g), dim3(256), 0, s, idx->n, nmaps, ldv, idx->d_band,
                           idx->d_bands, idx->d_v, idx->d_vmat64, idx->d_vmat32);
        if ((st = check_launch("k_group_values/k_value_matrix")) != Z3_OK) return st;
    }
    return Z3_OK;
}

z3_status update_values_impl(z3_index idx, const double *x, hipStream_t s)
{
    return fill_values(idx, idx->nmaps, x, s);
}

z3_status set_values_impl(z3_index idx, int nmaps, const double *x, hipStream_t s)
{
    z3_status st;
    if (!idx->d_v) {
        if ((st = check_hip(hipStreamSynchronize(s), "hipStreamSynchronize")) != Z3_OK) return st;
    } else {
        // earlier work, on any stream, may still read the old values
        if ((st = wait_device(idx->device)) != Z3_OK) return st;
        void *old[] = {idx->d_v, idx->d_rec, idx->d_vgrp, idx->d_vmat64, idx->d_vmat32};
        for (void *p : old) return_block(p, idx->device);
        idx->d_v = nullptr;
        idx->d_rec = nullptr;
        idx->d_vgrp = nullptr;
        idx->d_vmat64 = nullptr;
        idx->d_vmat32 = nullptr;
    }
    idx->nmaps = 0;
    idx->ngroups = 0;
    for (auto &row : idx->batch_shape_tuned)
        for (int &t : row) t = 0;
    size_t cnt = (size_t)nmaps * (size_t)idx->n;
    if ((st = dalloc(&idx->d_v, cnt, "alloc values")) != Z3_OK) return st;
    if ((st = dalloc(&idx->d_rec, 2 * cnt, "alloc records")) != Z3_OK) return st;
    if (nmaps > 1) {
        const int ng = (nmaps + kMapGroup - 1) / kMapGroup;
        if ((st = dalloc(&idx->d_vgrp, (size_t)ng * 2 * idx->n * kMapGroup, "alloc grouped values")) != Z3_OK)
            return st;
        idx->ngroups = ng;
        const int ldv = batch_ldv(nmaps);
        if ((st = dalloc(&idx->d_vmat64, (size_t)2 * idx->n * ldv, "alloc value matrix")) != Z3_OK) return st;
        if ((st = dalloc(&idx->d_vmat32, (size_t)2 * idx->n * ldv, "alloc value matrix")) != Z3_OK) return st;
    }
    if ((st = fill_values(idx, nmaps, x, s)) != Z3_OK) return st;
    idx->nmaps = nmaps;
    return Z3_OK;
}

}  // namespace z3
