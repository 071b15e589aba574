// Multipole launches: the one-map kernel (z3_multipoles_device.h) band by band, and the
// register-tiled kernel that carries several maps per lane.
#include "z3_multipoles_device.h"

namespace z3 {

// Groups of bins for a launch of nblk pivot blocks.  Up to kFillBlocks blocks in all (eight per
// resident slot, 256 CUs x 4 blocks): with fewer, SIMDs idle (20,000 pivots are 79 blocks) or a
// last round of long blocks runs on a part of the chip (490,000 pivots are 1.9 rounds); with
// more, the pivot set-up each group repeats costs more than the balance gives.  The groups
// are cut where the running cost of the bins passes each g / n of the total; a bin costs its
// pairs (its share of the annuli's area) and the band windows that even a sparse bin visits.
// Measured, one launch without and with the split: 4,000 pivots x 10 bins 528 -> 103 us, 20,000
// x 10 1342 -> 293 us, 150,000 x 15 3682 -> 2414 us, a plane of 491,000 x 15 3196 -> 2875 us,
// 786,000 x 15 2893 -> 2677 us; four maps per lane, 197,000 x 12, 1569 -> 1076 us.
constexpr int64_t kFillBlocks = 8192;

BinGroups bin_groups(const z3_index_s *idx, int64_t nblk)
{
    const int nb = idx->nbins;
    const int64_t want = nblk > 0 ? (kFillBlocks + nblk - 1) / nblk : 1;
    BinGroups q;
    q.n = (int)(want < nb ? want : nb);
    const double *e = idx->edges.e;
    double run = 0.0;
    for (int b = 0, g = 0; b < nb; ++b) {
        // a group starts here when its share is reached, or when every bin left must start one
        if (g < q.n && (run >= 1.5 * g / q.n || nb - b == q.n - g)) q.first[g++] = (unsigned char)b;
        run += (e[b + 1] - e[b]) / (e[nb] - e[0]) + 0.5 / nb;
    }
    q.first[q.n] = (unsigned char)nb;
    return q;
}

// ---- many maps over one set of positions -------------------------------------------------
//
// Same decomposition (one lane per pivot, bins in order, band windows), but every lane
// carries K maps of a group of kMapGroup (K = 3 when the caller reads at most the first three,
// else 4): the pair test, the bearing and the unit chain U_k(cos phi) are computed once per
// pair, and each map adds v U_k and v 2 sin(phi) U_k with two FMAs per k (the epilogue forms
// the harmonics' sums from T_m = (U_m - U_{m-2}) / 2 and sin(m phi) = sin(phi) U_{m-1}; the
// product basis of HarmonicSums would cost each map two more multiplications a pair).

struct MapArgs {
    const double *px, *py, *pz;   // index-order pivot positions
    const double4 *rec;           // doubled-band records (x, y, z used)
    const double *vgrp;           // [2n][kMapGroup] values of the map group
    const double *wdbl;           // doubled-band weights or null
    const int *cell_start;
    const Band *bands;
    int nbands;
    double inv_h;
    const EdgeTab *edges;
    int nb;
    int64_t p0, p1;
    void *A;                      // per map [m+1][2][nb][ldA], maps map_stride elements apart
    int64_t ldA;
    size_t map_stride;
    double *W;                    // [nb][ldA] W_{p,b} (shared by the maps), or null
    uint64_t *pair_total;
    int nblocks;
    BinGroups groups;             // bins of each blockIdx.y
};

template <int M>
constexpr int maps_waves_per_eu()
{
    return M <= 6 ? 3 : 2;
}

template <int M, bool F32OUT, int K>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(maps_waves_per_eu<M>())))
void k_multipoles_maps(MapArgs a)
{
    static_assert(K == 3 || K == kMapGroup, "three or four maps per lane");
    const int nblk = a.nblocks;
    const int bid = blockIdx.x;
    const int per = nblk / 8, rem = nblk % 8;
    const int xcd = bid % 8, k8 = bid / 8;
    const int lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k8;
    const int64_t wave0 = a.p0 + (int64_t)lb * kBlock + (threadIdx.x & ~(kWave - 1));
    if (__builtin_amdgcn_readfirstlane((int)(wave0 >= a.p1))) return;
    const int64_t p = a.p0 + (int64_t)lb * kBlock + threadIdx.x;
    const bool valid = p < a.p1;
    const int64_t pp = valid ? p : a.p1 - 1;

    const double xp = a.px[pp], yp = a.py[pp], zp = a.pz[pp];
    const double sinth = sqrt(xp * xp + yp * yp);
    const double th = atan2(sinth, zp);
    double ph = atan2(yp, xp);
    if (ph < 0.0) ph += kTwoPi;
    double sh, ch;
    sincos(0.5 * th, &sh, &ch);
    const float inv_sp = sinth > 0.0 ? (float)(1.0 / sinth) : INFINITY;
    const float phf = (float)ph;
    double nx = -zp * xp, ny = -zp * yp, nz = 1.0 - zp * zp;
    double nn = sqrt(nx * nx + ny * ny + nz * nz);
    if (nn < 1e-12) {
        nx = 1.0 - xp * xp; ny = -xp * yp; nz = -xp * zp;
        nn = sqrt(nx * nx + ny * ny + nz * nz);
    }
    nx /= nn; ny /= nn; nz /= nn;
    // east without its z component, as in k_multipoles
    const double ex = ny * zp - nz * yp, ey = nz * xp - nx * zp;

    const int64_t col = p - a.p0;
    const int nb = a.nb;
    const bool unit_w = a.wdbl == nullptr;
    uint64_t my_pairs = 0;

    const int grp = a.groups.n - 1 - (int)blockIdx.y;  // outermost bins first
    const int bin_end = a.groups.first[grp + 1];
    for (int bin = a.groups.first[grp]; bin < bin_end; ++bin) {
        const double elo = a.edges->e[bin], ehi = a.edges->e[bin + 1];
        const double hav_out = a.edges->hav_out[bin + 1], hav_in = a.edges->hav_in[bin];
        const double rad = a.edges->rad_out[bin + 1];
        int klo = (int)floor((th - rad) * a.inv_h);
        int khi = (int)floor((th + rad) * a.inv_h);
        klo = max(klo, 0);
        khi = min(khi, a.nbands - 1);
        klo = __builtin_amdgcn_readfirstlane(wave_min(klo));
        khi = __builtin_amdgcn_readfirstlane(wave_max(khi));

        // per map: SU_k = sum v U_k(cos phi), SV_k = sum v 2 sin(phi) U_k(cos phi), with one unit
        // chain U_k shared by the maps
        double SU[K][M + 1], SV[K][M + 1];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int m = 0; m <= M; ++m) { SU[k][m] = 0.0; SV[k][m] = 0.0; }
        double Wb = 0.0;
        int cnt = 0;

        for (int kb = klo; kb <= khi; ++kb) {
            const Band bd = a.bands[kb];
            if (bd.npts == 0) continue;
            int s0, l0, s1, l1;
            band_window(bd, a.cell_start, th, sh, ch, inv_sp, phf, hav_out, hav_in, s0, l0, s1, l1);
            const int base = 2 * bd.pt_start;
#pragma unroll
            for (int seg = 0; seg < 2; ++seg) {
                int j = base + (seg == 0 ? s0 : s1);
                const int jend = j + (seg == 0 ? l0 : l1);
                for (; j < jend; ++j) {
                    const double4 r = a.rec[j];
                    const double dx = r.x - xp, dy = r.y - yp, dz = r.z - zp;
                    const double d2 = (dx * dx + dy * dy) + dz * dz;
                    if (d2 >= elo && d2 < ehi) {
                        cnt += 1;
                        if (!unit_w) Wb += a.wdbl[j];
                        const double4 vv = *reinterpret_cast<const double4 *>(a.vgrp + (size_t)j * kMapGroup);
                        double v[K];
                        v[0] = vv.x; v[1] = vv.y; v[2] = vv.z;
                        if constexpr (K == 4) v[3] = vv.w;
                        const double u1 = fma(dx, nx, fma(dy, ny, dz * nz));
                        const double u2 = fma(dx, ex, dy * ey);
                        double tc, ts;  // 2 cos(phi), 2 sin(phi)
                        twice_unit_bearing(u1, u2, kBearingTiny, tc, ts);
#pragma unroll
                        for (int k = 0; k < K; ++k) SU[k][0] += v[k];
                        if constexpr (M >= 1) {
                            double vs[K];
#pragma unroll
                            for (int k = 0; k < K; ++k) {
                                vs[k] = ts * v[k];
                                SV[k][0] += vs[k];
                                SU[k][1] = fma(v[k], tc, SU[k][1]);
                            }
                            double ua = 1.0, ub = tc;  // U_0, U_1
#pragma unroll
                            for (int m = 2; m <= M; ++m) {
#pragma unroll
                                for (int k = 0; k < K; ++k) SV[k][m - 1] = fma(vs[k], ub, SV[k][m - 1]);
                                const double um = fma(tc, ub, -ua);
#pragma unroll
                                for (int k = 0; k < K; ++k) SU[k][m] = fma(v[k], um, SU[k][m]);
                                ua = ub; ub = um;
                            }
                        }
                    }
                }
            }
        }

        if (valid) {
            my_pairs += (uint64_t)cnt;
            if (unit_w) Wb = (double)cnt;
            const double inv = Wb > 0.0 ? 1.0 / Wb : 0.0;
            const double hinv = 0.5 * inv;
            if (a.W) a.W[(size_t)bin * (size_t)a.ldA + col] = Wb;
#pragma unroll
            for (int k = 0; k < K; ++k) {
#pragma unroll
                for (int m = 0; m <= M; ++m) {
                    const double y = m >= 2 ? SU[k][m] - SU[k][m >= 2 ? m - 2 : 0] : SU[k][m];
                    const double re = m == 0 ? y * inv : y * hinv;
                    const double im = m == 0 ? 0.0 : -SV[k][m >= 1 ? m - 1 : 0] * hinv;
                    const size_t ore = k * a.map_stride + ((size_t)(2 * m) * nb + bin) * (size_t)a.ldA + col;
                    const size_t oim = k * a.map_stride + ((size_t)(2 * m + 1) * nb + bin) * (size_t)a.ldA + col;
                    if constexpr (F32OUT) {
                        static_cast<float *>(a.A)[ore] = (float)re;
                        static_cast<float *>(a.A)[oim] = (float)im;
                    } else {
                        static_cast<double *>(a.A)[ore] = re;
                        static_cast<double *>(a.A)[oim] = im;
                    }
                }
            }
        }
    }

    if (a.pair_total) {
        const uint64_t tot = wave_sum_u64(valid ? my_pairs : 0);
        if ((threadIdx.x & (kWave - 1)) == 0 && tot) atomicAdd((unsigned long long *)a.pair_total, (unsigned long long)tot);
    }
}

template <int M>
static void launch_maps_m(bool f32out, bool three, const MapArgs &a, hipStream_t s)
{
    dim3 grid(a.nblocks, a.groups.n), block(kBlock);
    if (three) {
        if (f32out) hipLaunchKernelGGL((k_multipoles_maps<M, true, 3>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles_maps<M, false, 3>), grid, block, 0, s, a);
    } else {
        if (f32out) hipLaunchKernelGGL((k_multipoles_maps<M, true, kMapGroup>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles_maps<M, false, kMapGroup>), grid, block, 0, s, a);
    }
}

z3_status launch_multipoles_maps(const z3_index_s *idx, int group, int nslots, int m_max, int prec, int64_t p0,
                                 int64_t p1, void *A, int64_t ldA, size_t map_stride, double *W,
                                 uint64_t *pair_total, hipStream_t s)
{
    if (nslots < 1 || nslots > kMapGroup) return fail(Z3_ERR_INVALID_ARG, "map slots %d outside 1..%d", nslots, kMapGroup);
    int64_t nblk = (p1 - p0 + kBlock - 1) / kBlock;
    if (nblk > 0x7fffffff) return fail(Z3_ERR_OVERFLOW, "too many pivot blocks");
    MapArgs a;
    a.px = idx->d_x; a.py = idx->d_y; a.pz = idx->d_z;
    a.rec = idx->d_rec;
    a.vgrp = idx->d_vgrp + (size_t)group * 2 * idx->n * kMapGroup;
    a.wdbl = idx->unit_w ? nullptr : idx->d_wdbl;
    a.cell_start = idx->d_cell_start;
    a.bands = idx->d_bands;
    a.nbands = idx->nbands;
    a.inv_h = 1.0 / idx->band_h;
    a.edges = idx->d_edges;
    a.nb = idx->nbins;
    a.p0 = p0; a.p1 = p1;
    a.A = A; a.ldA = ldA; a.map_stride = map_stride;
    a.W = W;
    a.pair_total = pair_total;
    a.nblocks = (int)nblk;
    a.groups = bin_groups(idx, nblk);
    const bool f32 = prec == Z3_PREC_MIXED;
    hipEvent_t ev0;
    profile_begin(s, &ev0);
    switch (m_max) {
#define Z3_CASE(MM) case MM: launch_maps_m<MM>(f32, nslots <= 3, a, s); break;
        Z3_CASE(0) Z3_CASE(1) Z3_CASE(2) Z3_CASE(3) Z3_CASE(4) Z3_CASE(5) Z3_CASE(6) Z3_CASE(7)
        Z3_CASE(8) Z3_CASE(9) Z3_CASE(10) Z3_CASE(11) Z3_CASE(12) Z3_CASE(13) Z3_CASE(14)
        Z3_CASE(15) Z3_CASE(16)
#undef Z3_CASE
    default: return fail(Z3_ERR_UNSUPPORTED, "m_max=%d not compiled", m_max);
    }
    z3_status st = check_launch("k_multipoles_maps");
    profile_end(s, ev0);
    return st;
}

// The mixed path differs only in the output: FP32 multipoles for its split-FP32 contraction.
template <int M, bool PLANAR>
static void launch_mp(bool f32out, bool ids, bool self, const MultArgs &a, hipStream_t s)
{
    dim3 grid(a.nblocks, a.groups.n), block(kBlock);
    if (f32out) {
        if (ids) hipLaunchKernelGGL((k_multipoles<M, true, true, false, PLANAR, false>), grid, block, 0, s, a);
        else if (self) hipLaunchKernelGGL((k_multipoles<M, true, false, true, PLANAR, false>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles<M, true, false, false, PLANAR, false>), grid, block, 0, s, a);
    } else {
        if (ids) hipLaunchKernelGGL((k_multipoles<M, false, true, false, PLANAR, false>), grid, block, 0, s, a);
        else if (self) hipLaunchKernelGGL((k_multipoles<M, false, false, true, PLANAR, false>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles<M, false, false, false, PLANAR, false>), grid, block, 0, s, a);
    }
}

template <int M>
static void launch_m(bool planar, bool mixed, bool ids, bool self, const MultArgs &a, hipStream_t s)
{
    if (planar) launch_mp<M, true>(mixed, ids, self, a, s);
    else launch_mp<M, false>(mixed, ids, self, a, s);
}

// Whether the launch walks window lists: its windows hold few pairs on average.  The pairs of a
// pivot follow from the index's mean density, its windows from the bands that each bin's circle
// crosses, two a band.  Short windows gain because a lane need not wait for the longest window
// of every band; with long ones on a regular grid the lanes are even by themselves, and lanes
// that drift into different bands share fewer cache lines.  Measured (estimator calls, bands in
// lockstep / lists): HEALPix maps at 0.8 to 3.9 pairs a window 1.07-1.14 times faster on
// lists, 5.6: 1.02, 6.5: 1.05, 9.5: 0.99, 10.1: 0.99; random points on the full sky at 1.1-2.1:
// 1.29-1.33; caps of 2,500 to 1e6 random points, whose density over the colatitude range reads
// low: 1.04-1.32; jittered plane grids at 3.8: 1.14-1.20, 9.3: 1.03.  The line is set at 8.
constexpr double kShortWindow = 8.0;

static bool short_windows(const z3_index_s *idx)
{
    const EdgeTab &t = idx->edges;
    const int nb = idx->nbins;
    double windows = 0.0;
    for (int b = 1; b <= nb; ++b) windows += 4.0 * t.rad_out[b] / idx->band_h + 2.0;
    return idx->density * kPi * (t.e[nb] - t.e[0]) < kShortWindow * windows;
}

z3_status launch_multipoles(const z3_index_s *idx, Pivots piv, int map, int m_max, int prec, int norm,
                            int64_t p0, int64_t p1, void *A, int64_t ldA, double *W,
                            int64_t *counts, uint64_t *idhash, uint64_t *pair_total, hipStream_t s,
                            const double *self_pv, double *self_part)
{
    int64_t nblk = (p1 - p0 + kBlock - 1) / kBlock;
    if (nblk > 0x7fffffff) return fail(Z3_ERR_OVERFLOW, "too many pivot blocks");
    if ((self_part != nullptr) != (self_pv != nullptr) || (self_part && idhash))
        return fail(Z3_ERR_INVALID_ARG, "k_multipoles: the self-pair sums need pivot values and no fingerprints");
    MultArgs a;
    a.px = piv.x; a.py = piv.y; a.pz = piv.z;
    a.rec = idx->d_rec + (size_t)map * 2 * idx->n;
    a.wdbl = idx->unit_w ? nullptr : idx->d_wdbl;
    a.permdbl = idx->d_permdbl;
    a.cell_start = idx->d_cell_start;
    a.bands = idx->d_bands;
    a.nbands = idx->nbands;
    a.inv_h = 1.0 / idx->band_h;
    a.edges = idx->d_edges;
    a.nb = idx->nbins;
    a.p0 = p0; a.p1 = p1;
    a.norm = norm;
    a.A = A; a.ldA = ldA;
    a.W = W; a.counts = counts; a.idhash = idhash; a.pair_total = pair_total;
    a.pv = self_pv; a.self_part = self_part;
    a.px0 = idx->plane_x0; a.py0 = idx->plane_y0; a.psx = idx->plane_sx;
    a.tiny = kBearingTiny;
    a.nblocks = (int)nblk;
    a.groups = bin_groups(idx, nblk);
    const bool mixed = prec == Z3_PREC_MIXED, ids = idhash != nullptr, self = self_part != nullptr;
    hipEvent_t ev0;
    profile_begin(s, &ev0);
    if (!ids && short_windows(idx)) {
        const z3_status st = launch_multipoles_list(m_max, idx->planar, mixed, self, a, s);
        profile_end(s, ev0);
        return st;
    }
    switch (m_max) {
#define Z3_CASE(MM) case MM: launch_m<MM>(idx->planar, mixed, ids, self, a, s); break;
        Z3_CASE(0) Z3_CASE(1) Z3_CASE(2) Z3_CASE(3) Z3_CASE(4) Z3_CASE(5) Z3_CASE(6) Z3_CASE(7)
        Z3_CASE(8) Z3_CASE(9) Z3_CASE(10) Z3_CASE(11) Z3_CASE(12) Z3_CASE(13) Z3_CASE(14)
        Z3_CASE(15) Z3_CASE(16)
#undef Z3_CASE
    default: return fail(Z3_ERR_UNSUPPORTED, "m_max=%d not compiled", m_max);
    }
    z3_status st = check_launch("k_multipoles");
    profile_end(s, ev0);
    return st;
}

}  // namespace z3
