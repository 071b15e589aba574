// The register-tiled many-map kernel: several maps per lane over one set of positions.
#include "z3_multipoles_device.h"

namespace z3 {

// ---- many maps over one set of positions -------------------------------------------------
//
// Same decomposition and walks as k_multipoles (one lane per pivot, bins in order, window
// lists where windows are short), but every lane carries K maps of a group of kMapGroup: the
// pair test, the bearing and the unit chain U_k(cos phi) are computed once per pair, and each
// map adds v U_k and v 2 sin(phi) U_k with two FMAs per k (the epilogue forms the harmonics'
// sums from T_m = (U_m - U_{m-2}) / 2 and sin(m phi) = sin(phi) U_{m-1}; the product basis of
// HarmonicSums would cost each map two more multiplications a pair).
//
// At two waves per SIMD nothing hides a miss but the lane's own work, so a candidate's record
// and its group's values are both requested one candidate ahead.  Measured for four maps:
// Nside 512 at m_max = 10 139.6 -> 107.0 ms an estimate, Nside 128 2.39 -> 1.43 ms (there on
// lists, 1.58 band by band).
//
// Four maps' values requested ahead spill in the candidate loop from m_max 5 on at three waves per
// SIMD, and at m_max 11 on lists also at two; the first run at two waves from there, the last
// loads them when a pair is found (Nside 192, 5 bins of 28 to 300 pairs, four maps: m_max 5 2386 ->
// 1672 us, 6 3836 -> 1784 us, 11 4606 -> 3741 us).  Two maps at m_max 12 likewise (4390 -> 3602 us).
//
// K = 3 when the caller reads at most the first three maps of the group, else 4 up to m_max =
// kTileMmax; beyond, the 2 K (2 m_max + 1) registers of four maps' sums no longer fit beside the
// requests, and blockIdx.z takes the group two maps at a time (Nside 128, m_max = 16: 15.4 ->
// 2.5 ms; four maps a lane spill in the candidate loop).  Three maps keep their sums up to m_max
// = 16, but from 13 on not the values requested ahead (they are loaded when a pair is found),
// and from 15 on not the record either.
constexpr int kTileMmax = 11;
template <int M, int K, bool LIST> constexpr bool maps_values_ahead()
{
    return K == 2 || (K == 3 ? M <= 12 : M <= (LIST ? 10 : 11));
}
template <int M, int K> constexpr bool maps_record_ahead() { return K != 3 || M <= 14; }

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

template <int M, int K>
constexpr int maps_waves_per_eu()
{
    return M <= (K == 2 ? 11 : (K == 3 ? 6 : 4)) ? 3 : 2;
}

template <int M, bool F32OUT, int K, bool LIST>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(maps_waves_per_eu<M, K>())))
void k_multipoles_maps(MapArgs a)
{
    static_assert(K >= 2 && K <= kMapGroup, "two to four maps per lane");
    const int slot0 = K * (int)blockIdx.z;  // first map of the group that this block carries
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
    __shared__ uint2 lists[LIST ? kBlock / kWave : 1][LIST ? 2 * kWinBands + 1 : 1][kWave];
    uint2 *list = &lists[LIST ? threadIdx.x / kWave : 0][0][threadIdx.x & (kWave - 1)];  // this lane's windows

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
        double Wb = 0.0, wpend = 0.0;
        int cnt = 0;

        // one candidate: its record r, its byte offset o of the window's records and the group's
        // values, requested `ahead` or loaded when the pair is found
        constexpr bool AHEAD = maps_values_ahead<M, K, LIST>();
        auto cand = [&](const double4 &r, const double4 &ahead, uint32_t o, __amdgpu_buffer_rsrc_t vband,
                        __amdgpu_buffer_rsrc_t wband) __attribute__((always_inline)) {
            const double dx = r.x - xp, dy = r.y - yp, dz = r.z - zp;
            const double d2 = (dx * dx + dy * dy) + dz * dz;
            if (d2 >= elo && d2 < ehi) {
                cnt += 1;
                if (!unit_w) {  // wave-uniform; the weight is added at the next pair, as in k_multipoles
                    Wb += wpend;
                    wpend = load_f64(wband, o >> 2);
                }
                const double4 vv = AHEAD ? ahead : load_record(vband, o);
                double v[K];
                v[0] = vv.x; v[1] = vv.y;
                if constexpr (K >= 3) v[2] = vv.z;
                if constexpr (K >= 4) v[3] = vv.w;
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
        };
        // this block's values of the record at byte offset o
        auto load_values = [&](__amdgpu_buffer_rsrc_t v, uint32_t o) __attribute__((always_inline)) {
            if constexpr (!AHEAD) {
                return double4{};
            } else if constexpr (K == 2) {
                const double2 q = load_f64x2(v, o + 16u * (uint32_t)blockIdx.z);
                return make_double4(q.x, q.y, 0.0, 0.0);
            } else {
                return load_record(v, o);
            }
        };
        for (int kb = klo; kb <= khi;) {
            auto window = [&](const Band &bd, int &s0, int &l0, int &s1, int &l1) {
                band_window(bd, a.cell_start, th, sh, ch, inv_sp, phf, hav_out, hav_in, s0, l0, s1, l1);
            };
            if constexpr (LIST) {
                int base;
                const uint32_t span = list_windows(a.bands, kb, khi, list, base, window);
                const __amdgpu_buffer_rsrc_t rband = buffer_view(a.rec + base, span);
                const __amdgpu_buffer_rsrc_t vband = buffer_view(a.vgrp + (size_t)base * kMapGroup, span);
                const __amdgpu_buffer_rsrc_t wband = buffer_view(unit_w ? nullptr : a.wdbl + base, unit_w ? 0u : span >> 2);
                ListWalk walk(list);
                uint32_t oa = walk.first();
                if constexpr (!maps_record_ahead<M, K>()) {
                    for (; oa != kNoRecord; oa = walk.next(oa)) cand(load_record(rband, oa), double4{}, oa, vband, wband);
                    continue;
                }
                double4 ra = load_record(rband, oa), va = load_values(vband, oa);
                while (oa != kNoRecord) {
                    const uint32_t ob = walk.next(oa);
                    const double4 rb = load_record(rband, ob), vb = load_values(vband, ob);
                    cand(ra, va, oa, vband, wband);
                    if (ob == kNoRecord) break;
                    oa = walk.next(ob);
                    ra = load_record(rband, oa);
                    va = load_values(vband, oa);
                    cand(rb, vb, ob, vband, wband);
                }
            } else {
                const Band bd = a.bands[kb++];
                if (bd.npts == 0) continue;
                int s0, l0, s1, l1;
                window(bd, s0, l0, s1, l1);
                const int base = 2 * bd.pt_start;
                const uint32_t span = (uint32_t)bd.npts * 64u;
                const __amdgpu_buffer_rsrc_t rband = buffer_view(a.rec + base, span);
                const __amdgpu_buffer_rsrc_t vband = buffer_view(a.vgrp + (size_t)base * kMapGroup, span);
                const __amdgpu_buffer_rsrc_t wband = buffer_view(unit_w ? nullptr : a.wdbl + base, unit_w ? 0u : span >> 2);
#pragma unroll
                for (int seg = 0; seg < 2; ++seg) {
                    uint32_t off = (uint32_t)(seg == 0 ? s0 : s1) * 32u;
                    const uint32_t oend = off + (uint32_t)(seg == 0 ? l0 : l1) * 32u;
                    if constexpr (!maps_record_ahead<M, K>()) {
                        for (; off < oend; off += 32u) cand(load_record(rband, off), double4{}, off, vband, wband);
                        continue;
                    }
                    double4 ra = load_record(rband, off < oend ? off : 0u), va = load_values(vband, off < oend ? off : 0u);
                    for (; off < oend; off += 64u) {
                        const double4 rb = load_record(rband, off + 32u), vb = load_values(vband, off + 32u);
                        cand(ra, va, off, vband, wband);
                        if (off + 32u >= oend) break;
                        ra = load_record(rband, off + 64u);
                        va = load_values(vband, off + 64u);
                        cand(rb, vb, off + 32u, vband, wband);
                    }
                }
            }
        }
        Wb += wpend;

        if (valid) {
            my_pairs += (uint64_t)cnt;
            if (unit_w) Wb = (double)cnt;
            const double inv = Wb > 0.0 ? 1.0 / Wb : 0.0;
            const double hinv = 0.5 * inv;
            if (a.W && slot0 == 0) a.W[(size_t)bin * (size_t)a.ldA + col] = Wb;
#pragma unroll
            for (int k = 0; k < K; ++k) {
#pragma unroll
                for (int m = 0; m <= M; ++m) {
                    const double y = m >= 2 ? SU[k][m] - SU[k][m >= 2 ? m - 2 : 0] : SU[k][m];
                    const double re = m == 0 ? y * inv : y * hinv;
                    const double im = m == 0 ? 0.0 : -SV[k][m >= 1 ? m - 1 : 0] * hinv;
                    const size_t ore = (slot0 + k) * a.map_stride + ((size_t)(2 * m) * nb + bin) * (size_t)a.ldA + col;
                    const size_t oim = (slot0 + k) * a.map_stride + ((size_t)(2 * m + 1) * nb + bin) * (size_t)a.ldA + col;
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

    if (a.pair_total && slot0 == 0) {
        const uint64_t tot = wave_sum_u64(valid ? my_pairs : 0);
        if ((threadIdx.x & (kWave - 1)) == 0 && tot) atomicAdd((unsigned long long *)a.pair_total, (unsigned long long)tot);
    }
}

// Whether the launch walks window lists: as in k_multipoles, but four maps at m_max 11 and three at 16,
// which spill in the lists' candidate loop, only below one pair a window, and by the density where
// the points are.  Lists / band by band, three maps at 16 and four at 11, us: at 0.8 pairs a window
// (Nside 192) 1597 / 1662 and 1581 / 1527, at 1.2 3857 / 3902 and 3780 / 3489, at 4.6 3862 / 3295 and 3730 /
// 2833; on a pixelised patch of 54,000 points at 99 (7.5 by the density of the colatitude range) 5377 /
// 3689 and 5187 / 2887.
constexpr double kShortSpilled = 1.0;
static bool walk_lists(const z3_index_s *idx, int m_max, int nslots)
{
    const bool spills = nslots <= 3 ? m_max == 16 : m_max == 11;
    return spills ? pairs_a_window(idx, true) < kShortSpilled : short_windows(idx);
}

template <int M, bool LIST>
static void launch_maps_ml(bool f32out, int nslots, const MapArgs &a, hipStream_t s)
{
    const dim3 grid(a.nblocks, a.groups.n), block(kBlock);
    if (nslots <= 3) {
        if (f32out) hipLaunchKernelGGL((k_multipoles_maps<M, true, 3, LIST>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles_maps<M, false, 3, LIST>), grid, block, 0, s, a);
    } else if constexpr (M > kTileMmax) {
        const dim3 pairs(grid.x, grid.y, kMapGroup / 2);
        if (f32out) hipLaunchKernelGGL((k_multipoles_maps<M, true, 2, LIST>), pairs, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles_maps<M, false, 2, LIST>), pairs, block, 0, s, a);
    } else {
        if (f32out) hipLaunchKernelGGL((k_multipoles_maps<M, true, kMapGroup, LIST>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles_maps<M, false, kMapGroup, LIST>), grid, block, 0, s, a);
    }
}

template <int M>
static void launch_maps_m(bool f32out, int nslots, bool lists, const MapArgs &a, hipStream_t s)
{
    if (lists) launch_maps_ml<M, true>(f32out, nslots, a, s);
    else launch_maps_ml<M, false>(f32out, nslots, a, s);
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
    const bool lists = walk_lists(idx, m_max, nslots);
    hipEvent_t ev0;
    profile_begin(s, &ev0);
    switch (m_max) {
#define Z3_CASE(MM) case MM: launch_maps_m<MM>(f32, nslots, lists, a, s); break;
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

}  // namespace z3
