// Ball search + binning + multipole accumulation (eqs. Xm.binned and Ym/Zm.binned).
//
// Work decomposition: one lane per pivot, 64 consecutive index-order pivots per wave
// (neighbouring points of one latitude band, so their neighbour windows overlap and the
// lanes' loads of neighbour points fall on the same cache lines).  Each lane walks the
// radial bins in order; for bin b it visits, band by band, only the longitude window
// that can hold neighbours at chord-squared distance in [E_b, E_{b+1}), and keeps the
// bin's sums in registers:
//
//   Y_m = sum w_j x_j cos(m phi),  Z_m = sum w_j x_j sin(m phi),  W = sum w_j,  N = #pairs
//
// so a_{m,b} = Y_m - i Z_m.  There are no atomics and no cross-lane reductions, and the
// summation order of every (pivot, bin) is fixed, so results are bit-reproducible.
//
// Exactness of the pair decision: d2 = (dx*dx + dy*dy) + dz*dz in FP64 with every
// operation rounded separately (this file is compiled with -ffp-contract=off), compared
// with the caller's FP64 edges.  The longitude windows are conservative (rounding
// guards), so they never drop a pair that the d2 test accepts.
//
// Harmonics: the paper's remark after the binned estimator builds cos(m phi) and
// sin(m phi) from Chebyshev polynomials of cos(phi), so that no trigonometric function is
// evaluated per pair.  The 2 M + 1 sums of a bin need a basis of the trigonometric
// polynomials of degree M, not the harmonics themselves; HarmonicSums takes products of two
// short factors, whose sums cost one FMA each and whose factors are few (see there), and the
// bin's epilogue turns the sums into Y_m and Z_m by the product-to-sum identities.
//
// Pivots on a plane (PLANAR): the same loop over a strip x cell grid of (x, y, 0) records;
// the frame is fixed (angles from +y towards +x) and the windows are planar_window's.
//
// Optionally (SELF) the kernel also removes the k = j terms of the contraction's diagonal
// (the overcount the paper points out in the kappa^3 multipole-signal subsection): per
// (pivot, bin) it sums Q = sum_j (w_j x_j)^2 in FP64, forms v_p Q / W^2 (v_p Q for raw
// sums), adds that over the wave in a fixed order and writes one value per (wave, bin).
//
// Precision: both paths form the separation, the exact squared chord, the bearing (an
// FP32-seeded reciprocal square root refined by one FP64 Newton step) and the harmonics in
// FP64 and add them into FP64 bin sums; the mixed path stores the normalised multipoles in
// FP32 for its split-FP32 MFMA contraction.  An FP32 bearing or FP32 recurrences would carry
// an angle error of ~1e-7 per pair, which the m-th harmonic multiplies by m: ~1e-6 at
// m = 10 on fields whose 3PCF is a sum of terms of random sign.  On this hardware the FP32
// vector instructions (packed forms excluded) issue at the FP64 rate, so the FP64 harmonics
// cost the same instructions and are exact to ~1e-15.
#pragma once

#include "z3_internal.h"
#include "z3_device.h"

namespace z3 {

struct MultArgs {
    const double *px, *py, *pz;   // index-order positions (the pivots)
    const double4 *rec;           // doubled-band records {x, y, z, w x} of the map
    const double *wdbl;           // doubled-band weights, or null when all weights are 1
    const int *permdbl;           // doubled-band original indices (neighbour fingerprints)
    const int *cell_start;
    const Band *bands;
    int nbands;
    double inv_h;
    const EdgeTab *edges;
    int nb;
    int64_t p0, p1;
    int norm;
    void *A;
    int64_t ldA;
    double *W;
    int64_t *counts;
    uint64_t *idhash;
    uint64_t *pair_total;
    const double *pv;             // SELF: index-order pivot products w_p x_p
    double *self_part;            // SELF: [waves of the launch][nb] sums of v_p Q / W^2
    double px0, py0, psx;         // PLANAR: plane origin and cell-coordinate scale
    double tiny;                  // kBearingTiny, passed so that it sits in scalar registers
    int nblocks;
    BinGroups groups;             // bins of each blockIdx.y
};

// Sums over a bin's pairs of v times a basis of the trigonometric polynomials of degree <= M,
// v = w_j x_j.  With B_0 = 1, B_k = 2 T_k(cos phi) = 2 cos(k phi) (B_1 = t = 2 cos phi, B_2 = t t - 2,
// B_{k+1} = t B_k - B_{k-1}) and s = 2 sin phi the basis is
//   B_0..B_H,  B_H B_1..B_H B_{M-H},  s B_0..s B_{H-1},  s B_H B_0..s B_H B_{M-H-1},
// from H - 1 steps of the chain and the three weights v B_H, v s and v s B_H: H + 2 operations
// a pair beside the 2 M + 1 additions into the sums that any method needs, against M for one
// chain over all degrees (31 -> 28 FP64 instructions a pair at M = 10, 49 -> 43 at M = 16).
// H = ceil(M / 2); up to M = 4 the products save nothing and H = M leaves them out.  finish()
// recovers the harmonics from
//   B_H B_j = 2 (T_{H+j} + T_{H-j})  and  s B_k = 2 (sin (k+1) phi - sin (k-1) phi):
// every step adds sums of size sum |v| with factors of 1 or 1/2, so no bits are lost near
// phi = 0 and pi as in the second-kind basis (U_m ~ m + 1 there).  Measured against that one
// chain: Nside 512 at M = 16 65.6 -> 58.0 ms a launch (with 3 waves per SIMD in place of 2),
// half of Nside 1024 at M = 10 160.5 -> 156.7 ms, 786,000 pivots at M = 10 2669 -> 2617 us.
template <int M>
struct HarmonicSums {
    static constexpr int H = M <= 4 ? M : (M + 1) / 2;
    static constexpr int R = M - H;
    double c[M + 1];  // B_k (k <= H), B_H B_j at H + j
    double s[M + 1];  // s B_{k-1} at k (1 <= k <= H), s B_H B_j at H + 1 + j

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int m = 0; m <= M; ++m) { c[m] = 0.0; s[m] = 0.0; }
    }

    // one pair: tc = 2 cos phi, ts = 2 sin phi
    __device__ __forceinline__ void add(double v, double tc, double ts)
    {
        c[0] += v;
        if constexpr (M >= 1) {
            double B[H + 1];
            B[1] = tc;
            if constexpr (H >= 2) B[2] = fma(tc, tc, -2.0);
#pragma unroll
            for (int k = 3; k <= H; ++k) B[k] = fma(tc, B[k - 1], -B[k - 2]);
            const double vs = v * ts;
            s[1] += vs;
#pragma unroll
            for (int k = 1; k < H; ++k) {
                c[k] = fma(v, B[k], c[k]);
                s[k + 1] = fma(vs, B[k], s[k + 1]);
            }
            if constexpr (R == 0) {
                c[H] = fma(v, B[H], c[H]);
            } else {
                const double vg = v * B[H], vsg = vs * B[H];
                c[H] += vg;
                s[H + 1] += vsg;
#pragma unroll
                for (int j = 1; j <= R; ++j) {
                    c[H + j] = fma(vg, B[j], c[H + j]);
                    if (j < R) s[H + 1 + j] = fma(vsg, B[j], s[H + 1 + j]);
                }
            }
        }
    }

    // c[m] = sum v cos(m phi), s[m] = sum v sin(m phi)
    __device__ __forceinline__ void finish()
    {
#pragma unroll
        for (int k = 1; k <= H; ++k) {
            c[k] *= 0.5;
            s[k] = k >= 2 ? fma(0.5, s[k], s[k >= 2 ? k - 2 : 0]) : 0.5 * s[k];
        }
#pragma unroll
        for (int j = 1; j <= R; ++j) c[H + j] = fma(0.5, c[H + j], -c[H - j]);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            // s_{H+1+j} = S / 2 + s_{H+j-1} - s_{H-j+1} + s_{H-j-1}, the last two for j >= 1
            double t = fma(0.5, s[H + 1 + j], s[H + j - 1]);
            if (j >= 1) t = t - s[H - j + 1] + s[H - j - 1];
            s[H + 1 + j] = t;
        }
    }
};

// Occupancy target of the multipole kernel (waves per SIMD that the register allocation
// aims for).  Measured on MI355X at m_max = 10: 4 waves beat 3 by ~15% although up to 33
// registers of the band loop spill; from m_max = 11 the sums need more registers, and 3 waves hold
// them (a few of the band loop's spill from m_max = 12 on, 23 at 16).
#ifndef Z3_MULT_WAVES_PER_EU
#define Z3_MULT_WAVES_PER_EU 4
#endif
template <int M>
constexpr int mult_waves_per_eu()
{
    return M <= 10 ? Z3_MULT_WAVES_PER_EU : 3;
}

// LIST: the lanes list their windows of kWinBands bands and walk the lists on their own, else all
// lanes walk a band's windows before the next band's; the launch chooses (short_windows).
// Bands whose windows a lane lists before it walks them (17 x 512 B of LDS per wave: four blocks
// of four waves fit a CU).  A lane goes on to its next window while others are still in theirs,
// so a wave's trips follow its lanes' total numbers of candidates, not the longest window of
// every band, and the first records of a window are requested while the last of the one before
// are worked on.
constexpr int kWinBands = 8;
constexpr uint32_t kNoRecord = 0xffffffe0u;  // past any band's records (a multiple of 64 B below 2^32)

// Lists this lane's windows of the bands from k on, at most kWinBands of them (fewer when their
// records span 2^32 bytes) and up to khi: byte ranges of the doubled records from record `base`
// on, ended by kNoRecord.  Moves k past the bands listed; returns the bytes they span (every
// byte offset of the list lies below).  `window(band, s0, l0, s1, l1)` gives a band's windows.
template <class Window>
__device__ __forceinline__ uint32_t list_windows(const Band *bands, int &k, int khi, uint2 *list, int &base,
                                                 Window window)
{
    base = 2 * bands[k].pt_start;
    uint32_t span = 0;
    const int kend = min(khi + 1, k + kWinBands);
    for (; k < kend; ++k) {
        const Band bd = bands[k];
        if (bd.npts == 0) continue;
        // one band's records span less than 2^32 bytes (checked when the index is built)
        const uint64_t reach = (uint64_t)(2 * (int64_t)(bd.pt_start + bd.npts) - base) * 32u;
        if (reach > UINT32_MAX) break;
        span = (uint32_t)reach;
        int s0, l0, s1, l1;
        window(bd, s0, l0, s1, l1);
        const uint32_t first = (uint32_t)(2 * bd.pt_start - base);
        if (l0 > 0) {
            *list = make_uint2((first + s0) * 32u, (first + s0 + l0) * 32u);
            list += kWave;
        }
        if (l1 > 0) {
            *list = make_uint2((first + s1) * 32u, (first + s1 + l1) * 32u);
            list += kWave;
        }
    }
    *list = make_uint2(kNoRecord, kNoRecord);
    return span;
}

// The records of a list of windows, one after the other; kNoRecord after the last.
struct ListWalk {
    const uint2 *at;
    uint32_t end;
    __device__ __forceinline__ explicit ListWalk(const uint2 *list) : at(list), end(0) {}
    __device__ __forceinline__ uint32_t first() { return window(); }
    __device__ __forceinline__ uint32_t next(uint32_t o)
    {
        o += 32u;
        if (o >= end) o = window();
        return o;
    }
    __device__ __forceinline__ uint32_t window()
    {
        const uint2 w = *at;
        at += kWave;
        end = w.y;
        return w.x;
    }
};

template <int M, bool F32OUT, bool IDS, bool SELF, bool PLANAR, bool LIST>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(mult_waves_per_eu<M>())))
void k_multipoles(MultArgs a)
{
    // XCD-aware order: hardware hands consecutive block ids to the 8 XCDs in turn;
    // give each XCD a contiguous run of pivot tiles so neighbour data stays in its L2.
    const int nblk = a.nblocks;
    const int bid = blockIdx.x;
    const int per = nblk / 8, rem = nblk % 8;
    const int xcd = bid % 8, k8 = bid / 8;
    const int lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k8;
    const int64_t wave0 = a.p0 + (int64_t)lb * kBlock + (threadIdx.x & ~(kWave - 1));
    if (__builtin_amdgcn_readfirstlane((int)(wave0 >= a.p1))) return;  // whole wave past the end
    const int64_t p = a.p0 + (int64_t)lb * kBlock + threadIdx.x;
    const bool valid = p < a.p1;
    const int64_t pp = valid ? p : a.p1 - 1;  // idle lanes shadow the last pivot

    const double xp = a.px[pp], yp = a.py[pp], zp = a.pz[pp];
    double th, sh = 0.0, ch = 0.0, phd = 0.0;
    float inv_sp = 0.0f, phf = 0.0f;
    // local north n and east e.  Off the poles e = n x r_p = (-y, x, 0) / |n| has no z
    // component for any pivot length; in the pole fallback (north along x, |y| < 1e-12) its z
    // component is y / |n|, and leaving that term out of the east coordinate turns the
    // bearing by less than 1e-12 |dz| / |d| (dz ~ |d|^2 / 2 there).  So e_z is never used.
    double nx, ny, nz, ex, ey;
    if constexpr (PLANAR) {
        // plane: strips of y, cells of x; angles from +y ("north") towards +x ("east")
        th = yp - a.py0;
        phd = (xp - a.px0) * a.psx;
        nx = 0.0; ny = 1.0; nz = 0.0;
        ex = 1.0; ey = 0.0;
    } else {
        const double sinth = sqrt(xp * xp + yp * yp);
        th = atan2(sinth, zp);
        double ph = atan2(yp, xp);
        if (ph < 0.0) ph += kTwoPi;
        sincos(0.5 * th, &sh, &ch);
        inv_sp = sinth > 0.0 ? (float)(1.0 / sinth) : INFINITY;
        phf = (float)ph;
        // local north and east
        nx = -zp * xp; ny = -zp * yp; nz = 1.0 - zp * zp;
        double nn = sqrt(nx * nx + ny * ny + nz * nz);
        if (nn < 1e-12) {
            nx = 1.0 - xp * xp; ny = -xp * yp; nz = -xp * zp;
            nn = sqrt(nx * nx + ny * ny + nz * nz);
        }
        nx /= nn; ny /= nn; nz /= nn;
        ex = ny * zp - nz * yp; ey = nz * xp - nx * zp;
    }

    // External pivots need not be unit vectors (the index's points are, to within the
    // windows' guards).  For a pivot of length rho = 1 + d and a unit neighbour at angle t,
    // the chord test reads d2 = d^2 + rho 4 hav(t), so the pair lies in [E_lo, E_hi) iff
    // hav(t) lies in [(E_lo - d^2) / 4 rho, (E_hi - d^2) / 4 rho): the wave's windows then
    // use the envelope of those bounds over its lanes (wave-uniform, per bin).
    double dmin = 0.0, dmax = 0.0;
    if constexpr (!PLANAR) {
        const double dp = sqrt(xp * xp + yp * yp + zp * zp) - 1.0;
        dmin = dp; dmax = dp;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            dmin = fmin(dmin, __shfl_xor(dmin, o, kWave));
            dmax = fmax(dmax, __shfl_xor(dmax, o, kWave));
        }
        dmin = uniform_f64(dmin);
        dmax = uniform_f64(dmax);
    }
    const bool rescale = __builtin_amdgcn_readfirstlane((int)!(dmin >= -kPivotNormTol && dmax <= kPivotNormTol));

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
        double hav_out = a.edges->hav_out[bin + 1], hav_in = a.edges->hav_in[bin];
        double rad = a.edges->rad_out[bin + 1];
        if (rescale) {
            const double dsq = fmax(dmin * dmin, dmax * dmax);
            hav_out = 1.0 + fmin(dmin, 0.0) > 1e-3 ? fmin(hav_out / (1.0 + dmin) * (1.0 + 1e-15), 1.0 + 2e-9)
                                                   : 1.0 + 2e-9;
            hav_in = (hav_in - 0.25 * dsq) / (1.0 + fmax(dmax, 0.0)) * (1.0 - 1e-15) - 1e-300;
            rad = 2.0 * asin(fmin(1.0, sqrt(hav_out))) * (1.0 + 1e-9) + 1e-12;
            if (!(hav_in <= hav_out)) hav_in = -1.0;  // non-finite pivots: no inner exclusion
        }
        int klo = (int)floor((th - rad) * a.inv_h);
        int khi = (int)floor((th + rad) * a.inv_h);
        klo = max(klo, 0);
        khi = min(khi, a.nbands - 1);
        klo = __builtin_amdgcn_readfirstlane(wave_min(klo));
        khi = __builtin_amdgcn_readfirstlane(wave_max(khi));

        HarmonicSums<M> sums;
        sums.clear();
        // wpend: the weight of the lane's previous pair, added at its next pair (or after the
        // bin), so that its load overlaps a candidate's work instead of stalling the pair that
        // requested it; the additions keep their order
        double Wb = 0.0, Qb = 0.0, wpend = 0.0;
        int cnt = 0;
        uint64_t hsum = 0;

        // one candidate: its record r at byte offset o of the records from `base` on
        auto cand = [&](const double4 &r, uint32_t o, int base, __amdgpu_buffer_rsrc_t wband) __attribute__((always_inline)) {
            const double dx = r.x - xp, dy = r.y - yp;
            // on the plane both z are 0, and adding dz * dz = +0 to the
            // non-negative sum changes nothing: the same d2 without that term
            const double dz = PLANAR ? 0.0 : r.z - zp;
            const double d2 = PLANAR ? dx * dx + dy * dy : (dx * dx + dy * dy) + dz * dz;
            if (d2 >= elo && d2 < ehi) {
                cnt += 1;
                if constexpr (IDS) {
                    // record index from the byte offset, as an opaque shift so
                    // that the compiler keeps no second induction variable
                    uint32_t jo;
                    asm("v_lshrrev_b32 %0, 5, %1" : "=v"(jo) : "v"(o));
                    hsum += mix64((uint64_t)a.permdbl[base + (int)jo]);
                }
                if (!unit_w) {  // wave-uniform
                    Wb += wpend;
                    wpend = load_f64(wband, o >> 2);
                }
                const double v = r.w;
                if constexpr (SELF) Qb = fma(v, v, Qb);
                // plane: north +y, east +x, so the coordinates are dy and dx
                const double u1 = PLANAR ? dy : fma(dx, nx, fma(dy, ny, dz * nz));
                const double u2 = PLANAR ? dx : fma(dx, ex, dy * ey);
                double tc, ts;  // 2 cos(phi), 2 sin(phi)
                twice_unit_bearing(u1, u2, a.tiny, tc, ts);
                sums.add(v, tc, ts);
            }
        };
        if constexpr (LIST) {
            for (int k = klo; k <= khi;) {
                int base;
                const uint32_t span = list_windows(
                    a.bands, k, khi, list, base, [&](const Band &bd, int &s0, int &l0, int &s1, int &l1) {
                        if constexpr (PLANAR)
                            planar_window(bd, a.cell_start, th, phd, a.psx, hav_out, hav_in, s0, l0, s1, l1);
                        else
                            band_window(bd, a.cell_start, th, sh, ch, inv_sp, phf, hav_out, hav_in, s0, l0, s1, l1);
                    });
                // their doubled records (wave-uniform base), walked by byte offset, and doubled
                // weights (8 B per record: byte offset = record offset / 4)
                const __amdgpu_buffer_rsrc_t rband = buffer_view(a.rec + base, span);
                const __amdgpu_buffer_rsrc_t wband = buffer_view(unit_w ? nullptr : a.wdbl + base, unit_w ? 0u : span >> 2);
                // one candidate at a time, its record requested one candidate ahead so that an L2
                // or HBM miss overlaps the previous candidate's work; two candidates per trip with
                // two record registers in turn, so the record requested ahead needs no copy.  A
                // request at kNoRecord lies past the buffer's range and reads nothing.
                ListWalk walk(list);
                uint32_t oa = walk.first();
                double4 ra = load_record(rband, oa);
                while (oa != kNoRecord) {
                    const uint32_t ob = walk.next(oa);
                    const double4 rb = load_record(rband, ob);
                    cand(ra, oa, base, wband);
                    if (ob == kNoRecord) break;
                    oa = walk.next(ob);
                    ra = load_record(rband, oa);
                    cand(rb, ob, base, wband);
                }
            }
        } else {
            for (int k = klo; k <= khi; ++k) {
                const Band bd = a.bands[k];
                if (bd.npts == 0) continue;
                int s0, l0, s1, l1;
                if constexpr (PLANAR)
                    planar_window(bd, a.cell_start, th, phd, a.psx, hav_out, hav_in, s0, l0, s1, l1);
                else
                    band_window(bd, a.cell_start, th, sh, ch, inv_sp, phf, hav_out, hav_in, s0, l0, s1, l1);
                const int base = 2 * bd.pt_start;
                // the band's doubled records (wave-uniform base), walked by byte offset
                const __amdgpu_buffer_rsrc_t rband = buffer_view(a.rec + base, (uint32_t)bd.npts * 64u);
                // and its doubled weights (8 B per record: byte offset = record offset / 4)
                const __amdgpu_buffer_rsrc_t wband = buffer_view(unit_w ? nullptr : a.wdbl + base,
                                                                 unit_w ? 0u : (uint32_t)bd.npts * 16u);
#pragma unroll
                for (int seg = 0; seg < 2; ++seg) {
                    uint32_t off = (uint32_t)(seg == 0 ? s0 : s1) * 32u;
                    const uint32_t oend = off + (uint32_t)(seg == 0 ? l0 : l1) * 32u;
                    {
                        // one candidate at a time, its record requested one candidate ahead so
                        // that an L2 or HBM miss overlaps the previous candidate's work; two
                        // candidates per trip with two record registers in turn, so the record
                        // requested ahead needs no copy.  Past the window a request reads a
                        // record of the band that is never used (or, past the band, zeros from
                        // the buffer's range check).
                        double4 ra = load_record(rband, off < oend ? off : 0u);
                        for (; off < oend; off += 64u) {
                            const double4 rb = load_record(rband, off + 32u);
                            cand(ra, off, base, wband);
                            if (off + 32u >= oend) break;
                            ra = load_record(rband, off + 64u);
                            cand(rb, off + 32u, base, wband);
                        }
                    }
                }
            }
        }

        Wb += wpend;
        double self_t = 0.0;
        if (valid) {
            my_pairs += (uint64_t)cnt;
            if (unit_w) Wb = (double)cnt;
            double inv = 1.0;
            if (a.norm == Z3_NORM_BIN) inv = Wb > 0.0 ? 1.0 / Wb : 0.0;
            if constexpr (SELF) self_t = a.pv[p] * Qb * inv * inv;
            if (a.A) {
                sums.finish();
#pragma unroll
                for (int m = 0; m <= M; ++m) {
                    const double re = sums.c[m] * inv;
                    const double im = m == 0 ? 0.0 : -sums.s[m] * inv;
                    const size_t ore = ((size_t)(2 * m) * nb + bin) * (size_t)a.ldA + col;
                    const size_t oim = ((size_t)(2 * m + 1) * nb + bin) * (size_t)a.ldA + col;
                    if constexpr (F32OUT) {
                        static_cast<float *>(a.A)[ore] = (float)re;
                        static_cast<float *>(a.A)[oim] = (float)im;
                    } else {
                        static_cast<double *>(a.A)[ore] = re;
                        static_cast<double *>(a.A)[oim] = im;
                    }
                }
            }
            const size_t ob = (size_t)bin * (size_t)a.ldA + col;
            if (a.W) a.W[ob] = Wb;
            if (a.counts) a.counts[ob] = cnt;
            if constexpr (IDS) a.idhash[ob] = hsum;
        }
        if constexpr (SELF) {
            const double t = wave_sum_f64(self_t);
            if ((threadIdx.x & (kWave - 1)) == 0)
                a.self_part[(size_t)((wave0 - a.p0) / kWave) * nb + bin] = t;
        }
    }

    if (a.pair_total) {
        const uint64_t tot = wave_sum_u64(valid ? my_pairs : 0);
        if ((threadIdx.x & (kWave - 1)) == 0 && tot) atomicAdd((unsigned long long *)a.pair_total, (unsigned long long)tot);
    }
}

// Launch over window lists (z3_multipoles_list.hip).
z3_status launch_multipoles_list(int m_max, bool planar, bool mixed, bool self, const MultArgs &a, hipStream_t s);

}  // namespace z3
