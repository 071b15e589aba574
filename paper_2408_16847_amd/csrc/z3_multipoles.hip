// Launches of the one-map multipole kernel (z3_multipoles_device.h) and the rules they follow.
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
//
// The density is that of the whole colatitude range, which a catalogue on a part of the sky fills
// in part: such a catalogue reads shorter windows than it has.  Pixelised patches of 5 and 15 degrees
// (Nside 256 to 1024, 1,500 to 214,000 points, one map and four a lane) read 0.1 to 7.5 and walk lists:
// 1.01-1.66 times as fast as in lockstep at 4 to 22 real pairs a window, 0.89-1.35 at 40 to 176 (0.94 in
// the middle at 15 degrees, where there are enough blocks, 1.08 at 5, where few).  At the density
// where the points are (1/4 to 1/40 of the circle) all but the first would go in lockstep, and lose
// more than they gain.
constexpr double kShortWindow = 8.0;

double pairs_a_window(const z3_index_s *idx, bool occupied)
{
    const EdgeTab &t = idx->edges;
    const int nb = idx->nbins;
    double windows = 0.0;
    for (int b = 1; b <= nb; ++b) windows += 4.0 * t.rad_out[b] / idx->band_h + 2.0;
    return idx->density / (occupied ? idx->sky_part : 1.0) * kPi * (t.e[nb] - t.e[0]) / windows;
}

bool short_windows(const z3_index_s *idx) { return pairs_a_window(idx, false) < kShortWindow; }

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
