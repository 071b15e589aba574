// What the two many-map kernels on MFMA share: their arguments, block shapes and the harmonic row
// of a pair (internal).
#pragma once

#include "z3_batch_device.h"

namespace z3 {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct BatchArgs {
    const double4 *rec;           // [2n] doubled records (x, y, z, .)
    const void *vmat;             // [2n][ldv] doubled per-map values w * x (FP64 or FP32)
    int ldv;                      // maps padded to a multiple of 32 (zeros)
    const double *wdbl;           // [2n] doubled weights, or null for unit weights
    const int *cell_start;
    const Band *bands;
    int nbands;
    double inv_h;
    const EdgeTab *edges;
    int nb;
    const double *px, *py, *pz;   // pivots (index order)
    int64_t p0, p1;
    int nmaps;                    // maps written (rows >= nmaps are padding)
    int ntiles;                   // map tiles of one pivot (blocks per pivot)
    void *stage;                  // [P][nb][nmaps][2 (m+1)] pivot-major multipoles (re, im per m)
    double *W;                    // [nb][ldA] W_{p,b}, or null
    int64_t ldA;
    uint64_t *pair_total;
    int nblocks;
    uint32_t vmat_bytes;          // size of vmat, below 4 GiB (kernel over many bins only)
};

// Block shapes the library is built with: waves per block, 16-map tiles per wave.
struct BatchShape { int wpb, ti; };
constexpr BatchShape kBatchShapes[] = {{4, 1}, {2, 2}, {2, 1}, {4, 2}};
constexpr int kNumBatchShapes = sizeof(kBatchShapes) / sizeof(kBatchShapes[0]);

template <bool F32> struct BatchT { typedef double T; typedef v4d V4; };
template <> struct BatchT<true> { typedef float T; typedef v4f V4; };

// Harmonic row h[c] of a pair that is in a bin, from its separation (dx, dy, dz).
template <int M, class T>
__device__ __forceinline__ void harmonic_row(const PivotFrame &f, double dx, double dy, double dz, T (&h)[2 * M + 1])
{
    const double u1 = fma(dx, f.nx, fma(dy, f.ny, dz * f.nz));
    const double u2 = fma(dx, f.ex, dy * f.ey);
    double c1, sn1;
    unit_bearing(u1, u2, c1, sn1);
    // cos(m phi) = T_m(cos phi), sin(m phi) = sin phi U_{m-1}(cos phi): the
    // three-term recurrence in FP64 on both paths (as cheap as FP32 on this
    // hardware, and free of the recurrence's error growth in FP32); the mixed
    // path rounds each harmonic to FP32 once
    h[0] = T(1);
    if constexpr (M >= 1) {
        const double tc = c1 + c1;
        double t2 = 1.0, t1 = c1, u2s = 0.0, u1s = sn1;
        h[1] = (T)t1;
        h[M + 1] = (T)u1s;
#pragma unroll
        for (int m = 2; m <= M; ++m) {
            const double tm = fma(tc, t1, -t2);
            const double sm = fma(tc, u1s, -u2s);
            h[m] = (T)tm;
            h[M + m] = (T)sm;
            t2 = t1; t1 = tm;
            u2s = u1s; u1s = sm;
        }
    }
}

// The kernel over many bins at a time (z3_batch_bins.hip): whether the launch takes it, and the
// launch.
bool batch_many_bins(const z3_index_s *idx, bool f32);
z3_status launch_batch_bins(int m_max, bool f32, int shape, const BatchArgs &a, hipStream_t s);

}  // namespace z3
