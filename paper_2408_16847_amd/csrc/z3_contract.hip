// Contraction of the per-pivot multipoles (eqs. zetamEst, zetamEst2) on MFMA.
//
// For every m, with U_p = [Re X_m(0..nb-1; p), Im X_m(0..nb-1; p)] (length 2 nb):
//     G = sum_p v_p U_p U_p^T                       (2nb x 2nb real Gram matrix)
//     Re zeta_m(b1, b2) = G(r1, r2) + G(i1, i2),   Im zeta_m(b1, b2) = G(i1, r2) - G(r1, i2)
// (r = b, i = nb + b), which is sum_p v_p X(b1) conj(X(b2)) written in real arithmetic.
// The Gram matrix is a dense contraction over pivots, formed in 16 x 16 tiles over segments
// of pivots with v_mfma_f64_16x16x4f64 (FP64 path) or v_mfma_f32_16x16x4f32 (mixed path: FP32
// multipoles U; the scaled operand v_p U_i is formed in FP64 and split into FP32 hi + lo
// parts, two MFMAs per step; FP32 sums over 16 pivots are added into FP64 segment sums),
// from the pivot-minor layout of the one-map kernels (through LDS, k_pair_lds; on the mixed path
// up to 32 bins straight into registers, k_pair), or from the many-map kernel's pivot-major
// staging through LDS (k_gram_lds).
// Only tiles on or above the diagonal are formed; entries below are read from their
// mirror, so zeta(b2, b1) is exactly conj(zeta(b1, b2)) and Im zeta(b, b) is exactly 0.
// Segment partials are summed in FP64 in segment order (deterministic).
#include <algorithm>
#include <type_traits>

#include "z3_device.h"

namespace z3 {

// Pivots per segment: at most kSeg (a partial sum of 2 KB a tile pair is then small beside the
// pivots it sums), fewer when the launch would leave the chip idle (one block per segment and
// m: 20,000 pivots at m_max = 8 were 45 blocks of 4096 pivots, 146 us).  kContractUnits bounds
// the partial sums, (segment, map, m, tile pair), that shorter segments may bring, to 16 MB.
constexpr int kSeg = 4096, kSegMin = 128;
constexpr int kContractUnits = 8192;

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

static inline int tiles_for(int nbins) { return (2 * nbins + 15) / 16; }

// Pivots per segment for npiv pivots and `units` (map, m, tile pair) per segment: a multiple of
// kSegMin, with partial sums that fit `bytes` (at least least_bytes).
static int segment_pivots(int64_t npiv, int64_t units, size_t bytes)
{
    const int64_t room = (int64_t)std::min<size_t>(kContractUnits, bytes / (256 * sizeof(double)));
    const int64_t most = std::max<int64_t>(1, room / units);  // segments the bounds allow
    const int64_t len = (npiv + most - 1) / most;
    return (int)std::min<int64_t>(kSeg, (len + kSegMin - 1) / kSegMin * kSegMin);
}

// Bytes of the partial sums (segment, unit) of any call with up to npiv pivots and up to `units`
// per segment (a call's last chunk is shorter, its last group of maps smaller): what the shorter
// segments above take, and the least that a call works with, in segments of kSeg.
static size_t least_bytes(int64_t npiv, int64_t units)
{
    return (size_t)(std::max<int64_t>(1, (npiv + kSeg - 1) / kSeg) * units) * 256 * sizeof(double);
}

static PartialBytes partial_bytes(int64_t npiv, int64_t units)
{
    const int64_t shortest = (npiv + kSegMin - 1) / kSegMin;
    const int64_t n = std::min(shortest * units, std::max<int64_t>(kContractUnits, units));
    const size_t least = least_bytes(npiv, units);
    return PartialBytes{std::max(least, (size_t)n * 256 * sizeof(double)), least};
}

static int64_t contract_units(int m_max, int nbins, int nmaps)
{
    const int T = tiles_for(nbins);
    return (int64_t)nmaps * (m_max + 1) * (T * (T + 1) / 2);
}

PartialBytes contract_partial_bytes(int64_t npiv, int m_max, int nbins, int nmaps)
{
    return partial_bytes(npiv, contract_units(m_max, nbins, nmaps));
}

// Sums of the segments' partials, element by element, into segment 0 (in place: a block reads
// and writes its own 64 columns only).  16 threads of a column take every 16th segment, their
// sums are added in order.  k_gram_reduce alone walked the segments one after the other in
// each of its M1 nb^2 threads: 447 us for 768 segments at m_max = 16.
__global__ __launch_bounds__(1024) void k_segment_sum(double *part, int64_t nseg, int64_t columns)
{
    __shared__ double sh[16][64];
    const int e = threadIdx.x & 63, g = threadIdx.x >> 6;
    double *col = part + (int64_t)blockIdx.x * 64 + e;
    double acc = 0.0;
#pragma unroll 8
    for (int64_t s = g; s < nseg; s += 16) acc += col[s * columns];
    sh[g][e] = acc;
    __syncthreads();
    if (g == 0) {
#pragma unroll
        for (int k = 1; k < 16; ++k) acc += sh[k][e];
        col[0] = acc;
    }
}

// Segments up to which the final reduction takes them itself (one launch less).
constexpr int64_t kDirectSegments = 8;

static z3_status sum_segments(double *part, int64_t *nseg, int64_t columns, hipStream_t s)
{
    if (*nseg <= kDirectSegments) return Z3_OK;
    hipLaunchKernelGGL(k_segment_sum, dim3((unsigned)(columns / 64)), dim3(1024), 0, s, part, *nseg, columns);
    *nseg = 1;
    return check_launch("k_segment_sum");
}

// G(u, v) of one segment, read from the tile holding min/max of (u, v).
__device__ __forceinline__ double gram_at(const double *seg_m, int T, int u, int v)
{
    if (u > v) { int t = u; u = v; v = t; }
    const int I = u >> 4, J = v >> 4;
    const int tp = I * T - I * (I - 1) / 2 + (J - I);
    return seg_m[(size_t)tp * 256 + (u & 15) * 16 + (v & 15)];
}

__global__ void k_gram_reduce(const double *part, int64_t nseg, int nmaps, int M1, int nb, int T, int ntp,
                              double *zeta, size_t z_stride)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int total = nmaps * M1 * nb * nb;
    if (t >= total) return;
    const int mm = t / (nb * nb), rem = t % (nb * nb), b1 = rem / nb, b2 = rem % nb;
    const int map = mm / M1, m = mm % M1;
    const int r1 = b1, r2 = b2, i1 = nb + b1, i2 = nb + b2;
    double rr = 0.0, ii = 0.0, ir = 0.0, ri = 0.0;
    for (int64_t s = 0; s < nseg; ++s) {
        const double *g = part + (size_t)((s * nmaps + map) * M1 + m) * ntp * 256;
        rr += gram_at(g, T, r1, r2);
        ii += gram_at(g, T, i1, i2);
        ir += gram_at(g, T, i1, r2);
        ri += gram_at(g, T, r1, i2);
    }
    double *z = zeta + map * z_stride + ((size_t)(m * nb + b1) * nb + b2) * 2;
    z[0] += rr + ii;
    z[1] += ir - ri;
}

// ---- pair contraction over pivot-minor multipoles -------------------------------------------
// G = sum_p v_p U1_p U2_p^T per (map, m): with U1 = U2 the Gram matrix of one field (only the
// tile pairs on or above the diagonal), else the full product of two fields (the multi-field
// estimator: Re zeta_m(b1, b2) = G(r1, r2) + G(i1, i2), Im zeta_m(b1, b2) = G(i1, r2) -
// G(r1, i2), i.e. sum_p v_p X1(b1) conj(X2(b2))).

struct PairArgs {
    const void *A1, *A2;  // [map][m+1][2][nb][ldA] multipoles of the b1 and b2 fields (Gram: A1 only)
    int64_t ldA;
    int64_t npiv;
    const double *v;      // pivot products w_p x_p of the pivot field
    size_t a_stride;      // elements between the maps' multipoles (Gram of several maps)
    size_t v_stride;      // elements between the maps' pivot products
    int nb, T, M1, nmaps;
    int seg;              // pivots per segment
    int npairs;           // tile pairs per (map, m): T^2, or T (T + 1) / 2 for a Gram matrix
    int ldr;              // k_pair_lds: LDS row length
    double *part;         // [seg][map][m][npairs][256]
};

// k_pair, the mixed path up to T = 4 row tiles (T = 3 for the product of two fields): one block
// of four waves per (segment, map, m).  A wave takes every fourth group of 16 pivots and forms
// all tile pairs of it: lane (row r, quarter q) loads 4 consecutive pivots of row r of each row
// tile, the next group's loads in flight during the current group's MFMAs.  An operand is read
// and split once for all the tile pairs that take it, nothing goes through LDS and the waves
// meet only once, to add their sums in wave order.  The FP32 sums run over the pivots of a
// group in increasing order, four per MFMA (step s takes the pivots 4 s + q): the lanes'
// quadruples are transposed between the four quarters of the wave.
// At 20 bins, m_max = 10 and 6.3e6 pivots (5.5 GB) 5.9 ms, against 7.5 ms for tiles of pivots in
// LDS with one wave per tile pair.  Bound by issue: per group 48 MFMAs of 32 cycles (47% of the
// time) and the splits' conversions, which do not overlap them (counters).  On the FP64 path,
// without splits, the same form is slower than the LDS tiles (2.87 against 2.58 ms at 15 bins,
// m_max = 16, 12.8 GB: both near the copy rate).  The product of two fields, m_max = 10 and 786,000
// pivots, LDS tiles with the sum over segments / this form with its own: 8 bins 529 / 316 us, 15 770 /
// 734, 16 768 / 770, 20 1899 / 1671, 24 1919 / 1713.
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));  // rows start anywhere

// x[i] of quarter q = element 4 q + i  ->  x[s] of quarter q = element 4 s + q
__device__ __forceinline__ void transpose_quarters(float (&x)[4])
{
    auto swap16 = [](float &a, float &b) {
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    auto swap32 = [](float &a, float &b) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    swap16(x[0], x[1]);
    swap16(x[2], x[3]);
    swap32(x[0], x[2]);
    swap32(x[1], x[3]);
}

constexpr int kPairWaves = 4;

template <int T, bool SYM>
__global__ __launch_bounds__(kPairWaves * 64) void k_pair(PairArgs c)
{
    constexpr int NP = SYM ? T * (T + 1) / 2 : T * T;
    __shared__ double sums[kPairWaves][256];
    const int64_t unit = blockIdx.x;  // (segment, map, m)
    const int m = (int)(unit % c.M1);
    const int map = (int)((unit / c.M1) % c.nmaps);
    const int64_t seg = unit / ((int64_t)c.M1 * c.nmaps);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, q = lane >> 4;
    const int rows = 2 * c.nb;
    const size_t mo = (size_t)map * c.a_stride + (size_t)2 * m * c.nb * c.ldA;
    const double *v = c.v + (size_t)map * c.v_stride;
    const int64_t pbeg = seg * c.seg;
    const int64_t pend = min(c.npiv, pbeg + c.seg);

    // this lane's rows, one per row tile; a padding row reads row 0 and counts as zeros
    const float *src1[T], *src2[T];
    bool in[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int u = 16 * t + row;
        in[t] = u < rows;
        const size_t o = mo + (in[t] ? (size_t)u * c.ldA : 0);
        src1[t] = static_cast<const float *>(c.A1) + o;
        src2[t] = static_cast<const float *>(SYM ? c.A1 : c.A2) + o;
    }
    // this quarter's four pivots of group g: one load, or only those below pend
    auto load4 = [&](const float *s, int64_t g, bool whole, bool rin, float (&x)[4]) __attribute__((always_inline)) {
        const int64_t p = g + 4 * q;
        if (whole) {
            const f4_any r = *reinterpret_cast<const f4_any *>(s + p);
            x[0] = r.x; x[1] = r.y; x[2] = r.z; x[3] = r.w;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = p + i < pend ? s[p + i] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = rin ? x[i] : 0.0f;
    };
    float x1[T][4], x2[SYM ? 1 : T][4];
    double vk[4];
    auto fetch = [&](int64_t g) __attribute__((always_inline)) {
        const bool whole = g + 16 <= pend;  // wave-uniform
#pragma unroll
        for (int t = 0; t < T; ++t) {
            load4(src1[t], g, whole, in[t], x1[t]);
            if constexpr (!SYM) load4(src2[t], g, whole, in[t], x2[SYM ? 0 : t]);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int64_t p = g + 4 * s + q;
            vk[s] = whole || p < pend ? v[p] : 0.0;
        }
    };
    v4d acc[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) acc[j] = v4d{0.0, 0.0, 0.0, 0.0};
    int64_t g = pbeg + 16 * wave;
    if (g < pend) fetch(g);
    for (; g < pend; g += 16 * kPairWaves) {
        // operands: the scaled rows of field 1 as hi + lo, the rows of field 2
        float hi[T][4], lo[T][4], b[T][4];
#pragma unroll
        for (int t = 0; t < T; ++t) {
#pragma unroll
            for (int i = 0; i < 4; ++i) b[t][i] = SYM ? x1[t][i] : x2[SYM ? 0 : t][i];
            if constexpr (!SYM) transpose_quarters(x1[t]);
            transpose_quarters(b[t]);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double av = (double)(SYM ? b[t][s] : x1[t][s]) * vk[s];
                hi[t][s] = (float)av;
                lo[t][s] = (float)(av - (double)hi[t][s]);
            }
        }
        const int64_t gn = g + 16 * kPairWaves;
        if (gn < pend) fetch(gn);
        // FP32 products over 16 pivots, then into the FP64 sums
        v4f part[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) part[j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int I = 0, j = 0; I < T; ++I)
#pragma unroll
                for (int J = SYM ? I : 0; J < T; ++J, ++j)
                    part[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(hi[I][s], b[J][s], part[j], 0, 0, 0);
#pragma unroll
            for (int I = 0, j = 0; I < T; ++I)
#pragma unroll
                for (int J = SYM ? I : 0; J < T; ++J, ++j)
                    part[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(lo[I][s], b[J][s], part[j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][r] += (double)part[j][r];
    }
    double *out = c.part + (size_t)unit * (size_t)NP * 256;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        if (j) __syncthreads();
        // f32 16x16x4 result: register r of lane l is D[4 (l/16) + r][l % 16]
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[wave][(4 * q + r) * 16 + row] = acc[j][r];
        __syncthreads();
        double s = sums[0][tid];
#pragma unroll
        for (int w = 1; w < kPairWaves; ++w) s += sums[w][tid];
        out[(size_t)j * 256 + tid] = s;
    }
}

// k_pair_lds: one block per (segment, map, m) (and 16 tile pairs beyond T = 4).  Tiles of KP
// pivots of the fields' 2nb rows of that m are staged in LDS as [pivot][row], consecutive
// pivots of a row on consecutive lanes (one contiguous run of the pivot-minor layout), and the
// waves run the 16 x 16 tile pairs out of LDS, so every multipole is read from memory once per
// launch; the next tile's loads are in flight during the current tile's MFMAs.  The scaled
// operand v_p U1 is formed once per element when it is staged (on the mixed path as hi + lo),
// not once per tile pair that reads it.  The LDS row length is the least >= 2 nb that is 17 mod
// 32 (conflict-free staging writes, 16 pivots of a row 17 banks apart; operand reads of the
// four pivot groups nearly so).  Fixed-order FP64 sums.
//
// Pivots per tile: 32, but 16 for the Gram matrix of more than 64 FP64 rows, whose two tiles
// would otherwise take 74 KB of LDS (the two fields' product takes that).
constexpr int pair_kp(bool f32, bool sym, int T) { return !f32 && sym && T > 4 ? 16 : 32; }

// NW waves per block, one tile pair per wave, tile pairs blockIdx.y NW onwards; each thread
// stages up to ROWS rows of both fields per tile (2 nb <= 16 T <= ROWS x (64 NW / KP) for every
// shape launched).  SYM: a Gram matrix of one field (A2 = A1; only the tile pairs on or above
// the diagonal, the others are their mirror).
template <bool F32, int NW, int KP, int ROWS, bool SYM>
__global__ __launch_bounds__(NW * 64) void k_pair_lds(PairArgs c)
{
    typedef typename std::conditional<F32, float, double>::type E;
    constexpr int kThreads = NW * 64;
    extern __shared__ __align__(16) unsigned char smem[];
    const int ldr = c.ldr;
    E *ta = reinterpret_cast<E *>(smem);  // [KP][ldr] v_p U1 (mixed: its hi part)
    E *tb = ta + KP * ldr;                // [KP][ldr] U2
    E *tl = tb + KP * ldr;                // [KP][ldr] mixed: the lo part of v_p U1
    const int64_t unit = blockIdx.x;  // (segment, map, m)
    const int m = (int)(unit % c.M1);
    const int map = (int)((unit / c.M1) % c.nmaps);
    const int64_t seg = unit / ((int64_t)c.M1 * c.nmaps);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = lane & 15, kq = lane >> 4;
    const int two_nb = 2 * c.nb, T = c.T;
    const size_t mo = (size_t)map * c.a_stride + (size_t)2 * m * c.nb * c.ldA;
    const E *src1 = static_cast<const E *>(c.A1) + mo;
    const E *src2 = static_cast<const E *>(SYM ? c.A1 : c.A2) + mo;
    const double *v = c.v + (size_t)map * c.v_stride;

    const int tp = (int)blockIdx.y * NW + wave;
    int ua = -1, ub = -1;
    v4d acc = {0.0, 0.0, 0.0, 0.0};
    if (tp < c.npairs) {
        int I = tp / T, J = tp % T;
        if constexpr (SYM) {
            int r = tp;
            I = 0;
            while (r >= T - I) { r -= T - I; ++I; }
            J = I + r;
        }
        ua = I * 16 + row;
        ub = J * 16 + row;
    }
    const bool in_a = ua >= 0 && ua < two_nb, in_b = ub >= 0 && ub < two_nb;
    const int64_t pbeg = seg * c.seg;
    const int64_t pend = min(c.npiv, pbeg + c.seg);
    // staging: thread -> (row u, pivot k), KP pivots of a row on consecutive lanes; the next
    // tile's global loads are issued before the current tile's MFMAs
    const int k = tid % KP, u0 = tid / KP;
    constexpr int ustep = kThreads / KP;
    E a[ROWS], b[SYM ? 1 : ROWS];
    double vk = 0.0;
    auto fetch = [&](int64_t q0) {
        const bool kin = q0 + k < pend;
        vk = kin ? v[q0 + k] : 0.0;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int uu = u0 + i * ustep;
            const bool in = uu < two_nb && kin;
            a[i] = in ? src1[(size_t)uu * c.ldA + q0 + k] : E(0);
            if constexpr (!SYM) b[i] = in ? src2[(size_t)uu * c.ldA + q0 + k] : E(0);
        }
    };
    fetch(pbeg);
    for (int64_t p0 = pbeg; p0 < pend; p0 += KP) {
        __syncthreads();  // the previous tile is consumed
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int uu = u0 + i * ustep;
            if (uu < two_nb) {
                const double av = (double)a[i] * vk;
                const E hi = (E)av;
                ta[k * ldr + uu] = hi;
                if constexpr (F32) tl[k * ldr + uu] = (float)(av - (double)hi);
                tb[k * ldr + uu] = SYM ? a[i] : b[SYM ? 0 : i];
            }
        }
        __syncthreads();
        if (p0 + KP < pend) fetch(p0 + KP);
        if (ua < 0) continue;  // wave-uniform
#pragma unroll
        for (int h = 0; h < KP / 16; ++h) {
            if constexpr (F32) {
                // FP32 products over 16 pivots, then into the FP64 sum
                v4f part = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int base = (16 * h + 4 * ks + kq) * ldr;
                    const float ahi = in_a ? ta[base + ua] : 0.0f;
                    const float alo = in_a ? tl[base + ua] : 0.0f;
                    const float x2 = in_b ? tb[base + ub] : 0.0f;
                    part = __builtin_amdgcn_mfma_f32_16x16x4f32(ahi, x2, part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_16x16x4f32(alo, x2, part, 0, 0, 0);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] += (double)part[q];
            } else {
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int base = (16 * h + 4 * ks + kq) * ldr;
                    const double x1 = in_a ? ta[base + ua] : 0.0;
                    const double x2 = in_b ? tb[base + ub] : 0.0;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x2, acc, 0, 0, 0);
                }
            }
        }
    }
    if (ua < 0) return;
    double *out = c.part + ((size_t)unit * (size_t)c.npairs + tp) * 256;
    // f64 16x16x4 result: register q of lane l is D[4q + l/16][l % 16]; f32 as in k_pair
#pragma unroll
    for (int q = 0; q < 4; ++q) out[(F32 ? 4 * kq + q : 4 * q + kq) * 16 + row] = acc[q];
}

// NW waves, at most T row tiles
template <bool F32, int NW, int T, bool SYM>
static void launch_pair_lds(dim3 grid, size_t lds, const PairArgs &c, hipStream_t s)
{
    constexpr int KP = pair_kp(F32, SYM, T), kAtOnce = NW * 64 / KP;  // rows staged at a time
    hipLaunchKernelGGL((k_pair_lds<F32, NW, KP, (16 * T + kAtOnce - 1) / kAtOnce, SYM>), grid, dim3(NW * 64), lds, s, c);
}

// The kernel and its shape for c.T row tiles.
template <bool F32, bool SYM>
static z3_status launch_pair_shape(dim3 grid, const PairArgs &c0, hipStream_t s)
{
    PairArgs c = c0;
    const int T = c.T;
    if (F32 && T <= (SYM ? 4 : 3)) {
        const dim3 block(kPairWaves * 64);
        if (T == 1) hipLaunchKernelGGL((k_pair<1, SYM>), grid, block, 0, s, c);
        else if (T == 2) hipLaunchKernelGGL((k_pair<2, SYM>), grid, block, 0, s, c);
        else if (T == 3) hipLaunchKernelGGL((k_pair<3, SYM>), grid, block, 0, s, c);
        else if constexpr (SYM) hipLaunchKernelGGL((k_pair<4, SYM>), grid, block, 0, s, c);
        return check_launch("k_pair");
    }
    c.ldr = 2 * c.nb + ((17 - 2 * c.nb) % 32 + 32) % 32;
    const size_t lds = (size_t)pair_kp(F32, SYM, T) * c.ldr * (F32 ? 3 * sizeof(float) : 2 * sizeof(double));
    int dev = 0, lds_max = 0;
    z3_status st = check_hip(hipGetDevice(&dev), "hipGetDevice");
    if (st == Z3_OK)
        st = check_hip(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev), "LDS size");
    if (st != Z3_OK) return st;
    if (lds > (size_t)lds_max)
        return fail(Z3_ERR_UNSUPPORTED, "contraction of %d bins needs %zu bytes of LDS per block (%d)", c.nb, lds,
                    lds_max);
    // one tile pair per wave, as many waves as pairs up to T = 4 (6 or 9 waves at T = 3); beyond,
    // groups of 16 pairs in blocks of their own (grid.y), each staging the whole tile
    const dim3 grid16(grid.x, (unsigned)((c.npairs + 15) / 16));
    if constexpr (!F32) {
        if (T <= 2) launch_pair_lds<F32, 4, 2, SYM>(grid, lds, c, s);
        else if (T == 3) launch_pair_lds<F32, SYM ? 6 : 9, 3, SYM>(grid, lds, c, s);
        else if (T == 4) launch_pair_lds<F32, SYM ? 10 : 16, 4, SYM>(SYM ? grid : grid16, lds, c, s);
        else launch_pair_lds<F32, 16, 8, SYM>(grid16, lds, c, s);
    } else {
        launch_pair_lds<F32, 16, 8, SYM>(grid16, lds, c, s);
    }
    return check_launch("k_pair_lds");
}

// Pair contraction over pivot-minor multipoles: one block per (segment, map, m)
static z3_status launch_pair(const PairArgs &c, bool f32, bool sym, int64_t nseg, hipStream_t s)
{
    const int64_t nblk = nseg * c.nmaps * c.M1;
    if (nblk > (int64_t)(UINT32_MAX / 1024))
        return fail(Z3_ERR_OVERFLOW, "contraction of %lld pivot segments x %d maps", (long long)nseg, c.nmaps);
    const dim3 grid((unsigned)nblk);
    if (f32) return sym ? launch_pair_shape<true, true>(grid, c, s) : launch_pair_shape<true, false>(grid, c, s);
    return sym ? launch_pair_shape<false, true>(grid, c, s) : launch_pair_shape<false, false>(grid, c, s);
}

// ---- LDS-staged contraction of the pivot-major staging ------------------------------------
// One block of kGramWaves waves per (pivot segment, map).  Tiles of kGramKP pivots of the
// many-map kernel's pivot-major staging (one contiguous run of R = 2 (m_max + 1) rows per
// pivot and bin) are staged in LDS, (re, im) pairs on consecutive lanes.  Every wave then runs
// its (m, tile pair) units over the tile out of LDS, so each multipole is fetched once per
// block and the staging needs no transpose.
//
// What bounds it: 64 maps of 197,000 pivots (15 bins, m_max 10) are 16.6 GB in FP32, 3.5 ms, and
// 3.3 ms of MFMA, and the vector unit's split of v_p U_i costs about as much.  The tile's loads are
// requested one tile ahead, so that they pass beside the products; an operand of 4 k-steps is one
// 16-byte LDS read without bank conflicts instead of four scalar ones; and on the mixed path 2
// blocks fit a CU (126 VGPRs).  With loads, barrier and products in turn it took 11.3 ms, now 6.8;
// FP64 16.4 -> 9.5 ms.
constexpr int kGramWaves = 8;
constexpr int kGramThreads = kGramWaves * 64;
constexpr int kGramKP = 16;                      // pivots per LDS tile (4 MFMA k-steps)
constexpr size_t kGramLdsMax = 64 * 1024 - 256;  // tile + pivot values

static size_t gram_tile_bytes(int nb, int R, bool f32)
{
    return ((size_t)kGramKP * nb * R * (f32 ? 4 : 8) + 15) / 16 * 16;
}

// units per wave: the smallest compiled bound covering M1 x (tile pairs) units, else 0 (more
// accumulators than a wave can hold at two waves per SIMD without spilling).  A tile then has
// at most 7 or 9 (re, im) pairs per thread: 16 nb M1 <= 256 units / (T + 1), with T = 1 and at
// most 17 units (m_max 16), T = 2 and at most 51, T >= 3.
static int gram_upw(int nunits)
{
    for (int u : {5, 9})
        if (kGramWaves * u >= nunits) return u;
    return 0;
}

bool gram_lds_fits(int m_max, int nbins, int prec)
{
    const int T = tiles_for(nbins), ntp = T * (T + 1) / 2;
    const int R = 2 * (m_max + 1);
    return gram_upw((m_max + 1) * ntp) > 0 && R <= 64 &&
           gram_tile_bytes(nbins, R, prec == Z3_PREC_MIXED) + kGramKP * sizeof(double) <= kGramLdsMax;
}

// element (pivot p, bin b, row r) of map j: pivot-major staging at base + j map_stride + p sp + b sb + r,
// pivot-minor multipoles at base + j map_stride + (r nb + b) sb + p
struct GramSrc {
    const void *base;
    int64_t sp, sb;
    size_t map_stride;
};

struct GramArgs {
    GramSrc src;
    int64_t npiv;
    const double *v;
    size_t v_stride;
    int nb, R, T, ntp, M1, nmaps, nunits;
    int seg;             // pivots per segment
    size_t tile_bytes;
    double *part;        // [seg][map][m][tile pair][256]
};

// The tile in LDS: entry e = 2 m nb + u of U_m at 16 pivots, so that the rows of an operand are
// neighbours.  A lane's four pivots kq, 4 + kq, .. (one of each k-step) stand together, 16 bytes
// in FP32, 32 in FP64, and the 16-byte slots of an entry are permuted by e so that a read by 16
// rows touches every bank once.  gram_slot is the byte offset of pivot kq (in FP64: its slot of
// k-steps 0 and 1; that of 2 and 3 is the offset ^ 16).
template <bool F32>
__device__ __forceinline__ int gram_slot(int e, int kq)
{
    return F32 ? 64 * e + 16 * (kq ^ (e >> 2 & 3)) : 128 * e + 16 * ((2 * kq) ^ (e >> 1 & 7));
}

__device__ __forceinline__ void gram_entries(const unsigned char *smem, int at, float (&u)[4])
{
    const float4 q = *reinterpret_cast<const float4 *>(smem + at);
    u[0] = q.x; u[1] = q.y; u[2] = q.z; u[3] = q.w;
}

__device__ __forceinline__ void gram_entries(const unsigned char *smem, int at, double (&u)[4])
{
    const double2 q = *reinterpret_cast<const double2 *>(smem + at), r = *reinterpret_cast<const double2 *>(smem + (at ^ 16));
    u[0] = q.x; u[1] = q.y; u[2] = r.x; u[3] = r.y;
}

template <bool F32, int UPW>
__global__ __launch_bounds__(kGramThreads) __attribute__((amdgpu_waves_per_eu(F32 && UPW == 5 ? 4 : 2))) void k_gram_lds(GramArgs g)
{
    typedef typename std::conditional<F32, float, double>::type T;
    typedef typename std::conditional<F32, float2, double2>::type T2;
    constexpr int NLD = UPW == 5 ? 7 : 9;  // (re, im) pairs of a tile per thread, see gram_upw
    extern __shared__ __align__(16) unsigned char smem[];
    double *vt = reinterpret_cast<double *>(smem + g.tile_bytes);   // [kGramKP]
    const int nb = g.nb, R = g.R;
    // blocks are dealt round-robin to the 8 XCDs: each XCD gets a contiguous run of
    // (segment, map) units, so blocks reading neighbouring maps' runs share its L2
    const int64_t nblk = gridDim.x, bi = blockIdx.x, per = nblk / 8;
    const int64_t unit = bi < per * 8 ? (bi % 8) * per + bi / 8 : bi;
    const int64_t seg = unit / g.nmaps;
    const int map = (int)(unit - seg * g.nmaps);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = lane & 15, kq = lane >> 4;
    const T *src = static_cast<const T *>(g.src.base) + (size_t)map * g.src.map_stride;
    const double *v = g.v + (size_t)map * g.v_stride;

    // this wave's units (m, tile pair) and, for each, where in LDS this lane's entries of the A
    // and B operands stand (rows that pad a tile read entry 0: their results are never read)
    int um[UPW], offa[UPW], offb[UPW];
    v4d acc[UPW];
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        const int uu = wave + kGramWaves * j;
        um[j] = -1;
        offa[j] = offb[j] = gram_slot<F32>(0, kq);
        acc[j] = v4d{0.0, 0.0, 0.0, 0.0};
        if (uu < g.nunits) {
            const int m = uu / g.ntp;
            int r = uu - m * g.ntp, I = 0;
            while (r >= g.T - I) { r -= g.T - I; ++I; }
            const int J = I + r;
            const int ua = I * 16 + row, ub = J * 16 + row;
            um[j] = m;
            if (ua < 2 * nb) offa[j] = gram_slot<F32>(2 * m * nb + ua, kq);
            if (ub < 2 * nb) offb[j] = gram_slot<F32>(2 * m * nb + ub, kq);
        }
    }

    // (re, im) pairs tid, tid + kGramThreads, .. of a tile
    const int npr = nb * (R / 2);  // pairs of a pivot
    uint32_t off[NLD], at[NLD];  // in memory, from its first pivot's row; in LDS: re, im << 16
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int e = min(tid + i * kGramThreads, kGramKP * npr - 1), k = e / npr, b = (e - k * npr) / (R / 2);
        const int m = e - k * npr - b * (R / 2), ks = k >> 2;
        off[i] = tid + i * kGramThreads < kGramKP * npr ? (uint32_t)((k * g.src.sp + b * g.src.sb + 2 * m) * sizeof(T)) : 0xfffffff0u;
        const int re = gram_slot<F32>(2 * m * nb + b, k & 3), im = gram_slot<F32>((2 * m + 1) * nb + b, k & 3);
        const int part = F32 ? 4 * ks : 8 * (ks & 1), half = F32 ? 0 : 16 * (ks >> 1);
        at[i] = (uint32_t)((re ^ half) + part) | (uint32_t)((im ^ half) + part) << 16;
    }
    T2 val[NLD];
    double vval = 0.0;
    // reads past the tile's last pivot give zeros: their offsets are past the view's end
    auto load_tile = [&](int64_t p0, int np) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rows = buffer_view(src + p0 * g.src.sp, (uint32_t)(np * g.src.sp * sizeof(T)));
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            if constexpr (F32) val[i] = __builtin_bit_cast(T2, __builtin_amdgcn_raw_buffer_load_b64(rows, off[i], 0, 0));
            else val[i] = __builtin_bit_cast(T2, __builtin_amdgcn_raw_buffer_load_b128(rows, off[i], 0, 0));
        }
        if (tid < kGramKP) vval = tid < np ? v[p0 + tid] : 0.0;
    };

    const int64_t pbeg = seg * g.seg;
    const int64_t pend = min(g.npiv, pbeg + g.seg);
    load_tile(pbeg, (int)min((int64_t)kGramKP, pend - pbeg));
    for (int64_t p0 = pbeg; p0 < pend; p0 += kGramKP) {
        __syncthreads();  // the previous tile is consumed
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            if (tid + i * kGramThreads < kGramKP * npr) {
                *reinterpret_cast<T *>(smem + (at[i] & 0xffff)) = val[i].x;
                *reinterpret_cast<T *>(smem + (at[i] >> 16)) = val[i].y;
            }
        if (tid < kGramKP) vt[tid] = vval;
        __syncthreads();
        // the next tile is on its way while this one is multiplied
        if (p0 + kGramKP < pend) load_tile(p0 + kGramKP, (int)min((int64_t)kGramKP, pend - p0 - kGramKP));
        double vk[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) vk[ks] = vt[4 * ks + kq];
#pragma unroll
        for (int j = 0; j < UPW; ++j) {
            if (um[j] < 0) continue;  // wave-uniform
            T ua[4], ub[4];
            gram_entries(smem, offa[j], ua);
            gram_entries(smem, offb[j], ub);
            if constexpr (F32) {
                // FP32 products and sums over the tile's pivots, then into the FP64 sum; the
                // scaled operand v_p U_i is formed in FP64 and carried as FP32 hi + lo
                v4f part = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const double av = (double)ua[ks] * vk[ks];
                    const float ahi = (float)av;
                    const float alo = (float)(av - (double)ahi);
                    part = __builtin_amdgcn_mfma_f32_16x16x4f32(ahi, ub[ks], part, 0, 0, 0);
                    part = __builtin_amdgcn_mfma_f32_16x16x4f32(alo, ub[ks], part, 0, 0, 0);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[j][k] += (double)part[k];
            } else {
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ua[ks] * vk[ks], ub[ks], acc[j], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        if (um[j] < 0) continue;
        const int tp = wave + kGramWaves * j - um[j] * g.ntp;
        double *out = g.part + ((((size_t)seg * g.nmaps + map) * g.M1 + um[j]) * g.ntp + tp) * 256;
        // f64 16x16x4 result: register k of lane l is D[4k + l/16][l % 16];
        // f32 16x16x4 result: register k of lane l is D[4 (l/16) + k][l % 16]
#pragma unroll
        for (int k = 0; k < 4; ++k) out[(F32 ? 4 * kq + k : 4 * k + kq) * 16 + row] = acc[j][k];
    }
}

template <bool F32>
static void launch_gram_lds(int upw, dim3 grid, size_t lds, const GramArgs &g, hipStream_t s)
{
    if (upw == 5) hipLaunchKernelGGL((k_gram_lds<F32, 5>), grid, dim3(kGramThreads), lds, s, g);
    else hipLaunchKernelGGL((k_gram_lds<F32, 9>), grid, dim3(kGramThreads), lds, s, g);
}

static z3_status contract_src(int64_t npiv, int m_max, int nbins, int prec, int nmaps, const GramSrc &src, bool pm,
                              const double *piv_v, size_t v_stride, double *zeta, size_t z_stride, void *partials,
                              size_t partial_bytes, hipStream_t s)
{
    if (npiv <= 0 || nmaps <= 0) return Z3_OK;
    const int T = tiles_for(nbins), ntp = T * (T + 1) / 2;
    const int64_t units = contract_units(m_max, nbins, nmaps);
    if (least_bytes(npiv, units) > partial_bytes) return fail(Z3_ERR_INVALID_ARG, "contraction workspace too small");
    const int seg = segment_pivots(npiv, units, partial_bytes);
    int64_t nseg = (npiv + seg - 1) / seg;
    if (nseg > 65535) return fail(Z3_ERR_OVERFLOW, "too many pivots for one contraction (%lld)", (long long)npiv);
    if ((int64_t)nmaps * (m_max + 1) > 65535) return fail(Z3_ERR_OVERFLOW, "too many maps for one contraction");
    const bool f32 = prec == Z3_PREC_MIXED;
    z3_status st;
    if (pm) {
        if (!gram_lds_fits(m_max, nbins, prec))
            return fail(Z3_ERR_UNSUPPORTED, "pivot-major contraction for m_max=%d, %d bins", m_max, nbins);
        // one block per (segment, map): the dispatch stays below 2^32 work-items
        if (nseg * nmaps > (int64_t)(UINT32_MAX / kGramThreads))
            return fail(Z3_ERR_OVERFLOW, "contraction of %lld pivots x %d maps in one launch", (long long)npiv, nmaps);
        GramArgs g;
        g.src = src;
        g.npiv = npiv;
        g.v = piv_v;
        g.v_stride = v_stride;
        g.nb = nbins;
        g.R = 2 * (m_max + 1);
        g.T = T;
        g.ntp = ntp;
        g.M1 = m_max + 1;
        g.nmaps = nmaps;
        g.nunits = (m_max + 1) * ntp;
        g.seg = seg;
        g.tile_bytes = gram_tile_bytes(nbins, g.R, f32);
        g.part = static_cast<double *>(partials);
        const int upw = gram_upw(g.nunits);
        const dim3 grid((unsigned)(nseg * nmaps));
        const size_t lds = g.tile_bytes + kGramKP * sizeof(double);
        if (f32) launch_gram_lds<true>(upw, grid, lds, g, s);
        else launch_gram_lds<false>(upw, grid, lds, g, s);
        st = check_launch("k_gram_lds");
    } else {
        PairArgs c = {};
        c.A1 = src.base;
        c.ldA = src.sb;
        c.npiv = npiv;
        c.v = piv_v;
        c.a_stride = src.map_stride;
        c.v_stride = v_stride;
        c.nb = nbins;
        c.T = T;
        c.M1 = m_max + 1;
        c.nmaps = nmaps;
        c.npairs = ntp;
        c.seg = seg;
        c.part = static_cast<double *>(partials);
        st = launch_pair(c, f32, true, nseg, s);
    }
    if (st == Z3_OK)
        st = sum_segments(static_cast<double *>(partials), &nseg, units * 256, s);
    if (st != Z3_OK) return st;
    const int total = nmaps * (m_max + 1) * nbins * nbins;
    hipLaunchKernelGGL(k_gram_reduce, dim3((total + 127) / 128), dim3(128), 0, s,
                       static_cast<const double *>(partials), nseg, nmaps, m_max + 1, nbins, T, ntp, zeta, z_stride);
    return check_launch("k_gram_reduce");
}

z3_status launch_contract_maps(int64_t npiv, int m_max, int nbins, int prec, int nmaps, const void *A, int64_t ldA,
                               size_t a_stride, const double *piv_v, size_t v_stride, double *zeta, size_t z_stride,
                               void *partials, size_t partial_bytes, hipStream_t s)
{
    const GramSrc src{A, 1, ldA, a_stride};
    return contract_src(npiv, m_max, nbins, prec, nmaps, src, false, piv_v, v_stride, zeta, z_stride, partials,
                        partial_bytes, s);
}

z3_status launch_contract_staged(int64_t npiv, int m_max, int nbins, int prec, int nmaps, const void *stage,
                                 const double *piv_v, size_t v_stride, double *zeta, size_t z_stride, void *partials,
                                 size_t partial_bytes, hipStream_t s)
{
    const int64_t R = 2 * (m_max + 1);
    const GramSrc src{stage, (int64_t)nbins * nmaps * R, (int64_t)nmaps * R, (size_t)R};
    return contract_src(npiv, m_max, nbins, prec, nmaps, src, true, piv_v, v_stride, zeta, z_stride, partials,
                        partial_bytes, s);
}

z3_status launch_contract(int64_t npiv, int m_max, int nbins, int prec, const void *A, int64_t ldA,
                          const double *piv_v, double *zeta, void *partials, size_t partial_bytes,
                          hipStream_t s)
{
    return launch_contract_maps(npiv, m_max, nbins, prec, 1, A, ldA, 0, piv_v, 0, zeta, 0, partials, partial_bytes, s);
}

__device__ __forceinline__ double cross_at(const double *seg_m, int T, int u, int v)
{
    return seg_m[(size_t)((u >> 4) * T + (v >> 4)) * 256 + (u & 15) * 16 + (v & 15)];
}

__global__ void k_cross_reduce(const double *part, int64_t nseg, int M1, int nb, int T, double *zeta)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= M1 * nb * nb) return;
    const int m = t / (nb * nb), rem = t % (nb * nb), b1 = rem / nb, b2 = rem % nb;
    const int r1 = b1, r2 = b2, i1 = nb + b1, i2 = nb + b2;
    double rr = 0.0, ii = 0.0, ir = 0.0, ri = 0.0;
    for (int64_t s = 0; s < nseg; ++s) {
        const double *g = part + (size_t)(s * M1 + m) * (size_t)(T * T) * 256;
        rr += cross_at(g, T, r1, r2);
        ii += cross_at(g, T, i1, i2);
        ir += cross_at(g, T, i1, r2);
        ri += cross_at(g, T, r1, i2);
    }
    double *z = zeta + ((size_t)(m * nb + b1) * nb + b2) * 2;
    z[0] += rr + ii;
    z[1] += ir - ri;
}

PartialBytes cross_partial_bytes(int64_t npiv, int m_max, int nbins)
{
    const int T = tiles_for(nbins);
    return partial_bytes(npiv, (int64_t)(m_max + 1) * T * T);
}

z3_status launch_contract_cross(int64_t npiv, int m_max, int nbins, int prec, const void *A1, const void *A2,
                                int64_t ldA, const double *piv_v, double *zeta, void *partials,
                                size_t partial_bytes, hipStream_t s)
{
    if (npiv <= 0) return Z3_OK;
    const int T = tiles_for(nbins);
    const int64_t units = (int64_t)(m_max + 1) * T * T;
    if (least_bytes(npiv, units) > partial_bytes)
        return fail(Z3_ERR_INVALID_ARG, "multi-field contraction: partial buffer too small");
    const int seg = segment_pivots(npiv, units, partial_bytes);
    int64_t nseg = (npiv + seg - 1) / seg;
    PairArgs c = {};
    c.A1 = A1;
    c.A2 = A2;
    c.ldA = ldA;
    c.npiv = npiv;
    c.v = piv_v;
    c.nb = nbins;
    c.T = T;
    c.M1 = m_max + 1;
    c.nmaps = 1;
    c.npairs = T * T;
    c.seg = seg;
    c.part = static_cast<double *>(partials);
    z3_status st = launch_pair(c, prec == Z3_PREC_MIXED, false, nseg, s);
    if (st == Z3_OK) st = sum_segments(static_cast<double *>(partials), &nseg, units * 256, s);
    if (st != Z3_OK) return st;
    const int total = (m_max + 1) * nbins * nbins;
    hipLaunchKernelGGL(k_cross_reduce, dim3((total + 127) / 128), dim3(128), 0, s,
                       static_cast<const double *>(partials), nseg, m_max + 1, nbins, T, zeta);
    return check_launch("k_cross_reduce");
}

// ---- sum of pivot weights (fixed order) ------------------------------------------------

__global__ void k_sum_partials(const double *w, int64_t n, int64_t per_block, double *partial)
{
    __shared__ double sh[256];
    const int64_t beg = (int64_t)blockIdx.x * per_block;
    const int64_t end = min(n, beg + per_block);
    double acc = 0.0;
    for (int64_t i = beg + threadIdx.x; i < end; i += 256) acc += w[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

__global__ void k_sum_final(const double *partial, int nblk, double *out)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        double acc = 0.0;
        for (int b = 0; b < nblk; ++b) acc += partial[b];
        out[0] += acc;
    }
}

z3_status launch_weight_sum(const double *w, int64_t n, double *out, hipStream_t s)
{
    int64_t want = (n + 4095) / 4096;
    int nblk = (int)(want < 1024 ? want : 1024);
    if (nblk < 1) nblk = 1;
    const int64_t per = (n + nblk - 1) / nblk;
    void *part = nullptr;
    z3_status st = scratch_alloc(&part, nblk * sizeof(double), s);
    if (st != Z3_OK) return st;
    double *partial = static_cast<double *>(part);
    hipLaunchKernelGGL(k_sum_partials, dim3(nblk), dim3(256), 0, s, w, n, per, partial);
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(64), 0, s, partial, nblk, out);
    st = check_launch("k_sum");
    scratch_free(part, s);
    return st;
}

__global__ void k_pivot_values(const double *w, const double *x, int64_t n, double *v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = w ? w[i] * x[i] : x[i];
}

z3_status launch_pivot_values(const double *w, const double *x, int64_t n, double *v, hipStream_t s)
{
    if (n <= 0) return Z3_OK;
    hipLaunchKernelGGL(k_pivot_values, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, x, n, v);
    return check_launch("k_pivot_values");
}

__global__ void k_fill_value(double *p, int64_t n, double value)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// Fills with a kernel rather than a memset, so that the call can sit in a captured graph.
z3_status launch_fill(double *p, int64_t n, double value, hipStream_t s)
{
    if (n <= 0) return Z3_OK;
    hipLaunchKernelGGL(k_fill_value, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, value);
    return check_launch("k_fill_value");
}

__global__ void k_add_scalar(double *out, double value)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) out[0] += value;
}

z3_status launch_add_scalar(double *out, double value, hipStream_t s)
{
    hipLaunchKernelGGL(k_add_scalar, dim3(1), dim3(64), 0, s, out, value);
    return check_launch("k_add_scalar");
}

__global__ void k_finalize(double *zeta, int64_t count, const double *sum_w)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // an empty pivot set (sum of weights 0) leaves the (zero) sums unchanged
    if (i < count && sum_w[0] != 0.0) zeta[i] /= sum_w[0];
}

z3_status launch_finalize(int nmaps, int m_max, int nbins, double *zeta, const double *sum_w, hipStream_t s)
{
    const int64_t count = (int64_t)nmaps * (m_max + 1) * nbins * nbins * 2;
    hipLaunchKernelGGL(k_finalize, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, zeta, count, sum_w);
    return check_launch("k_finalize");
}

// Removal of the k = j terms: one block per bin adds the bin's column of the per-wave
// sums v_p Q / W^2 in a fixed order and subtracts the total from Re zeta_m(b, b) for every
// m (those terms are real and the same for every m).
__global__ void k_self_subtract(const double *part, int64_t nw, int nb, int M, double *zeta)
{
    __shared__ double sh[256];
    const int b = blockIdx.x;
    double acc = 0.0;
    for (int64_t w = threadIdx.x; w < nw; w += 256) acc += part[w * nb + b];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if ((int)threadIdx.x <= M) zeta[(((size_t)threadIdx.x * nb + b) * nb + b) * 2] -= sh[0];
}

z3_status launch_self_subtract(const double *part, int64_t nw, int m_max, int nbins, double *zeta, hipStream_t s)
{
    if (nw <= 0) return Z3_OK;
    hipLaunchKernelGGL(k_self_subtract, dim3(nbins), dim3(256), 0, s, part, nw, nbins, m_max, zeta);
    return check_launch("k_self_subtract");
}

// zeta(b1, b2, phi) = Re zeta_0 + 2 sum_{m>=1} (Re zeta_m cos(m phi) - Im zeta_m sin(m phi))
__global__ void k_resum(int M, int nb, const double *zeta, int nphi, const double *phi, double *out)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nb * nb * nphi) return;
    const int k = (int)(t % nphi);
    const int64_t bb = t / nphi;
    const double ph = phi[k];
    double acc = zeta[bb * 2];
    for (int m = 1; m <= M; ++m) {
        const double *z = zeta + ((size_t)m * nb * nb + bb) * 2;
        double sm, cm;
        sincos(m * ph, &sm, &cm);
        acc += 2.0 * (z[0] * cm - z[1] * sm);
    }
    out[t] = acc;
}

z3_status launch_resum(int m_max, int nbins, const double *zeta, int nphi, const double *phi, double *out,
                       hipStream_t s)
{
    const int64_t total = (int64_t)nbins * nbins * nphi;
    hipLaunchKernelGGL(k_resum, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, m_max, nbins, zeta, nphi,
                       phi, out);
    return check_launch("k_resum");
}

}  // namespace z3
