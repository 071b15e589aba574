// FFTLog evaluation of the line-of-sight integrals of the modelling appendix ("FFTLog for the
// line-of-sight integral"): the functions A_0, A_1, A_2 of a batch of models sharing P_L(k)
// and the angle grid, each with its own line-of-sight kernel F(chi) = q_A q_B q_C D_+^4.
//
//   c_s   = W_s k_min^{-nu - i eta_s} (1/N) sum_l P(k_l) (k_l/k_min)^{-nu} e^{-2 pi i s l/N}
//           (eqs. pklfft, pklfft_eta, cm; s = -N/2..N/2; one set per bias nu)
//   g(a)  = 2^{mt+a-1} Gamma((1+mt+a+n)/2) / (pi Gamma((1-a-mt+n)/2)),   a_s = 1 + nu + i eta_s
//           (the closed-form k integral of the appendix)
//   U_{is}= c_s g(a_s) theta_i^{-(1 + a_s + mt)}                         per factor (n, mt, nu)
//   A_{s1 s2} = int dchi F(chi) chi^{-a_s1 - a_s2 - 2}                  (trapezoid in ln chi)
//   I     = U1 A U2^T,   A_0 = I^{(0,0)}_{(0,0)},  A_1 = I^{(1,1)}_{(1,-1)} + transpose,
//           A_2 = I^{(2,0)}_{(2,0)}
//
// Two structural facts shape the evaluation:
//  * eta_s is linear in s (eta_s = s deta), so chi^{-a_s1 - a_s2} = chi^{-(2 + nu1 + nu2)}
//    e^{-i (s1 + s2) deta ln chi}: the stored matrix is a Hankel matrix, A_{s1 s2} = h(s1 + s2)
//    with only 2N + 1 distinct entries
//        h(t) = sum_j d_j chi_j^{-(2 + nu1 + nu2)} e^{-i t deta ln chi_j},   t = -N..N,
//    d_j the trapezoid weights in ln chi times F chi^{-1}; h(-t) = conj h(t).
//  * P is real, so c_{-s} = conj c_s, and with real nu every factor obeys U_{i,-s} = conj U_{is}:
//    the terms (s1, s2) and (-s1, -s2) are conjugate, I is real, and
//        I = Re sum_{s1 >= 0} omega_s1 sum_{s2} U1_{i s1} h(s1 + s2) U2_{j s2},
//    omega_0 = 1, omega_{s1 > 0} = 2 (the s1 = 0 column of U1 is real).
// So the library forms h for t >= 0 for every model and factor pair as one real-by-complex
// product over chi (E_{jt} = e^{-i t deta ln chi_j}, shared by all models), mirrors it to
// t < 0, then UA = (omega U1)_{s1 >= 0} H (H read straight from h) and Re(UA U2^T): complex
// FP64 matrix products on v_mfma_f64_16x16x4f64 through one strided batched kernel, 8 (N+1)
// (N/2+1) ntheta + 4 ntheta^2 (N+1) flop per function and model in place of the dense
// evaluation's 8 (N+1)^2 (nchi + ntheta) + 8 ntheta^2 (N+1).  The coefficient DFT and the Gamma
// ratios (complex log-Gamma: upward recurrence to Re z >= 12, then Stirling's series) run one
// wave per coefficient; the operands are elementwise kernels.
#include <type_traits>

#include "z3_fftlog_pass.h"
#include "z3_internal.h"

namespace z3 {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

__device__ __forceinline__ double2 cexp(double2 z)
{
    double s, c;
    sincos(z.y, &s, &c);
    const double e = exp(z.x);
    return make_double2(e * c, e * s);
}

__device__ __forceinline__ double2 clog(double2 z) { return make_double2(0.5 * log(z.x * z.x + z.y * z.y), atan2(z.y, z.x)); }

__device__ __forceinline__ double2 cdiv(double2 a, double2 b)
{
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

// log Gamma(z) for complex z away from the poles, up to a multiple of 2 pi i in the imaginary
// part (only exp of differences is used).  Upward recurrence log Gamma(z) = log Gamma(z + K) -
// log prod_{j<K} (z + j) until Re(z + K) >= 12 (the product kept as one complex number, one
// logarithm at the end), then Stirling's series with Bernoulli terms B_{2k} / (2k (2k-1)
// z^{2k-1}), k = 1..8.
__device__ double2 clgamma(double2 z)
{
    double2 prod = make_double2(1.0, 0.0);
    bool shifted = false;
    while (z.x < 12.0) {
        prod = cmul(prod, z);
        z.x += 1.0;
        shifted = true;
    }
    const double2 shift = shifted ? clog(prod) : make_double2(0.0, 0.0);
    const double2 lz = clog(z);
    const double2 zh = make_double2(z.x - 0.5, z.y);
    double2 r = cmul(zh, lz);
    r.x += -z.x + 0.91893853320467274178;  // ln(2 pi) / 2
    r.y += -z.y;
    const double2 iz = cdiv(make_double2(1.0, 0.0), z);
    const double2 iz2 = cmul(iz, iz);
    const double b[8] = {1.0 / 12.0, -1.0 / 360.0, 1.0 / 1260.0, -1.0 / 1680.0, 1.0 / 1188.0, -691.0 / 360360.0,
                         1.0 / 156.0, -3617.0 / 122400.0};
    double2 t = iz, s = make_double2(0.0, 0.0);
    for (int k = 0; k < 8; ++k) {
        s.x += b[k] * t.x;
        s.y += b[k] * t.y;
        t = cmul(t, iz2);
    }
    return make_double2(r.x + s.x - shift.x, r.y + s.y - shift.y);
}

struct FactorSpec {
    int n, mt;
    double nu;
};

struct FftlogArgs {
    int N;                    // samples of P (even); Ns = N + 1 coefficients s = 0..N (m = s - N/2)
    int Ns, ld, ldw, ldh;     // padded lengths: s (ld), s1 >= 0 half (ldw), t >= 0 half (ldh)
    const double *Pk;
    double k_min, k_max;
    FactorSpec f[4];          // (0,0), (1,1), (1,-1), (2,0)
    int nchi;
    double chi_min, dlnchi;
    int T;
    const double *theta;
    double2 *cg;              // [4][ld]: c_s g(a_s)
    double2 *a;               // [4][ld]: a_s
    double2 *U;               // [4][ld][T]
    double2 *Uw;              // [4][ldw][T]: omega_m U[N/2 + m][.], m = 0..N/2
    double2 *E;               // [nchi][ldh]: e^{-i t deta ln chi_j}, t = 0..N
};

__device__ __forceinline__ double fftlog_deta(int N, double k_min, double k_max)
{
    return (double)(N - 1) / N * 2.0 * kPi / log(k_max / k_min);
}

// c_s (eq. cm), a_s and c_s g(a_s): one wave per (s, factor), the DFT over l split across lanes
__global__ __launch_bounds__(64) void k_fftlog_coeffs(FftlogArgs g)
{
    const int s = blockIdx.x, f = blockIdx.y, lane = threadIdx.x;
    const int N = g.N, m = s - N / 2;
    const double nu = g.f[f].nu;
    const double L = log(g.k_max / g.k_min), dl = L / (N - 1);
    const int mm = ((m % N) + N) % N;
    double re = 0.0, im = 0.0;
    for (int l = lane; l < N; l += 64) {
        const double v = g.Pk[l] * exp(-nu * dl * l);
        const int q = (int)(((unsigned)mm * (unsigned)l) % (unsigned)N);  // exact residue (< 2^24 product)
        double sn, cs;
        sincospi(2.0 * q / N, &sn, &cs);
        re += v * cs;
        im -= v * sn;
    }
    for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o, 64);
        im += __shfl_xor(im, o, 64);
    }
    if (lane > 1) return;
    const double eta = fftlog_deta(N, g.k_min, g.k_max) * m;
    const double2 a = make_double2(1.0 + nu, eta);
    const int n = g.f[f].n, mt = g.f[f].mt;
    // lane 0: log Gamma((1 + mt + a + n)/2); lane 1: log Gamma((1 - a - mt + n)/2)
    const double2 lg = clgamma(lane == 0 ? make_double2(0.5 * (1.0 + mt + a.x + n), 0.5 * a.y)
                                         : make_double2(0.5 * (1.0 - a.x - mt + n), -0.5 * a.y));
    const double2 l1 = make_double2(__shfl(lg.x, 0, 64), __shfl(lg.y, 0, 64));
    const double2 l2 = make_double2(__shfl(lg.x, 1, 64), __shfl(lg.y, 1, 64));
    if (lane) return;
    const double w = (s == 0 || s == N) ? 0.5 : 1.0;
    const double2 pre = cexp(make_double2(-nu * log(g.k_min), -eta * log(g.k_min)));
    const double2 c = cmul(pre, make_double2(w * re / N, w * im / N));
    const double ln2 = 0.69314718055994530942;
    const double2 gl = make_double2((mt + a.x - 1.0) * ln2 + l1.x - l2.x, a.y * ln2 + l1.y - l2.y);
    double2 cg = cmul(c, cexp(gl));
    cg.x /= kPi;
    cg.y /= kPi;
    g.cg[(size_t)f * g.ld + s] = cg;
    g.a[(size_t)f * g.ld + s] = a;
}

// Two tables in one launch:
//   U[f][s][i] = c_s g(a_s) theta_i^{-(1 + a_s + mt)} and its weighted upper half Uw [f][m][i],
//   one thread per (factor, s < Ns, angle);
//   E[j][t] = e^{-i t deta ln chi_j}, t = 0..N, the threads after those.
__global__ void k_fftlog_tables(FftlogArgs g)
{
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nu = (int64_t)4 * g.T * g.Ns;
    if (t0 < nu) {
        const int i = (int)(t0 % g.T), s = (int)((t0 / g.T) % g.Ns), f = (int)(t0 / ((int64_t)g.Ns * g.T));
        const int mt = g.f[f].mt;
        const double2 cg = g.cg[(size_t)f * g.ld + s], a = g.a[(size_t)f * g.ld + s];
        const double lt = log(g.theta[i]);
        const double2 u = cmul(cg, cexp(make_double2(-(1.0 + a.x + mt) * lt, -a.y * lt)));
        g.U[((size_t)f * g.ld + s) * g.T + i] = u;
        const int m = s - g.N / 2;
        if (m >= 0) {
            const double om = m ? 2.0 : 1.0;
            g.Uw[((size_t)f * g.ldw + m) * g.T + i] = make_double2(om * u.x, om * u.y);
        }
    } else if (t0 - nu < (int64_t)g.nchi * (g.N + 1)) {
        const int64_t e = t0 - nu;
        const int t = (int)(e % (g.N + 1)), j = (int)(e / (g.N + 1));
        const double lc = log(g.chi_min) + j * g.dlnchi;
        double sn, cs;
        sincos(-(double)t * fftlog_deta(g.N, g.k_min, g.k_max) * lc, &sn, &cs);
        g.E[(size_t)j * g.ldh + t] = make_double2(cs, sn);
    }
}

// weights of each (factor pair q, model b): D[j][q][b] = w_j F_b(chi_j) chi_j^{-1} chi_j^{-(2 + nu1 + nu2)}
// (w_j the trapezoid weights in ln chi)
__global__ void k_fftlog_weights(const double *F, int nchi, int nmodels, double chi_min, double dlnchi,
                                 double3 nusum, double *D)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nchi * nmodels * 3) return;
    const int b = (int)(t % nmodels), q = (int)(t / nmodels % 3), j = (int)(t / ((int64_t)nmodels * 3));
    const double lc = log(chi_min) + j * dlnchi;
    const double w = (j == 0 || j == nchi - 1) ? 0.5 * dlnchi : dlnchi;
    const double e = q == 0 ? nusum.x : q == 1 ? nusum.y : nusum.z;
    D[t] = w * F[(size_t)b * nchi + j] * exp(-(3.0 + e) * lc);
}

// Batched FP64 matrix product C[q][b] = A[q][b] B[q][b] over the factor pairs q and the models b of
// a pass (blockIdx.z = q models + b), elements addressed by strides (a Hankel operand
// H_{ik} = h[i + k] is a_i = a_k = 1).  One launch takes all three factor pairs: one pair of 128
// models (640 blocks of four waves at N = 256, T = 64) left the chip a third empty and ended in
// a tail of its own.  A is complex; by TAG:
//   1: B real, C complex, and each row i of C also written, conjugated, at row -i (the mirror
//      h(-t) = conj h(t))
//   2: B and C complex
//   3: B complex, only Re C computed and stored (as double)
// Each wave computes a (16 RM) x 16 tile of C (RM 16 x 16 MFMA tiles sharing one B fragment).
// With KSPLIT the block's four waves share one tile and split the k range (runs of 8, wave w
// takes runs w, w + 4, ...; partial sums added through LDS in a fixed order, so results are
// deterministic): for products with few output tiles and a long k range.  Without it the four
// waves take neighbouring tiles of their own.  The fragments of the next k-steps are loaded
// before the current step's MFMAs.  Operand lane
// layout of v_mfma_f64_16x16x4f64: A row / B column = lane & 15, k = lane >> 4.  Every operand is
// laid out with its rows (A) or columns (B) contiguous: a 16-byte load then returns 64 bytes
// per cycle, where rows far apart return one lane's 16 (counters at 1024 models, rows apart: 55
// cycles per load, the data return 94% busy, the matrix cores 72%).  Waves of 32 x 16 tiles:
// 64 x 16 leave the last row tile of N + 1 = 257 a block of its own (128 models 255 us in all,
// 32 x 16 237 us).  Whole calls at N = 256, 512 chi, 64 angles, this and the form before: 4
// models 192 -> 98 us, 128 343 -> 237 us, 1024 1827 -> 1428 us.
struct CGemm {
    const double2 *A;
    int64_t a_i, a_k, a_b;
    const void *B;
    int64_t b_k, b_j, b_b;
    int64_t c_i, c_j;
    int M, N, K;
    int nb;                    // models
    int64_t a_q[3], b_q[3];    // operands of factor pair q
    void *c_q[3];              // results of factor pair q, models c_bq apart
    int64_t c_bq[3];
    int wc_shift;
};

template <int TAG, int RM, bool KSPLIT>
__global__ __launch_bounds__(256) void k_cgemm(CGemm g)
{
    constexpr bool BREAL = TAG == 1, CREAL = TAG == 3;
    typedef typename std::conditional<BREAL, double, double2>::type BT;
    __shared__ double red[3][8][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // without KSPLIT the block's waves are 2^wc_shift columns by 4 >> wc_shift rows of tiles
    const int wr = w >> g.wc_shift, wc = w & ((1 << g.wc_shift) - 1);
    const int j0 = (KSPLIT ? blockIdx.x : (blockIdx.x << g.wc_shift) + wc) * 16;
    const int i0 = (KSPLIT ? blockIdx.y : blockIdx.y * (4 >> g.wc_shift) + wr) * 16 * RM;
    if (!KSPLIT && (j0 >= g.N || i0 >= g.M)) return;  // no barrier in this mode
    const int fq = (int)blockIdx.z / g.nb, b = (int)blockIdx.z - fq * g.nb;
    const int r = lane & 15, q = lane >> 4;
    const int nrm = min(RM, (g.M - i0 + 15) / 16);  // block-uniform count of live row tiles
    const double2 *A = g.A + (size_t)b * g.a_b + g.a_q[fq];
    const BT *B = static_cast<const BT *>(g.B) + (size_t)b * g.b_b + g.b_q[fq];
    const int jb = j0 + r;
    const bool jin = jb < g.N;

    // per-lane row pointers of A and column pointer of B; k offsets stay 32-bit (k a_k and k b_k
    // < 2^31, see fftlog_most_models).  Rows and columns past the matrix read its first ones
    // and are not stored, so only the last k-step, past K, is masked: a zero B with the A of K - 1
    const double2 *Ar[RM];
#pragma unroll
    for (int u = 0; u < RM; ++u) {
        const int i = i0 + 16 * u + r;
        Ar[u] = A + (u < nrm && i < g.M ? (size_t)i * g.a_i : 0);
    }
    const BT *Bc = B + (jin ? (size_t)jb * g.b_j : 0);
    const int ak = (int)g.a_k, bk = (int)g.b_k;
    auto load = [&](int kb, double2 (&av)[RM], BT &bv) __attribute__((always_inline)) {
        if (kb + 4 <= g.K) {  // wave-uniform
            const int k = kb + q;
#pragma unroll
            for (int u = 0; u < RM; ++u) av[u] = Ar[u][k * ak];
            bv = Bc[k * bk];
        } else if (kb < g.K) {
            const int k = min(kb + q, g.K - 1);
#pragma unroll
            for (int u = 0; u < RM; ++u) av[u] = Ar[u][k * ak];
            bv = Bc[k * bk];
            if (kb + q >= g.K) bv = BT{};
        }
    };
    v4d re[RM], im[RM];
#pragma unroll
    for (int u = 0; u < RM; ++u) {
        re[u] = v4d{0.0, 0.0, 0.0, 0.0};
        im[u] = v4d{0.0, 0.0, 0.0, 0.0};
    }
    auto step = [&](const double2 (&av)[RM], const BT &bv) {
        if constexpr (BREAL) {
#pragma unroll
            for (int u = 0; u < RM; ++u)
                if (u < nrm) re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv, re[u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < RM; ++u)
                if (u < nrm) im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].y, bv, im[u], 0, 0, 0);
        } else if constexpr (CREAL) {
            const double nby = -bv.y;
#pragma unroll
            for (int u = 0; u < RM; ++u)
                if (u < nrm) re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv.x, re[u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < RM; ++u)
                if (u < nrm) re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].y, nby, re[u], 0, 0, 0);
        } else {
            const double nby = -bv.y;
#pragma unroll
            for (int u = 0; u < RM; ++u)
                if (u < nrm) {
                    re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv.x, re[u], 0, 0, 0);
                    im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].x, bv.y, im[u], 0, 0, 0);
                }
#pragma unroll
            for (int u = 0; u < RM; ++u)
                if (u < nrm) {
                    re[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].y, nby, re[u], 0, 0, 0);
                    im[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u].y, bv.x, im[u], 0, 0, 0);
                }
        }
    };
    // k-steps requested ahead: the single-tile product has two MFMAs a step, which hide little
    // (one step ahead it took 19 us at N = 256, 512 chi and 128 models)
    constexpr int PD = RM == 1 ? 8 : 2;
    double2 af[PD][RM];
    BT bf[PD];
    // step n of this wave starts at k = kat(n)
    auto kat = [&](int n) { return KSPLIT ? 32 * (n >> 1) + 8 * w + 4 * (n & 1) : 4 * n; };
#pragma unroll
    for (int d = 0; d < PD - 1; ++d) load(kat(d), af[d], bf[d]);
    for (int n = 0; kat(n) < g.K; n += PD) {
#pragma unroll
        for (int d = 0; d < PD; ++d) {
            load(kat(n + d + PD - 1), af[(d + PD - 1) % PD], bf[(d + PD - 1) % PD]);
            if (kat(n + d) < g.K) step(af[d], bf[d]);
        }
    }
    // partial sums of waves 1..3 added into wave 0's, one row tile at a time
    for (int u = 0; KSPLIT && u < RM; ++u) {
        if (u >= nrm) break;
        if (w > 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                red[w - 1][k][lane] = re[u][k];
                red[w - 1][4 + k][lane] = im[u][k];
            }
        }
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                re[u][k] = ((re[u][k] + red[0][k][lane]) + red[1][k][lane]) + red[2][k][lane];
                im[u][k] = ((im[u][k] + red[0][4 + k][lane]) + red[1][4 + k][lane]) + red[2][4 + k][lane];
            }
        }
        __syncthreads();
    }
    if ((KSPLIT && w > 0) || !jin) return;
    // v_mfma_f64_16x16x4f64 result layout: register k of lane l holds D[4k + l/16][l % 16]
#pragma unroll
    for (int u = 0; u < RM; ++u) {
        if (u >= nrm) break;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + 16 * u + 4 * k + q;
            if (i >= g.M) continue;
            const int64_t o = (size_t)b * g.c_bq[fq] + i * g.c_i + jb * g.c_j;
            if constexpr (CREAL) {
                static_cast<double *>(g.c_q[fq])[o] = re[u][k];
            } else {
                double2 *C = static_cast<double2 *>(g.c_q[fq]);
                C[o] = make_double2(re[u][k], im[u][k]);
                if constexpr (TAG == 1) C[o - 2 * i * g.c_i] = make_double2(re[u][k], -im[u][k]);
            }
        }
    }
}

template <int TAG, int RM, bool KSPLIT>
static z3_status cgemm(const CGemm &g0, int pairs, hipStream_t s)
{
    // waves side by side along the columns, as far as there are column tiles
    CGemm g = g0;
    g.wc_shift = g.N > 32 ? 2 : (g.N > 16 ? 1 : 0);
    const int cols = KSPLIT ? 16 : 16 << g.wc_shift, rows = 16 * RM * (KSPLIT ? 1 : 4 >> g.wc_shift);
    const dim3 grid((unsigned)((g.N + cols - 1) / cols), (unsigned)((g.M + rows - 1) / rows), (unsigned)(pairs * g.nb));
    hipEvent_t ev0 = nullptr;
    if (TAG == 2) profile_begin(s, &ev0);
    hipLaunchKernelGGL((k_cgemm<TAG, RM, KSPLIT>), grid, dim3(256), 0, s, g);
    if (TAG == 2) profile_end(s, ev0);
    return check_launch("k_cgemm");
}

// out[b][1] = I1 + I1^T (out [b][3][T][T], I1 [b][T][T]; the other two are written directly)
__global__ void k_fftlog_out(const double *I1, int T, int nmodels, double *out)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per = (int64_t)T * T;
    if (t >= per * nmodels) return;
    const int64_t b = t / per;
    const int ij = (int)(t % per), i = ij / T, j = ij % T;
    const double *Ib = I1 + (size_t)b * per;
    out[(size_t)(3 * b + 1) * per + ij] = Ib[ij] + Ib[(size_t)j * T + i];
}

z3_status fftlog_impl(int N, const double *Pk, double k_min, double k_max, const double *nu, int nchi, double chi_min,
                      double chi_max, int nmodels, const double *F, int T, const double *theta, double *out,
                      void *ws, int chunk, hipStream_t s)
{
    const FftlogLayout L = fftlog_layout(N);
    FftlogArgs g;
    g.N = N;
    g.Ns = N + 1;
    g.ld = (int)L.ld;
    g.ldw = (int)L.ldw;
    g.ldh = (int)L.ldh;
    g.Pk = Pk;
    g.k_min = k_min;
    g.k_max = k_max;
    const int ns[4] = {0, 1, 1, 2}, mts[4] = {0, 1, -1, 0};
    for (int f = 0; f < 4; ++f) g.f[f] = FactorSpec{ns[f], mts[f], nu[f]};
    g.nchi = nchi;
    g.chi_min = chi_min;
    g.dlnchi = log(chi_max / chi_min) / (nchi - 1);
    g.T = T;
    g.theta = theta;
    char *p = static_cast<char *>(ws);
    auto take = [&](size_t bytes) { char *q = p; p += (bytes + 255) / 256 * 256; return q; };
    g.cg = reinterpret_cast<double2 *>(take(4 * L.ld * sizeof(double2)));
    g.a = reinterpret_cast<double2 *>(take(4 * L.ld * sizeof(double2)));
    g.U = reinterpret_cast<double2 *>(take(4 * (size_t)T * L.ld * sizeof(double2)));
    g.Uw = reinterpret_cast<double2 *>(take(4 * (size_t)T * L.ldw * sizeof(double2)));
    g.E = reinterpret_cast<double2 *>(take((size_t)nchi * L.ldh * sizeof(double2)));
    double *D = reinterpret_cast<double *>(take((size_t)chunk * 3 * nchi * sizeof(double)));
    double2 *H = reinterpret_cast<double2 *>(take((size_t)chunk * 3 * L.ldt * sizeof(double2)));
    double2 *UA = reinterpret_cast<double2 *>(take((size_t)chunk * 3 * T * L.ld * sizeof(double2)));
    double *Ire = reinterpret_cast<double *>(take((size_t)chunk * 3 * T * T * sizeof(double)));

    hipLaunchKernelGGL(k_fftlog_coeffs, dim3((unsigned)g.Ns, 4), dim3(64), 0, s, g);
    z3_status st = check_launch("k_fftlog_coeffs");
    if (st != Z3_OK) return st;
    const int64_t ntab = (int64_t)4 * T * g.Ns + (int64_t)nchi * (N + 1);
    hipLaunchKernelGGL(k_fftlog_tables, dim3((unsigned)((ntab + 255) / 256)), dim3(256), 0, s, g);
    if ((st = check_launch("k_fftlog_tables")) != Z3_OK) return st;
    // factor pairs of A_0, A_1, A_2: (0,0)x(0,0), (1,1)x(1,-1), (2,0)x(2,0)
    const int f1[3] = {0, 1, 3}, f2[3] = {0, 2, 3};
    const double3 nusum = make_double3(nu[0] + nu[0], nu[1] + nu[2], nu[3] + nu[3]);
    const int64_t ld = (int64_t)L.ld, ldw = (int64_t)L.ldw, ldh = (int64_t)L.ldh, ldt = (int64_t)L.ldt;
    for (int b0 = 0; b0 < nmodels && st == Z3_OK; b0 += chunk) {
        const int nb = nmodels - b0 < chunk ? nmodels - b0 : chunk;
        const int64_t nw = (int64_t)nb * nchi * 3;
        hipLaunchKernelGGL(k_fftlog_weights, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, s,
                           F + (size_t)b0 * nchi, nchi, nb, chi_min, g.dlnchi, nusum, D);
        if ((st = check_launch("k_fftlog_weights")) != Z3_OK) break;
        // h[col][N + t] = sum_j E[j][t] D[col][j] for t = 0..N, mirrored to N - t; col = (q, b)
        CGemm mh{g.E, 1, ldh, 0, D, 3 * nb, 1, 0, 1, ldt, N + 1, 3 * nb, nchi, 1, {0, 0, 0}, {0, 0, 0},
                 {H + N, nullptr, nullptr}, {0, 0, 0}};
        if ((st = cgemm<1, 1, true>(mh, 1, s)) != Z3_OK) break;
        const int64_t TT = (int64_t)T * T, TL = (int64_t)T * ld, TW = (int64_t)T * ldw;
        double *ob = out + (size_t)b0 * 3 * TT;
        // UA[b][q][s2][i] = sum_{m >= 0} h[q][b][N/2 + m + s2] Uw_f1[m][i]
        CGemm m2{H + N / 2, 1, 1, ldt, g.Uw, T, 1, 0, T, 1, g.Ns, T, N / 2 + 1, nb,
                 {0, nb * ldt, 2 * nb * ldt}, {f1[0] * TW, f1[1] * TW, f1[2] * TW}, {UA, UA + TL, UA + 2 * TL},
                 {3 * TL, 3 * TL, 3 * TL}};
        if ((st = cgemm<2, 2, false>(m2, 3, s)) != Z3_OK) break;
        // I[b][q][i][j] = Re sum_s UA[b][q][s][i] U_f2[s][j]: A_0 and A_2 as they are, A_1 still to
        // be symmetrised
        CGemm m3{UA, 1, T, 3 * TL, g.U, T, 1, 0, (int64_t)T, 1, T, T, g.Ns, nb, {0, TL, 2 * TL},
                 {f2[0] * TL, f2[1] * TL, f2[2] * TL}, {ob, Ire, ob + 2 * TT}, {3 * TT, TT, 3 * TT}};
        if ((st = cgemm<3, 2, false>(m3, 3, s)) != Z3_OK) break;
        hipLaunchKernelGGL(k_fftlog_out, dim3((unsigned)((nb * TT + 255) / 256)), dim3(256), 0, s, Ire, T, nb, ob);
        st = check_launch("k_fftlog_out");
    }
    return st;
}

}  // namespace z3
