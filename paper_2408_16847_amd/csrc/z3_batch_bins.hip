// Many-map multipoles on MFMA, many bins at a time: the contraction of z3_batch.hip for bins of
// few pairs.
//
// Work split: as there, one block owns one pivot and 16 * TI * WPB maps.  The (bin, band) windows
// of as many bins as fit, one per thread, are laid end to end, each run of windows of one bin (up
// to 64 bands) starting on a multiple of four candidates.  Groups of 64 * WPB consecutive
// candidates, of however many bins, go one per thread: each thread tests its candidate against
// its own bin and writes its harmonic row to LDS (zeros when it is not in its bin); after a block
// barrier every wave runs the MFMA steps for its own maps over the whole group, 4 candidates of
// one bin per step, and writes a bin's sums when its last step is done.  The sums and their order
// are those of z3_batch.hip.
//
// What bounds it: with one bin at a time, a bin of 25 pairs fills a fifth of a group of 128 and
// pays the same four barriers and chain of dependent loads as a full one.  Measured, 64 maps,
// Nside 128, 15 bins of 25 pairs, m_max 10: 19.5 -> 13.5 ms mixed, 22.5 -> 17.9 ms FP64 (70 weighted
// maps 43.9 -> 33.2 ms); the map values' cache lines (256 B per candidate and wave) are what is left.
#include "z3_batch.h"

namespace z3 {

// Whether the launch takes many bins at a time: bins of few pairs, which the index's mean density
// (over the longitudes that hold points: a cap fills little of its colatitude range) and the
// bins' area give.  Larger bins fill groups by themselves and run faster with one bin's
// edges, window and flush points held for all of its groups.  Measured, one bin at a time / many:
// 12 pairs a bin (90 maps, FP32, m_max 3) 2147 / 1345 us; 25 pairs (64 maps, m_max 10) 19458 / 13543 us,
// in FP64 22470 / 17926; 83 (m_max 16) 35372 / 36872; 100 (m_max 10) 46122 / 44560; 187 (m_max 4,
// weights) 23820 / 22845; 400 111016 / 133761, in FP64 175719 / 188280.  The line is set at 64.  The
// value matrix is read through 32-bit offsets: one of 4 GiB and more takes one bin at a time.
constexpr double kFewPairs = 64.0;
constexpr size_t kMaxBinsBytes = 0xffffffff;

bool batch_many_bins(const z3_index_s *idx, bool f32)
{
    const EdgeTab &t = idx->edges;
    const int nb = idx->nbins;
    return idx->density / idx->sky_part * kPi * (t.e[nb] - t.e[0]) < kFewPairs * nb &&
           2 * (size_t)idx->n * batch_ldv(idx->nmaps) * (f32 ? 4 : 8) <= kMaxBinsBytes;
}

constexpr int kLastRun = 256;  // flag beside a bin number (Z3_MAX_NBINS = 64)

// Register budget: 3 waves per SIMD on the mixed path (measured faster than the
// compiler's own choice), 2 on the FP64 path.
template <int M, bool F32, int WPB, int TI>
__global__ __launch_bounds__(WPB * kWave) __attribute__((amdgpu_waves_per_eu(F32 ? 3 : 2)))
void k_multipoles_batch_bins(BatchArgs a)
{
    typedef typename BatchT<F32>::T T;
    typedef typename BatchT<F32>::V4 V4;
    constexpr int NC = 2 * M + 1;             // harmonic columns
    constexpr int NCT = (NC + 15) / 16;       // 16-column MFMA tiles
    constexpr int HS = (NC + 31) / 32 * 32;   // LDS row length of the harmonic rows
    constexpr int NCAND = WPB * kWave;        // candidates per group
    constexpr int SL = NCAND;                 // windows laid end to end at a time

    __shared__ int s_klo[Z3_MAX_NBINS], s_nk[Z3_MAX_NBINS];  // bands of each bin: first, number
    // windows: search key, end of the positions, and the records of a position p: a0 + p before
    // `split`, a1 + p from it on
    __shared__ int s_key[SL];
    __shared__ int4 s_win[SL];         // end of its positions, split, a0, a1
    __shared__ double2 s_winedge[SL];  // edges of the window's bin
    // runs of windows of one bin (up to 64 bands): first window, bin (kLastRun: the bin's last
    // run), first position and end of its candidates
    __shared__ int s_runw[kWave + 1], s_runbin[kWave], s_runpos[kWave + 1], s_runlim[kWave], s_runshift[kWave];
    __shared__ int s_wtot[WPB];
    __shared__ uint64_t s_in[WPB];    // which of the group's candidates are in their bins
    __shared__ uint32_t s_j[NCAND];   // byte offset of each candidate's value row
    __shared__ T s_h[NCAND * HS];
    __shared__ double s_wc[NCAND];    // weights of the group's candidates (0 outside the bin)

    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int tid = threadIdx.x;
    // logical block: XCD-contiguous; the map tiles of one pivot are adjacent
    const int lb = xcd_block(blockIdx.x, a.nblocks);
    const int mt = lb % a.ntiles;
    const int64_t p = a.p0 + lb / a.ntiles;
    if (p >= a.p1) return;  // uniform per block
    const int mb = (mt * WPB + wv) * 16 * TI;  // first map of this wave
    const bool has_maps = mb < a.nmaps;        // uniform per wave

    const PivotFrame f = uniform_frame(pivot_frame(a.px[p], a.py[p], a.pz[p]));
    const int64_t col = p - a.p0;
    const int nb = a.nb;
    const bool unit_w = a.wdbl == nullptr;
    const int r16 = lane & 15, g4 = lane >> 4;
    // this lane's maps of a candidate's value row, by the row's byte offset
    const __amdgpu_buffer_rsrc_t vbuf = buffer_view(a.vmat, a.vmat_bytes);
    const uint32_t vlane = (uint32_t)(has_maps ? mb + TI * r16 : 0) * sizeof(T);
    auto load_values = [&](uint32_t row, T (&v)[TI]) __attribute__((always_inline)) {
        constexpr int NB = TI * (int)sizeof(T) / 4;  // 4-byte words
        typedef unsigned int w2 __attribute__((ext_vector_type(2)));
        typedef unsigned int w4 __attribute__((ext_vector_type(4)));
        if constexpr (NB == 1) {
            v[0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(vbuf, row + vlane, 0, 0));
        } else if constexpr (NB == 2) {
            const w2 q = __builtin_amdgcn_raw_buffer_load_b64(vbuf, row + vlane, 0, 0);
            __builtin_memcpy(v, &q, sizeof(q));
        } else {
            const w4 q = __builtin_amdgcn_raw_buffer_load_b128(vbuf, row + vlane, 0, 0);
            __builtin_memcpy(v, &q, sizeof(q));
        }
    };
    // harmonic columns of this lane: LDS column, before the row's swizzle (hslot), of the MFMA
    // operand, and place in the output of a map: 2 m + (re, im), its sign in e^{-i m phi}
    int hcol[NCT], ocol[NCT];
    double osgn[NCT];
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
        const int c = 16 * t + r16;
        hcol[t] = c ^ ((g4 & 1) << 4) ^ (g4 >> 1);
        ocol[t] = c <= M ? 2 * c : (c < NC ? 2 * (c - M) + 1 : (c == NC ? 1 : -1));
        osgn[t] = c <= M ? 1.0 : -1.0;
    }
    uint64_t pairs_all = 0;

    if (tid < nb) {
        const double rad = a.edges->rad_out[tid + 1];
        const int klo = max((int)floor((f.th - rad) * a.inv_h), 0);
        const int khi = min((int)floor((f.th + rad) * a.inv_h), a.nbands - 1);
        s_klo[tid] = klo;
        s_nk[tid] = max(khi - klo + 1, 0);
    }
    __syncthreads();

    // sums of the current bin
    V4 acc[TI][NCT];
    double acc64[TI][NCT][4];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                acc[i][t] = V4{0, 0, 0, 0};
#pragma unroll
                for (int r = 0; r < 4; ++r) acc64[i][t][r] = 0.0;
            }
    };
    clear();
    double wslot = 0.0;  // weight sum of the candidates at positions lane, lane + 64, ...
    int cnt = 0;         // pairs of the current bin

    // the sums of bin `bin` are complete: normalise and write them
    auto write_bin = [&](int bin) {
        const double Wb = unit_w ? (double)cnt : wave_sum_f64(wslot);
        pairs_all += (uint64_t)cnt;
        if (has_maps) {
            const double inv = Wb > 0.0 ? 1.0 / Wb : 0.0;
            // pivot-major staging: the bin's values of all maps are one contiguous run, so the
            // block's stores fill whole cache lines
            T *out = static_cast<T *>(a.stage) + ((size_t)col * nb + bin) * (size_t)a.nmaps * (2 * (M + 1));
#pragma unroll
            for (int t = 0; t < NCT; ++t) {
                if (ocol[t] < 0) continue;
                const double scale = osgn[t] * inv;
                const bool zero = 16 * t + r16 == NC;  // Im X_0 = 0
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // f32 16x16x4 result: register r of lane l is D[4 (l/16) + r][l % 16];
                        // f64 16x16x4 result: register r of lane l is D[4 r + l/16][l % 16]
                        const int map = mb + TI * (F32 ? 4 * g4 + r : 4 * r + g4) + i;
                        if (map >= a.nmaps) continue;
                        const double s = F32 ? acc64[i][t][r] : (double)acc[i][t][r];
                        out[map * (2 * (M + 1)) + ocol[t]] = zero ? T(0) : (T)(s * scale);
                    }
            }
        }
        if (mt == 0 && tid == 0 && a.W) a.W[(size_t)bin * (size_t)a.ldA + col] = Wb;
        clear();
        wslot = 0.0;
        cnt = 0;
    };

    int bin = 0, kb = __builtin_amdgcn_readfirstlane(s_klo[0]);  // next window: band kb of bin `bin`
    while (bin < nb) {
        // the next runs: whole ones, as many as fit, this thread's window among them
        int nwin = 0, nrun = 0, wbin = 0, wband = 0, wrun = -1;
        while (bin < nb && nrun < kWave) {
            const int rest = __builtin_amdgcn_readfirstlane(s_klo[bin] + s_nk[bin]) - kb, take = min(rest, kWave);
            if (nwin + take > SL) break;
            if (tid >= nwin && tid < nwin + take) {
                wbin = bin;
                wband = kb + tid - nwin;
                wrun = nrun;
            }
            const bool last = take == rest;
            if (tid == 0) {
                s_runw[nrun] = nwin;
                s_runbin[nrun] = bin | (last ? kLastRun : 0);
            }
            nwin += take;
            ++nrun;
            kb += take;
            if (last && ++bin < nb) kb = __builtin_amdgcn_readfirstlane(s_klo[bin]);
        }
        if (tid == 0) s_runw[nrun] = nwin;
        int s0 = 0, l0 = 0, s1 = 0, l1 = 0, base = 0;
        if (wrun >= 0) {
            const Band bd = a.bands[wband];
            if (bd.npts > 0) {
                band_window(bd, a.cell_start, f.th, f.sh, f.ch, f.inv_sp, f.phf, a.edges->hav_out[wbin + 1],
                            a.edges->hav_in[wbin], s0, l0, s1, l1);
                base = 2 * bd.pt_start;
            }
        }
        // positions: inclusive sums over the windows, then every run moved to a multiple of 4
        const int len = l0 + l1;
        int incl = wave_incl_scan(len, lane);
        if (lane == kWave - 1) s_wtot[wv] = incl;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WPB - 1; ++w)
            if (w < wv) incl += s_wtot[w];
        s_key[tid] = incl;
        __syncthreads();
        if (wv == 0) {
            const int r = min(lane, nrun), r1 = min(lane + 1, nrun);
            const int w0 = s_runw[r], w1 = s_runw[r1];
            const int beg = w0 > 0 ? s_key[w0 - 1] : 0, n = (w1 > 0 ? s_key[w1 - 1] : 0) - beg;
            const int padded = (n + 3) & ~3;
            const int pend = wave_incl_scan(padded, lane), pos = pend - padded;
            if (lane < nrun) {
                s_runpos[lane] = pos;
                s_runlim[lane] = pos + n;
                s_runshift[lane] = pos - beg;
                s_runpos[lane + 1] = pend;  // the next lane writes the same value
            }
        }
        __syncthreads();
        if (wrun >= 0) {
            const int lim = incl + s_runshift[wrun], start = lim - len;
            // the padding belongs to the run's last window that holds candidates
            s_key[tid] = lim == s_runlim[wrun] ? s_runpos[wrun + 1] : lim;
            s_win[tid] = make_int4(lim, start + l0, base + s0 - start, base + s1 - (start + l0));
            s_winedge[tid] = make_double2(a.edges->e[wbin], a.edges->e[wbin + 1]);
        } else {
            s_key[tid] = 0x7fffffff;
        }
        __syncthreads();
        const int total = nrun ? __builtin_amdgcn_readfirstlane(s_runpos[nrun]) : 0;

        // `run` is being summed, n of its steps are done; runs that end by position p are finished
        int run = 0, n = 0;
        auto finish_runs = [&](int p) {
            while (run < nrun && __builtin_amdgcn_readfirstlane(s_runpos[run + 1]) <= p) {
                const int rb = __builtin_amdgcn_readfirstlane(s_runbin[run]);
                if (rb & kLastRun) write_bin(rb & ~kLastRun);
                ++run;
                n = 0;
            }
        };
        for (int f0 = 0; f0 < total; f0 += NCAND) {
            // locate this thread's candidate: window = first q with s_key[q] > p
            const int p = min(f0 + tid, total - 1);
            int q = 0;
#pragma unroll
            for (int step = SL / 2; step > 0; step >>= 1)
                if (s_key[q + step - 1] <= p) q += step;
            const int4 win = s_win[q];
            const double2 edge = s_winedge[q];
            const bool cand = f0 + tid < total && p < win.x;
            const int pc = min(p, win.x - 1);  // padding reads the run's last candidate
            const int j = pc < win.y ? win.z + pc : win.w + pc;

            const double4 rec = a.rec[j];
            const double dx = rec.x - f.xp, dy = rec.y - f.yp, dz = rec.z - f.zp;
            const double d2 = (dx * dx + dy * dy) + dz * dz;
            const bool in = cand && d2 >= edge.x && d2 < edge.y;
            const uint64_t inmask = __ballot(in);
            if (lane == 0) s_in[wv] = inmask;
            T h[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) h[c] = T(0);
            if (!unit_w) s_wc[tid] = in ? a.wdbl[j] : 0.0;
            if (in) harmonic_row<M>(f, dx, dy, dz, h);
#pragma unroll
            for (int c = 0; c < NC; ++c) s_h[hslot<HS>(tid, c)] = h[c];
            s_j[tid] = (uint32_t)j * (uint32_t)(a.ldv * sizeof(T));
            __syncthreads();

            // MFMA steps of 4 candidates over the group, in chunks of up to 8 steps of one run; the
            // map values of the next chunk are requested before the current one's steps.  The
            // mixed path adds its FP32 sums into the FP64 bin sums every 32 steps of a run (128
            // candidates) and at its end, the same points for every block shape, so no chunk
            // reaches over a multiple of 32.
            constexpr int CH = 8;
            const int nst = min(total - f0, NCAND) >> 2;
            T vcur[CH][TI], vnext[CH][TI];
            auto load_chunk = [&](int at, int len, T (&v)[CH][TI]) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < CH; ++u)
                    if (u < len) load_values(s_j[4 * (at + u) + g4], v[u]);
            };
            int st = 0, rend = 0, len = 0;
            // the pairs of the current run among the group's candidates
            auto count_run = [&](int beg, int end) __attribute__((always_inline)) {
#pragma unroll
                for (int w = 0; w < WPB; ++w) {
                    const int lo = min(max(4 * beg - kWave * w, 0), kWave), hi = min(max(4 * end - kWave * w, 0), kWave);
                    if (hi <= lo) continue;
                    const uint64_t bits = (hi - lo == kWave ? ~0ull : ((1ull << (hi - lo)) - 1)) << lo;
                    cnt += __popcll(s_in[w] & bits);
                }
            };
            finish_runs(f0);
            if (nst > 0) {
                rend = (__builtin_amdgcn_readfirstlane(s_runpos[run + 1]) - f0) >> 2;
                len = min(min(CH, 32 - (n & 31)), min(rend, nst));
                if (has_maps) load_chunk(0, len, vcur);
                count_run(0, min(rend, nst));
            }
            while (st < nst) {
                const int st2 = st + len;
                int rend2 = rend, len2 = 0;
                if (st2 < nst) {
                    int n2 = n + len;
                    for (int r = run + 1; rend2 <= st2; ++r) {
                        rend2 = (__builtin_amdgcn_readfirstlane(s_runpos[r + 1]) - f0) >> 2;
                        n2 = 0;
                    }
                    len2 = min(min(CH, 32 - (n2 & 31)), min(rend2, nst) - st2);
                    if (has_maps) load_chunk(st2, len2, vnext);
                }
                if (!unit_w) {
                    // the weight of the run's candidate i goes to lane i mod 64, in order
                    const int o = (lane - 4 * n) & (kWave - 1);
                    if (o < 4 * len) wslot += s_wc[4 * st + o];
                }
                n += len;
                if (has_maps) {
                    // operands of a step: rows 4 sp + g4; hslot's swizzle is that of hcol and the
                    // step's share.  They are read one step ahead.
                    auto row = [&](int sp, T (&hb)[NCT]) __attribute__((always_inline)) {
#pragma unroll
                        for (int t = 0; t < NCT; ++t) hb[t] = s_h[(4 * sp + g4) * HS + (hcol[t] ^ (2 * sp & 15))];
                    };
                    T ha[NCT], hn[NCT];
                    row(st, ha);
#pragma unroll
                    for (int u = 0; u < CH; ++u) {
                        if (u >= len) break;
                        row(min(st + u + 1, NCAND / 4 - 1), hn);
#pragma unroll
                        for (int i = 0; i < TI; ++i)
#pragma unroll
                            for (int t = 0; t < NCT; ++t) {
                                if constexpr (F32)
                                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vcur[u][i], ha[t], acc[i][t], 0, 0, 0);
                                else
                                    acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(vcur[u][i], ha[t], acc[i][t], 0, 0, 0);
                            }
#pragma unroll
                        for (int t = 0; t < NCT; ++t) ha[t] = hn[t];
                    }
                    if constexpr (F32) {
                        if ((n & 31) == 0 || st2 == rend) {
#pragma unroll
                            for (int i = 0; i < TI; ++i)
#pragma unroll
                                for (int t = 0; t < NCT; ++t) {
#pragma unroll
                                    for (int r = 0; r < 4; ++r) acc64[i][t][r] += (double)acc[i][t][r];
                                    acc[i][t] = V4{0, 0, 0, 0};
                                }
                        }
                    }
                }
                st = st2;
                if (st == rend) {
                    finish_runs(f0 + 4 * st);
                    if (st < nst) count_run(st, min(rend2, nst));
                }
                rend = rend2;
                len = len2;
#pragma unroll
                for (int u = 0; u < CH; ++u)
#pragma unroll
                    for (int i = 0; i < TI; ++i) vcur[u][i] = vnext[u][i];
            }
            __syncthreads();  // the next group overwrites the rows and indices
        }
        finish_runs(total);  // runs without candidates after the last group
        __syncthreads();     // the tables are rewritten next
    }
    if (mt == 0 && tid == 0 && a.pair_total && pairs_all)
        atomicAdd((unsigned long long *)a.pair_total, (unsigned long long)pairs_all);
}

template <int M, bool F32, int S>
static void launch_shape(const BatchArgs &a, hipStream_t s)
{
    constexpr int WPB = kBatchShapes[S].wpb, TI = kBatchShapes[S].ti;
    hipLaunchKernelGGL((k_multipoles_batch_bins<M, F32, WPB, TI>), dim3(a.nblocks), dim3(WPB * kWave), 0, s, a);
}

template <int M, bool F32>
static z3_status launch_bins_m(int shape, const BatchArgs &a, hipStream_t s)
{
    switch (shape) {
    case 0: launch_shape<M, F32, 0>(a, s); break;
    case 1: launch_shape<M, F32, 1>(a, s); break;
    case 2: launch_shape<M, F32, 2>(a, s); break;
    case 3: launch_shape<M, F32, 3>(a, s); break;
    default: return fail(Z3_ERR_UNSUPPORTED, "batch shape %d not compiled", shape);
    }
    return Z3_OK;
}

z3_status launch_batch_bins(int m_max, bool f32, int shape, const BatchArgs &a, hipStream_t s)
{
    switch (m_max) {
#define Z3_CASE(MM) \
    case MM: return f32 ? launch_bins_m<MM, true>(shape, a, s) : launch_bins_m<MM, false>(shape, a, s);
        Z3_CASE(0) Z3_CASE(1) Z3_CASE(2) Z3_CASE(3) Z3_CASE(4) Z3_CASE(5) Z3_CASE(6) Z3_CASE(7)
        Z3_CASE(8) Z3_CASE(9) Z3_CASE(10) Z3_CASE(11) Z3_CASE(12) Z3_CASE(13) Z3_CASE(14)
        Z3_CASE(15) Z3_CASE(16)
#undef Z3_CASE
    default: return fail(Z3_ERR_UNSUPPORTED, "m_max=%d not compiled", m_max);
    }
}

}  // namespace z3
