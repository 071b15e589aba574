// Sizes of an FFTLog evaluation: the padded lengths, the workspace and the models per pass
// (plain host code, no device types).
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace z3 {

// s (ld), s1 >= 0 half (ldw), t >= 0 half (ldh), all t (ldt)
struct FftlogLayout {
    size_t ld, ldw, ldh, ldt;
};

inline FftlogLayout fftlog_layout(int N)
{
    auto up16 = [](size_t v) { return (v + 15) / 16 * 16; };
    return FftlogLayout{up16((size_t)N + 1), up16((size_t)N / 2 + 1), up16((size_t)N + 1), up16(2 * (size_t)N + 1)};
}

inline size_t fftlog_workspace_bytes(int N, int nchi, int T, int chunk)
{
    // nine pieces, each rounded up to 256 bytes by the carving in fftlog_impl
    const FftlogLayout L = fftlog_layout(N);
    return 2 * sizeof(double) * (8 * L.ld + 4 * (size_t)T * (L.ld + L.ldw) + (size_t)nchi * L.ldh +
                                 (size_t)chunk * 3 * (L.ldt + (size_t)T * L.ld)) +
           sizeof(double) * (size_t)chunk * 3 * (nchi + (size_t)T * T) + 9 * 256;
}

// Most models of one pass, 0 if there is no such pass.  A pass has one grid z index per factor pair
// and model, and the products' offsets along k are 32-bit: over chi, (nchi - 1) ldh into the
// phases and (nchi - 1) 3 models into the weights; over s, at most N T into the other operands
// (2^24 at the largest N and T).
inline int fftlog_most_models(int N, int nchi)
{
    const int64_t top = INT32_MAX;
    if ((int64_t)nchi * (int64_t)fftlog_layout(N).ldh > top) return 0;
    const int64_t by_offset = top / (3 * (int64_t)nchi);
    return (int)(by_offset < 21845 ? by_offset : 21845);
}

// Models per pass for `nmodels` in all and a workspace of `budget` bytes (which even one model may
// exceed), 0 if there is no such pass.
inline int fftlog_pass_models(int N, int nchi, int T, int nmodels, size_t budget)
{
    const int most = fftlog_most_models(N, nchi);
    int chunk = nmodels < most ? nmodels : most;
    while (chunk > 1 && fftlog_workspace_bytes(N, nchi, T, chunk) > budget) chunk = (chunk + 1) / 2;
    return chunk;
}

}  // namespace z3
