// The FFTLog pass length (csrc/z3_fftlog_pass.h): for every size that the entry point takes, the
// products' offsets along k fit 32 bits, the workspace fits the budget, and a pass takes as many
// models as it may.  Exit status 0 when every check holds.
#include <stdio.h>

#include <initializer_list>

#include "z3_fftlog_pass.h"

using namespace z3;

int main()
{
    int failures = 0;
    const int top = INT32_MAX;
    for (int N : {4, 64, 256, 1000, 4096})
        for (int64_t nchi : {(int64_t)2, (int64_t)512, (int64_t)32767, (int64_t)32768, (int64_t)32770, (int64_t)65536,
                             (int64_t)521999, (int64_t)522247, (int64_t)523000, (int64_t)1 << 24, (int64_t)1 << 26,
                             (int64_t)1 << 27, (int64_t)715827882, (int64_t)top})
            for (int T : {1, 64, 4096})
                for (int models : {1, 2, 100, 21845, 21846, 65535, 1 << 20, top})
                    for (size_t budget : {(size_t)0, (size_t)1 << 30, (size_t)17 << 30, (size_t)40 << 30, SIZE_MAX}) {
                        const int c = fftlog_pass_models(N, (int)nchi, T, models, budget);
                        const bool phases = nchi * (int64_t)fftlog_layout(N).ldh <= top;
                        bool ok = c >= 0 && c <= models && c <= 21845 && (c > 0) == phases;
                        if (c > 0) {
                            // the last k-step's offsets into the phases and the weights
                            ok = ok && (nchi - 1) * (int64_t)fftlog_layout(N).ldh <= top && (nchi - 1) * 3 * (int64_t)c <= top;
                            ok = ok && (c == 1 || fftlog_workspace_bytes(N, (int)nchi, T, c) <= budget);
                            // without a budget's bound, one model more would not do
                            if (budget == SIZE_MAX && c < models && c < 21845) ok = ok && 3 * nchi * (c + 1) > top;
                        }
                        if (!ok) {
                            fprintf(stderr, "N %d nchi %lld T %d models %d budget %zu: %d models a pass\n", N,
                                    (long long)nchi, T, models, budget, c);
                            ++failures;
                        }
                    }
    if (!failures) printf("pass checks ok\n");
    return failures != 0;
}
