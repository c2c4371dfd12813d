// Host-only checks of the rules by which the library picks a way of computing
// (internal.h).  Built and run by tests/test_rules.py; prints "ok" and exits 0.
#include <cstdio>

#include "internal.h"

int main()
{
    // A layer's phase table never costs more sines and cosines than its
    // amplitudes would, fits its room, and is used wherever both hold.
    for (int prec = 0; prec < 2; ++prec)
        for (int n = 1; n <= 13 - prec; ++n)
            for (int64_t W : {0LL, 1LL, 126LL, 127LL, 128LL, 200LL, 1400LL, 1535LL, 1536LL, 3000LL, 3071LL, 3072LL, 1LL << 30}) {
                const int e = qs::small_table_entries(prec, n, W);
                const int64_t direct = n < 6 ? 64 : 1LL << n, table = (W + 2) / 2;
                const bool fits = W + 1 <= (prec == 0 ? 3072 : 1536);
                if (e != (fits && table <= direct ? W + 1 : 0)) {
                    std::printf("table of %d entries: precision %d, n = %d, W_t = %lld\n", e, prec, n, (long long)W);
                    return 1;
                }
            }
    std::printf("ok\n");
    return 0;
}
