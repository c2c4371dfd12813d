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
    // Shots: 16 lanes each below 2^17, one lane each wherever that is the faster
    // way (measured, see shot_lanes), and the same for every larger count once
    // the largest threshold is passed.
    struct Shots {
        int prec, n;
        int64_t shots;
        bool lanes;
    };
    const Shots want[] = {{0, 27, 100000, false}, {0, 13, 1, false},        {0, 13, 400000, true},  {0, 20, 400000, true},
                          {0, 14, 4000000, true}, {0, 16, 1000000, false},  {0, 24, 1 << 24, false}, {0, 27, 1 << 24, true},
                          {1, 14, 1000000, true}, {1, 20, 4000000, true},   {1, 24, 1000000, false}, {1, 27, 4000000, true},
                          {1, 24, 4000000, false}, {0, 28, 6000000, true},   {1, 25, 2000000, true},
                          {1, 34, 1LL << 39, true}};
    for (const Shots &w : want)
        if (qs::shot_lanes(w.prec, w.n, w.shots) != w.lanes) {
            std::printf("shots: precision %d, n = %d, %lld\n", w.prec, w.n, (long long)w.shots);
            return 1;
        }
    std::printf("ok\n");
    return 0;
}
