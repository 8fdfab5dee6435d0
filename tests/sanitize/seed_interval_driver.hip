// Host driver for the window form's arithmetic on one ranked seed (test infrastructure, no kernel and no GPU call): what it gives
// against every window written out, and, behind the last seed, with whatever memory may hold.
#include <stdio.h>

#include "seed_interval.h"

int main()
{
    int failures = 0;
    for (int len = 1; len <= 12; ++len)
        for (int reach = 0; reach <= 4; ++reach)
            for (int at = 0; at < len; ++at)
                for (int before = 1; before <= 13; ++before)
                    for (int behind = 1; behind <= 13; ++behind) {
                        // 13 stands for none, noted as the largest distance; a distance beyond the context's ends is none either
                        const uint32_t lo = before == 13 ? 0xFFFFu : (uint32_t)before, hi = behind == 13 ? 0xFFFFu : (uint32_t)behind;
                        const ilre::SeedInterval got = ilre::seed_interval(true, (uint32_t)at, hi << 16 | lo, (uint32_t)reach, (uint32_t)len);
                        int first = -1, last = -1;
                        for (int t = 0; t < len; ++t) {
                            const bool holds = t - reach <= at && at <= t + reach;
                            const bool outranked = (before != 13 && t - reach <= at - before) || (behind != 13 && at + behind <= t + reach);
                            if (holds && !outranked) {
                                if (first < 0) first = t;
                                last = t;
                            }
                        }
                        const bool same = first < 0 ? !got.some : got.some && got.first == (uint32_t)first && got.last == (uint32_t)last;
                        if (!same && ++failures < 10)
                            printf("len %d reach %d at %d before %d behind %d: %d %u..%u, wanted %d..%d\n", len, reach, at, before, behind, got.some,
                                   got.first, got.last, first, last);
                    }
    const uint32_t words[] = {0u, 1u, 0x7FFFFFFFu, 0x80000000u, 0x80000001u, 0xFFFFu, 0xFFFF0000u, 0xFFFFFFFFu, 0xDEADBEEFu};
    const uint32_t lens[] = {1u, 1000u, 0x7FFFFFFFu};
    for (uint32_t at : words)
        for (uint32_t dominators : words)
            for (uint32_t len : lens)
                for (uint32_t reach : {0u, 1u, 1023u}) {
                    const ilre::SeedInterval got = ilre::seed_interval(false, at, dominators, reach, len);
                    if (got.some || got.first || got.last) ++failures;
                }
    printf("%d failures\n", failures);
    return failures ? 1 : 0;
}
