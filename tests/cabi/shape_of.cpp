// The tiles that calls of the reduce take: reads lines "B width capacity P cus", with the
// workspace that such a call is told to bring, and prints "form kind slots" for each.
#include <cstdio>

#include "okt_sizes.h"

int main() {
    using namespace okt;
    static const char* const forms[] = {"wide5", "wide4", "narrow", "slim"};
    static const char* const kinds[] = {"dense", "ranked", "sparse"};
    unsigned long long B, width, capacity, P, cus;
    while (std::scanf("%llu %llu %llu %llu %llu", &B, &width, &capacity, &P, &cus) == 5) {
        const ReduceShape s = reduce_shape(B, width, capacity, (uint32_t)P, cus, reduce_ws_bytes(B, width, (uint32_t)P));
        std::printf("%s %s %u%s\n", forms[s.form], kinds[s.kind], s.slots,
                    reduce_counts_first(s, B, width, cus) ? " counted" : "");
    }
    return 0;
}
