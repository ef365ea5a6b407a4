// Host check of the searches' arithmetic at the top of 32 bits, on lists of up to 2^32 - 1
// entries that nobody has to build for it: only numbers go in and come out.  Prints the
// number of cases and exits 0, or prints the first violations and exits 1.
#include <cstdint>
#include <cstdio>
#include <random>

#include "okt_search.h"

static long bad = 0, cases = 0;
static void expect(bool ok, const char* what, uint64_t a, uint64_t b) {
    ++cases;
    if (ok) return;
    if (bad < 8) std::printf("%s: %llu, %llu\n", what, (unsigned long long)a, (unsigned long long)b);
    ++bad;
}

static void check_spread(uint32_t part, uint32_t room) {
    const okt::SpreadSample s = okt::spread_sample(part, room);
    expect(s.step > 0 && s.count > 0 && s.count <= room, "step or count", part, room);
    expect((uint64_t)(s.count - 1) * s.step < part && (uint64_t)s.count * s.step >= part, "does not cover", part, room);
}

int main() {
    std::mt19937_64 rng(32);
    for (const uint32_t room : {1u, 2u, 1000u, 1024u, 4096u})
        for (uint32_t d = 0; d < 20000; ++d) {
            check_spread(0xffffffffu - d, room);
            check_spread(1 + d, room);
            check_spread(1 + (uint32_t)(rng() % 0xffffffffull), room);
        }
    std::printf("%ld cases, %ld violations\n", cases, bad);
    return bad ? 1 : 0;
}
