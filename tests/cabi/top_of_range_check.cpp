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

// The line of a guess lies inside a list that is a line long or more, whatever the guess,
// and takes in the guess where that is in [lo, hi).
static void check_line(uint32_t from, uint32_t upto, uint32_t lo, uint32_t hi, uint32_t guess) {
    const uint32_t line = okt::line_of_guess(okt::LineSearch{lo, hi, guess}, from, upto);
    expect(line >= from && (uint64_t)line + okt::SEARCH_LINE <= upto, "line outside the list", line, upto);
    const uint32_t g = guess < lo ? lo : guess >= hi ? hi - 1 : guess;
    expect(line <= g && g - line < okt::SEARCH_LINE, "line without its guess", line, g);
}

int main() {
    std::mt19937_64 rng(32);
    for (const uint32_t room : {1u, 2u, 1000u, 1024u, 4096u})
        for (uint32_t d = 0; d < 20000; ++d) {
            check_spread(0xffffffffu - d, room);
            check_spread(1 + d, room);
            check_spread(1 + (uint32_t)(rng() % 0xffffffffull), room);
        }
    for (int rep = 0; rep < 400000; ++rep) {
        const uint32_t from = (uint32_t)(rng() % okt::SEARCH_LINE);
        const uint32_t upto = rng() % 2 ? 0xffffffffu - (uint32_t)(rng() % 100) : from + okt::SEARCH_LINE + (uint32_t)(rng() % 100);
        const uint32_t lo = rng() % 2 ? upto - 1 - (uint32_t)(rng() % okt::SEARCH_LINE) : from + (uint32_t)(rng() % (upto - from));
        const uint32_t hi = rng() % 2 ? upto : lo + 1 + (uint32_t)(rng() % (upto - lo));
        check_line(from, upto, lo, hi, rng() % 2 ? upto - (uint32_t)(rng() % 80) : (uint32_t)rng());
    }
    std::printf("%ld cases, %ld violations\n", cases, bad);
    return bad ? 1 : 0;
}
