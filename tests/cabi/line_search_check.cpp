// Host check of the search by whole lines (the boundaries of the reduce's tiles)
// against std::lower_bound: random sorted lists, with and without duplicates, narrow and
// wide value ranges, that begin anywhere in a line, guesses before, in and behind them,
// and boundaries searched in turn from the one before.  Unsorted lists: the search ends
// and its answer lies in the list.  Prints the number of cases and exits 0, or prints the
// first disagreements and exits 1.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "okt_search.h"

// What a team of lanes does: `from` as in LineSearch, `list` its first entry.
static uint32_t search(const std::vector<uint32_t>& list, uint32_t from, okt::LineSearch s, uint32_t x, bool* inside) {
    const uint32_t upto = from + (uint32_t)list.size();
    bool known = s.hi <= s.lo;
    for (int step = 0; !known && step < okt::SEARCH_GUESSES; ++step) {
        const uint32_t line = okt::line_of_guess(s, from, upto);
        if (line < from || (list.size() >= okt::SEARCH_LINE && line + okt::SEARCH_LINE > upto)) *inside = false;
        uint32_t below = 0, first = 0, last = 0;
        for (uint32_t i = line; i < line + okt::SEARCH_LINE; ++i) {
            const uint32_t e = i < upto ? list[i - from] : ~0u;
            if (i == line) first = e;
            last = e;
            below += e < x ? 1u : 0u;
        }
        known = okt::line_says(s, line, below, first, last, x);
    }
    return known ? s.lo : s.lo + (uint32_t)okt::lower_bound_idx(list.data() + (s.lo - from), 0, s.hi - s.lo, x);
}

int main() {
    std::mt19937_64 rng(20220118);
    long bad = 0, cases = 0;
    for (int rep = 0; rep < 200000; ++rep) {
        int n = (int)(rng() % 400);
        const uint32_t span = rng() % 3 == 0 ? 40u : rng() % 3 == 0 ? 0xffffffffu : 100000u;
        std::vector<uint32_t> v(n);
        for (auto& x : v) x = (uint32_t)(rng() % span);
        const bool sorted = rng() % 8 != 0;
        if (sorted) std::sort(v.begin(), v.end());
        if (sorted && rng() % 2) v.erase(std::unique(v.begin(), v.end()), v.end());
        n = (int)v.size();
        const uint32_t from = (uint32_t)(rng() % okt::SEARCH_LINE), upto = from + (uint32_t)n;
        std::vector<uint32_t> bounds(1 + rng() % 5);
        for (auto& x : bounds) x = rng() % 4 == 0 && n ? v[rng() % n] : (uint32_t)(rng() % span) + (uint32_t)(rng() % 3);
        std::sort(bounds.begin(), bounds.end());
        uint32_t lo = from;
        for (const uint32_t x : bounds) {
            bool inside = true;
            const uint32_t got = search(v, from, okt::LineSearch{lo, upto, (uint32_t)(rng() % (uint64_t)(n + 80))}, x, &inside);
            const uint32_t want = from + (uint32_t)(std::lower_bound(v.begin(), v.end(), x) - v.begin());
            ++cases;
            if (!inside || (sorted ? got != want : got < lo || got > upto)) {
                if (bad < 5) std::printf("n=%d from=%u lo=%u x=%u: want %u, got %u%s\n", n, from, lo, x, want, got, inside ? "" : ", read outside");
                ++bad;
            }
            lo = got;
        }
    }
    std::printf("%ld cases, %ld disagreements\n", cases, bad);
    return bad ? 1 : 0;
}
