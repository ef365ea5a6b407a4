// Searches in a sorted index list, written so that a host compiler can build them
// too (the CPU tests check them against std::lower_bound).
#ifndef OKT_SEARCH_H
#define OKT_SEARCH_H

#include <stdint.h>

#ifdef __HIPCC__
#define OKT_SEARCH_FN __host__ __device__ __forceinline__
#else
#define OKT_SEARCH_FN static inline
#endif

namespace okt {

// The first position in [lo, hi) whose entry is not below x, or hi.
OKT_SEARCH_FN uint64_t lower_bound_idx(const uint32_t* a, uint64_t lo, uint64_t hi, uint32_t x) {
    while (lo < hi) {
        const uint64_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Sixteen consecutive entries at any word address, read together.
struct __attribute__((packed, aligned(4))) SearchWindow { uint32_t v[16]; };

// The same answer - the first position in [lo, hi) whose entry is not below x, or
// hi - found from a guess: sixteen entries around the guess are read at once (one
// line of memory, or two) and, if x does not fall among them, the next guess is
// extrapolated from their spacing.  With indices spread evenly over the region the
// first guess is a few dozen entries off and the second one hits, so a boundary
// costs two or three lines and as many waits, where probes of one entry each (steps
// of doubling length from the guess, then a bisection) take eight waits in three or
// four lines.  After SEARCH_GUESSES misses, and in lists shorter than a window, what
// is left is bisected: any input ends.
constexpr int SEARCH_GUESSES = 4;
OKT_SEARCH_FN uint64_t lower_bound_near(const uint32_t* a, uint64_t lo, uint64_t hi, uint32_t x,
                                        uint64_t guess) {
    for (int miss = 0; miss < SEARCH_GUESSES; ++miss) {
        if (hi <= lo || hi - lo < 16) break;                 // the answer lies in [lo, hi]
        uint64_t w = guess < lo + 8 ? lo : guess - 8;
        if (w > hi - 16) w = hi - 16;
        const SearchWindow win = *reinterpret_cast<const SearchWindow*>(a + w);
        uint32_t below = 0;
        for (int j = 0; j < 16; ++j) below += win.v[j] < x ? 1u : 0u;
        if (below != 0 && below != 16) return w + below;
        const uint32_t first = win.v[0], last = win.v[15];
        const float per = 15.0f / (float)(last > first ? last - first : 1u);   // entries per index
        if (below == 0) {                                    // a[w] is not below x
            hi = w;
            const uint64_t back = (uint64_t)((float)(first - x) * per);
            guess = back < w ? w - back : 0;
        } else {
            lo = w + 16;
            guess = lo + (uint64_t)((float)(x - last) * per);
        }
    }
    return lower_bound_idx(a, lo, hi, x);
}

// The same again by whole lines of memory: the SEARCH_LINE entries of the aligned line
// that holds the guess are read at once (at the ends of a list the first or last as many),
// so that a guess costs one line and one wait and hits if it is some sixteen entries off.
// Positions count from the beginning of the line that holds the list's first entry, which
// is at `from`; the last one is before `upto`.
constexpr uint32_t SEARCH_LINE = 32;
struct LineSearch { uint32_t lo, hi, guess; };               // the answer lies in [lo, hi]

// Where the line of the guess begins (there is one: lo < hi), inside the list unless that
// is shorter than a line.
OKT_SEARCH_FN uint32_t line_of_guess(const LineSearch& s, uint32_t from, uint32_t upto) {
    const uint32_t g = s.guess < s.lo ? s.lo : s.guess >= s.hi ? s.hi - 1 : s.guess;
    const uint32_t line = g & ~(SEARCH_LINE - 1);
    return line < from || upto - from < SEARCH_LINE ? from : line > upto - SEARCH_LINE ? upto - SEARCH_LINE : line;
}

// What the line says: `below` of its entries are below x (an entry past the end of the
// list is not), `first` and `last` are its ends.  True if that is the answer, which is in
// lo then.  Every line takes the guess off [lo, hi], sorted or not.
OKT_SEARCH_FN bool line_says(LineSearch& s, uint32_t line, uint32_t below, uint32_t first, uint32_t last, uint32_t x) {
    const uint32_t at = line + below, lo = s.lo, hi = s.hi;
    const uint32_t in = at < lo ? lo : at > hi ? hi : at;
    if (below != 0 && below != SEARCH_LINE) {
        s.lo = in;
        return true;
    }
    const float per = (float)(SEARCH_LINE - 1) / (float)(last > first ? last - first : 1u);   // entries per index
    if (below == 0) {
        s.hi = in;
        const float back = (float)(first - x) * per;
        s.guess = back < (float)in ? in - (uint32_t)back : 0u;
    } else {
        s.lo = in;
        const float on = (float)(x - last) * per;
        s.guess = on < (float)(hi - in) ? in + (uint32_t)on : hi;
    }
    return s.hi <= s.lo;
}

// Every step-th of `part` > 0 elements, from the first on, at most `room` of them: count
// elements, (count - 1) * step < part <= count * step.  For every part below 2^32.
struct SpreadSample { uint32_t step, count; };
OKT_SEARCH_FN SpreadSample spread_sample(uint32_t part, uint32_t room) {
    const uint32_t step = (part - 1) / room + 1;             // (part + room - 1 may not fit)
    return SpreadSample{step, (part - 1) / step + 1};
}

// Boundary r (0 <= r <= R) of the balanced split of [0, n) by a sorted index list
// of nnz entries (Sec. 3.1.1), and the list position where region r begins:
// b[r] = idx[floor(r * nnz / R)], b[0] = 0, b[R] = n; without entries the equal
// split floor(r * n / R).  A count above n cannot come from a select over n
// elements - it is the all-ones word a failed call leaves in its counts - and is
// answered without reading idx: the equal split, every offset all ones, so that
// whatever consumes the offsets sees empty slices and the failure stays visible.
struct PartitionCut { uint32_t bound; uint64_t offset; };
OKT_SEARCH_FN PartitionCut partition_cut(const uint32_t* idx, uint64_t nnz, uint64_t n, uint32_t R,
                                         uint64_t r) {
    if (nnz > n) return PartitionCut{r == R ? (uint32_t)n : (uint32_t)((r * n) / R), ~0ull};
    if (r == 0) return PartitionCut{0u, 0ull};
    if (r == R) return PartitionCut{(uint32_t)n, nnz};
    if (nnz == 0) return PartitionCut{(uint32_t)((r * n) / R), 0ull};     // r, n < 2^32: no overflow
    const uint64_t at = (r * nnz) / R;                                     // r, nnz < 2^32
    const uint32_t b = idx[at];
    // in a list that ascends strictly, as a select's does, that is where b is first
    if (at == 0 || idx[at - 1] < b) return PartitionCut{b, at};
    return PartitionCut{b, lower_bound_idx(idx, 0, at, b)};
}

}  // namespace okt
#endif
