// Host check of the workspace arithmetic in okt_sizes.h: for vector lengths from 1
// to 2^32 - 1 and devices of 1 to 1024 compute units, the layout of the
// three-pass select (scan state, counts, places, list, slots) is in order, does
// not overlap, covers every tile, stays inside what okt_workspace_bytes-style
// bounds promise for any device, and the second pass's shape (tiles per thread,
// workgroups) covers all tiles within the limits its kernel assumes; and for random
// regions, that the reduce's tiles are ones its kernels hold and its workspace covers.  Prints the
// number of cases and exits 0, or the first violations and exits 1.
#include <cstdint>
#include <cstdio>
#include <random>

#include "okt_sizes.h"

int main() {
    using namespace okt;
    std::mt19937_64 rng(2201);
    long bad = 0, cases = 0;
    auto fail = [&](const char* what, uint64_t n, uint32_t cus) {
        if (bad < 8) std::printf("n=%llu cus=%u: %s\n", (unsigned long long)n, cus, what);
        ++bad;
    };
    const uint32_t cu_counts[] = {1, 2, 3, 7, 64, 104, 128, 228, 256, 304, 1000, 1024};
    for (int rep = 0; rep < 200000; ++rep) {
        uint64_t n;
        switch (rng() % 5) {
            case 0: n = 1 + rng() % 5000; break;
            case 1: n = 1 + rng() % (1ull << 22); break;
            case 2: n = (1ull << (10 + rng() % 22)) + (rng() % 3) - 1; break;
            case 3: n = 0xffffffffull - rng() % 4096; break;
            default: n = 1 + rng() % 0xffffffffull; break;
        }
        const uint32_t cus = cu_counts[rng() % (sizeof(cu_counts) / sizeof(cu_counts[0]))];
        const SlotPlan p = slot_plan(n, cus);
        ++cases;
        const uint64_t tiles = (n + SLOT_TILE - 1) / SLOT_TILE;
        if (p.ntiles != tiles) fail("tile count", n, cus);
        if (p.tpt < 1 || p.tpt > 63) fail("tiles per thread out of range", n, cus);
        if ((uint64_t)p.nseg * SLOT_SCAN_TILES * p.tpt < tiles) fail("second pass does not cover the tiles", n, cus);
        if (p.nseg > tiles / SLOT_SCAN_TILES + 1) fail("more workgroups than the scan state is sized for", n, cus);
        // scan state of the second pass: header, a descriptor per workgroup and per 64
        const size_t scan = 64 + 8 * ((size_t)p.nseg + ((size_t)p.nseg + 63) / 64);
        if (scan > p.counts_at) fail("scan state runs into the counts", n, cus);
        if (p.counts_at % 256 || p.place_at % 256 || p.dense_at % 256 || p.slots_at % 256) fail("misaligned part", n, cus);
        if (p.counts_at + 2 * tiles > p.place_at) fail("counts run into the places", n, cus);
        if (p.place_at + 4 * tiles > p.dense_at) fail("places run into the list", n, cus);
        if (p.dense_at + 4 * tiles > p.slots_at) fail("list runs into the slots", n, cus);
        const uint64_t groups = (tiles + SLOT_GROUP - 1) / SLOT_GROUP;
        if (p.slots_at + 8 * (uint64_t)SLOT_C * SLOT_GROUP * groups > p.bytes) fail("slots run past the end", n, cus);
        // the size a caller is told (computed for 256 compute units) holds for any device
        if (p.bytes > slot_ws_bytes(n)) fail("a device needs more than slot_ws_bytes says", n, cus);
        if (n >= RS_SAMPLE_MIN_N && refresh_ws_bytes(n) < threshold_ws_min_bytes() + refresh_scan_bytes(n) +
                                                             round_up_256(p.bytes) + 8 * (n / 16))
            fail("refresh workspace has no room for slots and n/16 candidates", n, cus);
        // the one-kernel form: a launch never has more workgroups than descriptors
        const SelectShape s = select_shape(n, cus);
        const size_t one = 64 + 8 * ((size_t)s.nseg + ((size_t)s.nseg + 63) / 64);
        if (one > select_ws_bytes(n)) fail("one-kernel scan state exceeds select_ws_bytes", n, cus);
        if ((uint64_t)s.nseg * SEL_WAVES * s.piece < n) fail("one-kernel pieces do not cover the vector", n, cus);
        if (s.piece > SEL_PIECE_MAX || s.piece % 256) fail("piece length", n, cus);
    }
    long forms[4][3] = {};
    // the reduce: every tile shape is one its kernels hold, and fits the workspace it was chosen for
    for (int rep = 0; rep < 200000; ++rep) {
        const uint64_t width = rng() % 3 ? 1 + rng() % (1ull << (1 + rng() % 27)) : rng() % 0xffffffffull;
        const uint64_t expected = rng() % 4 ? (uint64_t)((double)width * (rng() % 2000) / 1000.0) : rng() % (width + 2);
        const uint32_t P = 1 + rng() % (1u << (1 + rng() % 16)), Pc = P > 65535 ? 65535 : P;
        const uint64_t B = 1 + rng() % (1u << (rng() % 12));
        const uint32_t cus = cu_counts[rng() % (sizeof(cu_counts) / sizeof(cu_counts[0]))];
        ++cases;
        const size_t told = reduce_ws_bytes(B, width, Pc);
        const size_t least = reduce_ws_bytes_region(width, Pc, reduce_least_shape(width, expected, Pc).slots);
        if (least > 0xffffffffull) continue;                       // refused
        if (least * B > told) fail("a call asks for more than its callers are told", width, Pc);
        for (const size_t ws : {told, (least * B + told) / 2, least * B}) {
            const ReduceShape s = reduce_shape(B, width, expected, Pc, cus, ws);
            const size_t region = reduce_ws_bytes_region(width, Pc, s.slots);
            if (ws < region * B || region > 0xffffffffull) fail("reduce workspace too small for its tiles", width, Pc);
            ++forms[s.form][s.kind];
            uint32_t dense = ReduceWide5::C_DENSE, ranked = ReduceWide5::S_RANKED, sparse = ReduceWide5::S_SPARSE;
            if (s.form == RED_NARROW) dense = ReduceNarrow::C_DENSE, ranked = ReduceNarrow::S_RANKED, sparse = ReduceNarrow::S_SPARSE;
            if (s.form == RED_WIDE4) dense = ReduceWide4::C_DENSE, ranked = ReduceWide4::S_RANKED, sparse = ReduceWide4::S_SPARSE;
            if (s.form == RED_SLIM) {
                ranked = ReduceSlim::S_RANKED, sparse = ReduceSlim::S_SPARSE;
                if (s.kind == RED_DENSE) fail("a dense slim tile", width, Pc);
                if (Pc >= RED_SLIM_P || (double)expected / (double)width >= reduce_slim_to(Pc)) fail("a slim tile where the rule has none", width, Pc);
            }
            if (s.kind == RED_DENSE && s.slots != dense) fail("dense tile", width, Pc);
            if (s.kind == RED_RANKED && (s.slots > ranked || s.slots < RED_SLOTS_MIN || s.slots % 32)) fail("ranked tile", width, Pc);
            if (s.kind == RED_SPARSE && (s.slots > sparse || s.slots <= ranked || s.slots % 32)) fail("sparse tile", width, Pc);
        }
    }
    for (const auto form : {RED_WIDE5, RED_WIDE4, RED_NARROW, RED_SLIM})
        for (const auto kind : {RED_DENSE, RED_RANKED, RED_SPARSE})
            if (forms[form][kind] == 0 && !(form == RED_SLIM && kind == RED_DENSE)) fail("a kind of tile that no case takes", form, kind);
    std::printf("%ld cases, %ld violations\n", cases, bad);
    return bad ? 1 : 0;
}
