// Tile shapes and workspace sizes, shared by the host entry points.
#ifndef OKT_SIZES_H
#define OKT_SIZES_H

#include <math.h>
#include <stddef.h>
#include <stdint.h>

namespace okt {

// ---- threshold select + compaction ----
// A workgroup of SEL_BLOCK threads owns SEL_WAVES consecutive pieces of the
// vector, one per wave; a wave streams its piece in rounds of 256 elements,
// SEL_U rounds in flight.  The piece length (select_shape below) is never above
// SEL_PIECE_MAX, which keeps the selected entries of a piece inside the wave's
// LDS stash up to a local density of SEL_STASH / SEL_PIECE_MAX = 9.8 %.
constexpr int SEL_BLOCK = 1024;
constexpr int SEL_WAVES = SEL_BLOCK / 64;
constexpr int SEL_U = 4;
// The kernels need more than 64 registers, so a CU holds one workgroup at a time
// anyway: its stash takes nearly the whole LDS (16 waves x 1600 entries x 6 bytes
// = 150 KB of 160).  Gradients select unevenly - whole layers above the
// threshold next to layers with nothing - and a piece that overflows its stash
// is partly walked twice.
constexpr int SEL_STASH = 1600;                // entries per wave
constexpr uint32_t SEL_ROUND = 256u * SEL_U;
constexpr uint32_t SEL_PIECE_MAX = 16384;

struct SelectShape { uint32_t nseg, piece; };
// The select kernels run one 1024-thread workgroup per CU at a time, and a
// workgroup streams for tens of microseconds, so a last round of workgroups that
// fills only part of the chip costs as much as a full one.  The vector is
// therefore cut for whole rounds: `rounds` x `cus` workgroups of equal pieces
// (a multiple of 256 elements, at most SEL_PIECE_MAX), `cus` being the number of
// compute units of the device at hand (device_cus(), never above SEL_CUS_MAX).
constexpr uint32_t SEL_CUS_MAX = 1024;
inline uint64_t select_rounds(uint64_t n, uint32_t cus) {
    const uint64_t per_round = (uint64_t)cus * SEL_WAVES * SEL_PIECE_MAX;
    const uint64_t rounds = (n + per_round - 1) / per_round;
    return rounds ? rounds : 1;
}
inline SelectShape select_shape(uint64_t n, uint32_t cus) {
    const uint64_t waves = (uint64_t)cus * SEL_WAVES * select_rounds(n, cus);
    uint64_t piece = ((n + waves - 1) / waves + 255) / 256 * 256;
    if (piece < SEL_ROUND) piece = SEL_ROUND;
    const uint64_t per_wg = piece * SEL_WAVES;
    return SelectShape{(uint32_t)((n + per_wg - 1) / per_wg), (uint32_t)piece};
}
// Header, segment and group descriptors.  A bound for any device: a launch has at
// most cus x rounds <= n / (SEL_WAVES x SEL_PIECE_MAX) + 1 + cus workgroups.
inline size_t select_ws_bytes(uint64_t n) {
    const uint64_t t = n / ((uint64_t)SEL_WAVES * SEL_PIECE_MAX) + 1 + SEL_CUS_MAX;
    return 64 + 8 * (size_t)(t + (t + 63) / 64);
}

// ---- the same over a COO list ----
// Short lists need no scan across workgroups (okt_coo.hip): one workgroup up to
// COO_SMALL_N entries, a count a tile of 1024 up to COO_TILED_N, as many as the
// least workspace of a call has room for (two bytes each).
constexpr uint32_t COO_SMALL_N = 32768, COO_TILED_N = 4u << 20;

// Vectors longer than the 256 MB last-level cache are read, and where a kernel
// rewrites them densely written, with the non-temporal hint: nothing of them is
// found cached again, and what goes around the cache pushes nothing out.  Shorter
// ones are not: what one kernel writes the next still finds there (the select
// that follows an accumulate, the zeros that follow a refresh iteration's pass).
constexpr uint64_t STREAM_PAST_CACHE_N = 64u << 20;                          // 256 MiB of fp32 and up
inline bool stream_past_cache(uint64_t n) { return n >= STREAM_PAST_CACHE_N; }
// The passes that form the accumulator read the gradient for the last time, so from
// 32 MiB of it on (the size of all the L2s) they read it around the cache and leave the
// room to the residual, which the next pass or iteration reads again: accumulate and
// select in one pass at 20 M elements 57 -> 48 us, at 27 M 76 -> 72, the plain
// accumulate at 25 M 54 -> 46 us; at 1 M, where everything stays cached, 24 -> 26.
enum CacheUse { CACHED = 0, GRADIENT_PAST_CACHE = 1, ALL_PAST_CACHE = 2 };
constexpr uint64_t GRADIENT_PAST_CACHE_N = 8u << 20;
inline CacheUse accumulate_cache_use(uint64_t n) {
    return stream_past_cache(n) ? ALL_PAST_CACHE : n >= GRADIENT_PAST_CACHE_N ? GRADIENT_PAST_CACHE : CACHED;
}

// ---- the same through per-tile slots ----
// With a workspace that has room for them, the streaming pass of the selects
// writes what a tile of SLOT_TILE elements (one wave) selects into the tile's own
// slot of SLOT_C entries and counts it; a scan over the counts and a copy out of
// the slots follow as a short second pass, and the tiles that selected more than
// a slot holds (a local density above SLOT_C / SLOT_TILE = 12.5 %) are walked
// again by a third.  Gradients select unevenly - in the layered workloads three
// quarters of the selected entries sit in tiles that select 3 to 12 % - and a
// slot costs address space, not traffic: only the entries written are ever
// touched.  Workspace: a scan state, then per tile a 2-byte count, a 4-byte
// place, 4 bytes of the list of fuller and dense tiles and the slot, as many bytes
// as the vector has elements in all.
constexpr uint32_t SLOT_TILE = 1024;
constexpr uint32_t SLOT_C = 128;
constexpr uint32_t SLOT_GROUP = 4;                   // tiles whose slots are interleaved
constexpr uint32_t SLOT_SCAN_TILES = 1024;           // tiles per workgroup of the second pass and turn
struct SlotPlan {
    uint32_t ntiles;
    uint32_t tpt;                // tiles per thread of the second pass
    uint32_t nseg;               // workgroups of the second pass
    size_t counts_at, place_at, dense_at, slots_at, bytes;   // offsets into the workspace; its size
};
inline size_t round_up_256(size_t v) { return (v + 255) & ~(size_t)255; }
inline SlotPlan slot_plan(uint64_t n, uint32_t cus) {
    SlotPlan p;
    p.ntiles = (uint32_t)((n + SLOT_TILE - 1) / SLOT_TILE);
    // about half as many workgroups as compute units: the pass is short, and every
    // workgroup takes a ticket from one counter
    const uint64_t want = (uint64_t)SLOT_SCAN_TILES * (cus > 1 ? cus / 2 : 1);
    p.tpt = (uint32_t)((p.ntiles + want - 1) / want);
    if (p.tpt == 0) p.tpt = 1;
    if (p.tpt > 63) p.tpt = 63;              // a workgroup's tiles are counted in 16 bits
    const uint64_t per_seg = (uint64_t)SLOT_SCAN_TILES * p.tpt;
    p.nseg = (uint32_t)((p.ntiles + per_seg - 1) / per_seg);
    if (p.nseg == 0) p.nseg = 1;
    // the scan state is sized for the most workgroups any device gives (tpt = 1)
    const uint64_t segs_max = (uint64_t)p.ntiles / SLOT_SCAN_TILES + 1;
    const size_t scan = 64 + 8 * (size_t)(segs_max + (segs_max + 63) / 64);
    p.counts_at = round_up_256(scan);
    p.place_at = p.counts_at + round_up_256(2 * (size_t)p.ntiles);
    p.dense_at = p.place_at + round_up_256(4 * (size_t)p.ntiles);
    p.slots_at = p.dense_at + round_up_256(4 * (size_t)p.ntiles);
    p.bytes = p.slots_at + 8 * (size_t)SLOT_C * ((p.ntiles + SLOT_GROUP - 1) / SLOT_GROUP * SLOT_GROUP);
    return p;
}
inline size_t slot_ws_bytes(uint64_t n) { return slot_plan(n, 256).bytes; }
// Shorter vectors take the one-kernel form: the extra launches and their fixed few
// microseconds cost more than the leaner streaming pass saves there.  Measured
// crossover: the calls that form the accumulator on the way (12 bytes an element: the
// saving is three times the select's) gain from about 24 M elements on (accumulate and
// select, layered, 2 %, a gradient that is handed in again and lies partly in the
// last-level cache: 20 M 47 against 50 us, 27 M 73 against 72, 40 M 115 against 104; one
// that comes from memory: 25.6 M 65.2 against 61.7), the plain selects from about 100 M, where the vector no longer fits the last-level
// cache.
constexpr uint64_t SLOT_MIN_N_SELECT = 96u << 20;
constexpr uint64_t SLOT_MIN_N_ACCUMULATE = 24u << 20;

// ---- index intersection and residual restore ----
constexpr int RST_BLOCK = 1024, RST_WAVES = RST_BLOCK / 64;
constexpr int RST_ROWS = 1;                              // entries per thread
constexpr uint32_t RST_TILE = RST_BLOCK * RST_ROWS;      // local entries per workgroup
constexpr int RST_CHAINED_ROWS = 2;                      // the same in the form with a scan across workgroups
constexpr uint32_t RST_SAMPLES = 1024;                   // places of the global list that say where a tile's part of it lies
constexpr uint32_t RST_WINDOW = 4096;                    // elements of that part that a workgroup holds at a time
constexpr uint32_t RST_BETWEEN = 16;                     // elements between two of a longer part's that are read and compared
constexpr uint32_t RST_TABLE_BITS = 13, RST_TABLE = 1u << RST_TABLE_BITS;   // hash table of a tile's entries
constexpr uint32_t RST_DIRECT_TILES = 4096;              // up to here every workgroup adds up the counts before its tile
constexpr int RST_SCAN_BLOCK = 1024;
constexpr uint32_t RST_PER_CU = 2;                        // workgroups of a launch
inline uint64_t restore_tiles(uint64_t max_local) {
    return max_local == 0 ? 1 : (max_local + RST_TILE - 1) / RST_TILE;
}
// What a call asks for, more than a count per tile and one for all of them.
inline size_t restore_ws_bytes(uint64_t max_local) {
    const uint64_t t = restore_tiles(max_local);
    return 64 + 8 * (size_t)(t + (t + 63) / 64);
}
// Where a bit per entry goes behind the counts, in a workspace that has room for them
// (okt_workspace_bytes always does: about two bytes an entry).
inline size_t restore_masks_at(uint64_t max_local) { return (4 * (size_t)(restore_tiles(max_local) + 1) + 63) / 64 * 64; }

// ---- exact threshold (radix select over the 31-bit magnitude key) ----
constexpr int RS_BITS1 = 11, RS_BITS2 = 11, RS_BITS3 = 9;   // 11 + 11 + 9 = 31
constexpr int RS_MAX_BINS = 1 << 11;
constexpr size_t RS_STATE_BYTES = 256;
constexpr size_t RS_HIST_BYTES = 4 * RS_MAX_BINS * sizeof(uint32_t);   // the digits'
constexpr uint64_t RS_SAMPLE_MIN_N = 4u << 20;   // vectors whose workspace has room for slots
// A refresh iteration below this takes accumulate, threshold and select one after the other.
constexpr uint64_t RS_SAMPLE_FROM_N = 1u << 17;
// The exact threshold alone: collecting the candidates pays from the shortest length that
// does not fit one workgroup (digits over the vector from the bound up instead: 140,000
// elements 18.7 us against 15, 1 M 21 against 17, 2 M 25 against 22).  From k = n / 16 on,
// up to this length, it no longer does (400,000 elements: 21.2 against 20; 255,570 with
// most of them selected 4 us more); and with no room for candidates the two digits from
// the bound up beat three over everything up to here.
constexpr uint64_t BOUNDED_TO_N = 2u << 20;
constexpr uint32_t TINY_N = 65536;               // up to here one workgroup finds the threshold
inline size_t threshold_ws_min_bytes() { return RS_STATE_BYTES + RS_HIST_BYTES; }
inline size_t threshold_ws_bytes(uint64_t n) {
    // state + histograms + room for the candidate keys (a few percent of the vector)
    return threshold_ws_min_bytes() + 4 * (size_t)(n / 8 + 1024);
}
// A refresh iteration in one pass: the threshold's state and histograms, two scan
// states, candidates with their indices (8 bytes each, a sixteenth of the vector
// and some), and the slots through which a long vector's candidates are
// collected.  A shorter vector takes the three steps one after the other.
inline size_t refresh_scan_bytes(uint64_t n) { return (select_ws_bytes(n) + 255) & ~(size_t)255; }
inline size_t refresh_ws_bytes(uint64_t n) {
    if (n < RS_SAMPLE_FROM_N) return 0;
    return threshold_ws_min_bytes() + 2 * refresh_scan_bytes(n) + 8 * (size_t)(n / 8 + 1024) +
           (n < RS_SAMPLE_MIN_N ? 0 : round_up_256(slot_ws_bytes(n)));
}

// ---- sparse reduce ----
// A workgroup owns a tile of `slots` consecutive index slots of the region and
// sums into C fp64 accumulators in LDS.  In a region that is densely hit slot =
// accumulator.  In a sparsely hit region a tile is wider than that, up to S slots:
// the hit slots are marked in a bitmap, the popcount prefix of the bitmap ranks
// them, and the accumulators are indexed by rank, so the LDS holds hit slots only.
// Very sparsely hit regions trade accumulators for bitmap.
constexpr uint32_t RED_UNIT = 16;               // entries read by four lanes with one 16-byte load each
// Four forms of tile: two wide tiles to a CU (80 KB of LDS each), whose threads hold
// five units per four threads in registers (ROUNDS) or four, three slim ones, or four narrow ones.
enum ReduceForm { RED_WIDE5, RED_WIDE4, RED_NARROW, RED_SLIM };
struct ReduceWide5 {
    static constexpr int BLOCK = 512, ROUNDS = 5;
    static constexpr uint32_t C_DENSE = 9216, C_RANKED = 7968, S_RANKED = 65536, C_SPARSE = 7168, S_SPARSE = 98304;
    static constexpr double FILL = 0.93;
};
struct ReduceWide4 {
    static constexpr int BLOCK = 512, ROUNDS = 4;
    static constexpr uint32_t C_DENSE = 9216, C_RANKED = 8064, S_RANKED = 65536, C_SPARSE = 7168, S_SPARSE = 98304;
    static constexpr double FILL = 0.93;
};
// Three tiles to a CU (53 KB of LDS each), whose accumulators are floats and hold what a slot's
// first entry brings; the others go to a list of RED_SLIM_LIST (reduce_tile_kernel).
struct ReduceSlim {
    static constexpr int BLOCK = 512, ROUNDS = 4;
    static constexpr uint32_t C_DENSE = 0, C_RANKED = 6912, S_RANKED = 65536, C_SPARSE = 6912, S_SPARSE = 98304;
    static constexpr double FILL = 0.95;
};
constexpr uint32_t RED_SLIM_LIST = 2968;
struct ReduceNarrow {
    static constexpr int BLOCK = 512, ROUNDS = 2;
    static constexpr uint32_t C_DENSE = 4096, C_RANKED = 3968, S_RANKED = 32768, C_SPARSE = 3584, S_SPARSE = 49152;
    static constexpr double FILL = 0.9;
};
constexpr uint32_t RED_SLOTS_MIN = 4096;        // no tile is narrower
// Launches with fewer wide tiles than this take the narrow form: more, shorter tiles.
constexpr uint64_t RED_WIDE_TILES_PER_CU = 2;
// Regions of at least RED_PLACED_FROM narrow tiles, in launches of at most RED_PLACED_TILES_PER_CU
// of them per CU (as many as run at a time), count the hit slots of every tile first and take no
// tickets (see reduce_count_kernel).  A ticket is 30 ns, the second reading of the indices some two
// microseconds: 361 tiles 24.8 and 21.0 us; 75 tiles 18.3 and 19.7, six tiles even.
constexpr uint64_t RED_PLACED_FROM = 128, RED_PLACED_TILES_PER_CU = 4;
// So do regions of at most RED_NARROW_TILES narrow tiles with at most RED_FEW
// contributions: with four tiles to a CU one waits while three work, a tile that is hit
// more than the rest holds up less, and long slices fill half as many units as well.
// In batches of 16 M entries, 2 to 32 contributions in 200 K to 800 K slots, the narrow form
// is 1.2 to 1.3 times as fast where they are hit evenly (8 contributions, a tenth of 400 K
// slots hit: 61 against 76 us) and up to 1.5 times where most hits lie in a few layers.
// In longer regions the entries' cost decides: 490 regions of 16 contributions, 67 narrow
// tiles each, take 601 us narrow and 532 us wide; so do more contributions, whose slices
// are shorter: 373 regions of 64, 831 and 690 us.
constexpr uint32_t RED_FEW = 32, RED_NARROW_TILES = 48;
// Wide tiles have a fifth round for entries that share slots and for stretches that are
// hit somewhat more than the rest: batches of 8 contributions in 4 M slots, 30 % of their
// entries among the same tenth, are 1.06 times as fast as with tiles that read every slice
// twice, where four rounds are 0.77 times; 40 contributions that hit every other 12,500 of
// 400 K slots 1.18 and 0.78 times.  From RED_MANY contributions on four rounds lose
// nothing there, and their registers count: 373 regions of 64, 690 against 702 us.  Dense tiles
// have five rounds all the same: 150 regions of 200, 100 K slots, 72 us with four, 66 with
// five, 48 of 256 131.5 and 129.4, 80 of 100 80.3 and 81.2.
// A region is taken as densely hit where the ranked tile would be no wider than the
// dense one.  With RED_MANY contributions it is from a lower share on, as more
// entries than assumed share slots then: 48 regions of 256 contributions that hit 0.37
// of the slots take 152 us dense and 177 us ranked.  With fewer the ranked tile is ahead
// there: 93 regions of 40 contributions that hit 0.35 of 400 K slots, 70 against 100 us.
constexpr uint32_t RED_MANY = 64;
constexpr double RED_DENSE_FROM = 0.35;

// Tile shape for a region `width` wide whose union is expected to hold at most
// `expected` entries, from P contributions.  A tile is as wide - any multiple of
// 32 slots - as keeps the expected number of hit slots at FILL of the
// accumulators, and the units the entries make within what a chunk holds.  Its entries
// are more than its hit slots: P contributions of one length that hit `share` of the
// slots together, at random, hold 1 - (1 - share)^(1/P) of them each (1.8 entries a hit
// slot for 8 at 0.7), and half a unit is lost at the end of every slice, which
// is not minded where it is more than half of what the accumulators could hold.
// The hits of even tiles vary by 1 to 2 %.  Narrow tiles cover less of the region, so
// what differs between its parts averages out less: they have more room.
constexpr double RED_FILL_UNITS = 0.98;
// Slim tiles of fewer than RED_SLIM_EVEN contributions have room for the entries of regions that
// have 30 % of them in common, which wide tiles of so few hold in registers too (with more, neither
// does, and narrower tiles would cost even regions more): 4 contributions, 1.6 M slots, 0.2 hit,
// 30 % in common, 52 us wide, 68 us slim without and 51 with it; hit evenly 55, 48 and 50.
constexpr uint32_t RED_SLIM_EVEN = 8;
enum ReduceKind { RED_DENSE = 0, RED_RANKED = 1, RED_SPARSE = 2 };
struct ReduceShape {
    uint32_t slots;
    ReduceKind kind;
    ReduceForm form;
};
template <typename Form>
inline ReduceShape reduce_tile_shape_of(uint64_t width, uint64_t expected, uint32_t P, ReduceForm form) {
    if (width == 0 || expected == 0)
        return expected == 0 && width > Form::C_DENSE ? ReduceShape{Form::S_SPARSE, RED_SPARSE, form}
                                                      : ReduceShape{Form::C_DENSE, RED_DENSE, form};
    const double share = (double)expected < 0.999 * (double)width ? (double)expected / (double)width : 0.999;
    double per_slot = P * (1.0 - pow(1.0 - share, 1.0 / P)) / share;       // entries per hit slot
    if (form == RED_SLIM && P < RED_SLIM_EVEN) per_slot *= P / (0.3 + 0.7 * P);
    const double entries = (RED_FILL_UNITS * (Form::BLOCK / 4 * Form::ROUNDS) - 0.5 * P) * RED_UNIT;
    auto hits = [&](uint32_t c) {
        const double most = Form::FILL * c;
        return entries > 0.5 * c && entries < most * per_slot ? entries / per_slot : most;
    };
    const double per_hit = (double)width / (double)expected;          // slots per hit
    const double want = per_hit * hits(Form::C_RANKED);
    if (want <= Form::C_DENSE || (P >= RED_MANY && share >= RED_DENSE_FROM))
        return ReduceShape{Form::C_DENSE, RED_DENSE, form};
    if (want > Form::S_RANKED) {
        const double sparse = per_hit * hits(Form::C_SPARSE);
        if (sparse >= Form::S_SPARSE) return ReduceShape{Form::S_SPARSE, RED_SPARSE, form};
        const uint32_t slots = (uint32_t)sparse / 32 * 32;
        // narrower than the other shape's widest tile: that one holds more per tile
        return slots > Form::S_RANKED ? ReduceShape{slots, RED_SPARSE, form}
                                      : ReduceShape{Form::S_RANKED, RED_RANKED, form};
    }
    const uint32_t slots = (uint32_t)want / 32 * 32;
    return ReduceShape{slots < RED_SLOTS_MIN ? RED_SLOTS_MIN : slots, RED_RANKED, form};
}
inline uint64_t reduce_tiles(uint64_t width, uint32_t slots) { return (width + slots - 1) / slots; }
// per region: a 64-byte header, one descriptor per tile and one per 64 tiles,
// then the table of slice starts, (tiles + 1) x P uint32, padded to 64 bytes
inline size_t reduce_ws_bytes_region(uint64_t max_width, uint32_t P, uint32_t slots) {
    uint64_t t = reduce_tiles(max_width, slots);
    if (t == 0) t = 1;
    size_t bytes = 64 + 8 * (size_t)(t + (t + 63) / 64) + 4 * (size_t)(t + 1) * P;
    return (bytes + 63) & ~(size_t)63;
}
// The least a call asks of its workspace: the table of wide tiles as a region would have
// them that is hit evenly by entries that share no slots.  Such tiles are correct for any
// input, and are taken where the workspace has no room for more.
inline ReduceShape reduce_least_shape(uint64_t width, uint64_t expected, uint32_t P) {
    using Form = ReduceWide4;
    if (width == 0 || expected == 0) return reduce_tile_shape_of<Form>(width, expected, P, RED_WIDE4);
    const double per_hit = (double)width / (double)expected;
    const double entries = (0.95 * (Form::BLOCK / 4 * Form::ROUNDS) - 0.5 * P) * RED_UNIT;
    auto slots = [&](uint32_t c) { return per_hit * (entries < 0.9 * c && entries > 0.5 * c ? entries : 0.9 * c); };
    if ((double)expected >= RED_DENSE_FROM * (double)width) return ReduceShape{Form::C_DENSE, RED_DENSE, RED_WIDE4};
    double want = slots(Form::C_RANKED);
    if (want <= Form::S_RANKED)
        return ReduceShape{want < RED_SLOTS_MIN ? RED_SLOTS_MIN : (uint32_t)want / 32 * 32, RED_RANKED, RED_WIDE4};
    want = slots(Form::C_SPARSE);
    if (want >= Form::S_SPARSE) return ReduceShape{Form::S_SPARSE, RED_SPARSE, RED_WIDE4};
    return want >= Form::S_RANKED + 32 ? ReduceShape{(uint32_t)want / 32 * 32, RED_SPARSE, RED_WIDE4}
                                       : ReduceShape{Form::S_RANKED, RED_RANKED, RED_WIDE4};
}
// Whether slim tiles take the place of wide ones in a region.  Evenly hit regions are 1.1 to 1.25
// times as fast in them throughout; a tile that is hit more than planned, or by entries that share
// slots, goes by windows with half a wide tile's accumulators, and the rule is about those.  Measured
// on 49,500 batches of 6 to 24 M entries, 3 to 256 contributions, 40 K to 5.5 M slots, 0.02 to 0.5
// hit: evenly, 30 % in common to all contributions, every other of 32 stretches, layers of which a
// quarter is hit eight times as often, log-normal stretches of 10,000 (sigma 1), zipf (exponent 1.1, up to
// 500 K slots).  Below: median of the times in wide tiles over those in slim ones, and how many of
// the batches are more than 3 % slower in slim ones.  They are not taken
// - from 0.4 of the slots hit on, with fewer than RED_SLIM_EVEN contributions from 0.2 and with fewer than
//   RED_SLIM_FEW from 0.1 (reduce_slim_to): 16 contributions, 0.4 / 0.5 / 0.6 hit evenly, 1.08 / 1.05 / 1.00;
//   5 to 7, 0.2 to 0.3 hit, in common 0.97 to 1.00 (40 % slower), log-normal 1.03 (14 %), evenly 1.02 to
//   1.05; 3 and 4, 0.1 to 0.13 hit, in common 0.98 (41 %), log-normal 1.09 (18 %).  Below, 8 to 32 contributions that
//   hit 0.3 to 0.4: evenly 1.07, layers 1.06 (7 %), halves 1.05 (6 %), log-normal 1.01 (19 %); 0.2 to 0.3: 1.10,
//   1.07 (3 %), 1.07 (3 %), 1.03 (19 %), in common 1.05 (13 %); 0.1 to 0.2: 1.12, 1.08 (3 %), 1.10 (1 %), 1.05 (9 %), 1.06
//   (14 %).  (What is hit is what the capacity says, here 5 % more than it is; callers that leave more room have
//   narrower tiles, which go by windows less often);
// - with up to RED_FEW contributions where the bitmap limits wide tiles so that the entries of a region
//   with 30 % in common (RED_COMMON a hit slot) still fit their registers, and slim ones have no room for
//   as many: 17 to 32 contributions, 0.05 to 0.07 hit, in common 0.81 to 0.97;
// - with more, from RED_SLIM_HITS planned hits a tile on: up to there entries that collide (zipf, two a
//   hit slot) are 1.1 times as fast, above 0.77 to 0.96 (33 to 63 contributions, 53 to 97 % slower); full
//   tiles lose more: in common 1.04 (27 %), halves 1.06 (28 %), layers 1.07 (12 %, 0.67 at worst), log-normal 1.06 (16 %);
// - but from RED_MANY contributions on in all tiles that the bitmap limits, where the tiles are not
//   planned full: layers 1.13 (2 %), halves 1.16 (2 %), log-normal 1.14 (2 %), in common 1.05 (14 %), zipf 1.0
//   (38 %, 0.8 at worst); in full ones layers 1.08 (3 %), halves 1.07 (8 %), in common 0.98 (38 %), zipf 1.02 (28 %);
// - from RED_SLIM_P contributions on: their slices are short, and where they collide the windows of
//   a slim tile read little pieces of each (129 to 256, zipf 0.96 to 1.06, in common 0.91 to 0.96 from 0.05 hit on).
constexpr double RED_COMMON = 1.41, RED_SLIM_HITS = 3300;
constexpr uint32_t RED_SLIM_P = 129, RED_SLIM_FEW = 5;
constexpr double reduce_slim_to(uint32_t P) { return P < RED_SLIM_FEW ? 0.1 : P < RED_SLIM_EVEN ? 0.2 : 0.4; }
inline bool reduce_slim_pays(const ReduceShape& slim, const ReduceShape& wide, uint64_t width, uint64_t expected, uint32_t P) {
    if (wide.kind == RED_DENSE || slim.kind == RED_DENSE || P >= RED_SLIM_P) return false;
    const double share = (double)expected / (double)width, hits = slim.slots * share;
    if (share >= reduce_slim_to(P)) return false;
    if (P > RED_FEW)
        return hits <= RED_SLIM_HITS ||
               (P >= RED_MANY && slim.slots == (slim.kind == RED_SPARSE ? ReduceSlim::S_SPARSE : ReduceSlim::S_RANKED));
    static_assert(ReduceSlim::BLOCK == ReduceWide5::BLOCK, "units of both");
    auto entries = [&](int rounds) { return (RED_FILL_UNITS * (ReduceSlim::BLOCK / 4 * rounds) - 0.5 * P) * RED_UNIT; };
    return RED_COMMON * wide.slots * share > entries(ReduceWide5::ROUNDS) || RED_COMMON * hits <= entries(ReduceSlim::ROUNDS);
}
// A region that a narrower bitmap covers takes the tiles that have it: more is left for sums.
inline ReduceShape reduce_slim_shape(uint64_t width, uint64_t expected, uint32_t P) {
    const ReduceShape s = reduce_tile_shape_of<ReduceSlim>(width, expected, P, RED_SLIM);
    return s.kind == RED_SPARSE && width <= ReduceSlim::S_RANKED ? ReduceShape{ReduceSlim::S_RANKED, RED_RANKED, RED_SLIM} : s;
}
// The shape a call takes with a workspace of ws_bytes, at least what the least shape needs.
inline ReduceShape reduce_shape(uint64_t B, uint64_t max_width, uint64_t expected, uint32_t P, uint64_t cus,
                                size_t ws_bytes) {
    auto fits = [&](const ReduceShape& s) {
        const size_t region = reduce_ws_bytes_region(max_width, P, s.slots);
        return region <= 0xffffffffull && ws_bytes >= region * B;
    };
    const ReduceShape wide = P < RED_MANY
        ? reduce_tile_shape_of<ReduceWide5>(max_width, expected, P, RED_WIDE5)
        : reduce_tile_shape_of<ReduceWide4>(max_width, expected, P, RED_WIDE4);
    const ReduceShape narrow = reduce_tile_shape_of<ReduceNarrow>(max_width, expected, P, RED_NARROW);
    const bool fills = B * reduce_tiles(max_width, wide.slots) >= RED_WIDE_TILES_PER_CU * cus;
    const bool small = P <= RED_FEW && reduce_tiles(max_width, narrow.slots) <= RED_NARROW_TILES;
    if ((!fills || small) && fits(narrow)) return narrow;
    const ReduceShape slim = reduce_slim_shape(max_width, expected, P);
    if (reduce_slim_pays(slim, wide, max_width, expected, P) && fits(slim)) return slim;
    return fits(wide) ? wide : reduce_least_shape(max_width, expected, P);
}
inline bool reduce_counts_first(const ReduceShape& shape, uint64_t B, uint64_t max_width, uint64_t cus) {
    const uint64_t tiles = reduce_tiles(max_width, shape.slots);
    return shape.form == RED_NARROW && tiles >= RED_PLACED_FROM && B * tiles <= RED_PLACED_TILES_PER_CU * cus;
}
// Whether teams of lanes search for the ends of the slices: in regions of RED_TEAM_TILES tiles
// or more with slices of RED_TEAM_SLICE entries or more, as a region hit evenly has them (a
// capacity of the whole width or more cannot be a count of hit slots: it is one of entries;
// 3.4 M slots, 256 contributions of 15,900 entries, taken as 0.999 hit 43.2 us, so 41.4).
// Whole calls, a thread a cell and teams: slices of 100 entries, 54 tiles, 696 and 663 us; of
// 450, two tiles, 57 and 58; of 19, 25 tiles, 117 and 122; of 16 to 21 in dense tiles, 256
// contributions, 17 to 218 tiles, 2 to 7 % more with teams, of 30 to 50 even.
constexpr uint64_t RED_TEAM_TILES = 16;
constexpr double RED_TEAM_SLICE = 64;
inline bool reduce_by_teams(const ReduceShape& shape, uint64_t width, uint64_t expected, uint32_t P) {
    if (reduce_tiles(width, shape.slots) < RED_TEAM_TILES) return false;
    const double share = (double)expected / (double)width;
    const double hit_by_one = share < 1.0 ? 1.0 - pow(1.0 - share, 1.0 / P) : share / P;
    return shape.slots * hit_by_one >= RED_TEAM_SLICE;
}
// Boundaries that a team of the slice table's kernel finds in turn: as many as leave enough
// teams to fill the chip (1 and 4: 1.3 M cells 670 and 660 us a call, 72,000 cells 72 and 78).
inline uint32_t reduce_chain(uint64_t cells) {
    const uint64_t chain = cells >> 18;
    return chain < 1 ? 1u : chain > 4 ? 4u : (uint32_t)chain;
}
inline size_t reduce_ws_bytes(uint64_t B, uint64_t max_width, uint32_t P) {
    return (size_t)B * reduce_ws_bytes_region(max_width, P, RED_SLOTS_MIN);     // largest
}

}  // namespace okt
#endif
