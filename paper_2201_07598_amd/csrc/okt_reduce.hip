// okt_sparse_reduce / okt_sparse_reduce_batch: the local reduction of the P
// sparse contributions a worker receives for its region (Algorithm 1, line 8;
// Sec. 3.1.1).  Plain sum over the union of the supports.
//
// Two kernels per call.
//  1. The region is cut into tiles of `slots` consecutive index slots; for every (tile
//     boundary, contribution) the first launch finds, in the sorted contribution, where the
//     boundary falls, all searches side by side, so that their latency is paid once.  Four
//     kernels do it: a wave a boundary where there are few (reduce_slices_wave_kernel), a
//     thread a boundary (reduce_slices_kernel), teams of lanes that find several in turn
//     where slices are longer (reduce_slices_team_kernel), and a workgroup a tile, which
//     also counts the tile's hit slots, where all tiles run at a time (reduce_count_kernel).
//  2. reduce_tile_kernel: a workgroup owns one tile.  Its slice of every
//     contribution is known from the table, so all its entries are addressed up
//     front, read with 16-byte loads all in flight and kept in registers.  Entries are
//     summed with LDS fp64 atomic adds.  Where the region is densely hit the
//     accumulator of a slot is the slot itself.  Where it is sparsely hit the tile is
//     wider than the accumulator array: the hit slots are marked in a bitmap, the popcount prefix
//     of the bitmap ranks them, and the entries are summed into accumulator [rank]; in the
//     slim form only those of slots that several entries hit.
//     The tile is then written out in index order; its place in the output comes from the
//     two-level chained scan over tile counts, or is the sum of the counts before it.
// Traffic: every input entry is read once (tiles with more entries than registers
// hold read indices twice), every output entry is written once, plus 4 B per slot if
// the dense region is requested.
#include "okt_device.h"
#include "okt_search.h"
#include "okt_sizes.h"

#include <type_traits>

namespace okt {

struct RegionView {
    uint32_t lo, hi, width, ntiles;
    bool bad;
};
__device__ __forceinline__ RegionView region_view(const uint32_t* lo_hi, uint32_t lo0, uint32_t hi0,
                                                  uint32_t region, uint32_t max_width,
                                                  uint32_t slots) {
    RegionView r;
    r.lo = lo_hi ? lo_hi[2 * region] : lo0;
    r.hi = lo_hi ? lo_hi[2 * region + 1] : hi0;
    r.bad = r.hi < r.lo || r.hi - r.lo > max_width;
    r.width = r.bad ? 0u : r.hi - r.lo;
    r.ntiles = (uint32_t)(((uint64_t)r.width + slots - 1) / slots);
    return r;
}

// table[region][t][p] = number of entries of contribution p with index below
// lo + t * slots (clipped to hi), for t = 0 .. ntiles.
// Every search starts from a guess, which makes it two or three waits and lines of
// memory instead of a bisection's fifteen: 35 boundaries x 16 contributions x 490
// regions in 33 us against 49 with a gallop of single probes from the same guess; a
// lone region (317 x 32) takes as long as with plain bisections.
// Neighbouring threads search the same contribution for neighbouring boundaries: their
// probes share lines where its slices are short.  A contribution lies inside its region as
// a rule, and one entry says so: 868 regions of one tile, 88 contributions of 77 entries,
// 55.9 -> 53.5 us a call.
__global__ __launch_bounds__(256) void reduce_slices_kernel(
    const uint32_t* __restrict__ idx_cat, const uint64_t* __restrict__ seg_begin,
    const uint64_t* __restrict__ seg_end, uint32_t seg_stride,
    const uint32_t* __restrict__ lo_hi, uint32_t lo0, uint32_t hi0, uint32_t P,
    uint32_t max_width, uint32_t slots, char* ws, uint32_t ws_region_bytes,
    uint32_t table_offset, uint32_t spin_limit) {
    const uint32_t region = blockIdx.y;
    const RegionView r = region_view(lo_hi, lo0, hi0, region, max_width, slots);
    uint32_t* table = (uint32_t*)(ws + (size_t)region * ws_region_bytes + table_offset);
    // the scan state of the region (header and descriptors, in front of the table)
    // must be zero when the tile kernel starts
    uint64_t* scan_state = (uint64_t*)(ws + (size_t)region * ws_region_bytes);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < table_offset / 8;
         i += gridDim.x * blockDim.x)
        scan_state[i] = i == SCAN_SPIN_WORD ? (uint64_t)spin_limit : 0ull;
    const uint64_t* begin = seg_begin + (size_t)region * seg_stride;
    const uint64_t* end = seg_end + (size_t)region * seg_stride;
    const uint32_t cells = (r.ntiles + 1) * P;                // below 2^32
    const float per_index = r.width ? 1.0f / (float)r.width : 0.0f;
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < cells; c += gridDim.x * blockDim.x) {
        const uint32_t p = c / (r.ntiles + 1), t = c - p * (r.ntiles + 1);
        const uint32_t x = r.width < (uint64_t)t * slots ? r.hi : r.lo + t * slots;
        const uint64_t cb = begin[p], ce = end[p] > cb ? end[p] : cb;
        // from where the boundary would fall if the indices were spread evenly over the region
        uint64_t at;
        if (t == 0 && cb < ce && idx_cat[cb] >= x) at = cb;
        else if (t == r.ntiles && cb < ce && idx_cat[ce - 1] < x) at = ce;
        else at = lower_bound_near(idx_cat, cb, ce, x, cb + (uint64_t)((float)(ce - cb) * ((float)(x - r.lo) * per_index)));
        table[(size_t)t * P + p] = (uint32_t)(at - cb);
    }
}

// The same by teams of lanes, for regions of many tiles and longer slices: a cell costs
// lines of the index lists at random places, so lines are what is saved.  A team reads a
// whole line a guess and finds `chain` boundaries of a contribution in turn, each guessed
// from the one before (the end of a slice of 117 entries to about ten, where a guess from
// the contribution's ends is up to 36 off); neighbouring teams hold neighbouring
// contributions, whose cells share lines of the table.  A thread a cell -> teams:
//   373 regions, 64 contributions, 54 tiles, slices of 97 entries    98 -> 64 us
//   490 regions, 16 contributions, 33 tiles, 484 entries             31 -> 23
// (Whole calls of the first: 696 -> 663 us, with teams of four lanes 661, of eight 680.)
constexpr uint32_t TEAM = 2;
// Sum over the lanes of a team; every lane gets it.
__device__ __forceinline__ uint32_t team_sum(uint32_t v) {
    static_assert(TEAM == 2, "one exchange");
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false);     // quad_perm: the neighbour
}

__global__ __launch_bounds__(256) void reduce_slices_team_kernel(
    const uint32_t* __restrict__ idx_cat, const uint64_t* __restrict__ seg_begin,
    const uint64_t* __restrict__ seg_end, uint32_t seg_stride,
    const uint32_t* __restrict__ lo_hi, uint32_t lo0, uint32_t hi0, uint32_t P,
    uint32_t max_width, uint32_t slots, char* ws, uint32_t ws_region_bytes,
    uint32_t table_offset, uint32_t spin_limit, uint32_t chain) {
    const uint32_t region = blockIdx.y;
    const RegionView r = region_view(lo_hi, lo0, hi0, region, max_width, slots);
    uint32_t* table = (uint32_t*)(ws + (size_t)region * ws_region_bytes + table_offset);
    uint64_t* scan_state = (uint64_t*)(ws + (size_t)region * ws_region_bytes);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < table_offset / 8;
         i += gridDim.x * blockDim.x)
        scan_state[i] = i == SCAN_SPIN_WORD ? (uint64_t)spin_limit : 0ull;
    const uint64_t* begin = seg_begin + (size_t)region * seg_stride;
    const uint64_t* end = seg_end + (size_t)region * seg_stride;
    constexpr uint32_t QUADS = SEARCH_LINE / 4 / TEAM;        // loads of a lane, its team's side by side
    const uint32_t lane = (uint32_t)lane_id(), sub = lane & (TEAM - 1);
    const uint32_t units = P * (r.ntiles / chain + 1);        // fewer than cells, which are below 2^32
    for (uint32_t u = (blockIdx.x * blockDim.x + threadIdx.x) / TEAM; u < units;
         u += gridDim.x * (blockDim.x / TEAM)) {              // a team is in or out together
        const uint32_t c = u / P, p = u - c * P, t_end = min((c + 1) * chain, r.ntiles + 1);
        uint32_t t = c * chain;
        const uint64_t cb = begin[p], ce = end[p];
        const uint32_t* const list = idx_cat + cb;
        const uint32_t skew = (uint32_t)((uintptr_t)list / sizeof(uint32_t)) & (SEARCH_LINE - 1);
        auto bound_of = [&](uint32_t tile) {
            return r.hi - r.lo < (uint64_t)tile * slots ? r.hi : r.lo + tile * slots;
        };
        if (ce > cb && ce - cb > 0xffffffffull - SEARCH_LINE) {       // positions would not fit 32 bits
            for (; t < t_end; ++t)
                table[(size_t)t * P + p] = (uint32_t)(lower_bound_idx(idx_cat, cb, ce, bound_of(t)) - cb);
            continue;
        }
        const uint32_t len = ce > cb ? (uint32_t)(ce - cb) : 0u;
        const uint32_t* const a = list - skew;                // positions count from here
        const uint32_t upto = len + skew;
        uint32_t x = bound_of(t);
        // as if the contribution's indices were spread evenly over the region
        LineSearch s{skew, upto, skew + (r.width ? (uint32_t)((float)len * ((float)(x - r.lo) / (float)r.width)) : 0u)};
        for (int guesses = 0;;) {
            bool known = s.hi <= s.lo;
            if (!known && guesses == 0) {
                if (t == 0 && list[0] >= x) {
                    known = true;
                } else if (t == r.ntiles && list[len - 1] < x) {
                    s.lo = upto;
                    known = true;
                }
            }
            if (!known && guesses == SEARCH_GUESSES) {        // any input ends
                s.lo = (uint32_t)lower_bound_idx(a, s.lo, s.hi, x);
                known = true;
            } else if (!known) {
                const uint32_t line = line_of_guess(s, skew, upto);
                uint32_t v[QUADS][4], below = 0;
                if (len >= SEARCH_LINE) {                     // alike in a team
#pragma unroll
                    for (uint32_t q = 0; q < QUADS; ++q) {
                        const QuadAt4 quad = *reinterpret_cast<const QuadAt4*>(a + line + 4 * (q * TEAM + sub));
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j) v[q][j] = quad.v[j];
                    }
                } else {
#pragma unroll
                    for (uint32_t q = 0; q < QUADS; ++q)
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j) {
                            const uint32_t at = line + 4 * (q * TEAM + sub) + j;
                            v[q][j] = at < upto ? a[at] : ~0u;
                        }
                }
#pragma unroll
                for (uint32_t q = 0; q < QUADS; ++q)
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j) below += v[q][j] < x ? 1u : 0u;
                below = team_sum(below);
                uint32_t first = 0, last = 0;
                if (below == 0 || below == SEARCH_LINE) {     // alike in a team
                    first = __shfl(v[0][0], (int)(lane & ~(TEAM - 1)), WAVE);
                    last = __shfl(v[QUADS - 1][3], (int)(lane | (TEAM - 1)), WAVE);
                }
                known = line_says(s, line, below, first, last, x);
                ++guesses;
            }
            if (!known) continue;
            if (sub == 0) table[(size_t)t * P + p] = s.lo - skew;
            if (++t == t_end) break;
            // the next boundary lies at or behind this one, as far on as if the rest were spread evenly
            const uint32_t rest = r.hi - x, step = rest < slots ? rest : slots;
            x += step;
            s.hi = upto;
            s.guess = s.lo + (uint32_t)((float)(upto - s.lo) * ((float)step / (float)rest));
            guesses = 0;
        }
    }
}

// The same table for launches with few cells (a lone region): one WAVE per cell,
// 64 evenly spaced probes per step, so a boundary is found in about log64 of the
// contribution's length dependent round trips instead of log2 - this kernel is
// nothing but that latency.  (For many regions the extra probes would cost more
// memory traffic than the latency they save.)
__global__ __launch_bounds__(256) void reduce_slices_wave_kernel(
    const uint32_t* __restrict__ idx_cat, const uint64_t* __restrict__ seg_begin,
    const uint64_t* __restrict__ seg_end, uint32_t seg_stride,
    const uint32_t* __restrict__ lo_hi, uint32_t lo0, uint32_t hi0, uint32_t P,
    uint32_t max_width, uint32_t slots, char* ws, uint32_t ws_region_bytes,
    uint32_t table_offset, uint32_t spin_limit) {
    const uint32_t region = blockIdx.y;
    const RegionView r = region_view(lo_hi, lo0, hi0, region, max_width, slots);
    uint32_t* table = (uint32_t*)(ws + (size_t)region * ws_region_bytes + table_offset);
    uint64_t* scan_state = (uint64_t*)(ws + (size_t)region * ws_region_bytes);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < table_offset / 8;
         i += gridDim.x * blockDim.x)
        scan_state[i] = i == SCAN_SPIN_WORD ? (uint64_t)spin_limit : 0ull;
    const uint64_t* begin = seg_begin + (size_t)region * seg_stride;
    const uint64_t* end = seg_end + (size_t)region * seg_stride;
    const uint64_t cells = (uint64_t)(r.ntiles + 1) * P;
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / WAVE);
    for (uint64_t c = (uint64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE; c < cells;
         c += waves) {
        const uint32_t p = (uint32_t)(c / (r.ntiles + 1)), t = (uint32_t)(c % (r.ntiles + 1));
        uint64_t bound = (uint64_t)r.lo + (uint64_t)t * slots;
        if (bound > r.hi) bound = r.hi;
        const uint32_t x = (uint32_t)bound;                 // bound <= hi < 2^32
        const uint64_t cb = begin[p];
        uint64_t lo = cb, hi = end[p] > cb ? end[p] : cb;   // the answer lies in [lo, hi]
        while (hi - lo > (uint64_t)WAVE) {
            const uint64_t step = (hi - lo + WAVE - 1) / WAVE;
            const uint64_t at = lo + lane * step;
            const bool below = at < hi && idx_cat[at] < x;
            const uint32_t n_below = (uint32_t)__popcll(__ballot(below));   // lanes 0 .. n_below-1
            if (n_below == 0) { hi = lo; break; }                           // idx_cat[lo] >= x
            const uint64_t next = lo + (uint64_t)n_below * step;            // first probe not below x
            lo = lo + (uint64_t)(n_below - 1) * step + 1;
            if (next < hi) hi = next;
        }
        if (hi > lo) {
            const bool below = lo + lane < hi && idx_cat[lo + lane] < x;
            lo += (uint64_t)__popcll(__ballot(below));
        }
        if (lane == 0) table[(size_t)t * P + p] = (uint32_t)(lo - cb);
    }
}

// ---- launches whose tiles are all in flight together ----
// A lone region takes as long as one tile, and every step of that is latency.  Tickets
// on one counter are served one at a time, 30 ns each - 361 tiles, 11 us - and each tile waits for
// the counts of those before it.  So the table, and a count of every tile's hit slots, are made
// by workgroups with a tile each, which read the indices once more than the scan does, and
// reduce_tile_kernel<PLACED> adds up the counts before its tile: no ticket, no
// descriptors to clear, no wait.  One region of 3.4 M slots, 32 contributions, 1.1 M entries:
// 8.0 us for the table and 16.5 for the tiles with tickets, 10.0 and 11.2 so.
// It pays up to PLACED_P contributions: with more, two searches for each of them in every
// tile and short slices cost more than the tickets (whole calls with tickets and so, 3.4 M
// slots, 0.4 to 0.78 hit: 96 contributions 31 to 42 and 25 to 39 us, 128 31 to 42 and 28 to 43,
// 160 32 to 43 and 30 to 46, 256 34 to 47 and 38 to 56).  It does not pay where a few tiles
// hold most of the entries, as the first launch then lasts as long as the busiest: with
// log-normal stretches (sigma 1.5), 0.4 hit, 32 contributions 77 and 92 us; layers of which a
// quarter is hit eight times as often as the rest come out even (73 to 80, 55 and 56).
constexpr int COUNT_BLOCK = 512;
constexpr uint32_t PLACED_P = 96;
static_assert(4 * PLACED_P <= COUNT_BLOCK, "two lanes at least for each end of a slice");

// lower_bound_near by `lanes` consecutive lanes (a power of two, at most 16) that all
// have the same arguments: each reads sixteen entries of one window around the guess.
__device__ __forceinline__ uint64_t lower_bound_lanes(const uint32_t* __restrict__ a, uint64_t lo, uint64_t hi,
                                                      uint32_t x, uint64_t guess, uint32_t lanes) {
    const uint32_t sub = (uint32_t)lane_id() & (lanes - 1), window = 16 * lanes;
    for (int miss = 0; miss < SEARCH_GUESSES; ++miss) {
        if (hi <= lo) return lo;
        uint64_t w = guess < lo + window / 2 ? lo : guess - window / 2;
        if (w + window > hi) w = hi < lo + window ? lo : hi - window;
        const uint64_t at = w + 16 * sub;
        uint32_t v[16], below = 0;
        if (at + 16 <= hi) {
            const SearchWindow win = *reinterpret_cast<const SearchWindow*>(a + at);
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = win.v[j];
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = at + j < hi ? a[at + j] : ~0u;   // past the end counts as not below
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) below += v[j] < x ? 1u : 0u;
        uint32_t first = v[0], last = v[15];
        for (uint32_t s = 1; s < lanes; s <<= 1) below += __shfl_xor(below, (int)s, WAVE);
        first = __shfl(first, (int)((uint32_t)lane_id() & ~(lanes - 1)), WAVE);
        last = __shfl(last, (int)((uint32_t)lane_id() | (lanes - 1)), WAVE);
        const bool whole = w + window <= hi;
        const bool up = whole && below == window && w + window < hi, down = below == 0 && w > lo;
        if (!up && !down) return w + below;
        const float per = (float)(window - 1) / (float)(whole && last > first ? last - first : 1u);   // entries per index
        if (down) {
            hi = w;
            const uint64_t back = (uint64_t)((float)(first - x) * per);
            guess = back < w ? w - back : 0;
        } else {
            lo = w + window;
            guess = lo + (uint64_t)((float)(x - last) * per);
        }
    }
    return lower_bound_idx(a, lo, hi, x);
}

template <uint32_t S_MAX>
__global__ __launch_bounds__(COUNT_BLOCK) void reduce_count_kernel(
    const uint32_t* __restrict__ idx_cat, const uint64_t* __restrict__ seg_begin,
    const uint64_t* __restrict__ seg_end, uint32_t seg_stride, const uint32_t* __restrict__ lo_hi, uint32_t lo0,
    uint32_t hi0, uint32_t P, uint32_t max_width, uint32_t slots, char* ws, uint32_t ws_region_bytes,
    uint32_t table_offset) {
    constexpr uint32_t WORDS_MAX = S_MAX / 32;
    __shared__ __attribute__((aligned(16))) uint32_t s_bits[WORDS_MAX];
    __shared__ uint64_t s_from[PLACED_P], s_upto[PLACED_P];
    __shared__ uint32_t s_wave[COUNT_BLOCK / WAVE];
    const uint32_t tid = threadIdx.x, region = blockIdx.y, tile = blockIdx.x;
    const RegionView r = region_view(lo_hi, lo0, hi0, region, max_width, slots);
    if (tile >= r.ntiles) return;
    char* const region_ws = ws + (size_t)region * ws_region_bytes;
    uint32_t* const table = (uint32_t*)(region_ws + table_offset);
    const uint64_t* begin = seg_begin + (size_t)region * seg_stride;
    const uint64_t* end = seg_end + (size_t)region * seg_stride;
    const uint32_t a = r.lo + tile * slots, tslots = (r.hi - a) < slots ? (r.hi - a) : slots;
    for (uint32_t w = tid; w < WORDS_MAX / 4; w += COUNT_BLOCK) reinterpret_cast<uint4*>(s_bits)[w] = uint4{0, 0, 0, 0};
    // ---- where the tile begins and ends in every contribution ----
    uint32_t lanes = 1;
    while (lanes < 16 && 4 * P * lanes <= (uint32_t)COUNT_BLOCK) lanes <<= 1;
    {
        const uint32_t team = tid / lanes, p = team >> 1, which = team & 1u;
        if (p < P) {                                 // a team is in or out together
            const uint64_t cb = begin[p], ce = end[p] > cb ? end[p] : cb;
            const uint64_t bound = (uint64_t)a + (which ? tslots : 0u);
            const uint64_t guess = cb + (ce - cb) * (bound - r.lo) / r.width;    // both factors are below 2^32
            const uint64_t at = bound > 0xffffffffull ? ce : lower_bound_lanes(idx_cat, cb, ce, (uint32_t)bound, guess, lanes);
            if (tid % lanes == 0) {
                (which ? s_upto : s_from)[p] = at;
                if (!which) table[(size_t)tile * P + p] = (uint32_t)(at - cb);
                else if (tile == r.ntiles - 1) table[(size_t)(tile + 1) * P + p] = (uint32_t)(at - cb);
            }
        }
    }
    __syncthreads();
    // ---- the hit slots ----
    uint32_t share = 0;                              // 2^share threads read a slice
    while (share < 8 && (P << (share + 1)) <= (uint32_t)COUNT_BLOCK) ++share;
    const uint32_t member = tid & ((1u << share) - 1u), q = tid >> share;
    if (q < P) {
        constexpr int FLIGHT = 4;
        const uint64_t from = s_from[q], upto = s_upto[q], step = 4ull << share;
        for (uint64_t i0 = from + 4 * member; i0 < upto; i0 += FLIGHT * step) {
            uint32_t v[FLIGHT][4];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) {
                const uint64_t i = i0 + u * step;
                if (i + 4 <= upto) {
                    const QuadAt4 x = *reinterpret_cast<const QuadAt4*>(idx_cat + i);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[u][j] = x.v[j];
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[u][j] = i + j < upto ? idx_cat[i + j] : a + tslots;
                }
            }
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t s = v[u][j] - a;
                    if (s < tslots)
                        __hip_atomic_fetch_or(&s_bits[s >> 5], 1u << (s & 31), __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
                }
        }
    }
    __syncthreads();
    uint32_t hits = 0;
    for (uint32_t w = tid; w < WORDS_MAX; w += COUNT_BLOCK) hits += (uint32_t)__popc(s_bits[w]);
    hits = wave_sum(hits);
    if (tid % WAVE == 0) s_wave[tid / WAVE] = hits;
    __syncthreads();
    if (tid == 0) {
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < COUNT_BLOCK / WAVE; ++w) total += s_wave[w];
        ((uint32_t*)(region_ws + SCAN_HEADER_BYTES))[tile] = total;
    }
}

// From one count per wave of the workgroup in LDS: the counts of the waves before
// the calling one, and of all.
struct WaveSums { uint32_t before, total; };
template <int WAVES>
__device__ __forceinline__ WaveSums sum_of_waves(const uint32_t* s_wave) {
    const int lane = threadIdx.x & (WAVE - 1), wave = (int)uniform(threadIdx.x >> 6);
    const uint32_t incl = wave_inclusive_scan_u32(lane < WAVES ? s_wave[lane] : 0u);
    return WaveSums{wave ? (uint32_t)__builtin_amdgcn_readlane((int)incl, wave - 1) : 0u,
                    (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVES - 1)};
}

// Exclusive prefix over the popcounts of `words` bitmap words into s_wprefix;
// returns the total (to every thread).  Called by the whole workgroup.
// A tile of more than 65,536 slots may have prefixes that 16 bits do not hold: the
// first word with such a prefix goes to *s_wrap (all ones if there is none).
template <int BLOCK, uint32_t WORDS_MAX>
__device__ __forceinline__ uint32_t bitmap_prefix(const uint32_t* s_bits, uint16_t* s_wprefix,
                                                  uint32_t words, uint32_t* s_wave, uint32_t* s_wrap) {
    static_assert(WORDS_MAX * 32 < 2 * 65536, "prefixes wrap once at most");
    constexpr uint32_t PER = (WORDS_MAX + BLOCK - 1) / BLOCK;           // words per thread (1 to 6)
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t w = tid * PER + j;
        c[j] = w < words ? (uint32_t)__popc(s_bits[w]) : 0u;
        sum += c[j];
    }
    const uint32_t incl = wave_inclusive_scan_u32(sum);
    if (lane == WAVE - 1) s_wave[wave] = incl;
    __syncthreads();
    const WaveSums sums = sum_of_waves<BLOCK / WAVE>(s_wave);
    uint32_t before = sums.before + incl - sum;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t w = tid * PER + j;
        if (w < words) s_wprefix[w] = (uint16_t)before;
        if (WORDS_MAX > 2048 && w < words && before > 0xffffu) atomicMin(s_wrap, w);
        before += c[j];
    }
    __syncthreads();
    return sums.total;
}

// grid = (tiles of the widest region, B).  Region j: chunk offsets at seg_begin /
// seg_end + j * seg_stride; bounds from lo_hi[2j..] if lo_hi != NULL else (lo0, hi0).
//
// A tile's entries are read in UNITS of RED_UNIT consecutive entries of one slice:
// a unit belongs to four lanes, each of which reads four entries of it with one
// 16-byte load, so a wave reads sixteen units - of as many slices, if they are
// short - with one load instruction, and only the last unit of a slice is partly
// empty.  The threads that hold the slice table write the units' places to LDS, so
// that finding a thread's entries is one LDS read.  ROUNDS units per four
// threads make a chunk.  A tile that is one chunk (the host sizes tiles so that
// this is the rule) keeps all its entries in registers: they are read from memory
// once, both arrays at once, and the marking, the summing and the writing of the
// indices need nothing more from memory.
//
// A tile with more entries (slots that several contributions hit, a stretch that is
// hit more than the rest of the region) is marked from all of them and then summed from
// all of them, read again.  If it has more hit slots than accumulators too, it is cut
// into windows of the bitmap with as many hit slots as there are accumulators, and only
// the pieces of the slices that lie in a window are read for it: one pass over
// the entries in all, where a pass over all of them for every window took 183 us
// instead of 117 for 382 regions of 8 contributions with most hits in a quarter
// of the region.
//
// What bounds it: a tile is a chain of phases - ticket, slice table, entries, marks,
// ranks, sums, place, output - of some 14 us with two tiles of 8,000 entries to a
// CU, of which about half wait for memory and half are LDS work (two reads and an
// fp64 atomic add at random places an entry), and LDS (ten bytes a hit slot) is what
// limits the tiles in flight.  490 regions of 16 contributions (1.9 GB in and out):
// 575 us with slices read in blocks of 64 entries, twice, by 8-wave workgroups of
// half this size, 519 us as it is here; 373 regions of 64 contributions: 734 and 599 us,
// the longer slices of the wider tile counting for as much as the rest.  The narrow form
// is held to 64 registers, for four tiles to a CU: 16 contributions, a tenth of 400 K slots
// hit, 380 regions, 65 us against 84 with slices read twice and 78 in wide tiles.
//
// SLIM: a sparsely hit region's slots are hit by one entry as a rule, which is the sum then.  So
// the marking notes which entries find their slot marked already; the first of every slot puts
// its value, a float, at the slot's rank, and the others go to a list, where each slot that has
// any gets an fp64 accumulator - in the list entry of the one that gets there first - with all of
// the slot's values added.  The list takes the place of the units, the bitmap and the prefixes,
// which nobody needs once the ranks are known.  So a hit slot takes four bytes of LDS instead of
// eight, and three tiles of 6,566 planned hits run on a CU where two of 7,410 did; no entry but the
// listed ones needs an LDS atomic on a double.  Held to 80 registers: what the compiler spills for it,
// four vector registers, it stores and reloads where a tile goes by windows.  490 regions of 16
// contributions 507 -> 423 us a call, 373 of 64 634 -> 515; neither
// a look at the descriptors before the list, nor four narrower tiles to a CU (452 us), nor the
// slice table made in the same launch by workgroups between the tiles (433 to 482 us: they wait
// for memory in places that tiles could have), nor stores of the outputs past the last-level cache
// (930 MB of them 417.9 us without and 419.9 with, 970 MB 508.8 and 510.5) makes it any faster.
// A tile with more hits, entries or listed
// entries than there is room for goes by windows, as others do, with fp64 accumulators in all
// that the bitmap leaves free; those are half as many as in a wide tile, and where regions are
// hit unevenly that costs more than the third tile to a CU gives.  Which launches that is, and both sides
// measured, stands at reduce_slim_pays; no change to the windows made up for it (accumulators in the units'
// place too, 12 % more of them: layers 1 to 2 % faster, entries that collide 1 to 2 % slower; three or four
// quads of a slice in flight instead of two: even to 4 % slower; tiles planned 15 to 35 % narrower: uneven
// regions as slow at worst, even ones 5 to 10 % slower).
//
// Tried and not kept: 16 waves with 8 entries a thread and the same tile (spills at
// 64 registers), several regions' tiles in turn per workgroup with the next slice table
// fetched ahead (what it hides, its registers and the extra barriers cost), tiles of
// several regions in turn in the grid (their inputs share no lines), the tile's windows
// each searched before its turn (a chain of searches instead of one).
// A thread's entries of a chunk: QUADS of four.
template <int QUADS>
struct TileEntries {
    static constexpr int ROUNDS = QUADS;
    uint32_t slot[ROUNDS][4];    // slot in the tile, later rank << SLOT_BITS | slot; from S_MAX on: no entry
    float value[ROUNDS][4];
    uint32_t have;               // bit 4u + j: there is such an entry
    bool last;                   // the wave has units in the last round (uniform): a chunk is seldom full
};

template <int BLOCK, int ROUNDS, uint32_t C, uint32_t S_MAX, bool PLACED = false, bool SLIM = false>
__global__ __launch_bounds__(BLOCK, SLIM ? 6 : ROUNDS == 2 ? 8 : 4) void reduce_tile_kernel(
    const uint32_t* __restrict__ idx_cat, const float* __restrict__ val_cat,
    const uint64_t* __restrict__ seg_begin, const uint64_t* __restrict__ seg_end,
    uint32_t seg_stride, const uint32_t* __restrict__ lo_hi, uint32_t lo0,
    uint32_t hi0, uint32_t P, uint32_t max_width, uint32_t slots,
    uint32_t* __restrict__ idx_out, float* __restrict__ val_out, uint64_t capacity,
    uint64_t* __restrict__ nnz_out, float* __restrict__ dense_out, char* ws,
    uint32_t ws_region_bytes, uint32_t table_offset) {
    constexpr int WAVES = BLOCK / WAVE;
    constexpr bool DENSE = S_MAX == C;            // accumulator = slot, always
    constexpr uint32_t WORDS_MAX = S_MAX / 32;
    constexpr uint32_t UNITS = BLOCK / 4 * ROUNDS, WINDOWS_MAX = SLIM ? 29 : 15;
    // A tile of at most EXCESS chunks is marked and summed chunk by chunk, the units spread
    // over all threads; a longer one goes slice by slice, without a barrier between chunks.
    // The narrow form keeps the first chunk in registers also then: beside a second chunk
    // the wide form has none for it.
    constexpr uint32_t EXCESS = 2;
    constexpr bool KEEP = ROUNDS == 2;
    // Lanes without an entry work on a slot, a rank and an accumulator of their own
    // past the end (one of SPARE), so that the loops over the entries have no branch.
    constexpr uint32_t SPARE = 32, SLOT_BITS = 17, SLOT_MASK = (1u << SLOT_BITS) - 1u;
    static_assert(S_MAX + 32 * SPARE <= SLOT_MASK && C + SPARE <= 1u << (32 - SLOT_BITS), "a slot and a rank share a word");
    // LDS: accumulators | units | bitmap | prefixes.  SLIM: the list lies behind the C values, over
    // the rest; the fp64 accumulators of a tile that goes by windows have what the rest leaves free.
    constexpr uint32_t FIXED = 8 * UNITS + 6 * (WORDS_MAX + SPARE), VALUES = 4 * (C + SPARE);
    constexpr uint32_t LIST = SLIM ? RED_SLIM_LIST : 1;
    static_assert(!SLIM || (FIXED <= 8 * LIST && (VALUES + 8 * LIST - FIXED + 8 * UNITS) % 16 == 0), "the list holds the rest");
    constexpr uint32_t ACC = SLIM ? ((VALUES + 8 * LIST - FIXED) / 8 - SPARE) & ~1u : C;    // fp64 accumulators
    static_assert(S_MAX <= WINDOWS_MAX * (ACC - 32), "windows of a tile");
    static_assert(!SLIM || ACC > RED_SLIM_HITS, "one window for as many hits");
    static_assert(ACC % 2 == 0 && WORDS_MAX % 4 == 0, "cleared 16 bytes at a time");
    constexpr uint32_t UNITS_AT = SLIM ? VALUES + 8 * LIST - FIXED : 8 * (C + SPARE);
    __shared__ __attribute__((aligned(16))) char s_mem[UNITS_AT + FIXED];
    double* const s_sum = (double*)s_mem;
    uint64_t* const s_unit = (uint64_t*)(s_mem + UNITS_AT);   // first entry << 6 | whole unit readable << 5 | entries
    uint32_t* const s_bits = (uint32_t*)(s_mem + UNITS_AT + 8 * UNITS);
    uint16_t* const s_wprefix = (uint16_t*)(s_mem + UNITS_AT + 8 * UNITS + 4 * (WORDS_MAX + SPARE));
    uint64_t* const s_list = (uint64_t*)(s_mem + VALUES);
    constexpr uint32_t MORE = SLIM ? (C + SPARE + 31) / 32 : 1;
    __shared__ uint32_t s_more[MORE], s_again;    // SLIM: ranks that have an fp64 sum, listed entries
    __shared__ uint32_t s_wave[2][WAVES], s_placed[WAVES];
    __shared__ uint32_t s_tile, s_before[2], s_wrap, s_cut[WINDOWS_MAX + 1], s_cut_rank[WINDOWS_MAX + 1];

    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = (int)uniform((uint32_t)tid >> 6);
    const uint32_t region = blockIdx.y;
    char* region_ws = ws + (size_t)region * ws_region_bytes;
    ScanHeader* hdr = (ScanHeader*)region_ws;
    uint64_t* tile_desc = (uint64_t*)(region_ws + SCAN_HEADER_BYTES);
    uint64_t* group_desc = tile_desc + gridDim.x;
    if (tid == 0) {
        if (!PLACED) s_tile = atomicAdd(&hdr->ticket, 1u);
        s_wrap = ~0u;
        if (SLIM) s_again = 0;
    }
    if (SLIM && tid < (int)MORE) s_more[tid] = 0;
    if (tid < (int)SPARE) s_wprefix[WORDS_MAX + tid] = (uint16_t)(C + tid);
    const RegionView r = region_view(lo_hi, lo0, hi0, region, max_width, slots);
    uint64_t* nnz = nnz_out + 2 * (size_t)region;
    // the bitmap and the accumulators are cleared while the ticket is under way
    for (uint32_t w = tid; w < WORDS_MAX / 4; w += BLOCK) reinterpret_cast<uint4*>(s_bits)[w] = uint4{0, 0, 0, 0};
    if (!SLIM)
        for (uint32_t s = tid; s < ACC / 2; s += BLOCK) reinterpret_cast<double2*>(s_sum)[s] = double2{0.0, 0.0};
    __syncthreads();
    const uint32_t tile = PLACED ? blockIdx.x : uniform(s_tile);
    if (r.ntiles == 0) {
        if (tile == 0 && tid == 0) {
            nnz[0] = r.bad ? ~0ull : 0ull;
            nnz[1] = r.bad ? ~0ull : 0ull;
        }
        return;
    }
    if (tile >= r.ntiles) return;
    const uint32_t a = r.lo + tile * slots;                       // first index of the tile
    const uint32_t tslots = (r.hi - a) < slots ? (r.hi - a) : slots;
    const uint32_t words = (tslots + 31) / 32;
    const uint32_t* row = (const uint32_t*)(region_ws + table_offset) + (size_t)tile * P;   // slice starts, then ends
    const uint64_t* off = seg_begin + (size_t)region * seg_stride;
    const uint64_t* off_end = seg_end + (size_t)region * seg_stride;
    idx_out += (size_t)region * capacity;
    val_out += (size_t)region * capacity;
    float* const dense = dense_out ? dense_out + (size_t)region * max_width + (size_t)tile * slots : nullptr;
    if (dense && !DENSE)
        for (uint32_t s = tid; s < tslots; s += BLOCK) dense[s] = 0.0f;   // the sums go on top, several barriers later

    // ---- the slice table: 2^share threads hold one slice ----
    // (several where contributions are few, so that the units of long slices are
    // written by many threads); BLOCK contributions at most at a time
    uint32_t share = 0;
    while (share < 6 && (P << (share + 1)) <= (uint32_t)BLOCK) ++share;
    const uint32_t member = (uint32_t)tid & ((1u << share) - 1u);
    uint64_t sl_start = 0;              // this thread's slice: its place in the input,
    uint32_t sl_len = 0, sl_readable = 0, sl_unit0 = 0;   // entries, entries up to the end of the contribution, first unit
    auto fetch_slices = [&](uint32_t p0) {
        const uint32_t q = p0 + ((uint32_t)tid >> share);
        sl_start = 0;
        sl_len = sl_readable = 0;
        if (q < P) {
            const uint32_t b = row[q], e = row[P + q];
            const uint64_t begin = off[q], end = off_end[q];
            sl_start = begin + b;
            sl_len = e > b ? e - b : 0u;                          // e < b, or a slice without end, only for
            if (sl_len > (1u << 26)) sl_len = 1u << 26;           // unsorted input: the units' numbers stay in 32 bits
            const uint64_t readable = end > sl_start ? end - sl_start : 0ull;
            sl_readable = readable < 0xffffffffull ? (uint32_t)readable : 0xffffffffu;
        }
    };
    uint32_t units = 0;                 // of the contributions fetched last
    auto number_slices = [&]() {                                  // one barrier
        const uint32_t mine = (sl_len + RED_UNIT - 1) / RED_UNIT;
        const uint32_t incl = wave_inclusive_scan_u32(member == 0 ? mine : 0u);
        if (lane == WAVE - 1) s_wave[0][wave] = incl;
        __syncthreads();
        const WaveSums sums = sum_of_waves<WAVES>(s_wave[0]);
        sl_unit0 = sums.before + incl - mine;                     // the members of a slice agree
        units = sums.total;
    };
    auto write_units = [&](uint32_t u0) {                         // units u0 .. u0 + UNITS - 1
        const uint32_t mine = (sl_len + RED_UNIT - 1) / RED_UNIT;
        uint32_t i = member;
        if (sl_unit0 + i < u0) i += (u0 - sl_unit0 - i + (1u << share) - 1u) >> share << share;
        for (; i < mine && sl_unit0 + i < u0 + UNITS; i += 1u << share) {
            const uint32_t o = i * RED_UNIT, left = sl_len - o;
            const uint64_t whole = o + RED_UNIT <= sl_readable ? 1u : 0u;
            s_unit[sl_unit0 + i - u0] =
                (sl_start + o) << 6 | whole << 5 | (left < RED_UNIT ? left : RED_UNIT);
        }
    };
    // ---- this thread's entries of a chunk ----
    using Chunk = TileEntries<ROUNDS>;
    using Streamed = TileEntries<SLIM ? 2 : ROUNDS>;
    const uint32_t nowhere = S_MAX + 32u * ((uint32_t)lane % SPARE);
    // Quad u of a chunk: the first `left` of the four entries at `from`, read with 16-byte
    // loads if all four lie inside the contribution (past the slice's end though they may be).
    auto load_entries = [&](auto& c, int u, uint64_t from, uint32_t left, bool whole, auto with_values) {
        constexpr bool VALUES = decltype(with_values)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c.slot[u][j] = 0;
            c.value[u][j] = 0.0f;
        }
        if (left == 0) return;
        if (whole) {
            const QuadAt4 i4 = *reinterpret_cast<const QuadAt4*>(idx_cat + from);
#pragma unroll
            for (int j = 0; j < 4; ++j) c.slot[u][j] = i4.v[j];
            if (VALUES) {
                const QuadAt4 v4 = *reinterpret_cast<const QuadAt4*>(val_cat + from);
#pragma unroll
                for (int j = 0; j < 4; ++j) c.value[u][j] = __uint_as_float(v4.v[j]);
            }
        } else {
            // Other loads than those, relaxed atomic ones, or the compiler makes one of what the
            // two branches begin or end with and reads a quad in two parts (373 regions of 64
            // contributions 663 us a call, 637 so; 490 of 16, 525 and 507).
            auto apart = [](const auto* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((uint32_t)j < left) {
                    c.slot[u][j] = apart(idx_cat + from + j);
                    if (VALUES) c.value[u][j] = apart(val_cat + from + j);
                }
        }
    };
    auto settle = [&](auto& c, const auto& left) {            // indices -> slots of the tile
        constexpr int QUADS = std::remove_reference_t<decltype(c)>::ROUNDS;
        c.have = 0;
#pragma unroll
        for (int u = 0; u < QUADS; ++u) c.have |= (left[u] < 4 ? (1u << left[u]) - 1u : 15u) << (4 * u);
#pragma unroll
        for (int u = 0; u < QUADS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t s = c.slot[u][j] - a;
                c.slot[u][j] = (uint32_t)j < left[u] && s < tslots ? s : nowhere;   // beyond tslots: unsorted input only
            }
    };
    auto load_chunk = [&](Chunk& c, uint32_t in_chunk, auto with_values) {
        uint32_t left[ROUNDS];
        c.last = in_chunk > (uint32_t)(ROUNDS - 1) * (BLOCK / 4) + (uint32_t)wave * (WAVE / 4);
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u) {
            const uint32_t unit = ((uint32_t)tid >> 2) + u * (BLOCK / 4);
            const uint64_t d = unit < in_chunk ? s_unit[unit] : 0ull;
            const uint32_t len = (uint32_t)d & 31u, first = 4u * ((uint32_t)tid & 3u);
            left[u] = len > first ? len - first : 0u;
            load_entries(c, u, (d >> 6) + first, left[u], ((uint32_t)d & 32u) != 0, with_values);
        }
        settle(c, left);
    };
    // The slices at hand, each read by the threads that hold it: no table of units and no
    // barrier, so a wave goes on to its next entries by itself.
    auto stream_slices = [&](auto with_values, auto&& body) {
        constexpr int QUADS = Streamed::ROUNDS;
        const uint32_t step = 4u << share;
        for (uint32_t i0 = 4u * member; i0 < sl_len; i0 += QUADS * step) {
            Streamed c;
            uint32_t left[QUADS];
            c.last = true;
#pragma unroll
            for (int u = 0; u < QUADS; ++u) {
                const uint32_t i = i0 + u * step;
                left[u] = i < sl_len ? sl_len - i : 0u;
                load_entries(c, u, sl_start + i, left[u], i + 4 <= sl_readable, with_values);
            }
            settle(c, left);
            body(c);
        }
    };
    using Yes = std::true_type;
    using No = std::false_type;
    auto for_each_chunk = [&](auto&& body) {
        for (uint32_t p0 = 0; p0 < P; p0 += BLOCK) {
            fetch_slices(p0);
            number_slices();
            for (uint32_t u0 = 0; u0 < units; u0 += UNITS) {
                write_units(u0);
                __syncthreads();
                Chunk c;
                load_chunk(c, units - u0 < UNITS ? units - u0 : UNITS, Yes{});
                body(c);
                __syncthreads();                              // s_unit and s_wave are free again
            }
            if (units == 0) __syncthreads();
        }
    };
    auto mark = [&](const auto& c) {
        constexpr int QUADS = std::remove_reference_t<decltype(c)>::ROUNDS;
#pragma unroll
        for (int u = 0; u < QUADS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (u < QUADS - 1 || c.last)
                    __hip_atomic_fetch_or(&s_bits[c.slot[u][j] >> 5], 1u << (c.slot[u][j] & 31), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // Hit slots of the tile below bitmap word w.  MAY_WRAP: there may be more than
    // 65,535 of them (a chunk's entries alone never make as many).
    auto hits_below = [&](uint32_t w, auto may_wrap) -> uint32_t {
        return (uint32_t)s_wprefix[w] + (decltype(may_wrap)::value && WORDS_MAX > 2048 && w >= s_wrap ? 65536u : 0u);
    };
    // Sums the entries and notes every entry's rank.  GENERAL: only those whose rank
    // lies in [r0, r0 + C).
    auto add = [&](auto& c, uint32_t r0, auto general) {
        constexpr int QUADS = std::remove_reference_t<decltype(c)>::ROUNDS;
        constexpr bool GENERAL = decltype(general)::value;
#pragma unroll
        for (int u = 0; u < QUADS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (u == QUADS - 1 && !c.last) break;
                const uint32_t s = c.slot[u][j];
                const uint32_t below = s_bits[s >> 5] & ((1u << (s & 31)) - 1u);
                uint32_t rank = hits_below(s >> 5, general) + (uint32_t)__popc(below);
                if (GENERAL) rank = s < S_MAX ? rank - r0 : ACC;
                else c.slot[u][j] = rank << SLOT_BITS | s;
                float x = c.value[u][j];
                asm volatile("" : "+v"(x));      // widened here, not where it was loaded: registers
                if (!GENERAL || rank < ACC)
                    __hip_atomic_fetch_add(&s_sum[rank], (double)x, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            }
    };

    // SLIM: marks the entries and notes those whose slot was marked before them.
    auto mark_again = [&](const Chunk& c, uint32_t& again) {
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u) {
            if (u == ROUNDS - 1 && !c.last) break;
            uint32_t was[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                was[j] = __hip_atomic_fetch_or(&s_bits[c.slot[u][j] >> 5], 1u << (c.slot[u][j] & 31), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int j = 0; j < 4; ++j) again |= (was[j] >> (c.slot[u][j] & 31) & 1u) << (4 * u + j);
        }
        again &= c.have;
    };
    // SLIM: ranks the entries and leaves the slots' sums, as floats, where the accumulators are.
    auto sum_slim = [&](Chunk& c, uint32_t again, uint32_t at, uint32_t listed) {
        uint32_t* const s_val = reinterpret_cast<uint32_t*>(s_sum);
        const uint32_t spare = C + (uint32_t)lane % SPARE;
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (u == ROUNDS - 1 && !c.last) break;
                uint32_t s = c.slot[u][j];
                asm volatile("" : "+v"(s));      // addresses are formed here, not kept from the marking: registers
                const uint32_t below = s_bits[s >> 5] & ((1u << (s & 31)) - 1u);
                const uint32_t rank = (uint32_t)s_wprefix[s >> 5] + (uint32_t)__popc(below);
                c.slot[u][j] = rank << SLOT_BITS | s;
                s_val[again >> (4 * u + j) & 1u ? spare : rank] = __float_as_uint(c.value[u][j]);
            }
        if (listed == 0) return;
        __syncthreads();                              // ranks are known: the list takes the place of what told them
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (again >> (4 * u + j) & 1u)
                    s_list[at++] = (uint64_t)__float_as_uint(c.value[u][j]) << 32 | c.slot[u][j] >> SLOT_BITS;
        __syncthreads();
        // The first of a slot's entries to get here starts the sum in its own place and says in
        // the slot's value where that is; the others add to it; the first rounds it.
        constexpr int TURNS = (int)((LIST + BLOCK - 1) / BLOCK);
        uint32_t rank[TURNS], first = 0;
#pragma unroll
        for (int t = 0; t < TURNS; ++t) {
            rank[t] = 0;
            const uint32_t i = (uint32_t)tid + t * BLOCK;
            if (i < listed) {
                const uint64_t e = s_list[i];
                const uint32_t r = rank[t] = (uint32_t)e, bit = 1u << (r & 31);
                if (!(__hip_atomic_fetch_or(&s_more[r >> 5], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit)) {
                    first |= 1u << t;
                    const double sum = (double)__uint_as_float(s_val[r]) + (double)__uint_as_float((uint32_t)(e >> 32));
                    s_list[i] = (uint64_t)__double_as_longlong(sum);
                    s_val[r] = i;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < TURNS; ++t) {
            const uint32_t i = (uint32_t)tid + t * BLOCK;
            if (i < listed && !(first >> t & 1u))
                __hip_atomic_fetch_add(reinterpret_cast<double*>(s_list) + s_val[rank[t]],
                                       (double)__uint_as_float((uint32_t)(s_list[i] >> 32)), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < TURNS; ++t)
            if (first >> t & 1u)
                s_val[rank[t]] = __float_as_uint((float)__longlong_as_double((long long)s_list[(uint32_t)tid + t * BLOCK]));
    };

    // Both waves of the chained scan; every thread gets the count of all tiles
    // before this one.  What the two waves look at first is asked for early
    // (look_back) and, as a rule, there by the time it is needed.
    const uint32_t group = tile / SCAN_GROUP;
    if constexpr (PLACED) {
        // the count before this tile, as reduce_count_kernel found it
        const uint32_t* counts = (const uint32_t*)(region_ws + SCAN_HEADER_BYTES);
        uint32_t sum = 0;
        for (uint32_t t = tid; t < tile; t += BLOCK) sum += counts[t];
        sum = wave_sum(sum);
        if (lane == 0) s_placed[wave] = sum;
    }
    uint64_t seen = 0;
    auto look_back = [&]() {
        if (PLACED) return;
        seen = 0;
        if (wave == 0 && (uint32_t)lane < tile % SCAN_GROUP) seen = desc_load(tile_desc + group * SCAN_GROUP + lane);
        if (wave == 1 && (uint32_t)lane < group) seen = desc_load(group_desc + (group - 1 - lane));
    };
    auto place_tile = [&](uint32_t count) -> uint32_t {
        if constexpr (PLACED) {
            __syncthreads();
            return sum_of_waves<WAVES>(s_placed).total;
        }
        if (wave == 0) {
            const uint32_t before = scan_within_group(hdr, tile_desc, group_desc, tile, count, seen);
            if (lane == 0) s_before[0] = before;
        } else if (wave == 1) {
            const uint32_t before = scan_across_groups(hdr, group_desc, group, seen);
            if (lane == 0) s_before[1] = before;
        }
        __syncthreads();
        const uint32_t before = uniform(s_before[0] + s_before[1]);
        if (tid == 0 && group != 0 && tile % SCAN_GROUP == SCAN_GROUP - 1)
            scan_close_group(group_desc, group, before + count);
        return before;
    };
    uint32_t distinct = 0, exclusive = 0;

    auto finish = [&]() {
        if (tile != r.ntiles - 1 || tid != 0) return;
        const uint64_t total = (uint64_t)exclusive + distinct;
        const bool failed =
            !PLACED && __hip_atomic_load(&hdr->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        nnz[0] = failed ? ~0ull : (total < capacity ? total : capacity);
        nnz[1] = failed ? ~0ull : total;
    };
    if constexpr (DENSE) {
        // ---- densely hit region: accumulator = slot, one sweep ----
        for_each_chunk([&](Chunk& c) {
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (c.slot[u][j] < S_MAX)
                        __hip_atomic_fetch_add(&s_sum[c.slot[u][j]], (double)c.value[u][j], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
            mark(c);
        });
        distinct = bitmap_prefix<BLOCK, WORDS_MAX>(s_bits, s_wprefix, words, s_wave[1], &s_wrap);
        if (!PLACED && tid == 0) scan_publish_early(tile_desc, tile, distinct);
        look_back();
        // The sums leave LDS, and the hit slots' come back in output order with their indices, while
        // the counts of the tiles before this one arrive; whole lines go out.  (Each thread storing the
        // hits of four slots where they belong, once the place was known, took 6,700 clocks of a
        // tile's 52,700 to wait and 7,700 to store: 48 regions of 256 colliding contributions 137 us a
        // call, so 131; 8 of 16 that hit 0.8 of 2 M slots 108 and 95; a lone one 13.8 and 13.1.)
        constexpr int PER = (int)(C / BLOCK);
        static_assert(C % BLOCK == 0, "a thread's slots");
        float x[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) x[i] = (float)s_sum[tid + i * BLOCK];
        uint32_t* const s_idx = reinterpret_cast<uint32_t*>(s_sum);
        float* const s_val = reinterpret_cast<float*>(s_idx + C);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t slot = (uint32_t)tid + i * BLOCK;
            if (slot < tslots) {
                if (dense) dense[slot] = x[i];
                const uint32_t word = s_bits[slot >> 5];
                if (word >> (slot & 31) & 1u) {
                    const uint32_t rank = s_wprefix[slot >> 5] + (uint32_t)__popc(word & ((1u << (slot & 31)) - 1u));
                    s_idx[rank] = a + slot;
                    s_val[rank] = x[i];
                }
            }
        }
        exclusive = place_tile(distinct);                 // a barrier
        const uint64_t room = capacity > exclusive ? capacity - exclusive : 0;
        const uint32_t out = distinct < room ? distinct : (uint32_t)room;
        uint32_t* const to_idx = idx_out + exclusive;
        float* const to_val = val_out + exclusive;
        for (uint32_t k = tid; k < out; k += BLOCK) {
            to_idx[k] = s_idx[k];
            to_val[k] = s_val[k];
        }
    } else {
        // ---- sparsely hit region: mark, rank, then sum into accumulator [rank] ----
        uint32_t* s_idx = reinterpret_cast<uint32_t*>(s_sum);   // takes over once the sums are read
        auto rank_tile = [&]() {
            distinct = bitmap_prefix<BLOCK, WORDS_MAX>(s_bits, s_wprefix, words, s_wave[1], &s_wrap);
            // the count is known before the sums: publish it now, wait for the others later
            if (!PLACED && tid == 0) scan_publish_early(tile_desc, tile, distinct);
        };
        // The sums of ranks r0 .. r0 + in_round - 1 leave LDS, the indices take their
        // place, and both go out in output order; the wait for the tiles before this
        // one lies in between.
        auto write_out = [&](uint32_t r0, uint32_t in_round, const auto* sums, auto&& put_indices) {
            constexpr int PER = (int)(((sizeof(*sums) == sizeof(float) ? C : ACC) + BLOCK - 1) / BLOCK);
            float x[PER];
            uint32_t k0 = (uint32_t)tid;
            asm volatile("" : "+v"(k0));             // addresses are formed here, not kept from before
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t k = k0 + i * BLOCK;
                x[i] = k < in_round ? (float)sums[k] + 0.0f : 0.0f;     // a lone -0 becomes +0, as 0 + -0 does
            }
            __syncthreads();
            put_indices();
            if (r0 == 0) exclusive = place_tile(distinct);
            else __syncthreads();
            const uint64_t first = (uint64_t)exclusive + r0, room = capacity > first ? capacity - first : 0;
            const uint32_t out = in_round < room ? in_round : (uint32_t)room;
            uint32_t* const to_idx = idx_out + first;
            float* const to_val = val_out + first;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t k = k0 + i * BLOCK;
                if (k < out) {
                    to_idx[k] = s_idx[k];
                    to_val[k] = x[i];
                }
                if (dense && k < in_round) dense[s_idx[k] - a] = x[i];
            }
        };
        fetch_slices(0);
        number_slices();
        // the units from u0 on, a chunk at a time
        auto chunks = [&](uint32_t u0, auto with_values, auto&& body) {
            for (; u0 < units; u0 += UNITS) {
                __syncthreads();                              // s_unit has been read
                write_units(u0);
                __syncthreads();
                Chunk c;
                load_chunk(c, units - u0 < UNITS ? units - u0 : UNITS, with_values);
                body(c);
            }
        };
        const bool by_chunk = P <= (uint32_t)BLOCK && (units <= EXCESS * UNITS || share < 3);
        if (by_chunk && (KEEP || units <= UNITS)) {
            // The first chunk, which is all there is as a rule, stays in registers from the
            // marking to the writing of the indices; what lies beyond it is read for each.
            write_units(0);
            __syncthreads();
            Chunk mine;
            load_chunk(mine, units < UNITS ? units : UNITS, Yes{});
            if constexpr (SLIM) {
                uint32_t again = 0, at = 0;                  // listed entries, the first one's place in the list
                mark_again(mine, again);
                {
                    const uint32_t n = (uint32_t)__popc(again), incl = wave_inclusive_scan_u32(n);
                    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
                    if (total) {
                        uint32_t base = 0;
                        if (lane == 0) base = __hip_atomic_fetch_add(&s_again, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        at = uniform(base) + incl - n;
                    }
                }
                __syncthreads();
                rank_tile();
                const uint32_t listed = uniform(s_again);
                if (distinct <= C && listed <= LIST) {
                    sum_slim(mine, again, at, listed);
                    __syncthreads();
                    look_back();
                    write_out(0, distinct, reinterpret_cast<const float*>(s_sum), [&]() {
#pragma unroll
                        for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
                            for (int j = 0; j < 4; ++j)       // every hit of a slot writes the same
                                if (u < ROUNDS - 1 || mine.last)
                                    s_idx[mine.slot[u][j] >> SLOT_BITS] = a + (mine.slot[u][j] & SLOT_MASK);
                    });
                    finish();
                    return;
                }
            } else {
                mark(mine);
                if (KEEP) chunks(UNITS, No{}, mark);
                __syncthreads();
                rank_tile();
            }
            if (!SLIM && distinct <= C) {
                add(mine, 0, No{});
                if (KEEP) chunks(UNITS, Yes{}, [&](Chunk& c) { add(c, 0, No{}); });
                __syncthreads();
                look_back();
                write_out(0, distinct, s_sum, [&]() {
                    if (KEEP && units > UNITS) {
                        for (uint32_t w = tid; w < words; w += BLOCK) {
                            uint32_t bits = s_bits[w], rank = hits_below(w, No{});
                            for (; bits; bits &= bits - 1, ++rank) s_idx[rank] = a + w * 32u + (uint32_t)(__ffs(bits) - 1);
                        }
                        return;
                    }
#pragma unroll
                    for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j)           // every hit of a slot writes the same
                            if (u < ROUNDS - 1 || mine.last)
                                s_idx[mine.slot[u][j] >> SLOT_BITS] = a + (mine.slot[u][j] & SLOT_MASK);
                });
                finish();
                return;
            }
        } else {
            if (!KEEP && by_chunk) {
                chunks(0, No{}, mark);
            } else {
                for (uint32_t p0 = 0; p0 < P; p0 += BLOCK) {
                    if (p0) fetch_slices(p0);
                    stream_slices(No{}, mark);
                }
            }
            __syncthreads();
            rank_tile();
        }
        {
            // More entries than registers hold, or more hit slots than accumulators: the tile
            // is cut, at words of the bitmap, into windows of at most C hit slots, and every
            // window's entries are read, summed and written in turn.  Window k ends in the word
            // that holds hit slot (k + 1) distinct / windows, up to 31 hit slots early.
            const uint32_t windows = distinct > ACC ? (distinct + ACC - 33) / (ACC - 32) : 1u;
            if (SLIM)
                for (uint32_t i = tid; i < ACC; i += BLOCK) s_sum[i] = 0.0;
            for (uint32_t w = tid; w < words; w += BLOCK) {
                const uint32_t here = hits_below(w, Yes{}), next = w + 1 < words ? hits_below(w + 1, Yes{}) : distinct;
                for (uint32_t k = 1; k < windows; ++k) {
                    const uint32_t target = k * distinct / windows;
                    if (here <= target && target < next) {        // one word for every k
                        s_cut[k] = w;
                        s_cut_rank[k] = here;
                    }
                }
            }
            if (tid == 0) {
                s_cut[0] = s_cut_rank[0] = 0;
                s_cut[windows] = words;
                s_cut_rank[windows] = distinct;
            }
            __syncthreads();
            if (SLIM) fetch_slices(0);                       // read again, not kept in registers until here
            // A slice is sorted, so a window's entries are a piece of it, whose end is searched
            // from where it would lie if the slice were spread as the tile's hits are: by the
            // threads that hold the slice, one window each, where LDS has room for the ends,
            // else when the window's turn comes.  (With more contributions than threads every
            // window reads all entries; those of other windows fall out by their rank.)
            const uint32_t slice = (uint32_t)tid >> share;
            const uint64_t whole_start = sl_start;
            const uint32_t whole_len = sl_len, whole_readable = sl_readable;
            auto window_end = [&](uint32_t k, uint32_t from) -> uint32_t {
                if (k == windows || whole_len == 0) return whole_len;
                const uint64_t guess = whole_start + (uint64_t)whole_len * s_cut_rank[k] / distinct;
                return (uint32_t)(lower_bound_near(idx_cat, whole_start + from, whole_start + whole_len,
                                                   a + s_cut[k] * 32u, guess) - whole_start);
            };
            uint32_t* const s_end = reinterpret_cast<uint32_t*>(s_unit);
            const bool whole = !KEEP && by_chunk && windows <= 1;
            const bool ends_kept = P <= (uint32_t)BLOCK && P * windows <= 2 * UNITS && !whole;
            if (ends_kept) {
                if (slice < P)
                    for (uint32_t k = member + 1; k <= windows; k += 1u << share) s_end[slice * windows + k - 1] = window_end(k, 0);
                __syncthreads();
            }
            uint32_t begin = 0;
            for (uint32_t k = 0; k < windows; ++k) {
                const uint32_t w0 = uniform(s_cut[k]), w1 = uniform(s_cut[k + 1]);
                const uint32_t r0 = uniform(s_cut_rank[k]), r1 = uniform(s_cut_rank[k + 1]);
                auto sum = [&](auto& c) { add(c, r0, Yes{}); };
                if (whole) {
                    chunks(0, Yes{}, sum);
                } else if (P <= (uint32_t)BLOCK) {
                    const uint32_t end = !ends_kept ? window_end(k + 1, begin) : slice < P ? s_end[slice * windows + k] : 0u;
                    sl_start = whole_start + begin;
                    sl_len = end > begin ? end - begin : 0u;
                    sl_readable = whole_readable > begin ? whole_readable - begin : 0u;
                    begin = end > begin ? end : begin;
                    stream_slices(Yes{}, sum);
                } else {
                    for (uint32_t p0 = 0; p0 < P; p0 += BLOCK) {
                        fetch_slices(p0);
                        stream_slices(Yes{}, sum);
                    }
                }
                __syncthreads();
                if (k == 0) look_back();
                write_out(r0, r1 - r0, s_sum, [&]() {
                    for (uint32_t w = w0 + tid; w < w1; w += BLOCK) {
                        uint32_t bits = s_bits[w], rank = hits_below(w, Yes{}) - r0;
                        for (; bits; bits &= bits - 1, ++rank)
                            if (rank < ACC) s_idx[rank] = a + w * 32u + (uint32_t)(__ffs(bits) - 1);
                    }
                });
                if (k + 1 == windows) break;
                __syncthreads();                              // sums and indices fully read
                for (uint32_t i = tid; i < ACC; i += BLOCK) s_sum[i] = 0.0;
                __syncthreads();
            }
        }
    }
    finish();
}

// traffic_only: the measurement entry point okt_stream_gather - the same tiles and
// the same slice table, but the tile kernel is replaced by one that only moves
// the entries (d_nnz_out and d_dense are not used then).
int reduce_launch(const uint32_t* d_idx_cat, const float* d_val_cat,
                  const uint64_t* d_seg_begin, const uint64_t* d_seg_end,
                  uint32_t seg_stride, const uint32_t* d_lo_hi, uint32_t lo,
                  uint32_t hi, uint32_t B, uint32_t P, uint32_t max_width,
                  uint32_t* d_idx_out, float* d_val_out, uint64_t capacity,
                  uint64_t* d_nnz_out, float* d_dense, void* d_ws, size_t ws_bytes,
                  hipStream_t s, bool traffic_only) {
    if (!d_idx_cat || !d_val_cat || !d_seg_begin || !d_seg_end || (!d_nnz_out && !traffic_only))
        return OKT_ERR_INVALID_ARG;
    if (P == 0 || P > 65535 || B == 0 || B > 65535) return OKT_ERR_INVALID_ARG;
    if (capacity > 0 && (!d_idx_out || !d_val_out)) return OKT_ERR_INVALID_ARG;
    if (!aligned(d_idx_cat, 4) || !aligned(d_val_cat, 4) || !aligned(d_seg_begin, 8) || !aligned(d_seg_end, 8) ||
        !aligned(d_nnz_out, 8) || !aligned(d_idx_out, 4) || !aligned(d_val_out, 4) ||
        !aligned(d_dense, 4) || !aligned(d_lo_hi, 4))
        return OKT_ERR_INVALID_ARG;
    // the caller's bound on the size of the union doubles as the density estimate
    const size_t least = reduce_ws_bytes_region(max_width, P, reduce_least_shape(max_width, capacity, P).slots);
    if (least > 0xffffffffull) return OKT_ERR_INVALID_ARG;
    if (!d_ws || !aligned(d_ws, 256) || ws_bytes < least * B) return OKT_ERR_WORKSPACE;
    const ReduceShape shape = reduce_shape(B, max_width, capacity, P, (uint64_t)device_cus(), ws_bytes);
    // (and contributions whose ends a workgroup finds side by side)
    const bool placed = !traffic_only && P <= PLACED_P && reduce_counts_first(shape, B, max_width, device_cus());
    const uint32_t slots = shape.slots;
    const size_t region_bytes = reduce_ws_bytes_region(max_width, P, slots);
    uint64_t tiles = reduce_tiles(max_width, slots);
    if (tiles == 0) tiles = 1;
    const uint32_t table_offset = (uint32_t)(64 + 8 * (tiles + (tiles + 63) / 64));
    const uint64_t cells = (tiles + 1) * P;
    if (placed) {
        auto* count = shape.kind == RED_DENSE    ? reduce_count_kernel<ReduceNarrow::C_DENSE>
                      : shape.kind == RED_RANKED ? reduce_count_kernel<ReduceNarrow::S_RANKED>
                                                 : reduce_count_kernel<ReduceNarrow::S_SPARSE>;
        hipLaunchKernelGGL(count, dim3((unsigned)tiles, B), dim3(COUNT_BLOCK), 0, s, d_idx_cat, d_seg_begin,
                           d_seg_end, seg_stride, d_lo_hi, lo, hi, P, max_width, slots, (char*)d_ws,
                           (uint32_t)region_bytes, table_offset);
    } else if (cells * B <= 4096) {
        // few cells: a wave each
        hipLaunchKernelGGL(reduce_slices_wave_kernel, dim3((unsigned)((cells + 3) / 4), B),
                           dim3(256), 0, s, d_idx_cat, d_seg_begin, d_seg_end, seg_stride, d_lo_hi,
                           lo, hi, P, max_width, slots, (char*)d_ws, (uint32_t)region_bytes,
                           table_offset, spin_limit_setting());
    } else {
        const uint32_t chain = reduce_chain(cells * B);
        const bool teams = reduce_by_teams(shape, max_width, capacity, P);
        const uint64_t threads = teams ? P * (tiles / chain + 1) * TEAM : cells;
        const dim3 grid((unsigned)(threads < 4096 * 256 ? (threads + 255) / 256 : 4096), B);
        if (teams)
            hipLaunchKernelGGL(reduce_slices_team_kernel, grid, dim3(256), 0, s, d_idx_cat, d_seg_begin, d_seg_end,
                               seg_stride, d_lo_hi, lo, hi, P, max_width, slots, (char*)d_ws, (uint32_t)region_bytes,
                               table_offset, spin_limit_setting(), chain);
        else
            hipLaunchKernelGGL(reduce_slices_kernel, grid, dim3(256), 0, s, d_idx_cat, d_seg_begin, d_seg_end,
                               seg_stride, d_lo_hi, lo, hi, P, max_width, slots, (char*)d_ws, (uint32_t)region_bytes,
                               table_offset, spin_limit_setting());
    }
    if (traffic_only) {
        timing_before(s);
        hipLaunchKernelGGL(gather_ceiling_kernel, dim3((unsigned)tiles, B), dim3(512), 0, s,
                           d_idx_cat, d_val_cat, d_seg_begin, seg_stride, d_lo_hi, P, max_width, slots,
                           d_idx_out, d_val_out, capacity, (const char*)d_ws, (uint32_t)region_bytes,
                           table_offset);
        timing_after(s);
        return launch_status();
    }
    timing_before(s);
    auto launch = [&](auto* tile_kernel, uint32_t block) {
        hipLaunchKernelGGL(tile_kernel, dim3((unsigned)tiles, B), dim3(block), 0, s, d_idx_cat, d_val_cat,
                           d_seg_begin, d_seg_end, seg_stride, d_lo_hi, lo, hi, P, max_width, slots,
                           d_idx_out, d_val_out, capacity, d_nnz_out, d_dense, (char*)d_ws,
                           (uint32_t)region_bytes, table_offset);
    };
    if (placed) {
        using F = ReduceNarrow;
        if (shape.kind == RED_DENSE) launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_DENSE, F::C_DENSE, true>, F::BLOCK);
        else if (shape.kind == RED_RANKED) launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_RANKED, F::S_RANKED, true>, F::BLOCK);
        else launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_SPARSE, F::S_SPARSE, true>, F::BLOCK);
        timing_after(s);
        return launch_status();
    }
    if (shape.form == RED_SLIM) {
        using F = ReduceSlim;
        if (shape.kind == RED_RANKED) launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_RANKED, F::S_RANKED, false, true>, F::BLOCK);
        else launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_SPARSE, F::S_SPARSE, false, true>, F::BLOCK);
        timing_after(s);
        return launch_status();
    }
    auto launch_form = [&](auto form) {
        using F = decltype(form);
        if constexpr (!std::is_same<F, ReduceWide4>::value)      // its dense tiles hold five units as well
            if (shape.kind == RED_DENSE) return launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_DENSE, F::C_DENSE>, F::BLOCK);
        if (shape.kind == RED_RANKED) launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_RANKED, F::S_RANKED>, F::BLOCK);
        else launch(reduce_tile_kernel<F::BLOCK, F::ROUNDS, F::C_SPARSE, F::S_SPARSE>, F::BLOCK);
    };
    if (shape.form == RED_WIDE5 || (shape.form == RED_WIDE4 && shape.kind == RED_DENSE)) launch_form(ReduceWide5{});
    else if (shape.form == RED_WIDE4) launch_form(ReduceWide4{});
    else launch_form(ReduceNarrow{});
    timing_after(s);
    return launch_status();
}

}  // namespace okt

extern "C" int okt_sparse_reduce(const uint32_t* d_idx_cat, const float* d_val_cat,
                                 const uint64_t* d_chunk_off, uint32_t P, uint32_t lo, uint32_t hi,
                                 uint32_t* d_idx_out, float* d_val_out, uint64_t capacity,
                                 uint64_t* d_nnz_out, float* d_dense_out_or_null, void* d_ws,
                                 size_t ws_bytes, void* stream) {
    if (lo > hi) return OKT_ERR_INVALID_ARG;
    if (!d_chunk_off) return OKT_ERR_INVALID_ARG;
    // contribution p = [off[p], off[p+1]): the same vector is the begins and, one on, the ends
    return okt::reduce_launch(d_idx_cat, d_val_cat, d_chunk_off, d_chunk_off + 1, P + 1, nullptr,
                              lo, hi, 1, P, hi - lo,
                              d_idx_out, d_val_out, capacity, d_nnz_out, d_dense_out_or_null,
                              d_ws, ws_bytes, (hipStream_t)stream, false);
}

extern "C" int okt_sparse_reduce_batch(const uint32_t* d_idx_cat, const float* d_val_cat,
                                       const uint64_t* d_chunk_off, const uint32_t* d_lo_hi,
                                       uint32_t B, uint32_t P, uint32_t max_width,
                                       uint32_t* d_idx_out, float* d_val_out, uint64_t capacity,
                                       uint64_t* d_nnz_out, float* d_dense_out_or_null,
                                       void* d_ws, size_t ws_bytes, void* stream) {
    if (!d_lo_hi || !d_chunk_off) return OKT_ERR_INVALID_ARG;
    return okt::reduce_launch(d_idx_cat, d_val_cat, d_chunk_off, d_chunk_off + 1, P + 1, d_lo_hi,
                              0, 0, B, P, max_width,
                              d_idx_out, d_val_out, capacity, d_nnz_out, d_dense_out_or_null,
                              d_ws, ws_bytes, (hipStream_t)stream, false);
}

extern "C" int okt_stream_gather(const uint32_t* d_idx_cat, const float* d_val_cat,
                                 const uint64_t* d_chunk_off, const uint32_t* d_lo_hi, uint32_t B,
                                 uint32_t P, uint32_t max_width, uint32_t* d_idx_out,
                                 float* d_val_out, uint64_t capacity, void* d_ws, size_t ws_bytes,
                                 void* stream) {
    if (!d_lo_hi || !d_chunk_off || !d_idx_out || !d_val_out) return OKT_ERR_INVALID_ARG;
    return okt::reduce_launch(d_idx_cat, d_val_cat, d_chunk_off, d_chunk_off + 1, P + 1, d_lo_hi,
                              0, 0, B, P, max_width, d_idx_out, d_val_out, capacity, nullptr, nullptr,
                              d_ws, ws_bytes, (hipStream_t)stream, true);
}

extern "C" int okt_sparse_reduce_segments(const uint32_t* d_idx_cat, const float* d_val_cat,
                                          const uint64_t* d_seg_begin, const uint64_t* d_seg_end,
                                          uint32_t P, uint32_t lo, uint32_t hi,
                                          uint32_t* d_idx_out, float* d_val_out, uint64_t capacity,
                                          uint64_t* d_nnz_out, float* d_dense_out_or_null,
                                          void* d_ws, size_t ws_bytes, void* stream) {
    if (lo > hi) return OKT_ERR_INVALID_ARG;
    return okt::reduce_launch(d_idx_cat, d_val_cat, d_seg_begin, d_seg_end, P, nullptr, lo, hi, 1, P,
                              hi - lo, d_idx_out, d_val_out, capacity, d_nnz_out,
                              d_dense_out_or_null, d_ws, ws_bytes, (hipStream_t)stream, false);
}
