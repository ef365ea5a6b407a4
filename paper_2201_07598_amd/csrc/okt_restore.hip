// okt_index_intersect_restore / okt_index_intersect_zero: indexes = local top-k
// indexes intersected with the global top-k indexes (Algorithm 1, line 14), and
// the residual update eps = acc - acc(indexes) (Algorithm 2, line 6), either
// completed on a residual whose locally selected entries were all zeroed by the
// select (the entries that did not reach the global top-k are put back) or
// applied to the untouched accumulator (the entries of the intersection are
// zeroed).
//
// Work proportional to the local list (about k entries), far below the dense
// passes of an iteration, and all of it latency.  A workgroup takes a tile of
// consecutive local entries and looks them up in the global list (tile_members).
// A second launch writes the matched indices in ascending order: the first left which
// of a tile's entries matched (a bit each) and how many, and every workgroup adds up
// the counts of the tiles before its own.  A call whose workspace has no room for the bits,
// or that writes over its inputs, finds a tile's place with a scan across workgroups instead.
#include "okt_device.h"
#include "okt_search.h"
#include "okt_select_kernel.h"
#include "okt_sizes.h"

namespace okt {

struct RestoreMemory {
    union {
        struct { uint32_t key[RST_TABLE]; uint8_t hit[RST_TABLE]; } table;
        uint32_t window[RST_WINDOW];
    };
    uint32_t below[2][RST_WAVES];
};
template <int ROWS>                                  // entries of a thread
struct Membership {
    uint32_t idx[ROWS];
    bool active[ROWS], member[ROWS];
};
__device__ __forceinline__ uint32_t entries_of(const uint64_t* d_nnz, uint32_t most) {
    const uint64_t have = *d_nnz;
    return have < most ? (uint32_t)have : most;
}
template <int ROWS>
__device__ __forceinline__ uint32_t tiles_of(uint32_t entries) {
    constexpr uint32_t TILE = ROWS * RST_BLOCK;
    return entries / TILE + (entries % TILE ? 1u : 0u);
}

// at[c] + the number of s[at[c] .. top[c]) that are below x[c], for the entries of a thread.
// No branch: every step of every search is one read, and a thread's reads of a step are
// under way together.  `most`: no search is over more elements (uniform).
template <int ROWS>
__device__ __forceinline__ void lower_bounds(const uint32_t* s, uint32_t (&at)[ROWS], const uint32_t (&top)[ROWS],
                                             const uint32_t (&x)[ROWS], uint32_t most) {
    for (uint32_t half = most ? 1u << (31 - __clz(most)) : 0u; half; half >>= 1) {
        uint32_t v[ROWS];
#pragma unroll
        for (int c = 0; c < ROWS; ++c) v[c] = s[at[c] + half <= top[c] ? at[c] + half - 1 : 0u];
#pragma unroll
        for (int c = 0; c < ROWS; ++c)
            if (at[c] + half <= top[c] && v[c] < x[c]) at[c] += half;
    }
}

// Which of the tile's entries [base, end), base < end, are in the global list: a chain of
// as few trips to memory and LDS as it can do with, as nothing else is left to save here.
// Both lists ascend, so all that the tile can match lies in one part of the global list.
// RST_SAMPLES places spread over the list are asked for together with the entries;
// how many of them lie below the first entry and the last says where that part begins
// and ends, to within their distance.  A part of up to RST_WINDOW elements is read
// at once, while the tile's entries go to a hash table in LDS, and every element is
// looked up there.  Of a longer one every s-th element is staged in LDS and searched
// for every entry, and what lies between two is read and compared.
// What it measured, whole call: 180,000 layered entries in a list of 350,000 15.9 us, 10,500
// in 14,000 9.8 us.  With the ends found by a 64-ary search, a binary search in LDS (or in
// memory, of longer parts) for every entry, and tickets and a scan across workgroups
// instead of the second launch: 30.2 and 13.5 us.  A workgroup alone on its compute unit waits out
// every LDS access (ten steps of a binary search 2.5 us), so sixteen waves share the
// work of a tile (four waves, four entries a thread: 13.6 and 8.4 us for the first launch,
// 11.9 and 6.2 so), and the table is eight times the entries (four times: 6.8).
template <int ROWS>
__device__ __forceinline__ Membership<ROWS> tile_members(const uint32_t* __restrict__ local_idx, uint32_t base,
                                                         uint32_t end, const uint32_t* __restrict__ global_idx,
                                                         uint32_t ng, RestoreMemory& lds) {
    constexpr uint32_t EMPTY = ~0u;                  // no index: vectors are shorter than 2^32
    static_assert(4 * ROWS * RST_BLOCK <= RST_TABLE, "a quarter of the table");
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    Membership<ROWS> m;
    constexpr int PER = RST_SAMPLES / RST_BLOCK;
    const uint32_t apart = ng / RST_SAMPLES + 1;
    uint32_t sample[PER];
    uint64_t place[PER];
#pragma unroll
    for (int c = 0; c < ROWS; ++c) {
        const uint32_t j = base + c * RST_BLOCK + tid;
        m.active[c] = j < end;
        m.idx[c] = m.active[c] ? local_idx[j] : EMPTY;
        m.member[c] = false;
    }
    const uint32_t first = local_idx[base], last = local_idx[end - 1];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        place[u] = (uint64_t)apart * (u * RST_BLOCK + tid);
        sample[u] = place[u] < ng ? global_idx[place[u]] : 0u;
    }
    for (uint32_t i = tid; i < RST_TABLE / 4; i += RST_BLOCK) {
        reinterpret_cast<uint4*>(lds.table.key)[i] = uint4{EMPTY, EMPTY, EMPTY, EMPTY};
        reinterpret_cast<uint32_t*>(lds.table.hit)[i] = 0;
    }
    uint32_t below[2] = {0, 0};                      // places whose element is below the first entry; not above the last
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        below[0] += (uint32_t)__popcll(__ballot(place[u] < ng && sample[u] < first));
        below[1] += (uint32_t)__popcll(__ballot(place[u] < ng && sample[u] <= last));
    }
    if (lane < 2) lds.below[lane][wave] = below[lane];
    __syncthreads();
    below[0] = below[1] = 0;
#pragma unroll
    for (int w = 0; w < RST_WAVES; ++w) {
        below[0] += lds.below[0][w];
        below[1] += lds.below[1][w];
    }
    const uint32_t w0 = below[0] ? (below[0] - 1) * apart + 1 : 0u;              // all before it are below the first entry
    const uint64_t upto = (uint64_t)below[1] * apart;                           // all from it on are above the last
    const uint32_t w1 = upto < ng ? (uint32_t)upto : ng;
    const uint32_t part = w1 > w0 ? w1 - w0 : 0u;    // nothing: only if the lists do not ascend, or match nowhere
    if (part == 0) return m;
    if (part <= RST_WINDOW) {
        constexpr int FLIGHT = RST_WINDOW / RST_BLOCK;
        uint32_t v[FLIGHT];
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) {
            const uint32_t i = u * RST_BLOCK + tid;
            v[u] = i < part ? global_idx[w0 + i] : EMPTY;
        }
        auto slot_of = [](uint32_t key) { return key * 2654435769u >> (32 - RST_TABLE_BITS); };
        uint32_t slot[ROWS];
#pragma unroll
        for (int c = 0; c < ROWS; ++c) {
            slot[c] = slot_of(m.idx[c]);
            if (m.active[c])
                while (true) {                       // a quarter of the table is filled at most, so it ends
                    const uint32_t found = atomicCAS(&lds.table.key[slot[c]], EMPTY, m.idx[c]);
                    if (found == EMPTY || found == m.idx[c]) break;
                    slot[c] = (slot[c] + 1) % RST_TABLE;
                }
        }
        __syncthreads();
        // four look-ups of a thread at a time, step by step together
        constexpr int TOGETHER = 4;
#pragma unroll
        for (int u0 = 0; u0 < FLIGHT; u0 += TOGETHER)
            if (u0 * RST_BLOCK < part) {
                uint32_t at[TOGETHER], key[TOGETHER];
                bool busy = false;
#pragma unroll
                for (int u = 0; u < TOGETHER; ++u) at[u] = slot_of(v[u0 + u]);
                do {
#pragma unroll
                    for (int u = 0; u < TOGETHER; ++u) key[u] = lds.table.key[at[u]];
                    busy = false;
#pragma unroll
                    for (int u = 0; u < TOGETHER; ++u) {
                        const bool on = key[u] != EMPTY && key[u] != v[u0 + u] && v[u0 + u] != EMPTY;
                        at[u] = on ? (at[u] + 1) % RST_TABLE : at[u];
                        busy |= on;
                    }
                } while (busy);
#pragma unroll
                for (int u = 0; u < TOGETHER; ++u)
                    if (key[u] == v[u0 + u] && key[u] != EMPTY) lds.table.hit[at[u]] = 1;
            }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < ROWS; ++c) m.member[c] = m.active[c] && lds.table.hit[slot[c]] != 0;
        return m;
    }
    // ---- a long part ----
    __syncthreads();                                 // the table has been cleared: its place is taken
    const SpreadSample sample_of_part = spread_sample(part, RST_WINDOW);
    const uint32_t step = sample_of_part.step, staged = sample_of_part.count;
    {
        constexpr int FLIGHT = RST_WINDOW / RST_BLOCK;
        uint32_t v[FLIGHT];
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) {
            const uint32_t i = u * RST_BLOCK + tid;
            v[u] = global_idx[w0 + (i < staged ? i : 0u) * step];
        }
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) lds.window[u * RST_BLOCK + tid] = v[u];
    }
    __syncthreads();
    uint32_t at[ROWS], top[ROWS], lo[ROWS], hi[ROWS];
#pragma unroll
    for (int c = 0; c < ROWS; ++c) {
        at[c] = 0;
        top[c] = m.active[c] ? staged : 0u;
    }
    lower_bounds<ROWS>(lds.window, at, top, m.idx, staged);
#pragma unroll
    for (int c = 0; c < ROWS; ++c) {
        m.member[c] = m.active[c] && at[c] < staged && lds.window[at[c]] == m.idx[c];
        lo[c] = at[c] ? w0 + (at[c] - 1) * step + 1 : w0;                        // elements lo .. hi - 1 are left
        const uint64_t next = (uint64_t)w0 + (uint64_t)at[c] * step;
        hi[c] = next < w1 ? (uint32_t)next : w1;
        if (!m.active[c] || m.member[c] || hi[c] < lo[c]) hi[c] = lo[c];
    }
    if (step > RST_BETWEEN + 1) {                    // a part of more than 70,000
#pragma unroll
        for (int c = 0; c < ROWS; ++c)
            while (hi[c] - lo[c] > RST_BETWEEN) {
                const uint32_t mid = lo[c] + ((hi[c] - lo[c]) >> 1), x = global_idx[mid];
                if (x < m.idx[c]) {
                    lo[c] = mid + 1;
                } else {
                    m.member[c] |= x == m.idx[c];
                    hi[c] = x == m.idx[c] ? lo[c] : mid;
                }
            }
    }
    // Equal is a member, wherever it stands, so a read may reach past both ends of what is left.
    constexpr uint32_t QUADS = RST_BETWEEN / 4;
    QuadAt4 v[QUADS][ROWS];
#pragma unroll
    for (uint32_t q = 0; q < QUADS; ++q)
#pragma unroll
        for (int c = 0; c < ROWS; ++c)
            v[q][c] = *reinterpret_cast<const QuadAt4*>(global_idx + (lo[c] < ng - 4 * (q + 1) ? lo[c] + 4 * q : ng - 4));
#pragma unroll
    for (uint32_t q = 0; q < QUADS; ++q)
#pragma unroll
        for (int c = 0; c < ROWS; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) m.member[c] |= m.active[c] && v[q][c].v[j] == m.idx[c];
    return m;
}

// The tile's entries looked up and the vector put right.  ZERO_MEMBERS false: the vector has
// every local entry zeroed already, the entries outside the intersection get their value
// back.  true: the vector is the untouched accumulator, the entries of the intersection
// are zeroed (local_val is not read).
template <int ROWS, bool ZERO_MEMBERS>
__device__ __forceinline__ Membership<ROWS> restore_tile(float* residual, uint32_t n, const uint32_t* local_idx,
                                                         const float* local_val, uint32_t base, uint32_t end,
                                                         const uint32_t* global_idx, uint32_t ng, RestoreMemory& lds) {
    float value[ROWS];
    if (!ZERO_MEMBERS) {
#pragma unroll
        for (int c = 0; c < ROWS; ++c) {
            const uint32_t j = base + c * RST_BLOCK + threadIdx.x;
            value[c] = j < end ? local_val[j] : 0.0f;
        }
    }
    const Membership<ROWS> m = tile_members<ROWS>(local_idx, base, end, global_idx, ng, lds);
#pragma unroll
    for (int c = 0; c < ROWS; ++c)
        if (m.active[c] && m.member[c] == ZERO_MEMBERS && m.idx[c] < n)
            residual[m.idx[c]] = ZERO_MEMBERS ? 0.0f : value[c];
    return m;
}

// `masks`, if the matched indices are wanted: a bit per entry, the tile's ballots row by row
// and wave by wave.
template <bool ZERO_MEMBERS>
__global__ __launch_bounds__(RST_BLOCK) void intersect_kernel(
    float* __restrict__ residual, uint32_t n, const uint32_t* __restrict__ local_idx,
    const float* __restrict__ local_val, const uint64_t* __restrict__ d_local_nnz,
    uint32_t max_local, const uint32_t* __restrict__ global_idx,
    const uint64_t* __restrict__ d_global_nnz, uint32_t max_global, uint32_t* __restrict__ counts,
    uint64_t* __restrict__ masks) {
    __shared__ RestoreMemory s_memory;
    __shared__ uint32_t s_count[RST_WAVES];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const uint32_t nl = entries_of(d_local_nnz, max_local), ng = entries_of(d_global_nnz, max_global);
    const uint32_t used = tiles_of<RST_ROWS>(nl);
    // The room a caller has, which sizes the launch, is often several times the entries there
    // are, and a workgroup of sixteen waves costs something also where it finds nothing to
    // do: no more are launched than run at a time.
    for (uint32_t tile = blockIdx.x; tile < used; tile += gridDim.x) {
        const uint32_t base = tile * RST_TILE, end = nl - base > RST_TILE ? base + RST_TILE : nl;
        const Membership<RST_ROWS> m = restore_tile<RST_ROWS, ZERO_MEMBERS>(residual, n, local_idx, local_val, base, end,
                                                                            global_idx, ng, s_memory);
        uint32_t found = 0;
#pragma unroll
        for (int c = 0; c < RST_ROWS; ++c) {
            const uint64_t ballot = __ballot(m.member[c]);
            if (masks && lane == 0) masks[(size_t)tile * (RST_TILE / WAVE) + c * RST_WAVES + wave] = ballot;
            found += (uint32_t)__popcll(ballot);
        }
        if (lane == 0) s_count[wave] = found;
        __syncthreads();
        if (tid == 0) {
            uint32_t total = 0;
#pragma unroll
            for (int w = 0; w < RST_WAVES; ++w) total += s_count[w];
            counts[tile] = total;
        }
        __syncthreads();                             // LDS is free again
    }
}

// The matched indices of a tile from the waves' ballots (s_row has a word per row and wave):
// tile_count says how many there are (one barrier), emit_tile writes them from `at` on.
template <int ROWS>
__device__ __forceinline__ uint32_t tile_count(const uint64_t (&ballot)[ROWS], uint32_t (&s_row)[ROWS][RST_WAVES]) {
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < ROWS; ++c)
        if (lane == 0) s_row[c][wave] = (uint32_t)__popcll(ballot[c]);
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int c = 0; c < ROWS; ++c)
#pragma unroll
        for (int w = 0; w < RST_WAVES; ++w) total += s_row[c][w];
    return total;
}
template <int ROWS>
__device__ __forceinline__ void emit_tile(const uint32_t (&idx)[ROWS], const uint64_t (&ballot)[ROWS],
                                          const uint32_t (&s_row)[ROWS][RST_WAVES], uint32_t at, uint32_t* indexes_out) {
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < ROWS; ++c) {
#pragma unroll
        for (int w = 0; w < RST_WAVES; ++w) {
            if (w == wave && (ballot[c] >> lane & 1u)) indexes_out[at + mask_rank(ballot[c])] = idx[c];
            at += s_row[c][w];
        }
    }
}

// The same in one launch, a tile's place from a scan across the workgroups: for a workspace
// without room for a bit per entry, and for outputs that take the place of an input: what a
// tile writes, the indices and the count, goes out when it and all tiles before it have
// read theirs, where the second launch of the other form reads the local list and its
// length again.  A ticket is 30 ns and they are served one at a time, so
// a tile has twice the entries here, and workgroups without entries leave before they take
// one.  1.1 M entries in a list of 1.6 M 33.8 us a call, 4.3 M in 5.0 M 114; looking everything
// up again in the second launch instead 52.2 and 189, workgroups that take several tiles of
// 1024 in turn 54.2 and 179.
template <bool ZERO_MEMBERS>
__global__ __launch_bounds__(RST_BLOCK) void intersect_chained_kernel(
    float* residual, uint32_t n, const uint32_t* local_idx, const float* local_val, const uint64_t* d_local_nnz,
    uint32_t max_local, const uint32_t* global_idx, const uint64_t* d_global_nnz, uint32_t max_global,
    uint32_t* indexes_out, uint64_t* count_out, ScanHeader* hdr, uint64_t* tile_desc, uint64_t* group_desc) {
    constexpr int ROWS = RST_CHAINED_ROWS;
    constexpr uint32_t TILE = ROWS * RST_BLOCK;
    __shared__ RestoreMemory s_memory;
    __shared__ uint32_t s_row[ROWS][RST_WAVES];
    __shared__ uint32_t s_tile, s_before[2];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const uint32_t nl = entries_of(d_local_nnz, max_local), ng = entries_of(d_global_nnz, max_global);
    const uint32_t used = tiles_of<ROWS>(nl);
    if (used == 0 && blockIdx.x == 0 && tid == 0) *count_out = 0;
    if (blockIdx.x >= used) return;
    if (tid == 0) s_tile = atomicAdd(&hdr->ticket, 1u);
    __syncthreads();
    const uint32_t tile = uniform(s_tile), base = tile * TILE, end = nl - base > TILE ? base + TILE : nl;
    const Membership<ROWS> m = restore_tile<ROWS, ZERO_MEMBERS>(residual, n, local_idx, local_val, base, end, global_idx,
                                                                ng, s_memory);
    uint64_t ballot[ROWS];
#pragma unroll
    for (int c = 0; c < ROWS; ++c) ballot[c] = __ballot(m.member[c]);
    const uint32_t aggregate = tile_count(ballot, s_row), group = tile / SCAN_GROUP;
    if (wave == 0) {
        const uint32_t before = scan_within_group(hdr, tile_desc, group_desc, tile, aggregate);
        if (lane == 0) s_before[0] = before;
    } else if (wave == 1) {
        const uint32_t before = scan_across_groups(hdr, group_desc, group);
        if (lane == 0) s_before[1] = before;
    }
    __syncthreads();
    const uint32_t exclusive = s_before[0] + s_before[1];
    if (tid == 0 && group != 0 && tile % SCAN_GROUP == SCAN_GROUP - 1)
        scan_close_group(group_desc, group, exclusive + aggregate);
    if (tile == used - 1 && tid == 0) {
        const bool failed = __hip_atomic_load(&hdr->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        *count_out = failed ? ~0ull : (uint64_t)exclusive + aggregate;
    }
    if (indexes_out) emit_tile(m.idx, ballot, s_row, exclusive, indexes_out);
}

// Sum over the workgroup (one barrier; s_wave has a word per wave).
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* s_wave) {
    v = wave_sum(v);
    if ((threadIdx.x & (WAVE - 1)) == 0) s_wave[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < RST_WAVES; ++w) total += s_wave[w];
    return total;
}

// The matched indices, in order: a tile's place is the sum of the counts before it
// (adding up RST_DIRECT_TILES counts takes a workgroup two microseconds; of more tiles
// than that intersect_scan_kernel has made prefixes of the counts).
template <bool PREFIXES>
__global__ __launch_bounds__(RST_BLOCK) void intersect_emit_kernel(
    const uint32_t* __restrict__ local_idx, const uint64_t* __restrict__ d_local_nnz, uint32_t max_local,
    const uint32_t* __restrict__ counts, const uint64_t* __restrict__ masks,
    uint32_t* __restrict__ indexes_out, uint64_t* __restrict__ count_out) {
    __shared__ uint32_t s_sum[RST_WAVES];
    __shared__ uint32_t s_row[RST_ROWS][RST_WAVES];
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t nl = entries_of(d_local_nnz, max_local), used = tiles_of<RST_ROWS>(nl);
    if (used == 0 && blockIdx.x == 0 && tid == 0) *count_out = 0;
    for (uint32_t tile = blockIdx.x; tile < used; tile += gridDim.x) {
        const uint32_t base = tile * RST_TILE, end = nl - base > RST_TILE ? base + RST_TILE : nl;
        uint32_t idx[RST_ROWS];
        uint64_t ballot[RST_ROWS];
        if (indexes_out) {
#pragma unroll
            for (int c = 0; c < RST_ROWS; ++c) {
                const uint32_t j = base + c * RST_BLOCK + tid;
                idx[c] = j < end ? local_idx[j] : 0u;
                ballot[c] = masks[(size_t)tile * (RST_TILE / WAVE) + c * RST_WAVES + wave];
            }
        }
        uint32_t before;
        if (PREFIXES) {
            before = counts[tile];
        } else {
            uint32_t sum = 0;
            for (uint32_t t = tid; t < tile; t += RST_BLOCK) sum += counts[t];
            before = block_sum(sum, s_sum);
        }
        if (tile == used - 1 && tid == 0) *count_out = (uint64_t)before + (PREFIXES ? counts[tile + 1] - before : counts[tile]);
        if (!indexes_out) {
            __syncthreads();                             // s_sum has been read
            continue;
        }
        tile_count(ballot, s_row);
        emit_tile(idx, ballot, s_row, before, indexes_out);
        __syncthreads();                                 // LDS is free again
    }
}

// Counts of up to 2^22 tiles -> the counts before each, and of all behind the last.
__global__ __launch_bounds__(RST_SCAN_BLOCK) void intersect_scan_kernel(
    const uint64_t* __restrict__ d_local_nnz, uint32_t max_local, uint32_t* __restrict__ counts) {
    __shared__ uint32_t s_wave[RST_SCAN_BLOCK / WAVE];
    const uint32_t tid = threadIdx.x, wave = tid >> 6, used = tiles_of<RST_ROWS>(entries_of(d_local_nnz, max_local));
    uint32_t before = 0;
    for (uint32_t t0 = 0; t0 < used; t0 += RST_SCAN_BLOCK) {
        const uint32_t c = t0 + tid < used ? counts[t0 + tid] : 0u;
        const uint32_t incl = wave_inclusive_scan_u32(c);
        if ((tid & (WAVE - 1)) == WAVE - 1) s_wave[wave] = incl;
        __syncthreads();
        uint32_t first = before;
#pragma unroll
        for (uint32_t w = 0; w < RST_SCAN_BLOCK / WAVE; ++w) {
            if (w == wave && t0 + tid < used) counts[t0 + tid] = first + incl - c;
            first += s_wave[w];
        }
        before = first;
        __syncthreads();
    }
    if (tid == 0) counts[used] = before;
}

template <bool ZERO_MEMBERS>
static int launch_intersect(float* d_vec, uint64_t n, const uint32_t* d_local_idx,
                            const float* d_local_val, const uint64_t* d_local_nnz,
                            uint64_t max_local, const uint32_t* d_global_idx,
                            const uint64_t* d_global_nnz, uint64_t max_global,
                            uint32_t* d_indexes_out_or_null, uint64_t* d_count_out, void* d_ws,
                            size_t ws_bytes, hipStream_t s) {
    if (!d_count_out || !aligned(d_count_out, 8)) return OKT_ERR_INVALID_ARG;
    if (n > 0xffffffffull || max_local > 0xffffffffull || max_global > 0xffffffffull)
        return OKT_ERR_INVALID_ARG;
    if (!d_local_nnz || !d_global_nnz || !aligned(d_local_nnz, 8) || !aligned(d_global_nnz, 8))
        return OKT_ERR_INVALID_ARG;
    if (max_local > 0 && (!d_vec || !d_local_idx || !aligned(d_vec, 4) || !aligned(d_local_idx, 4)))
        return OKT_ERR_INVALID_ARG;
    if (max_local > 0 && !ZERO_MEMBERS && (!d_local_val || !aligned(d_local_val, 4)))
        return OKT_ERR_INVALID_ARG;
    if (max_global > 0 && (!d_global_idx || !aligned(d_global_idx, 4))) return OKT_ERR_INVALID_ARG;
    if (d_indexes_out_or_null && !aligned(d_indexes_out_or_null, 4)) return OKT_ERR_INVALID_ARG;
    const uint32_t ntiles = (uint32_t)restore_tiles(max_local);
    if (!d_ws || !aligned(d_ws, 256) || ws_bytes < restore_ws_bytes(max_local))
        return OKT_ERR_WORKSPACE;
    const bool room = ws_bytes >= restore_masks_at(max_local) + (size_t)ntiles * (RST_TILE / 8);
    const size_t out_bytes = d_indexes_out_or_null ? 4 * (size_t)max_local : 0;
    const bool over_input = overlap(d_count_out, 8, d_local_nnz, 8) || overlap(d_count_out, 8, d_global_nnz, 8) ||
                            overlap(d_indexes_out_or_null, out_bytes, d_local_idx, 4 * (size_t)max_local) ||
                            overlap(d_indexes_out_or_null, out_bytes, d_global_idx, 4 * (size_t)max_global);
    if (over_input || (d_indexes_out_or_null && !room)) {
        constexpr uint64_t TILE = RST_CHAINED_ROWS * RST_BLOCK;
        const uint32_t tiles = max_local ? (uint32_t)((max_local + TILE - 1) / TILE) : 1u;
        uint64_t* tile_desc = (uint64_t*)((char*)d_ws + SCAN_HEADER_BYTES);
        if (launch_clear_scan_state(d_ws, scan_ws_bytes(tiles) / 8, s) != hipSuccess) return OKT_ERR_HIP;
        timing_before(s);
        hipLaunchKernelGGL(intersect_chained_kernel<ZERO_MEMBERS>, dim3(tiles), dim3(RST_BLOCK), 0, s, d_vec,
                           (uint32_t)n, d_local_idx, d_local_val, d_local_nnz, (uint32_t)max_local, d_global_idx,
                           d_global_nnz, (uint32_t)max_global, d_indexes_out_or_null, d_count_out,
                           (ScanHeader*)d_ws, tile_desc, tile_desc + tiles);
        timing_after(s);
        return launch_status();
    }
    const uint32_t grid = ntiles < RST_PER_CU * device_cus() ? ntiles : RST_PER_CU * device_cus();
    uint32_t* counts = (uint32_t*)d_ws;                              // one more than there are tiles
    uint64_t* masks = d_indexes_out_or_null ? (uint64_t*)((char*)d_ws + restore_masks_at(max_local)) : nullptr;
    timing_before(s);
    hipLaunchKernelGGL(intersect_kernel<ZERO_MEMBERS>, dim3(grid), dim3(RST_BLOCK), 0, s, d_vec,
                       (uint32_t)n, d_local_idx, d_local_val, d_local_nnz, (uint32_t)max_local,
                       d_global_idx, d_global_nnz, (uint32_t)max_global, counts, masks);
    timing_after(s);
    const bool prefixes = ntiles > RST_DIRECT_TILES;
    if (prefixes)
        hipLaunchKernelGGL(intersect_scan_kernel, dim3(1), dim3(RST_SCAN_BLOCK), 0, s, d_local_nnz,
                           (uint32_t)max_local, counts);
    hipLaunchKernelGGL(prefixes ? intersect_emit_kernel<true> : intersect_emit_kernel<false>, dim3(grid),
                       dim3(RST_BLOCK), 0, s, d_local_idx, d_local_nnz, (uint32_t)max_local, counts, masks,
                       d_indexes_out_or_null, d_count_out);
    return launch_status();
}

}  // namespace okt

extern "C" int okt_index_intersect_restore(
    float* d_residual_inout, uint64_t n, const uint32_t* d_local_idx, const float* d_local_val,
    const uint64_t* d_local_nnz, uint64_t max_local, const uint32_t* d_global_idx,
    const uint64_t* d_global_nnz, uint64_t max_global, uint32_t* d_indexes_out_or_null,
    uint64_t* d_count_out, void* d_ws, size_t ws_bytes, void* stream) {
    return okt::launch_intersect<false>(d_residual_inout, n, d_local_idx, d_local_val, d_local_nnz,
                                        max_local, d_global_idx, d_global_nnz, max_global,
                                        d_indexes_out_or_null, d_count_out, d_ws, ws_bytes,
                                        (hipStream_t)stream);
}

extern "C" int okt_index_intersect_zero(
    float* d_acc_inout, uint64_t n, const uint32_t* d_local_idx, const uint64_t* d_local_nnz,
    uint64_t max_local, const uint32_t* d_global_idx, const uint64_t* d_global_nnz,
    uint64_t max_global, uint32_t* d_indexes_out_or_null, uint64_t* d_count_out, void* d_ws,
    size_t ws_bytes, void* stream) {
    return okt::launch_intersect<true>(d_acc_inout, n, d_local_idx, nullptr, d_local_nnz, max_local,
                                       d_global_idx, d_global_nnz, max_global,
                                       d_indexes_out_or_null, d_count_out, d_ws, ws_bytes,
                                       (hipStream_t)stream);
}
