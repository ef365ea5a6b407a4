// okt_topk_threshold_exact: the exact k-th largest |acc| (Algorithm 1, lines
// 2-4, th_re_evaluate; Sec. 3.1.3).  The paper sorts; this is an exact
// selection on the 31-bit magnitude key that reads the vector about once.
//
//   1. A strided sample gives a key that lies, with a margin, below the k-th largest.
//   2. One streaming pass over the whole vector copies every key at or above
//      that bound, a little more than k of them, to the workspace (the select
//      kernel's loop: one compare per element, per-wave LDS stash, one global
//      atomic per workgroup for what the stashes hold at the end).
//   3. If at least k keys were collected (always, unless the sample misled),
//      rank k is among them, and an exact MSD radix select of two digits from the
//      bound up runs over the candidates only.  Otherwise, if the sample misled, a radix
//      select of 11 + 11 + 9 bits runs over the whole vector in the same launch.
// Where step 2 is known beforehand not to pay (no room for the candidates, or a large
// k), a longer vector takes three streaming launches, a digit each, and one of up to
// BOUNDED_TO_N elements the sample and the two digits from its bound up over all of it.
// One launch up to TINY_N elements, else two to four.
// Either way the answer is the exact order statistic: all arithmetic is integer
// counting, the sample only decides how much is read.  State lives in the
// workspace on the device; the host never waits.
//
// okt_accumulate_topk_select: a whole refresh iteration (Algorithm 2, lines 4-6,
// with the threshold re-evaluated) that reads the gradient and the residual
// once.  The sample is formed on the fly from both; the pass that collects the
// candidates is the fused accumulate+select kernel run against the sample's
// bound, writing the accumulator over the residual and the candidates, in index
// order with their indices, to the workspace; the radix select runs over the
// candidate values; and the final select, in the same launch, walks the candidates
// instead of the vector, zeroing the residual where an entry goes out.  If the sample misled,
// the last two steps run over the whole vector instead: same results.
#include "okt_device.h"
#include "okt_select_kernel.h"
#include "okt_sizes.h"
#include "okt_slots.h"

#include <stddef.h>

namespace okt {

constexpr int PHASES_MAX = 4;      // digits of resolve_kernel: one from a bound and three general ones at most
constexpr int BOUNDS = 16;         // workgroups of the sample
static_assert(SLOT_BOUNDS == BOUNDS, "the slots' first pass reads every bound");
constexpr uint32_t HIST_WORDS = 4 * RS_MAX_BINS;

struct RadixState {
    uint32_t bound[BOUNDS];           // the sample's: every key >= their least is a candidate
    unsigned long long cand_count;    // candidates found by the collect pass
    uint64_t collected[2];            // ordered collection (refresh iteration): candidates written, found
    uint32_t done[PHASES_MAX];        // shares of a phase of resolve_kernel that are finished
    uint32_t ticket;
    uint32_t base, k_rem, above;      // of digit_kernel's launches: what the digits so far say
    uint32_t spin_limit;              // polls a wait of resolve_kernel may take; 0 = SPIN_LIMIT
};
constexpr uint32_t STATE_SPIN_WORD = offsetof(RadixState, spin_limit) / 4;
static_assert(sizeof(RadixState) <= RS_STATE_BYTES, "state fits its slot");

__device__ __forceinline__ uint32_t cand_bound(const RadixState* state) {
    uint32_t lo = state->bound[0];
#pragma unroll
    for (int i = 1; i < BOUNDS; ++i) lo = state->bound[i] < lo ? state->bound[i] : lo;
    return lo;
}
// What the collecting passes test against.  A bound of zero (a vector with fewer than
// k elements that are not) is no bound: nothing is collected then, rather than
// everything that the candidates have room for, and the digits run over the vector.
__device__ __forceinline__ uint32_t collect_bound(const RadixState* state) {
    const uint32_t lo = cand_bound(state);
    return lo != 0 ? lo : ABS_MASK;
}

// Find the bin that holds rank k_rem counting from the top bin down.  Of BLOCK threads,
// thread t owns the `per` bins below the t * per highest ones; an inclusive scan
// over the threads' sums names the owner, who walks its own few bins.  The
// owner (exactly one thread, if the bins hold that many) stores (bin, keys above the
// bin, keys in it) to s_result, whose first word is all ones otherwise.
template <bool ELSEWHERE, int BLOCK = 1024>     // ELSEWHERE: the counts were added by other workgroups
__device__ __forceinline__ void pick_bin(const uint32_t* hist, uint32_t bins, uint32_t k_rem,
                                         uint32_t* s_wave, uint32_t* s_result) {
    constexpr int PER_MAX = 8;
    const int t = threadIdx.x, lane = t & (WAVE - 1), wave = t >> 6;
    const uint32_t per = bins > BLOCK ? bins / BLOCK : 1;             // bins is a power of two, at most 8 BLOCK
    const bool owner = (uint32_t)t * per < bins;
    uint32_t c[PER_MAX], mine = 0;
#pragma unroll
    for (int j = 0; j < PER_MAX; ++j) {
        c[j] = 0;
        if (owner && (uint32_t)j < per) {
            const uint32_t* at = hist + (bins - 1 - ((uint32_t)t * per + j));   // j = 0 is the thread's highest bin
            c[j] = ELSEWHERE ? __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *at;
        }
        mine += c[j];
    }
    const uint32_t incl = wave_inclusive_scan_u32(mine);
    if (lane == WAVE - 1) s_wave[wave] = incl;
    if (t == 0) s_result[0] = ~0u;
    __syncthreads();
    uint32_t before = incl - mine;
#pragma unroll
    for (int w = 0; w < BLOCK / WAVE; ++w)
        if (w < wave) before += s_wave[w];
    if (before < k_rem && k_rem <= before + mine) {  // true for at most one thread
        uint32_t above = before, in_bin = c[0], j = 0;
#pragma unroll
        for (int i = 0; i < PER_MAX - 1; ++i)
            if ((uint32_t)i == j && above + c[i] < k_rem) {
                above += c[i];
                in_bin = c[i + 1];
                ++j;
            }
        s_result[0] = bins - 1 - ((uint32_t)t * per + j);
        s_result[1] = above;                         // above < k_rem <= above + in_bin
        s_result[2] = in_bin;
    }
    __syncthreads();
}

// The key of rank k_rem among n <= FEW keys in LDS, how many of them are larger and how
// many equal: every wave works it out for itself.  A key costs some 45 ns, the histogram that
// is saved 0.6 us: 300 candidates, 1 to 16 keys 12.8 to 13.2 us a call and 13.5 with the
// histogram, 33 keys 14.0 and 13.4.
constexpr uint32_t FEW = 16;
struct KeyRank { uint32_t key, above, equal; };
__device__ __forceinline__ KeyRank rank_of_few(const uint32_t* s_keys, uint32_t n, uint32_t k_rem) {
    const uint32_t lane = (uint32_t)lane_id(), mine = lane < n ? s_keys[lane] : 0u;
    uint32_t larger = 0, same = 0;
    for (uint32_t j = 0; j < n; ++j) {
        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)j);
        larger += v > mine ? 1u : 0u;
        same += v == mine ? 1u : 0u;
    }
    // the lanes whose key it is hold the same
    const uint64_t is = __ballot(lane < n && larger < k_rem && k_rem <= larger + same);
    const int at = __ffsll((unsigned long long)is) - 1;
    return KeyRank{(uint32_t)__builtin_amdgcn_readlane((int)mine, at), (uint32_t)__builtin_amdgcn_readlane((int)larger, at),
                   (uint32_t)__builtin_amdgcn_readlane((int)same, at)};
}

// ---------------------------------------------------------------------------
// the sample
// ---------------------------------------------------------------------------
// A bound that lies, with a margin, below the k-th largest key, from a sample of
// 131,072 elements: 8192 blocks of 16 (a line of memory each), spread evenly.  Each
// of the BOUNDS workgroups histograms every sixteenth of them (13 bits of the key: a
// bin is a thirty-second of an octave), and its own bound is the bottom of the bin
// that holds the sample rank k' + sqrt(k'), k' = 8192 k / n: one standard
// deviation below the target rank.  The least of the sixteen is the one that counts:
// all of them lie above the k-th largest key with a probability of 0.16 ^ 16, and
// still one in a hundred million where neighbours are so alike that a count
// deviates twice as far.  About 1.3 k elements pass it at k = 1 % of a vector, 2 k at
// 0.1 %.  (One histogram over all the workgroups needs cleared memory and a last
// workgroup to read it: two launches, 16 us, against 6 us for this one.)
//
// The same launch clears what the later ones need cleared: the radix state, the
// histograms and up to two scan states.  With `grad` set the sampled values are
// eps + lr * G formed on the fly (`acc` is then the residual before the accumulate).
constexpr int SAMPLE_BLOCK = 1024;
constexpr uint32_t SAMPLE_RUN = 16, SAMPLE_RUNS = 8192, SAMPLE_RUNS_PER_WG = SAMPLE_RUNS / BOUNDS;
constexpr uint32_t SAMPLE_BINS = 8192;
constexpr int SAMPLE_SHIFT = 31 - 13;
// (A vector shorter than the sample has its blocks sampled more than once, evenly.)
static_assert(TINY_N >= SAMPLE_RUN, "a block to sample");

__global__ __launch_bounds__(SAMPLE_BLOCK) void sample_bound_kernel(
    const float* __restrict__ acc, const float* __restrict__ grad, float lr, uint32_t n, uint32_t k,
    RadixState* state, uint32_t* __restrict__ hist, uint64_t* __restrict__ scan_a, uint32_t words_a,
    uint64_t* __restrict__ scan_b, uint32_t words_b, uint32_t spin_limit, uint32_t digit_spin_limit) {
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[SAMPLE_BINS];
    __shared__ uint32_t s_wave[SAMPLE_BLOCK / WAVE], s_result[3];
    const uint32_t tid = threadIdx.x, wg = blockIdx.x;
    constexpr uint32_t PER = SAMPLE_RUNS_PER_WG * 4 / SAMPLE_BLOCK;
    float4 v[PER], g[PER];
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
        const uint32_t run = wg + BOUNDS * (u * (SAMPLE_BLOCK / 4) + (tid >> 2));
        const uint64_t at = (uint64_t)run * (n / SAMPLE_RUN) / SAMPLE_RUNS * 4 + (tid & 3u);   // in quads
        v[u] = reinterpret_cast<const float4*>(acc)[at];
        if (grad) g[u] = reinterpret_cast<const float4*>(grad)[at];
    }
    for (uint32_t b = tid; b < SAMPLE_BINS / 4; b += SAMPLE_BLOCK) reinterpret_cast<uint4*>(s_hist)[b] = uint4{0, 0, 0, 0};
    const uint32_t i = wg * SAMPLE_BLOCK + tid;
    for (uint32_t w = i; w < HIST_WORDS; w += BOUNDS * SAMPLE_BLOCK) hist[w] = 0;
    for (uint32_t w = i; w < words_a; w += BOUNDS * SAMPLE_BLOCK) scan_a[w] = w == SCAN_SPIN_WORD ? (uint64_t)spin_limit : 0ull;
    for (uint32_t w = i; w < words_b; w += BOUNDS * SAMPLE_BLOCK) scan_b[w] = w == SCAN_SPIN_WORD ? (uint64_t)spin_limit : 0ull;
    if (i >= BOUNDS && i < sizeof(RadixState) / 4)                                              // behind the bounds
        reinterpret_cast<uint32_t*>(state)[i] = i == STATE_SPIN_WORD ? digit_spin_limit : 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
        if (grad) {
            v[u].x = __fadd_rn(v[u].x, __fmul_rn(lr, g[u].x));
            v[u].y = __fadd_rn(v[u].y, __fmul_rn(lr, g[u].y));
            v[u].z = __fadd_rn(v[u].z, __fmul_rn(lr, g[u].z));
            v[u].w = __fadd_rn(v[u].w, __fmul_rn(lr, g[u].w));
        }
        atomicAdd(&s_hist[magnitude_key(v[u].x) >> SAMPLE_SHIFT], 1u);
        atomicAdd(&s_hist[magnitude_key(v[u].y) >> SAMPLE_SHIFT], 1u);
        atomicAdd(&s_hist[magnitude_key(v[u].z) >> SAMPLE_SHIFT], 1u);
        atomicAdd(&s_hist[magnitude_key(v[u].w) >> SAMPLE_SHIFT], 1u);
    }
    __syncthreads();
    constexpr uint32_t sample = SAMPLE_RUNS_PER_WG * SAMPLE_RUN;
    const uint32_t kp = (uint32_t)(((uint64_t)k * sample + n / 2) / n);       // at most `sample`
    uint32_t rank = kp + (uint32_t)(__builtin_sqrtf((float)kp) + 0.5f);
    rank = rank < 1 ? 1 : rank > sample ? sample : rank;
    pick_bin<false>(s_hist, SAMPLE_BINS, rank, s_wave, s_result);
    if (tid == 0) state->bound[wg] = s_result[0] << SAMPLE_SHIFT;
}

constexpr int CNT_BLOCK = SEL_BLOCK;
constexpr int CNT_WAVES = CNT_BLOCK / WAVE;
constexpr int CNT_STASH = 1024;                  // keys per wave between flushes
constexpr int CNT_U = 4;

// The counting pass, with the select kernel's one-compare-per-element test.  A workgroup's
// elements are dealt out to its waves batch by batch, so that it reads one place of the
// vector at a time: nothing has to be in order here, and sixteen waves with a piece each read
// sixteen (whole calls on vectors from memory, a piece a wave and so: 64 M elements 69.4 and 67.6 us,
// 133 M 119.5 and 113.3, 200 M 167 and 160, 110 M and 336 M even, 14 to 40 M 1 to 2 % less; even as well where
// the vector was written just before: accumulate, threshold and select of 133 M 491.6 and 491.3; pieces
// of a half or a quarter, for more workgroups than fit at a time, lose it again).  Every key at or above the bound is
// a candidate and is copied to `cand`, in any order (per-wave LDS stash; a stash
// that fills up is flushed with an atomic of its own, the rest of a workgroup
// with one atomic at the end).
template <bool NT, typename Test>
__device__ __forceinline__ void collect_body(const float* __restrict__ acc, uint32_t n,
                                             uint32_t piece, RadixState* state,
                                             uint32_t* __restrict__ cand, uint64_t cand_cap,
                                             Test test, uint32_t (*s_stash)[CNT_STASH],
                                             uint32_t* s_left, unsigned long long* s_base) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr uint64_t BATCH = 256 * CNT_U;
    const uint64_t first = (uint64_t)blockIdx.x * CNT_WAVES * piece;
    const uint64_t end = first + (uint64_t)CNT_WAVES * piece < n ? first + (uint64_t)CNT_WAVES * piece : n;
    uint32_t* mine = s_stash[wave];
    uint32_t stashed = 0;                        // wave-uniform

    auto flush = [&]() {
        if (stashed == 0) return;
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&state->cand_count, (unsigned long long)stashed);
        base = __shfl(base, 0, WAVE);
        for (uint32_t j = lane; j < stashed; j += WAVE)
            if (base + j < cand_cap) cand[base + j] = mine[j];
        stashed = 0;
    };
    auto round = [&](const float4& v, bool cx, bool cy, bool cz, bool cw) {
        if (stashed > (uint32_t)(CNT_STASH - 256)) flush();     // room for a whole round
        stashed = select_round(0u, v, cx, cy, cz, cw, stashed,
                               [&](uint32_t rank, uint32_t, float x) { mine[rank] = magnitude_key(x); });
    };

    const uint64_t whole = (end - first) / BATCH;         // batches, dealt out to the waves
    for (uint64_t b = wave; b < whole; b += CNT_WAVES) {
        const float4* src = reinterpret_cast<const float4*>(acc + first + b * BATCH) + lane;
        float4 v[CNT_U];
#pragma unroll
        for (int u = 0; u < CNT_U; ++u) v[u] = load_quad<NT>(src + u * WAVE);
#pragma unroll
        for (int u = 0; u < CNT_U; ++u)
            round(v[u], test(v[u].x), test(v[u].y), test(v[u].z), test(v[u].w));
    }
    uint64_t r = first + whole * BATCH + 256u * wave;     // what is left, a round a wave
    if (r + 256 <= end) {
        const float4 v = load_quad<NT>(reinterpret_cast<const float4*>(acc + r) + lane);
        round(v, test(v.x), test(v.y), test(v.z), test(v.w));
    } else if (r < end) {                                 // the ragged end of the vector
        const uint64_t i = r + 4u * (uint32_t)lane;
        float e[4];
        bool c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool inside = i + j < end;
            e[j] = inside ? acc[i + j] : 0.0f;
            c[j] = inside && test(e[j]);
        }
        round(make_float4(e[0], e[1], e[2], e[3]), c[0], c[1], c[2], c[3]);
    }
    // What is left goes out with ONE atomic per workgroup: atomics on a single
    // address retire one after the other, and one per wave (tens of thousands on a
    // long vector) would outlast the whole pass.
    if (lane == 0) s_left[wave] = stashed;
    __syncthreads();
    if (tid == 0) {
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < CNT_WAVES; ++w) total += s_left[w];
        *s_base = total ? atomicAdd(&state->cand_count, (unsigned long long)total) : 0ull;
    }
    __syncthreads();
    unsigned long long base = *s_base;
    for (uint32_t w = 0; w < wave; ++w) base += s_left[w];
    for (uint32_t j = lane; j < stashed; j += WAVE)
        if (base + j < cand_cap) cand[base + j] = mine[j];
}

template <bool NT>
__global__ __launch_bounds__(CNT_BLOCK) void collect_kernel(
    const float* __restrict__ acc, uint32_t n, uint32_t piece, RadixState* state,
    uint32_t* __restrict__ cand, uint64_t cand_cap) {
    __shared__ uint32_t s_stash[CNT_WAVES][CNT_STASH];
    __shared__ uint32_t s_left[CNT_WAVES];
    __shared__ unsigned long long s_base;
    const uint32_t lo_key = collect_bound(state);
    const float lo = __uint_as_float(lo_key);               // a key below the Inf/NaN range, or NaN
    if (lo == lo)
        collect_body<NT>(acc, n, piece, state, cand, cand_cap, TestFloat{lo}, s_stash, s_left, &s_base);
    else
        collect_body<NT>(acc, n, piece, state, cand, cand_cap, TestKey{lo_key}, s_stash, s_left, &s_base);
}

__global__ void radix_init_kernel(RadixState* state, uint32_t* hist) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < HIST_WORDS) hist[i] = 0;
    if (i < sizeof(RadixState) / 4) reinterpret_cast<uint32_t*>(state)[i] = 0;
}

// Whether CROWD lanes of the wave share a bin (see digit_kernel), and the add that serves
// all the lanes that share the first one's; `take` does the others.
constexpr uint32_t CROWD = 16;
__device__ __forceinline__ bool crowded(uint32_t bin, uint32_t bins) {
    const uint32_t lead = uniform(bin);
    return lead < bins && (uint32_t)__popcll(__ballot(bin == lead)) >= CROWD;
}
template <typename Take>
__device__ __forceinline__ void add_crowd(uint32_t* s_hist, uint32_t bin, uint32_t bins, Take&& take) {
    const uint32_t lead = uniform(bin);
    const uint64_t same = __ballot(bin == lead);
    if (lead < bins && bin == lead) {
        if (mask_rank(same) == 0) atomicAdd(&s_hist[lead], (uint32_t)__popcll(same));
    } else {
        take();
    }
}

// ---------------------------------------------------------------------------
// a digit over the whole vector, a launch each
// ---------------------------------------------------------------------------
// Where it is known beforehand that the digits run over all of a long vector, each is a
// streaming launch of its own: small workgroups, four 16-byte loads of a thread in
// flight, a histogram in LDS; the workgroup that hands in its counts last picks the bin
// and leaves what the next launch needs.  resolve_kernel below could do it as well, with
// one workgroup of 1024 threads per compute unit and contiguous shares by ticket, and is
// slower at it (its shares dealt out row by row instead: 400 us at 110 M, every row on a
// page of its own).  Two workgroups per compute unit: each adds up to 2048 bins to the
// total, and eight of them cost more there than they save in the pass.  Exact threshold
// with a workspace that has no room for candidates, layered values, cold:
//              resolve_kernel   8 per unit   2 per unit
//   25.6 M          137 us         125 us        82 us
//   60 M            250            164          140
//   110 M           260            240          231
//   336 M           697            661          613
// Keys that share a bin queue for one word of LDS, some seven cycles each.  Where one key
// a lane, looked at before a batch, finds CROWD of the wave's lanes in one bin, the batch
// is counted with one add for all the lanes that share the first one's bin (a vector of
// zeros, all but a thousandth of them: 25.6 M elements 281 us without this, 112 so).
constexpr int DIG_BLOCK = 256, DIG_QUADS = 4, DIG_PER_CU = 2;
constexpr uint32_t DIG_STEP = DIG_BLOCK * 4 * DIG_QUADS;

template <uint32_t SHIFT, int BITS, int PASS, bool NT>
__global__ __launch_bounds__(DIG_BLOCK) void digit_kernel(const float* __restrict__ acc, uint32_t n, uint32_t k,
                                                          RadixState* state, uint32_t* __restrict__ hist,
                                                          float* threshold_out, uint64_t* count_ge_out) {
    constexpr uint32_t BINS = 1u << BITS;
    constexpr bool FIRST = PASS == 0, LAST = SHIFT == 0;
    __shared__ uint32_t s_hist[BINS], s_wave[DIG_BLOCK / WAVE], s_result[3], s_last;
    const uint32_t tid = threadIdx.x;
    for (uint32_t b = tid; b < BINS; b += DIG_BLOCK) s_hist[b] = 0;
    const uint32_t base = FIRST ? 0u : state->base, k_rem = FIRST ? k : state->k_rem, above = FIRST ? 0u : state->above;
    __syncthreads();
    const uint32_t prefix = base >> (SHIFT + BITS);
    auto take = [&](float x) {
        const uint32_t key = magnitude_key(x);
        if (FIRST || key >> (SHIFT + BITS) == prefix) atomicAdd(&s_hist[(key >> SHIFT) & (BINS - 1)], 1u);
    };
    auto take_crowd = [&](float x) { add_crowd(s_hist, (magnitude_key(x) - base) >> SHIFT, BINS, [&]() { take(x); }); };
    const uint64_t stride = (uint64_t)gridDim.x * DIG_STEP;
    for (uint64_t r = (uint64_t)blockIdx.x * DIG_STEP; r < n; r += stride) {
        if (r + DIG_STEP <= n) {
            const float4* src = reinterpret_cast<const float4*>(acc + r) + tid;
            float4 v[DIG_QUADS];
#pragma unroll
            for (int u = 0; u < DIG_QUADS; ++u) v[u] = load_quad<NT>(src + u * DIG_BLOCK);
            // all four go out before the first is looked at (the compiler would otherwise wait
            // for the first behind the second)
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t first = (magnitude_key(v[0].x) - base) >> SHIFT;
            if (crowded(first, BINS)) {
#pragma unroll
                for (int u = 0; u < DIG_QUADS; ++u) {
                    take_crowd(v[u].x); take_crowd(v[u].y);
                    take_crowd(v[u].z); take_crowd(v[u].w);
                }
            } else {
#pragma unroll
                for (int u = 0; u < DIG_QUADS; ++u) {
                    take(v[u].x); take(v[u].y);
                    take(v[u].z); take(v[u].w);
                }
            }
        } else {
            for (uint64_t i = r + tid; i < n; i += DIG_BLOCK) take(acc[i]);
        }
    }
    __syncthreads();
    uint32_t* total = hist + RS_MAX_BINS * PASS;
    uint32_t seen = 0;
#pragma unroll
    for (uint32_t b = tid; b < BINS; b += DIG_BLOCK) {               // all out first, then one wait
        const uint32_t c = s_hist[b];
        if (c) seen |= atomicAdd(&total[b], c);
    }
    asm volatile("" ::"v"(seen));       // an atomic that has returned has been carried out (see resolve_kernel)
    __syncthreads();
    if (tid == 0) s_last = atomicAdd(&state->done[PASS], 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (s_last == 0) return;
    pick_bin<true, DIG_BLOCK>(total, BINS, k_rem, s_wave, s_result);
    if (tid != 0) return;
    const uint32_t key = base + (s_result[0] << SHIFT);
    if (LAST) {
        *threshold_out = __uint_as_float(key);
        *count_ge_out = (uint64_t)above + s_result[1] + s_result[2];
    } else {
        state->base = key;
        state->k_rem = k_rem - s_result[1];
        state->above = above + s_result[1];
    }
}

template <bool NT>
static void launch_digits(const float* acc, uint64_t n, uint64_t k, RadixState* state, uint32_t* hist,
                          float* d_threshold_out, uint64_t* d_count_ge_out, hipStream_t s) {
    const uint64_t steps = (n + DIG_STEP - 1) / DIG_STEP, most = (uint64_t)DIG_PER_CU * device_cus();
    const dim3 grid((unsigned)(steps < most ? steps : most)), block(DIG_BLOCK);
    hipLaunchKernelGGL((digit_kernel<20, RS_BITS1, 0, NT>), grid, block, 0, s, acc, (uint32_t)n, (uint32_t)k, state,
                       hist, d_threshold_out, d_count_ge_out);
    hipLaunchKernelGGL((digit_kernel<9, RS_BITS2, 1, NT>), grid, block, 0, s, acc, (uint32_t)n, (uint32_t)k, state,
                       hist, d_threshold_out, d_count_ge_out);
    hipLaunchKernelGGL((digit_kernel<0, RS_BITS3, 2, NT>), grid, block, 0, s, acc, (uint32_t)n, (uint32_t)k, state,
                       hist, d_threshold_out, d_count_ge_out);
}

// ---------------------------------------------------------------------------
// the exact threshold, and the select that uses it, in one launch
// ---------------------------------------------------------------------------
// An MSD radix select on the magnitude key, digit by digit, and (SELECT) the
// compaction of what lies at or above the result, as phases of one kernel.  A phase
// is cut into equal shares; a workgroup takes tickets, and ticket t is share t mod
// shares of phase t / shares.  A digit's counts go to a histogram in memory; who has
// a ticket of a later phase waits until all shares of the digit are counted, reads
// the complete histogram and works out for itself what the next phase is.  All
// shares of earlier phases are held by running workgroups that wait only for still
// earlier ones, so every wait ends, with however few workgroups running; the waits
// are bounded all the same.
//
// With a bound from the sample two digits do: the keys up to an octave above it in
// 2048 bins (and one for all that lie higher), then the 4096 keys of one of those
// bins.  If the answer lies higher, or the bound was not below it, the digits are the
// general ones, 11 + 11 + 9 bits from the top; they run over the candidates if rank k
// is among them, else over the whole vector.  The counts go out with atomics whose
// result is waited for: an atomic that has returned has been carried out where every
// compute unit sees it, which a release fence would only achieve by writing the whole
// L2 back.
//
// One launch takes the place of four (three digits of 6 to 14 us and a select of 10
// to 17 us; 31 us in all at 14.7 M elements and 2 %, 41 us at 336 M and 0.1 %, 28 and
// 34 us here; with the sample's two launches made one, a refresh iteration of 1 Mi
// elements went from 45 to 27 us, of 14.7 M from 84 to 74).  A phase boundary costs about four microseconds (counts out, last share
// noticed, histogram read), a launch five.  Tickets on one counter are served one at
// a time, some 30 ns each, so candidates are cut into SHARES_AIM shares or so (510
// shares: 33 us for two digits over 1.7 M candidates, 21 us with 69).  What fits into a
// single share is resolved from registers, without an exchange: by one workgroup, or, where
// a select follows, by each of several that share out the stores.
constexpr uint32_t BOUND_SHIFT = 12, BOUND_LOG_BINS = 11;   // first digit from a bound: 2^12 keys a bin
constexpr uint32_t SHARES_AIM = 64;
constexpr int RES_BLOCK = SEL_BLOCK;
constexpr int RES_WAVES = RES_BLOCK / WAVE;
static_assert(RES_BLOCK == 1024, "pick_bin is written for 1024 threads");
constexpr int ROWS_MAX = 6;                        // quads of a thread in a share of candidates
// Up to SINGLE_ROWS rows of candidates (ROWS_MAX of the threshold alone) are a single share,
// if they are spread: every workgroup of HELPERS holds all of them in registers, finds the
// answer for itself and writes out a part.
constexpr int SINGLE_ROWS = 10;
constexpr uint32_t HELPERS = 32, ALIKE = 10;
constexpr uint32_t ROW = RES_BLOCK * 4;

// What the digits run over: the keys of candidates in any order (cand_count of them);
// the values of candidates in index order, with their indices (collected); the whole
// vector, with a bound.
enum ResolveOver { OVER_KEYS = 1, OVER_COLLECTED = 2, OVER_BOUNDED = 3 };

struct Digit {                                     // a digit, or its result
    uint32_t base, shift, bins;                    // keys base .. base + (bins << shift) - 1
    bool higher;                                   // keys above those are counted too
    uint32_t k_rem, above;                         // rank to find among them and higher ones; keys above all that
    bool found;                                    // base is the key of the answer,
    uint32_t equal;                                // which so many keys share
};
__device__ __forceinline__ Digit general_digit(uint32_t k) { return Digit{0u, 20u, 1u << RS_BITS1, false, k, 0u, false, 0u}; }
__device__ __forceinline__ Digit bound_digit(uint32_t bound, uint32_t k) {
    return Digit{bound, BOUND_SHIFT, 1u << BOUND_LOG_BINS, true, k, 0u, false, 0u};
}
// What follows a digit whose histogram is complete (`higher`: its count of higher
// keys).  Called by the whole workgroup; uniform.
template <bool ELSEWHERE>
__device__ __forceinline__ Digit next_digit(const Digit& d, const uint32_t* hist, uint32_t higher, uint32_t k,
                                            uint32_t* s_wave, uint32_t* s_result) {
    const uint32_t beyond = d.higher ? higher : 0u;
    const uint32_t want = d.k_rem > beyond ? d.k_rem - beyond : 0u;
    pick_bin<ELSEWHERE>(hist, d.bins, want, s_wave, s_result);
    const uint32_t bin = uniform(s_result[0]), above = uniform(s_result[1]);
    if (bin == ~0u) return general_digit(k);      // more than an octave above the bound, or below it
    Digit r = d;
    r.base += bin << d.shift;
    r.k_rem = want - above;
    r.above += beyond + above;
    r.equal = uniform(s_result[2]);
    r.found = d.shift == 0;
    r.higher = false;
    r.bins = d.shift == BOUND_SHIFT ? 1u << BOUND_SHIFT : d.shift == 20 ? 1u << RS_BITS2 : 1u << RS_BITS3;
    r.shift = d.shift == 20 ? 9u : 0u;
    return r;
}

// A share of candidates in registers: rows of 4096, four consecutive ones a thread.
template <bool INDICES>
struct CandRows {
    uint32_t key[ROWS_MAX][4];                     // the value's bits
    uint32_t idx[INDICES ? ROWS_MAX : 1][4];
    uint32_t have;                                 // bit 4 row + c: there is one
    __device__ __forceinline__ void load(const uint32_t* __restrict__ vals, const uint32_t* __restrict__ indices,
                                         uint32_t start, uint32_t end) {
        // No branch between the loads: rows past the end read the last quad again (the
        // arrays have room for whole quads).
        const uint32_t last = (end - 1) / 4 * 4;
        have = 0;
#pragma unroll
        for (int r = 0; r < ROWS_MAX; ++r) {
            const uint32_t i = start + r * ROW + 4u * threadIdx.x, q = i < last ? i : last;
            const uint4 v = *reinterpret_cast<const uint4*>(vals + q);
            key[r][0] = v.x; key[r][1] = v.y; key[r][2] = v.z; key[r][3] = v.w;
            if (INDICES) {
                const uint4 j = *reinterpret_cast<const uint4*>(indices + q);
                idx[r][0] = j.x; idx[r][1] = j.y; idx[r][2] = j.z; idx[r][3] = j.w;
            }
            const uint32_t n = i < end ? (end - i < 4 ? end - i : 4u) : 0u;
            have |= ((1u << n) - 1u) << (4 * r);
        }
    }
};

// `vec`: the whole vector; the residual if SELECT.
template <bool SELECT>
__global__ __launch_bounds__(RES_BLOCK) void resolve_kernel(
    float* __restrict__ vec, uint32_t n, uint32_t k, RadixState* state, uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ cand_idx, float* __restrict__ cand, uint64_t cand_cap, int over,
    float* threshold_out, uint64_t* count_ge_out, uint32_t* __restrict__ idx_out,
    float* __restrict__ val_out, uint64_t capacity, uint64_t* __restrict__ nnz_out, ScanHeader* hdr,
    uint64_t* seg_desc, uint64_t* group_desc, uint32_t nseg, uint32_t piece) {
    constexpr uint32_t BINS_MAX = 4096;
    constexpr int STASH = SELECT ? SEL_STASH : 1;
    // the histogram of a digit and the stashes of the select are never in use together
    constexpr size_t LDS = SELECT ? sizeof(StashMemory<RES_WAVES, STASH>) : BINS_MAX * 4;
    static_assert(LDS >= BINS_MAX * 4, "room for a histogram");
    __shared__ __attribute__((aligned(16))) unsigned char s_memory[LDS];
    __shared__ uint32_t s_count[RES_WAVES], s_result[3], s_before[2], s_rows[ROWS_MAX][RES_WAVES];
    __shared__ uint32_t s_ticket, s_last, s_higher, s_give_up, s_few;
    uint32_t* s_hist = reinterpret_cast<uint32_t*>(s_memory);
    const uint32_t tid = threadIdx.x;

    // ---- alike in every workgroup ----
    const uint32_t bound = cand_bound(state);
    const uint64_t found = over == OVER_COLLECTED ? state->collected[1]
                         : over == OVER_KEYS ? (uint64_t)state->cand_count : 0ull;
    const bool use_cand = k <= found && found <= cand_cap;                   // rank k is among the candidates
    const bool bounded = use_cand || over == OVER_BOUNDED;
    const uint32_t len = use_cand ? (uint32_t)found : n;
    float* walked = use_cand ? cand : vec;
    uint32_t per_share = piece * (uint32_t)RES_WAVES;                        // the launch's, for the whole vector
    if (bounded) {
        // whole rows: as many as make SHARES_AIM shares; of candidates at most ROWS_MAX, which
        // registers hold
        uint32_t rows = (uint32_t)(((uint64_t)len + SHARES_AIM * ROW - 1) / (SHARES_AIM * ROW));
        if (use_cand && rows > (uint32_t)ROWS_MAX) rows = ROWS_MAX;
        // no more shares than the launch has descriptors for
        const uint32_t least = (uint32_t)(((uint64_t)len + (uint64_t)nseg * ROW - 1) / ((uint64_t)nseg * ROW));
        if (rows < least) rows = least;
        per_share = rows * ROW;
    }
    const uint32_t used = (uint32_t)(((uint64_t)len + per_share - 1) / per_share);
    // There is work for as many workgroups as there are shares.  Of a single share all find
    // the answer for themselves, from registers and LDS, and each writes out a part: no
    // exchange, which costs some eight microseconds a digit, and not all of the stores, most of
    // them to lines of their own, from one compute unit.  Refresh iterations, us:
    //                               digits across workgroups   one workgroup   32, the last digit gathered
    //   1 M, 1 % (13,600 candidates)                              33.4         25.6
    //   1 M, 2 % (26,400)                     35.2                             30.9
    //   2 M, 1 % (26,600)                     37.3                             34.9
    //   4 M, 1 % (52,000)                     41.0                             42.2 (with room for 81,920)
    bool single = use_cand && len <= (SELECT ? SINGLE_ROWS : ROWS_MAX) * ROW;
    if (single && len > ROWS_MAX * ROW) {
        // More than ROWS_MAX rows are a single share only if their keys are spread.  Keys that share
        // a bin queue for one word of LDS, some seven cycles each, and ten rows of them in one
        // workgroup take longer than a row in each of ten; so does the threshold alone (!SELECT),
        // as it has no stores to share out.  The first row, which all workgroups see alike,
        // says it: one of four lanes of some wave is among more than ALIKE in a bin.  Refresh
        // iterations of 1 M elements (27,000 and 40,000 candidates), us, shares / single / as the
        // first row says: spread 37.3 / 28.2 / 30.2 and 37.8 / 31.3 / 32.8, of four values
        // 38.3 / 41.0 / 39.1 and 38.7 / 49.8 / 39.4, half of them equal 40.2 / 47.4 / 40.9.
        const uint32_t bin = (magnitude_key(cand[4u * tid]) - bound) >> BOUND_SHIFT;
        uint32_t alike = 0;
#pragma unroll
        for (int l = 0; l < WAVE; l += WAVE / 4) {
            const uint32_t here = (uint32_t)__popcll(__ballot(bin == (uint32_t)__builtin_amdgcn_readlane((int)bin, l)));
            alike = here > alike ? here : alike;
        }
        single = !__syncthreads_or(alike > ALIKE);
    }
    const uint32_t helpers = !SELECT || !single ? 1u : gridDim.x < HELPERS ? gridDim.x : HELPERS;
    if (blockIdx.x >= (single ? helpers : used)) return;
    // A bound of zero over the whole vector: fewer than k elements, as far as the sample
    // saw, that are not, so the answer is zero most likely, which the digits from there
    // find in two (1 M elements, all but a thousandth of them zero: 36 us, general ones 42).
    Digit d = bounded || bound == 0 ? bound_digit(bound, k) : general_digit(k);

    // this share's counts of a digit
    uint32_t higher = 0;
    auto clear_hist = [&]() {
        higher = 0;
        for (uint32_t b = tid; b < d.bins; b += RES_BLOCK) s_hist[b] = 0;
        if (tid == 0) s_higher = 0;
        __syncthreads();
    };
    auto take = [&](uint32_t key) {
        const uint32_t bin = (key - d.base) >> d.shift;              // below the base: wraps to the far end
        if (bin < d.bins) atomicAdd(&s_hist[bin], 1u);
        else if ((int32_t)key >= (int32_t)d.base) ++higher;          // (all ones: no candidate)
    };
    // `crowd`: many of the wave's share a bin.  (Ties at the top of the candidates, 1 % of
    // 1 M elements: 47.7 us for the exact threshold with one add an element, 33 so.)
    auto crowd_of = [&](uint32_t key) { return crowded((key - d.base) >> d.shift, d.bins); };
    auto take_crowd = [&](uint32_t key) {
        add_crowd(s_hist, (key - d.base) >> d.shift, d.bins, [&]() { take(key); });
    };
    auto take_quad = [&](const float4& v, bool crowd) {
        const uint32_t a = magnitude_key(v.x), b = magnitude_key(v.y), e = magnitude_key(v.z), f = magnitude_key(v.w);
        if (crowd) {
            take_crowd(a); take_crowd(b); take_crowd(e); take_crowd(f);
        } else {
            take(a); take(b); take(e); take(f);
        }
    };
    auto counted = [&]() {
        if (d.higher) {
            higher = wave_sum(higher);
            if ((tid & (WAVE - 1)) == 0 && higher) atomicAdd(&s_higher, higher);
        }
        __syncthreads();
    };
    // The candidates of a share at or above the threshold: their places from a scan over
    // rows and waves, and over the shares before; stores straight from registers.
    auto compact = [&](const auto& rows, uint32_t share) {
        uint32_t chosen = 0, packed[2] = {0, 0};                     // per row: ten bits hold a wave's 256
#pragma unroll
        for (int r = 0; r < ROWS_MAX; ++r) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if ((rows.key[r][c] & ABS_MASK) >= d.base) chosen |= 1u << (4 * r + c);
        }
        chosen &= rows.have;
#pragma unroll
        for (int r = 0; r < ROWS_MAX; ++r) packed[r / 3] += (uint32_t)__popc(chosen >> (4 * r) & 15u) << (10 * (r % 3));
        const uint32_t incl[2] = {wave_inclusive_scan_u32(packed[0]), wave_inclusive_scan_u32(packed[1])};
        const int wave = (int)uniform(tid >> 6), lane = tid & (WAVE - 1);
        if (lane == WAVE - 1)
#pragma unroll
            for (int r = 0; r < ROWS_MAX; ++r) s_rows[r][wave] = incl[r / 3] >> (10 * (r % 3)) & 1023u;
        __syncthreads();
        if (wave == 0) {
            constexpr int CELLS = ROWS_MAX * RES_WAVES;
            static_assert(CELLS <= 2 * WAVE && CELLS % 2 == 0, "two cells a lane");
            uint32_t* cells = &s_rows[0][0];
            const bool in = 2 * lane < CELLS;
            const uint32_t c0 = in ? cells[2 * lane] : 0u, c1 = in ? cells[2 * lane + 1] : 0u;
            const uint32_t upto = wave_inclusive_scan_u32(c0 + c1);
            const uint32_t aggregate = (uint32_t)__builtin_amdgcn_readlane((int)upto, WAVE - 1);
            const uint32_t before = scan_within_group(hdr, seg_desc, group_desc, share, aggregate);
            if (lane == 0) {
                s_before[0] = before;
                s_count[0] = aggregate;
            }
            if (in) {
                cells[2 * lane] = upto - c0 - c1;
                cells[2 * lane + 1] = upto - c1;
            }
        } else if (wave == 1) {
            const uint32_t before = scan_across_groups(hdr, group_desc, share / SCAN_GROUP);
            if (lane == 0) s_before[1] = before;
        }
        __syncthreads();
        const uint32_t exclusive = uniform(s_before[0] + s_before[1]), aggregate = uniform(s_count[0]);
        if (tid == 0 && share / SCAN_GROUP != 0 && share % SCAN_GROUP == SCAN_GROUP - 1)
            scan_close_group(group_desc, share / SCAN_GROUP, exclusive + aggregate);
#pragma unroll
        for (int r = 0; r < ROWS_MAX; ++r) {
            uint64_t pos = (uint64_t)exclusive + s_rows[r][wave] +
                           ((incl[r / 3] - packed[r / 3]) >> (10 * (r % 3)) & 1023u);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (chosen >> (4 * r + c) & 1u) {
                    if (pos < capacity) {
                        idx_out[pos] = rows.idx[r][c];
                        val_out[pos] = __uint_as_float(rows.key[r][c]);
                        vec[rows.idx[r][c]] = 0.0f;
                    }
                    ++pos;
                }
        }
        if (share == used - 1 && tid == 0) {
            const uint64_t total = (uint64_t)exclusive + aggregate;
            const bool failed =
                __hip_atomic_load(&hdr->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            nnz_out[0] = failed ? ~0ull : (total < capacity ? total : capacity);
            nnz_out[1] = failed ? ~0ull : total;
        }
    };

    if (single) {
        // ---- one share: no exchange with other workgroups ----
        const uint32_t* vals = reinterpret_cast<const uint32_t*>(cand);
        const uint32_t rows = (len + ROW - 1) / ROW, last = (len - 1) / 4 * 4;
        const int wave = (int)uniform(tid >> 6), lane = tid & (WAVE - 1);
        uint32_t key[SINGLE_ROWS][4];                                // all ones: none, and in no digit's bins
#pragma unroll
        for (int r = 0; r < SINGLE_ROWS; ++r)
            if ((uint32_t)r < rows) {
                const uint32_t i = r * ROW + 4u * tid;
                const uint4 v = *reinterpret_cast<const uint4*>(vals + (i < last ? i : last));
                key[r][0] = v.x; key[r][1] = v.y; key[r][2] = v.z; key[r][3] = v.w;
            }
        // the first row whose 256 candidates this wave writes out
        uint32_t own = ((uint32_t)blockIdx.x + HELPERS * helpers - (uint32_t)wave) % helpers;
        uint4 own_val = uint4{0, 0, 0, 0}, own_idx = uint4{0, 0, 0, 0};
        auto load_own = [&]() {
            const uint32_t i = own * ROW + 4u * tid, q = i < last ? i : last;
            own_val = *reinterpret_cast<const uint4*>(vals + q);
            own_idx = *reinterpret_cast<const uint4*>(cand_idx + q);
        };
        if (SELECT && own < rows) load_own();
#pragma unroll
        for (int r = 0; r < SINGLE_ROWS; ++r)
            if ((uint32_t)r < rows) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    key[r][c] = r * ROW + 4u * tid + c < len ? key[r][c] & ABS_MASK : ~0u;
            }
        if (tid == 0) s_few = 0;
        while (!d.found) {
            __syncthreads();
            if (d.shift == 0 && d.equal <= FEW) {
                // The last digit of so few keys needs no histogram: they are gathered, and
                // every wave counts for each how many are larger.
#pragma unroll
                for (int r = 0; r < SINGLE_ROWS; ++r)
                    if ((uint32_t)r < rows) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (key[r][c] - d.base < d.bins) s_hist[atomicAdd(&s_few, 1u)] = key[r][c];
                    }
                __syncthreads();
                const KeyRank few = rank_of_few(s_hist, uniform(s_few), d.k_rem);
                d.base = few.key;
                d.above += few.above;
                d.equal = few.equal;
                d.found = true;
                break;
            }
            clear_hist();
            auto take_rows = [&](auto&& take_one) {
#pragma unroll
                for (int r = 0; r < SINGLE_ROWS; ++r)
                    if ((uint32_t)r < rows) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) take_one(key[r][c]);
                    }
            };
            if (crowd_of(key[0][0])) take_rows(take_crowd);
            else take_rows(take);
            counted();
            d = next_digit<false>(d, s_hist, s_higher, k, s_count, s_result);
        }
        if (tid == 0 && blockIdx.x == 0) {
            *threshold_out = __uint_as_float(d.base);
            *count_ge_out = (uint64_t)d.above + d.equal;
        }
        if constexpr (SELECT) {
            // how many of every row's and wave's 256 go out, and how many before them
            __shared__ uint32_t s_cell[SINGLE_ROWS * RES_WAVES];
#pragma unroll
            for (int r = 0; r < SINGLE_ROWS; ++r)
                if ((uint32_t)r < rows) {
                    uint32_t chosen = 0;
#pragma unroll
                    for (int c = 0; c < 4; ++c) chosen += (uint32_t)__popcll(__ballot((int32_t)key[r][c] >= (int32_t)d.base));
                    if (lane == 0) s_cell[r * RES_WAVES + wave] = chosen;
                }
            __syncthreads();
            const uint32_t cells = rows * RES_WAVES;
            if (wave == 0) {
                constexpr int PER = (SINGLE_ROWS * RES_WAVES + WAVE - 1) / WAVE;
                uint32_t c[PER], sum = 0;
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    const uint32_t i = (uint32_t)lane * PER + j;
                    c[j] = i < cells ? s_cell[i] : 0u;
                    sum += c[j];
                }
                uint32_t before = wave_inclusive_scan_u32(sum) - sum;
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    const uint32_t i = (uint32_t)lane * PER + j;
                    if (i < cells) s_cell[i] = before;
                    before += c[j];
                }
                if (lane == WAVE - 1 && blockIdx.x == 0) {
                    nnz_out[0] = before < capacity ? before : capacity;
                    nnz_out[1] = before;
                }
            }
            __syncthreads();
            while (own < rows) {
                const uint32_t i = own * ROW + 4u * tid;
                const uint32_t val[4] = {own_val.x, own_val.y, own_val.z, own_val.w};
                const uint32_t idx[4] = {own_idx.x, own_idx.y, own_idx.z, own_idx.w};
                uint32_t chosen = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (i + c < len && (val[c] & ABS_MASK) >= d.base) chosen |= 1u << c;
                const uint32_t mine = (uint32_t)__popc(chosen);
                uint64_t pos = s_cell[own * RES_WAVES + wave] + wave_inclusive_scan_u32(mine) - mine;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (chosen >> c & 1u) {
                        if (pos < capacity) {
                            idx_out[pos] = idx[c];
                            val_out[pos] = __uint_as_float(val[c]);
                            vec[idx[c]] = 0.0f;
                        }
                        ++pos;
                    }
                own += helpers;
                if (own < rows) load_own();
            }
        }
        return;
    }

    // phase q's histogram: RS_MAX_BINS words, the last digit from a bound twice that; the
    // last word of all counts the keys above a bound's octave
    uint32_t* const total_higher = hist + HIST_WORDS - 1;
    auto next_of = [&](uint32_t q) {
        const uint32_t up = d.higher ? __hip_atomic_load(total_higher, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        d = next_digit<true>(d, hist + RS_MAX_BINS * q, up, k, s_count, s_result);
    };
    uint32_t at = 0, ticket = 0;                           // the phase that d is
    if (tid == 0) ticket = atomicAdd(&state->ticket, 1u);
    for (;;) {
        __syncthreads();                                   // LDS of the share before is free
        if (tid == 0) {
            s_ticket = ticket;
            s_give_up = 0;
            ticket = atomicAdd(&state->ticket, 1u);        // asked for while this one is worked on
        }
        __syncthreads();
        const uint32_t p = uniform(s_ticket) / used, share = uniform(s_ticket) % used;
        while (at < p && !d.found) {
            if (!SELECT && d.shift == 0) return;           // nothing follows the last digit
            if (tid == 0) {
                uint32_t polls = 0;
                const uint32_t limit = state->spin_limit ? state->spin_limit : SPIN_LIMIT;
                while (__hip_atomic_load(&state->done[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != used) {
                    if (++polls > limit) {                 // give up: every count says so
                        *count_ge_out = ~0ull;
                        if (SELECT) {
                            __hip_atomic_store(&hdr->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            nnz_out[0] = nnz_out[1] = ~0ull;
                        }
                        s_give_up = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __syncthreads();
            if (uniform(s_give_up)) return;
            next_of(at++);
        }
        if (d.found) {
            // phase `at` is the select; a ticket beyond it is the end
            if (!SELECT || p > at) return;
            if constexpr (SELECT) {
                if (share == 0 && tid == 0) {
                    *threshold_out = __uint_as_float(d.base);
                    *count_ge_out = (uint64_t)d.above + d.equal;
                }
                if (use_cand && per_share <= ROWS_MAX * ROW) {
                    CandRows<true> rows;
                    const uint32_t start = share * per_share;
                    rows.load(reinterpret_cast<const uint32_t*>(cand), cand_idx, start,
                              len - start < per_share ? len : start + per_share);
                    compact(rows, share);
                } else {
                    StashMemory<RES_WAVES, STASH>& s_stash = *reinterpret_cast<StashMemory<RES_WAVES, STASH>*>(s_memory);
                    const CandidateSource source{use_cand ? cand_idx : nullptr, vec};
                    select_body<RES_BLOCK, SEL_U, STASH, false>(
                        walked, len, TestKey{d.base}, source, idx_out, val_out, capacity, nnz_out, hdr, seg_desc,
                        group_desc, used, per_share / RES_WAVES, share, s_stash, s_count, s_before);
                }
            }
            continue;
        }

        // ---- a digit ----
        clear_hist();
        const uint64_t start = (uint64_t)share * per_share;
        const uint64_t end = start + per_share < len ? start + per_share : len;
        // a pass over the whole of a vector longer than the last-level cache finds nothing
        // of it there
        const bool around_cache = !use_cand && len >= STREAM_PAST_CACHE_N;
        // of candidates, which are a few rows a share, the first row says it; of a vector
        // the first row of every four
        bool crowd = false;
        uint64_t r = start;
        for (; r + 4 * ROW <= end; r += 4 * ROW) {
            const float4* src = reinterpret_cast<const float4*>(walked + r) + tid;
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v[u] = around_cache ? load_quad<true>(src + u * RES_BLOCK) : load_quad<false>(src + u * RES_BLOCK);
            __builtin_amdgcn_sched_barrier(0);             // all out before the first is looked at
            if (!use_cand || r == start) crowd = crowd_of(magnitude_key(v[0].x));
#pragma unroll
            for (int u = 0; u < 4; ++u) take_quad(v[u], crowd);
        }
        for (; r < end; r += ROW) {
            const uint64_t i = r + 4u * tid;
            if (i + 4 <= end) {
                const float4 v = *reinterpret_cast<const float4*>(walked + i);
                if (r == start) crowd = crowd_of(magnitude_key(v.x));
                take_quad(v, crowd);
            } else {
                for (uint64_t j = i; j < end; ++j) take(magnitude_key(walked[j]));
            }
        }
        counted();
        uint32_t* total = hist + RS_MAX_BINS * p;
        uint32_t seen = 0;
        for (uint32_t b = tid; b < d.bins; b += RES_BLOCK) {           // all out first, then one wait
            const uint32_t c = s_hist[b];
            if (c) seen |= atomicAdd(&total[b], c);
        }
        if (d.higher && tid == 0 && s_higher) seen |= atomicAdd(total_higher, s_higher);
        asm volatile("" ::"v"(seen));
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(&state->done[p], 1u) == used - 1 ? 1u : 0u;
        if (!SELECT) {
            // nothing follows the last digit: the workgroup that finishes it writes the answer
            __syncthreads();
            if (uniform(s_last) && d.shift == 0) {
                next_of(p);
                if (tid == 0) {
                    *threshold_out = __uint_as_float(d.base);
                    *count_ge_out = (uint64_t)d.above + d.equal;
                }
                return;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// refresh iteration in one pass over the gradient
// ---------------------------------------------------------------------------
// The fused accumulate+select kernel run against the sample's bound: the
// residual becomes the accumulator (no zeros), every element at or above the
// bound goes, in index order, to the candidate list, whose length (written,
// found) lands in state->collected.
template <int BLOCK, int U, int STASH, int CACHE>
__global__ __launch_bounds__(BLOCK) void accumulate_collect_kernel(
    const float* __restrict__ grad, float* __restrict__ res, float lr, uint32_t n, RadixState* state,
    uint32_t* __restrict__ cand_idx, float* __restrict__ cand_val, uint64_t cand_cap,
    ScanHeader* hdr, uint64_t* seg_desc, uint64_t* group_desc, uint32_t nseg, uint32_t piece) {
    constexpr int WAVES = BLOCK / WAVE;
    __shared__ StashMemory<WAVES, STASH> s_stash;
    __shared__ uint32_t s_count[WAVES];
    __shared__ uint32_t s_seg;
    __shared__ uint32_t s_before[2];
    if (threadIdx.x == 0) s_seg = atomicAdd(&hdr->ticket, 1u);
    __syncthreads();
    const uint32_t seg = s_seg;
    const uint32_t lo_key = collect_bound(state);
    const float lo = __uint_as_float(lo_key);               // a key below the Inf/NaN range, or NaN
    if (lo == lo) {
        accumulate_select_body<BLOCK, U, STASH, false, CACHE>(
            grad, res, lr, n, TestFloat{lo}, cand_idx, cand_val, cand_cap, state->collected, hdr,
            seg_desc, group_desc, nseg, piece, seg, s_stash, s_count, s_before);
    } else {
        accumulate_select_body<BLOCK, U, STASH, false, CACHE>(
            grad, res, lr, n, TestKey{lo_key}, cand_idx, cand_val, cand_cap, state->collected, hdr,
            seg_desc, group_desc, nseg, piece, seg, s_stash, s_count, s_before);
    }
}

// The exact threshold of a short array in one workgroup and one launch: the keys stay
// in registers, the digits' histograms in LDS.  A call at 17,000 elements takes 8.8 us, at
// 30,000 9.1 us, at 65,536 15 us; the launches it replaces take 17 to 19 us, and at twice
// that length a thread's keys would no longer fit its registers.
constexpr int TINY_BLOCK = 1024;
template <uint32_t TINY_PER>                   // elements per thread
__global__ __launch_bounds__(TINY_BLOCK) void tiny_threshold_kernel(const float* __restrict__ acc, uint32_t n,
                                                                    uint32_t k, float* threshold_out,
                                                                    uint64_t* count_ge_out) {
    __shared__ uint32_t s_hist[RS_MAX_BINS];
    __shared__ uint32_t s_wave[TINY_BLOCK / WAVE], s_result[3];
    const uint32_t tid = threadIdx.x;
    uint32_t key[TINY_PER];                        // all ones: no element
#pragma unroll
    for (uint32_t u = 0; u < TINY_PER / 4; ++u) {
        const uint32_t i = 4 * (u * TINY_BLOCK + tid);
        if (i + 4 <= n) {
            const float4 v = *reinterpret_cast<const float4*>(acc + i);
            key[4 * u] = magnitude_key(v.x);
            key[4 * u + 1] = magnitude_key(v.y);
            key[4 * u + 2] = magnitude_key(v.z);
            key[4 * u + 3] = magnitude_key(v.w);
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) key[4 * u + j] = i + j < n ? magnitude_key(acc[i + j]) : ~0u;
        }
    }
    uint32_t base = 0, above = 0, k_rem = k;
#pragma unroll
    for (int digit = 0; digit < 3; ++digit) {
        const uint32_t shift = digit == 0 ? 20u : digit == 1 ? 9u : 0u;
        const uint32_t bins = digit == 2 ? 1u << RS_BITS3 : 1u << RS_BITS1;
        for (uint32_t b = tid; b < bins; b += TINY_BLOCK) s_hist[b] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < TINY_PER; ++j) {
            const uint32_t bin = (key[j] - base) >> shift;           // no element: beyond every bin
            if (bin < bins) atomicAdd(&s_hist[bin], 1u);
        }
        __syncthreads();
        pick_bin<false>(s_hist, bins, k_rem, s_wave, s_result);
        base += s_result[0] << shift;
        above += s_result[1];
        k_rem -= s_result[1];
        if (digit == 2 && tid == 0) {
            *threshold_out = __uint_as_float(base);
            *count_ge_out = (uint64_t)above + s_result[2];
        }
        __syncthreads();
    }
}

}  // namespace okt

namespace okt {

// Whether the candidates of a sampled bound are worth collecting: a vector long
// enough for the sample, and room for them - about 1.1 k where k is some percent of n,
// 2 k where it is a thousandth.  A larger share than a workspace of
// okt_workspace_bytes holds (9 % of n) is found as quickly by digits over the whole.
static bool sample_pays(uint64_t n, uint64_t k, uint64_t cand_cap) {
    return cand_cap >= k + k / 4 + n / 64;
}

template <bool SELECT>
static void launch_resolve(float* vec, uint64_t n, uint64_t k, RadixState* state, uint32_t* hist,
                           const uint32_t* cand_idx, float* cand, uint64_t cand_cap, int over,
                           float* d_threshold_out, uint64_t* d_count_ge_out, uint32_t* d_idx_out,
                           float* d_val_out, uint64_t capacity, uint64_t* d_nnz_out, char* scan,
                           const SelectShape& shape, hipStream_t s) {
    ScanHeader* hdr = (ScanHeader*)scan;
    uint64_t* seg_desc = scan ? (uint64_t*)(scan + SCAN_HEADER_BYTES) : nullptr;
    uint64_t* group_desc = scan ? seg_desc + shape.nseg : nullptr;
    // workgroups stay and take tickets: one per compute unit is all that LDS has room for
    const uint32_t grid = shape.nseg < device_cus() ? shape.nseg : device_cus();
    hipLaunchKernelGGL(resolve_kernel<SELECT>, dim3(grid), dim3(RES_BLOCK), 0, s, vec, (uint32_t)n, (uint32_t)k,
                       state, hist, cand_idx, cand, cand_cap, over, d_threshold_out, d_count_ge_out,
                       d_idx_out, d_val_out, capacity, d_nnz_out, hdr, seg_desc, group_desc, shape.nseg,
                       shape.piece);
}

}  // namespace okt

extern "C" int okt_topk_threshold_exact(const float* d_acc, uint64_t n, uint64_t k,
                                        float* d_threshold_out, uint64_t* d_count_ge_out,
                                        void* d_ws, size_t ws_bytes, void* stream) {
    using namespace okt;
    hipStream_t s = (hipStream_t)stream;
    if (!d_acc || !d_threshold_out || !d_count_ge_out) return OKT_ERR_INVALID_ARG;
    if (n == 0 || n > 0xffffffffull || k == 0 || k > n) return OKT_ERR_INVALID_ARG;
    if (!aligned(d_acc, 16) || !aligned(d_threshold_out, 4) || !aligned(d_count_ge_out, 8))
        return OKT_ERR_INVALID_ARG;
    if (!d_ws || !aligned(d_ws, 256) || ws_bytes < threshold_ws_min_bytes())
        return OKT_ERR_WORKSPACE;
    if (n <= TINY_N) {
        auto* tiny = n <= TINY_N / 4   ? tiny_threshold_kernel<TINY_N / 4 / TINY_BLOCK>
                     : n <= TINY_N / 2 ? tiny_threshold_kernel<TINY_N / 2 / TINY_BLOCK>
                                       : tiny_threshold_kernel<TINY_N / TINY_BLOCK>;
        hipLaunchKernelGGL(tiny, dim3(1), dim3(TINY_BLOCK), 0, s, d_acc, (uint32_t)n, (uint32_t)k,
                           d_threshold_out, d_count_ge_out);
        return launch_status();
    }
    RadixState* state = (RadixState*)d_ws;
    uint32_t* hist = (uint32_t*)((char*)d_ws + RS_STATE_BYTES);
    uint32_t* cand = hist + HIST_WORDS;
    const uint64_t cand_cap = ((ws_bytes - threshold_ws_min_bytes()) / 4) & ~(uint64_t)3;   // whole quads
    const SelectShape shape = select_shape(n, device_cus());
    const bool collect = sample_pays(n, k, cand_cap) && (n > BOUNDED_TO_N || k <= n / 16);
    if (!collect && n > BOUNDED_TO_N) {
        hipLaunchKernelGGL(radix_init_kernel, dim3(HIST_WORDS / 256), dim3(256), 0, s, state, hist);
        if (stream_past_cache(n)) launch_digits<true>(d_acc, n, k, state, hist, d_threshold_out, d_count_ge_out, s);
        else launch_digits<false>(d_acc, n, k, state, hist, d_threshold_out, d_count_ge_out, s);
        return launch_status();
    }
    hipLaunchKernelGGL(sample_bound_kernel, dim3(BOUNDS), dim3(SAMPLE_BLOCK), 0, s, d_acc,
                       (const float*)nullptr, 0.0f, (uint32_t)n, (uint32_t)k, state, hist,
                       (uint64_t*)nullptr, 0u, (uint64_t*)nullptr, 0u, 0u, digit_spin_limit_setting());
    if (collect) {
        static_assert(CNT_WAVES == SEL_WAVES, "the collect pass is cut like the select");
        timing_before(s);
        hipLaunchKernelGGL(stream_past_cache(n) ? collect_kernel<true> : collect_kernel<false>,
                           dim3(shape.nseg), dim3(CNT_BLOCK), 0, s, d_acc, (uint32_t)n, shape.piece,
                           state, cand, cand_cap);
        timing_after(s);
    }
    launch_resolve<false>(const_cast<float*>(d_acc), n, k, state, hist, nullptr, (float*)cand, cand_cap,
                          collect ? OVER_KEYS : OVER_BOUNDED, d_threshold_out, d_count_ge_out, nullptr,
                          nullptr, 0, nullptr, nullptr, shape, s);
    return launch_status();
}

extern "C" int okt_accumulate_topk_select(const float* d_grad, float* d_residual_inout, float lr,
                                          uint64_t n, uint64_t k, float* d_threshold_out,
                                          uint64_t* d_count_ge_out, uint32_t* d_idx_out,
                                          float* d_val_out, uint64_t capacity, uint64_t* d_nnz_out,
                                          void* d_ws, size_t ws_bytes, void* stream) {
    using namespace okt;
    hipStream_t s = (hipStream_t)stream;
    if (!d_grad || !d_residual_inout || d_grad == d_residual_inout || !d_threshold_out ||
        !d_count_ge_out || !d_nnz_out)
        return OKT_ERR_INVALID_ARG;
    if (n == 0 || n > 0xffffffffull || k == 0 || k > n) return OKT_ERR_INVALID_ARG;
    if (!aligned(d_grad, 16) || !aligned(d_residual_inout, 16) || !aligned(d_threshold_out, 4) ||
        !aligned(d_count_ge_out, 8) || !aligned(d_nnz_out, 8))
        return OKT_ERR_INVALID_ARG;
    if (capacity > 0 && (!d_idx_out || !d_val_out || !aligned(d_idx_out, 4) ||
                         !aligned(d_val_out, 4)))
        return OKT_ERR_INVALID_ARG;
    const size_t separate = threshold_ws_min_bytes() > select_ws_bytes(n) ? threshold_ws_min_bytes()
                                                                           : select_ws_bytes(n);
    if (!d_ws || !aligned(d_ws, 256) || ws_bytes < separate) return OKT_ERR_WORKSPACE;

    const SelectShape shape = select_shape(n, device_cus());
    const size_t scan_bytes = refresh_scan_bytes(n);
    // The collection of the candidates goes through per-tile slots where the vector
    // is long enough and the workspace has room for them next to the candidates;
    // else through the chained scan of the one-kernel select.
    const SlotPlan plan = slot_plan(n, device_cus());
    const size_t slot_bytes = round_up_256(plan.bytes);
    bool slots = n >= slot_min_n(true) && ws_bytes > threshold_ws_min_bytes() + scan_bytes + slot_bytes;
    size_t fixed = threshold_ws_min_bytes() + scan_bytes + (slots ? slot_bytes : scan_bytes);
    uint64_t cand_cap = ws_bytes > fixed ? ((ws_bytes - fixed) / 8) & ~(uint64_t)63 : 0;
    if (slots && cand_cap < n / 16) {
        slots = false;
        fixed = threshold_ws_min_bytes() + 2 * scan_bytes;
        cand_cap = ws_bytes > fixed ? ((ws_bytes - fixed) / 8) & ~(uint64_t)63 : 0;
    }
    if (n < RS_SAMPLE_FROM_N || !sample_pays(n, k, cand_cap)) {
        // short vector, large k, or a workspace without room for candidates: the three steps
        // one after the other, each with the workspace to itself
        int rc = okt_residual_accumulate(d_grad, d_residual_inout, lr, n, stream);
        if (rc != OKT_OK) return rc;
        rc = okt_topk_threshold_exact(d_residual_inout, n, k, d_threshold_out, d_count_ge_out, d_ws,
                                      ws_bytes, stream);
        if (rc != OKT_OK) return rc;
        return okt_threshold_select(d_residual_inout, n, d_threshold_out, d_idx_out, d_val_out,
                                    capacity, d_nnz_out, d_ws, ws_bytes, stream);
    }

    RadixState* state = (RadixState*)d_ws;
    uint32_t* hist = (uint32_t*)((char*)d_ws + RS_STATE_BYTES);
    char* scan_b = (char*)d_ws + threshold_ws_min_bytes();          // the final select's
    char* scan_a = scan_b + scan_bytes;                             // the collection's, or the slots
    float* cand_val = (float*)(scan_a + (slots ? slot_bytes : scan_bytes));
    uint32_t* cand_idx = (uint32_t*)(cand_val + cand_cap);
    auto header = [](char* p) { return (ScanHeader*)p; };
    auto segs = [](char* p) { return (uint64_t*)(p + SCAN_HEADER_BYTES); };

    const uint32_t words_b = (uint32_t)(scan_ws_bytes(shape.nseg) / 8);
    const uint32_t words_a = slots ? (uint32_t)(scan_ws_bytes(plan.nseg) / 8) : words_b;
    hipLaunchKernelGGL(sample_bound_kernel, dim3(BOUNDS), dim3(SAMPLE_BLOCK), 0, s, d_residual_inout, d_grad, lr,
                       (uint32_t)n, (uint32_t)k, state, hist, (uint64_t*)scan_a, words_a, (uint64_t*)scan_b,
                       words_b, spin_limit_setting() ? spin_limit_setting() : digit_spin_limit_setting(),
                       digit_spin_limit_setting());
    const CacheUse use = accumulate_cache_use(n);
    if (slots) {
        // the sample's bounds are magnitude keys, so their bits read as fp32 are the
        // bounds themselves: the slot kernels take the least for their threshold
        const float* bound = reinterpret_cast<const float*>(state->bound);
        timing_before(s);
        auto* fill = use == ALL_PAST_CACHE        ? slot_fill_accumulate_kernel<false, ALL_PAST_CACHE>
                     : use == GRADIENT_PAST_CACHE ? slot_fill_accumulate_kernel<false, GRADIENT_PAST_CACHE>
                                                  : slot_fill_accumulate_kernel<false, CACHED>;
        constexpr uint32_t per_wg = SLOT_FILL_BLOCK / WAVE;
        hipLaunchKernelGGL(fill, dim3((plan.ntiles + per_wg - 1) / per_wg), dim3(SLOT_FILL_BLOCK), 0,
                           s, d_grad, d_residual_inout, lr, (uint32_t)n, bound,
                           (uint16_t*)(scan_a + plan.counts_at), (SlotEntry*)(scan_a + plan.slots_at),
                           plan.ntiles, (uint64_t*)nullptr, 0u, 0u);      // sample_bound_kernel cleared it
        timing_after(s);
        const int rc = launch_slot_finish(d_residual_inout, n, bound, plan, scan_a, SLOT_KEEP,
                                          cand_idx, cand_val, cand_cap, state->collected, s, BOUNDS);
        if (rc != OKT_OK) return rc;
    } else {
        timing_before(s);
        auto* collect =
            use == ALL_PAST_CACHE        ? accumulate_collect_kernel<SEL_BLOCK, SEL_U, SEL_STASH, ALL_PAST_CACHE>
            : use == GRADIENT_PAST_CACHE ? accumulate_collect_kernel<SEL_BLOCK, SEL_U, SEL_STASH, GRADIENT_PAST_CACHE>
                                         : accumulate_collect_kernel<SEL_BLOCK, SEL_U, SEL_STASH, CACHED>;
        hipLaunchKernelGGL(collect, dim3(shape.nseg), dim3(SEL_BLOCK), 0, s, d_grad, d_residual_inout,
                           lr, (uint32_t)n, state, cand_idx, cand_val, cand_cap, header(scan_a),
                           segs(scan_a), segs(scan_a) + shape.nseg, shape.nseg, shape.piece);
        timing_after(s);
    }

    launch_resolve<true>(d_residual_inout, n, k, state, hist, cand_idx, cand_val, cand_cap, OVER_COLLECTED, d_threshold_out,
                         d_count_ge_out, d_idx_out, d_val_out, capacity, d_nnz_out, scan_b, shape, s);
    return launch_status();
}
