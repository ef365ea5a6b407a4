// okt_coo_threshold_select: the threshold selection over a sorted COO list instead of a
// dense vector (Algorithm 1, line 13, the local part; Sec. 3.1.2).
//
// 4 B read per entry plus 12 B per selected entry; the lists are short (k entries or
// so), so a call is made of launches and latency.
#include "okt_select_kernel.h"
#include "okt_sizes.h"

namespace okt {

// ---- short COO lists ----
// A list of up to COO_SMALL_N entries is selected by one workgroup in one launch, one of
// up to COO_TILED_N by many in two: the first counts what every tile selects, the
// second adds up the counts before its tile, tests its entries again and writes them.
// No scan across workgroups, so nothing to clear and no tickets: 11,700 entries 5.0 us
// (clearing and the kernel for long lists 1.4 + 6.6), 256,000 entries 3.8 + 3.6 us (4.2 + 9.8).
constexpr int COO_BLOCK = 256;
constexpr uint32_t COO_TILE = COO_BLOCK * 4;

// A thread's quad of the list: four values, and which of them are there and selected.
struct CooQuad {
    float v[4];
    uint32_t sel;
    __device__ __forceinline__ void load(const float* __restrict__ val_in, uint32_t i, uint32_t most) {
        if (i + 4 <= most) {
            const float4 x = *reinterpret_cast<const float4*>(val_in + i);
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = i + c < most ? val_in[i + c] : 0.0f;
        }
    }
    __device__ __forceinline__ void test(uint32_t i, uint32_t n, uint32_t th_key) {
        sel = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (i + c < n && magnitude_key(v[c]) >= th_key) sel |= 1u << c;
    }
};
__device__ __forceinline__ void coo_load_indices(uint32_t (&idx)[4], const uint32_t* __restrict__ idx_in, uint32_t i,
                                                 uint32_t most) {
    if (i + 4 <= most) {
        const QuadAt4 x = *reinterpret_cast<const QuadAt4*>(idx_in + i);
#pragma unroll
        for (int c = 0; c < 4; ++c) idx[c] = x.v[c];
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) idx[c] = i + c < most ? idx_in[i + c] : 0u;
    }
}
__device__ __forceinline__ uint32_t coo_length(const uint64_t* d_nnz_in, uint32_t max_nnz) {
    const uint64_t have = *d_nnz_in;
    return have < max_nnz ? (uint32_t)have : max_nnz;
}

constexpr int COO_SMALL_BLOCK = 1024;
template <int ROWS>                              // quads per thread
__global__ __launch_bounds__(COO_SMALL_BLOCK) void coo_small_kernel(
    const uint32_t* idx_in, const float* val_in, const uint64_t* d_nnz_in, uint32_t max_nnz, const float* d_threshold,
    uint32_t* idx_out, float* val_out, uint64_t capacity, uint64_t* nnz_out) {
    constexpr int WAVES = COO_SMALL_BLOCK / WAVE, CELLS = ROWS * WAVES;
    static_assert(CELLS <= 2 * WAVE && CELLS % 2 == 0, "two cells a lane");
    __shared__ uint32_t s_cell[CELLS + 1];
    const uint32_t tid = threadIdx.x;
    const int lane = tid & (WAVE - 1), wave = (int)uniform(tid >> 6);
    // Everything is asked for at once, up to the host's bound, and read before anything is
    // written: outputs may take the place of inputs.
    CooQuad q[ROWS];
    uint32_t idx[ROWS][4], incl[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) q[r].load(val_in, 4 * (r * COO_SMALL_BLOCK + tid), max_nnz);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) coo_load_indices(idx[r], idx_in, 4 * (r * COO_SMALL_BLOCK + tid), max_nnz);
    const uint32_t n = coo_length(d_nnz_in, max_nnz), th_key = magnitude_key(*d_threshold);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        q[r].test(4 * (r * COO_SMALL_BLOCK + tid), n, th_key);
        incl[r] = wave_inclusive_scan_u32((uint32_t)__popc(q[r].sel));
        if (lane == WAVE - 1) s_cell[r * WAVES + wave] = incl[r];
    }
    __syncthreads();
    if (wave == 0) {
        const bool in = 2 * lane < CELLS;
        const uint32_t c0 = in ? s_cell[2 * lane] : 0u, c1 = in ? s_cell[2 * lane + 1] : 0u;
        const uint32_t upto = wave_inclusive_scan_u32(c0 + c1);
        if (in) {
            s_cell[2 * lane] = upto - c0 - c1;
            s_cell[2 * lane + 1] = upto - c1;
        }
        if (lane == WAVE - 1) s_cell[CELLS] = upto;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        uint64_t pos = s_cell[r * WAVES + wave] + incl[r] - (uint32_t)__popc(q[r].sel);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (q[r].sel >> c & 1u) {
                if (pos < capacity) {
                    idx_out[pos] = idx[r][c];
                    val_out[pos] = q[r].v[c];
                }
                ++pos;
            }
    }
    if (tid == 0) {
        const uint64_t total = s_cell[CELLS];
        nnz_out[0] = total < capacity ? total : capacity;
        nnz_out[1] = total;
    }
}

__global__ __launch_bounds__(COO_BLOCK) void coo_count_kernel(
    const float* __restrict__ val_in, const uint64_t* __restrict__ d_nnz_in, uint32_t max_nnz,
    const float* __restrict__ d_threshold, uint16_t* __restrict__ counts) {
    __shared__ uint32_t s_wave[COO_BLOCK / WAVE];
    const uint32_t tid = threadIdx.x, i = blockIdx.x * COO_TILE + 4 * tid;
    CooQuad q;
    q.load(val_in, i, max_nnz);
    q.test(i, coo_length(d_nnz_in, max_nnz), magnitude_key(*d_threshold));
    const uint32_t sum = wave_sum((uint32_t)__popc(q.sel));
    if ((tid & (WAVE - 1)) == 0) s_wave[tid >> 6] = sum;
    __syncthreads();
    if (tid == 0) {
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < COO_BLOCK / WAVE; ++w) total += s_wave[w];
        counts[blockIdx.x] = (uint16_t)total;
    }
}

__global__ __launch_bounds__(COO_BLOCK) void coo_emit_kernel(
    const uint32_t* __restrict__ idx_in, const float* __restrict__ val_in, const uint64_t* __restrict__ d_nnz_in,
    uint32_t max_nnz, const float* __restrict__ d_threshold, const uint16_t* __restrict__ counts,
    uint32_t* __restrict__ idx_out, float* __restrict__ val_out, uint64_t capacity, uint64_t* __restrict__ nnz_out) {
    constexpr int WAVES = COO_BLOCK / WAVE;
    __shared__ uint32_t s_before[WAVES], s_wave[WAVES];
    const uint32_t tid = threadIdx.x, tile = blockIdx.x, i = tile * COO_TILE + 4 * tid;
    const int lane = tid & (WAVE - 1), wave = (int)uniform(tid >> 6);
    uint32_t before = 0;
    for (uint32_t t = tid; t < tile; t += COO_BLOCK) before += counts[t];
    CooQuad q;
    q.load(val_in, i, max_nnz);
    uint32_t idx[4];
    coo_load_indices(idx, idx_in, i, max_nnz);
    q.test(i, coo_length(d_nnz_in, max_nnz), magnitude_key(*d_threshold));
    before = wave_sum(before);
    const uint32_t mine = (uint32_t)__popc(q.sel), incl = wave_inclusive_scan_u32(mine);
    if (lane == WAVE - 1) {
        s_before[wave] = before;
        s_wave[wave] = incl;
    }
    __syncthreads();
    uint32_t first = 0, in_tile = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        first += s_before[w] + (w < wave ? s_wave[w] : 0u);
        in_tile += s_wave[w];
    }
    uint64_t pos = (uint64_t)first + incl - mine;
    if (tile == gridDim.x - 1 && tid == 0) {                        // wave 0: `first` is all before the tile
        const uint64_t total = (uint64_t)first + in_tile;
        nnz_out[0] = total < capacity ? total : capacity;
        nnz_out[1] = total;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (q.sel >> c & 1u) {
            if (pos < capacity) {
                idx_out[pos] = idx[c];
                val_out[pos] = q.v[c];
            }
            ++pos;
        }
}

// ---- long COO lists ----
// The same selection over the values of a sorted COO list whose length is on the
// device (at most max_nnz): entries at or above the threshold are copied, in
// order, with their indices; the input is not modified.
template <int BLOCK, int U, int STASH>
__global__ __launch_bounds__(BLOCK) void coo_select_kernel(
    const uint32_t* __restrict__ idx_in, const float* __restrict__ val_in,
    const uint64_t* __restrict__ d_nnz_in, uint32_t max_nnz,
    const float* __restrict__ d_threshold, uint32_t* __restrict__ idx_out,
    float* __restrict__ val_out, uint64_t capacity, uint64_t* __restrict__ nnz_out,
    ScanHeader* hdr, uint64_t* seg_desc, uint64_t* group_desc, uint32_t nseg, uint32_t piece) {
    constexpr int WAVES = BLOCK / WAVE;
    __shared__ StashMemory<WAVES, STASH> s_stash;
    __shared__ uint32_t s_count[WAVES];
    __shared__ uint32_t s_seg;
    __shared__ uint32_t s_before[2];
    if (threadIdx.x == 0) s_seg = atomicAdd(&hdr->ticket, 1u);
    __syncthreads();
    const uint32_t seg = s_seg;
    const uint64_t have = *d_nnz_in;
    const uint32_t n = have < max_nnz ? (uint32_t)have : max_nnz;
    float* vals = const_cast<float*>(val_in);         // CooSource never writes
    const float th = *d_threshold;
    if (th == th) {
        select_body<BLOCK, U, STASH, false>(vals, n, TestFloat{__builtin_fabsf(th)},
                                             CooSource{idx_in}, idx_out, val_out, capacity,
                                             nnz_out, hdr, seg_desc, group_desc, nseg, piece, seg,
                                             s_stash, s_count, s_before);
    } else {
        select_body<BLOCK, U, STASH, false>(vals, n, TestKey{magnitude_key(th)},
                                             CooSource{idx_in}, idx_out, val_out, capacity,
                                             nnz_out, hdr, seg_desc, group_desc, nseg, piece, seg,
                                             s_stash, s_count, s_before);
    }
}

}  // namespace okt

extern "C" int okt_coo_threshold_select(const uint32_t* d_idx_in, const float* d_val_in,
                                        const uint64_t* d_nnz_in, uint64_t max_nnz,
                                        const float* d_threshold, uint32_t* d_idx_out,
                                        float* d_val_out, uint64_t capacity, uint64_t* d_nnz_out,
                                        void* d_ws, size_t ws_bytes, void* stream) {
    using namespace okt;
    hipStream_t s = (hipStream_t)stream;
    if (!d_nnz_out || !aligned(d_nnz_out, 8)) return OKT_ERR_INVALID_ARG;
    if (max_nnz > 0xffffffffull) return OKT_ERR_INVALID_ARG;
    if (max_nnz == 0) {
        hipLaunchKernelGGL(select_empty_kernel, dim3(1), dim3(1), 0, s, d_nnz_out);
        return launch_status();
    }
    if (!d_idx_in || !d_val_in || !d_nnz_in || !d_threshold || !aligned(d_idx_in, 4) ||
        !aligned(d_val_in, 16) || !aligned(d_nnz_in, 8) || !aligned(d_threshold, 4))
        return OKT_ERR_INVALID_ARG;
    if (capacity > 0 && (!d_idx_out || !d_val_out || !aligned(d_idx_out, 4) ||
                         !aligned(d_val_out, 4)))
        return OKT_ERR_INVALID_ARG;
    const SelectShape shape = select_shape(max_nnz, device_cus());
    if (!d_ws || !aligned(d_ws, 256) || ws_bytes < select_ws_bytes(max_nnz))
        return OKT_ERR_WORKSPACE;
    if (max_nnz <= COO_SMALL_N) {
        auto* small = max_nnz <= COO_SMALL_N / 2 ? coo_small_kernel<(int)(COO_SMALL_N / 2 / (4 * COO_SMALL_BLOCK))>
                                                 : coo_small_kernel<(int)(COO_SMALL_N / (4 * COO_SMALL_BLOCK))>;
        timing_before(s);
        hipLaunchKernelGGL(small, dim3(1), dim3(COO_SMALL_BLOCK), 0, s, d_idx_in, d_val_in, d_nnz_in,
                           (uint32_t)max_nnz, d_threshold, d_idx_out, d_val_out, capacity, d_nnz_out);
        timing_after(s);
        return launch_status();
    }
    // The second launch by tiles reads the length and the values again while other workgroups
    // already write: outputs that take their place are for the kernel for long lists.
    const uint64_t most_out = capacity < max_nnz ? capacity : max_nnz;
    const bool over_input = overlap(d_nnz_out, 16, d_nnz_in, 8) || overlap(d_val_out, 4 * most_out, d_val_in, 4 * max_nnz);
    if (max_nnz <= COO_TILED_N && !over_input) {
        uint16_t* counts = (uint16_t*)d_ws;
        const dim3 grid((unsigned)((max_nnz + COO_TILE - 1) / COO_TILE));
        hipLaunchKernelGGL(coo_count_kernel, grid, dim3(COO_BLOCK), 0, s, d_val_in, d_nnz_in, (uint32_t)max_nnz,
                           d_threshold, counts);
        timing_before(s);
        hipLaunchKernelGGL(coo_emit_kernel, grid, dim3(COO_BLOCK), 0, s, d_idx_in, d_val_in, d_nnz_in,
                           (uint32_t)max_nnz, d_threshold, counts, d_idx_out, d_val_out, capacity, d_nnz_out);
        timing_after(s);
        return launch_status();
    }
    ScanHeader* hdr = (ScanHeader*)d_ws;
    uint64_t* seg_desc = (uint64_t*)((char*)d_ws + SCAN_HEADER_BYTES);
    uint64_t* group_desc = seg_desc + shape.nseg;
    if (launch_clear_scan_state(d_ws, scan_ws_bytes(shape.nseg) / 8, s) != hipSuccess)
        return OKT_ERR_HIP;
    timing_before(s);
    hipLaunchKernelGGL((coo_select_kernel<SEL_BLOCK, SEL_U, SEL_STASH>),
                       dim3(shape.nseg), dim3(SEL_BLOCK), 0, s, d_idx_in, d_val_in, d_nnz_in,
                       (uint32_t)max_nnz, d_threshold, d_idx_out, d_val_out, capacity, d_nnz_out,
                       hdr, seg_desc, group_desc, shape.nseg, shape.piece);
    timing_after(s);
    return launch_status();
}
