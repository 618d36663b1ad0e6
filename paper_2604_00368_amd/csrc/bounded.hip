// Bounded, pipelined staging (Section 4.1 of the paper: the payload is partitioned into chunks that
// pass through an intermediate buffer of fixed size).  The payload -- the transfers' bytes laid end to
// end in declaration order -- is cut into chunks of chunk_bytes; chunks pass through the staging
// arena one after the other, in one launch each where the batch allows one-pass copies (see copy.hip), else as gather
// of the chunk, then scatter of the chunk.  Inside the arena every rail keeps one contiguous region per chunk (chunk
// c lives in slot c mod slots of the arena, so that with two slots and two passes a chunk can be gathered while its
// predecessor is still being scattered): the chunk's bytes on rail d form an interval
// [lo_d, hi_d) of the rail's staging offsets, they sit at region_base_d + (offset - lo_d), and the
// region bases are the exclusive sum of the interval lengths rounded up to 256 bytes.
//
// All copies walk the chunk's tiles in declaration order (a chunk is a contiguous range of that
// enumeration), so a chunk's launch touches only its own table entries.
//
// Geometry whose lengths are no multiple of the tile size has no such enumeration.  There the same
// steps run over the payload in ranges of 1 KiB, one wavefront per range: the first step finds the
// slice that holds the range's first byte (transfers are laid end to end, so slices start at ascending
// payload positions) and keeps it, and the copies go through the slices that intersect the range, byte-exactly.
#include "copy_generic.h"

namespace tent {
namespace {

constexpr uint64_t kNoTile = ~0ull;
constexpr uint64_t kRegMask = (1ull << 56) - 1;
constexpr int kBothLanes = 512;

__global__ void __launch_bounds__(256) bounded_clear_kernel(BatchDev b, uint32_t n_chunks)
{
    const uint32_t at = blockIdx.x * blockDim.x + threadIdx.x;
    if (at < n_chunks * TENT_MAX_RAILS) {
        b.ch_lo[at] = kNoTile;
        b.ch_hi[at] = 0;
    }
    if (at == 0) b.plan->bounded_overflow = 0;
}

// Per tile (declaration order): rail and staging offset of its first byte, or kNoTile when its slice is
// not BOUND; per (chunk, rail): the interval of staging offsets the chunk touches.  A workgroup covers
// 256 consecutive tiles, which lie in one chunk because a chunk holds a multiple of 256 tiles.
__global__ void __launch_bounds__(256) bounded_tiles_kernel(BatchDev b, uint64_t chunk_tiles, uint64_t* staged)
{
    __shared__ unsigned long long lo[TENT_MAX_RAILS], hi[TENT_MAX_RAILS];
    if (threadIdx.x < TENT_MAX_RAILS) { lo[threadIdx.x] = kNoTile; hi[threadIdx.x] = 0; }
    __syncthreads();
    const uint64_t first = ((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256;
    const uint64_t q = first + threadIdx.x;
    if (q < b.n_sc_tiles) {
        const uint32_t i = b.ga_slice[q];
        uint64_t code = kNoTile;
        if (b.s_state[i] == TENT_SLICE_BOUND) {
            const uint32_t d = b.s_rail[i];
            const uint64_t reg = b.s_stage_off[i] + b.ga_x[q];
            code = ((uint64_t)d << 56) | reg;
            atomicMin(&lo[d], (unsigned long long)reg);
            atomicMax(&hi[d], (unsigned long long)(reg + b.tile_bytes));
        }
        staged[q] = code;
    }
    __syncthreads();
    if (first < b.n_sc_tiles && threadIdx.x < TENT_MAX_RAILS && lo[threadIdx.x] != kNoTile) {
        const uint64_t c = first / chunk_tiles;
        atomicMin((unsigned long long*)&b.ch_lo[c * TENT_MAX_RAILS + threadIdx.x], lo[threadIdx.x]);
        atomicMax((unsigned long long*)&b.ch_hi[c * TENT_MAX_RAILS + threadIdx.x], hi[threadIdx.x]);
    }
}

// One wavefront per chunk: region bases of the rails inside the arena for that chunk.
__global__ void __launch_bounds__(64) bounded_bases_kernel(BatchDev b, uint64_t slot_bytes)
{
    const uint64_t row = (uint64_t)blockIdx.x * TENT_MAX_RAILS + threadIdx.x;
    const uint64_t lo = b.ch_lo[row], hi = b.ch_hi[row];
    const uint64_t need = (lo != kNoTile && hi > lo) ? ((hi - lo + 255) & ~255ull) : 0;
    uint64_t inc = need;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t up = (uint64_t)__shfl_up((unsigned long long)inc, d, 64);
        if ((int)threadIdx.x >= d) inc += up;
    }
    b.ch_base[row] = inc - need;
    if (threadIdx.x == 63 && inc > slot_bytes) atomicAdd((unsigned long long*)&b.plan->bounded_overflow, 1ull);
}

// Turn every tile's (rail, staging offset) into its address inside the slot of its chunk (0 = tile not
// to be moved), so that the copy kernels need no dependent look-ups.
__global__ void __launch_bounds__(256) bounded_resolve_kernel(BatchDev b, uint64_t chunk_tiles, uint8_t* arena,
                                                              uint64_t slot_bytes, uint32_t slots, uint64_t* staged)
{
    const uint64_t q = ((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
    if (q >= b.n_sc_tiles) return;
    const uint64_t c = staged[q];
    uint64_t addr = 0;
    if (c != kNoTile) {
        const uint64_t chunk = q / chunk_tiles;
        const uint64_t row = chunk * TENT_MAX_RAILS + (c >> 56);
        addr = (uint64_t)arena + (chunk % slots) * slot_bytes + b.ch_base[row] + ((c & kRegMask) - b.ch_lo[row]);
    }
    staged[q] = addr;
}

// Copy the tiles [q_begin, q_end) of one chunk between their paged side and the arena.
template <bool kGather>
__global__ void __launch_bounds__(kOrderedLanes) bounded_copy_kernel(const uint64_t* __restrict__ paged,
                                                           const uint64_t* __restrict__ staged,
                                                           const uint64_t* __restrict__ overflow,
                                                           uint64_t q_begin, uint64_t q_end, uint32_t tile_shift)
{
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t at = w * (kOrderedLanes * 16) + (uint64_t)threadIdx.x * 16;
    const uint64_t q = q_begin + (at >> tile_shift);
    if (q >= q_end) return;
    const uint64_t near_tile = staged[q];
    const uint64_t far_tile = paged[q];
    if (near_tile == 0 || *overflow != 0) return;
    const uint64_t in_tile = at & ((1ull << tile_shift) - 1);
    const uint64_t far = far_tile + in_tile, near = near_tile + in_tile;
    typedef vec4u_dev vec4u_any;                                  // device memory, any alignment
    // the paged side is streamed (nontemporal); the arena side uses ordinary accesses so that a slot
    // small enough for the memory-side cache can be served from it when the chunk is scattered
    if (kGather) {
        const vec4u v = __builtin_nontemporal_load((const vec4u_any*)far);
        *(vec4u_any*)near = v;
    } else {
        const vec4u v = *(const vec4u_any*)near;
        __builtin_nontemporal_store(v, (vec4u_any*)far);
    }
}

// Both directions of a chunk in one launch, where the batch allows one-pass copies (see copy.hip): source -> slot and
// destination.  Chunks stay ordered by their launches, so the arena ends as with two launches per chunk.
__global__ void __launch_bounds__(kBothLanes) bounded_both_kernel(const uint64_t* __restrict__ from, const uint64_t* __restrict__ staged,
                                                           const uint64_t* __restrict__ to, const uint64_t* __restrict__ overflow,
                                                           uint64_t q_begin, uint64_t q_end, uint32_t tile_shift)
{
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t at = w * (kBothLanes * 16) + (uint64_t)threadIdx.x * 16;
    const uint64_t q = q_begin + (at >> tile_shift);
    if (q >= q_end) return;
    const uint64_t src = from[q];
    const uint64_t lin = staged[q];
    const uint64_t dst = to[q];
    if (lin == 0 || *overflow != 0) return;
    const uint64_t in_tile = at & ((1ull << tile_shift) - 1);
    const vec4u v = *(const vec4u_dev*)(src + in_tile);
    __builtin_nontemporal_store(v, (vec4u_dev*)(lin + in_tile));
    __builtin_nontemporal_store(v, (vec4u_dev*)(dst + in_tile));
}

// ---- geometry without a tile enumeration: ranges of 1 KiB of the payload -----------------------
constexpr uint32_t kRangeBytes = 1024;

// Per range the slice of its first byte, and per (chunk, rail) the interval of staging offsets that the BOUND bytes of the chunk touch.
// A workgroup takes kRangeSlices slices, a group of lanes (a power of two, up to a wavefront) one at a time.  Nearly all of them lie in
// the first one's chunk, whose intervals are put together in LDS.  (By a wavefront per range, with a search for its slice and a
// workgroup's intervals sent off every four ranges, 956 MB took 1640 us on MI355X, nearly all of it for atomics on the same few
// words; now 9.)
constexpr uint32_t kRangeSlices = 16;
__global__ void __launch_bounds__(256) bounded_ranges_kernel(BatchDev b, uint64_t chunk_bytes, uint32_t group_shift)
{
    __shared__ unsigned long long lo[TENT_MAX_RAILS], hi[TENT_MAX_RAILS];
    if (threadIdx.x < TENT_MAX_RAILS) { lo[threadIdx.x] = kNoTile; hi[threadIdx.x] = 0; }
    __syncthreads();
    const uint64_t first = (uint64_t)blockIdx.x * kRangeSlices, c_first = b.s_pos[first] / chunk_bytes;
    const uint32_t group = 1u << group_shift, t0 = threadIdx.x & (group - 1);
    for (uint64_t i = first + (threadIdx.x >> group_shift); i < first + kRangeSlices && i < b.n_slices; i += 256u >> group_shift) {
        const uint64_t at = b.s_pos[i], end = at + b.s_len[i];
        for (uint64_t r = (at + kRangeBytes - 1) / kRangeBytes + t0; r * kRangeBytes < end; r += group) b.range_slice[r] = (uint32_t)i;
        if (t0 != 0 || b.s_state[i] != TENT_SLICE_BOUND) continue;
        const uint32_t d = b.s_rail[i];
        const uint64_t off = b.s_stage_off[i];
        for (uint64_t c = at / chunk_bytes; c * chunk_bytes < end; ++c) {
            const uint64_t from = at > c * chunk_bytes ? at : c * chunk_bytes, to = end < (c + 1) * chunk_bytes ? end : (c + 1) * chunk_bytes;
            unsigned long long* const row_lo = c == c_first ? lo : (unsigned long long*)&b.ch_lo[c * TENT_MAX_RAILS];
            unsigned long long* const row_hi = c == c_first ? hi : (unsigned long long*)&b.ch_hi[c * TENT_MAX_RAILS];
            atomicMin(&row_lo[d], (unsigned long long)(off + (from - at)));
            atomicMax(&row_hi[d], (unsigned long long)(off + (to - at)));
        }
    }
    __syncthreads();
    if (threadIdx.x < TENT_MAX_RAILS && lo[threadIdx.x] != kNoTile) {
        atomicMin((unsigned long long*)&b.ch_lo[c_first * TENT_MAX_RAILS + threadIdx.x], lo[threadIdx.x]);
        atomicMax((unsigned long long*)&b.ch_hi[c_first * TENT_MAX_RAILS + threadIdx.x], hi[threadIdx.x]);
    }
}

// Where bytes [x0, x1) of a slice, at most kRangeBytes of them, start on a side whose tile table this is; false if they may be cut into
// several extents.
__device__ __forceinline__ bool one_piece(const uint64_t* tiles, uint32_t x0, uint32_t x1, uint64_t* paged)
{
    const uint32_t t0 = x0 / kRangeBytes, t1 = (x1 - 1) / kRangeBytes;
    const uint64_t a = tiles[t0], z = tiles[t1];
    *paged = a + x0 % kRangeBytes;
    return ((a | z) & kTileSlow) == 0 && z - a == (uint64_t)(t1 - t0) * kRangeBytes;
}

// Move the BOUND bytes of payload positions [c_lo, c_hi) -- one chunk -- between their paged side and the
// chunk's slot, one wavefront per range of 1 KiB (one-pass copies: both ways at once).  A piece of the range that has one address on
// either side goes straight through registers; otherwise its bytes pass through 1 KiB of LDS, and the side that is cut into
// several extents is walked piece by piece.
// What bounds it is loads that wait for one another, then memory.  When every range searched the transfers by halves, copied at
// the arena's alignment and read back from the arena what it had just written there, 956 MB of transfers of 256-byte tokens took
// 2920 us on MI355X; with the range's slice from a table, the slices' tile tables and LDS 1050.
template <bool kGather, bool kScatter>
__global__ void __launch_bounds__(256) bounded_ranges_copy_kernel(BatchDev b, uint64_t c_lo, uint64_t c_hi,
                                                                  uint8_t* slot, uint64_t row)
{
    __shared__ vec4u bounce[256];
    const uint64_t w = ((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * 4 + (threadIdx.x >> 6);
    const uint64_t p0 = c_lo + w * kRangeBytes;
    if (p0 >= c_hi || b.plan->bounded_overflow != 0) return;
    const uint64_t p1 = p0 + kRangeBytes < c_hi ? p0 + kRangeBytes : c_hi;
    vec4u* mine = &bounce[threadIdx.x & ~63u];                    // this wavefront's 1 KiB
    uint8_t* my_bytes = (uint8_t*)mine;
    const uint32_t lane = threadIdx.x & 63u;
    for (uint64_t i = b.range_slice[p0 / kRangeBytes];; ++i) {
        const uint64_t at = b.s_pos[i], end = at + b.s_len[i];
        if (b.s_state[i] == TENT_SLICE_BOUND) {
            const uint32_t x0 = (uint32_t)((at > p0 ? at : p0) - at), x1 = (uint32_t)((end < p1 ? end : p1) - at);
            const uint32_t d = b.s_rail[i];
            const uint64_t staged = (uint64_t)slot + b.ch_base[row + d] + (b.s_stage_off[i] + x0 - b.ch_lo[row + d]);
            uint64_t src = staged, dst = 0;
            const bool src_cut = kGather && !one_piece(b.src_tile + i * b.tiles_per_slice, x0, x1, &src);
            const bool dst_cut = kScatter && !one_piece(b.dst_tile + i * b.tiles_per_slice, x0, x1, &dst);
            // whole vectors, one per lane, and the bytes behind them
            const uint32_t n = x1 - x0, o = lane * 16, o_tail = (n & ~15u) + lane;
            const bool whole = o + 16 <= n, tail = o_tail < n;
            vec4u v;
            uint8_t t = 0;
            if (src_cut) {
                walk_cut_side<true>(b, i, x0, x1, mine);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                v = mine[lane];
                if (tail) t = my_bytes[o_tail];
            } else {
                if (whole) v = *(const vec4u_dev*)(src + o);
                if (tail) t = *(const byte_dev*)(src + o_tail);
                if (dst_cut) {
                    if (whole) mine[lane] = v;
                    if (tail) my_bytes[o_tail] = t;
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                }
            }
            if (kGather) {
                // (alone, the arena is written with ordinary stores: a slot small enough for the memory-side cache is then
                // served from it when the chunk is scattered)
                if (whole) { if (kScatter) __builtin_nontemporal_store(v, (vec4u_dev*)(staged + o)); else *(vec4u_dev*)(staged + o) = v; }
                if (tail) *(byte_dev*)(staged + o_tail) = t;
            }
            if (kScatter && dst_cut) {
                walk_cut_side<false>(b, i, x0, x1, mine);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");           // (before the next piece is written over it)
            } else if (kScatter) {
                if (whole) __builtin_nontemporal_store(v, (vec4u_dev*)(dst + o));
                if (tail) *(byte_dev*)(dst + o_tail) = t;
            }
        }
        if (end >= p1) break;
    }
}

__global__ void __launch_bounds__(256) mark_done_bounded_kernel(BatchDev b)
{
    if (b.plan->bounded_overflow != 0) return;                      // nothing moved: leave the slices BOUND
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride)
        if (b.s_state[i] == TENT_SLICE_BOUND) b.s_state[i] = TENT_SLICE_DONE;
}

bool grid_for(uint64_t blocks, dim3* grid)
{
    const uint32_t gx = blocks < 65536 ? (uint32_t)blocks : 65536u;
    const uint64_t gy = (blocks + gx - 1) / gx;
    if (gy > 0x7FFFFFFFull) return false;
    *grid = dim3(gx, (uint32_t)gy);
    return true;
}

}  // namespace

hipError_t launch_bounded_prepare(const BatchDev& b, uint64_t chunk_bytes, uint32_t n_chunks, uint64_t slot_bytes,
                                  uint32_t slots, uint8_t* arena, hipStream_t s)
{
    const uint32_t cells = n_chunks * TENT_MAX_RAILS;
    hipLaunchKernelGGL(bounded_clear_kernel, dim3((cells + 255) / 256), dim3(256), 0, s, b, n_chunks);
    dim3 grid;
    if (b.n_sc_tiles == 0) {                                  // no tile enumeration: ranges of the payload
        uint32_t group_shift = 0;
        while (group_shift < 6 && (1u << group_shift) < b.tiles_per_slice) ++group_shift;
        const uint64_t blocks = (b.n_slices + kRangeSlices - 1) / kRangeSlices;
        if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(bounded_ranges_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, chunk_bytes, group_shift);
        hipLaunchKernelGGL(bounded_bases_kernel, dim3(n_chunks), dim3(64), 0, s, b, slot_bytes);
        return hipGetLastError();
    }
    if (!grid_for((b.n_sc_tiles + 255) / 256, &grid)) return hipErrorInvalidValue;
    uint64_t* staged = b.one_pass ? b.op_lin : b.ga_lin;
    hipLaunchKernelGGL(bounded_tiles_kernel, grid, dim3(256), 0, s, b, chunk_bytes / b.tile_bytes, staged);
    hipLaunchKernelGGL(bounded_bases_kernel, dim3(n_chunks), dim3(64), 0, s, b, slot_bytes);
    hipLaunchKernelGGL(bounded_resolve_kernel, grid, dim3(256), 0, s, b, chunk_bytes / b.tile_bytes, arena, slot_bytes,
                       slots, staged);
    return hipGetLastError();
}

hipError_t launch_bounded_copy(const BatchDev& b, bool gather, uint32_t chunk, uint64_t payload, uint64_t chunk_bytes,
                               uint64_t slot_bytes, uint32_t slots, uint8_t* arena, hipStream_t s)
{
    if (b.n_sc_tiles == 0) {
        const uint64_t c_lo = (uint64_t)chunk * chunk_bytes;
        if (c_lo >= payload) return hipSuccess;
        const uint64_t c_hi = c_lo + chunk_bytes < payload ? c_lo + chunk_bytes : payload;
        dim3 grid;
        if (!grid_for((c_hi - c_lo + 4 * kRangeBytes - 1) / (4 * kRangeBytes), &grid)) return hipErrorInvalidValue;
        uint8_t* slot = arena + (chunk % slots) * slot_bytes;
        const uint64_t row = (uint64_t)chunk * TENT_MAX_RAILS;
        if (b.one_pass)
            hipLaunchKernelGGL((bounded_ranges_copy_kernel<true, true>), grid, dim3(256), 0, s, b, c_lo, c_hi, slot, row);
        else if (gather)
            hipLaunchKernelGGL((bounded_ranges_copy_kernel<true, false>), grid, dim3(256), 0, s, b, c_lo, c_hi, slot, row);
        else
            hipLaunchKernelGGL((bounded_ranges_copy_kernel<false, true>), grid, dim3(256), 0, s, b, c_lo, c_hi, slot, row);
        return hipGetLastError();
    }
    uint32_t tile_shift = 0;
    while ((1u << tile_shift) < b.tile_bytes) ++tile_shift;
    const uint64_t chunk_tiles = chunk_bytes >> tile_shift;
    const uint64_t q_begin = (uint64_t)chunk * chunk_tiles;
    if (q_begin >= b.n_sc_tiles) return hipSuccess;
    const uint64_t q_end = q_begin + chunk_tiles < b.n_sc_tiles ? q_begin + chunk_tiles : b.n_sc_tiles;
    const uint64_t bytes = (q_end - q_begin) << tile_shift;
    dim3 grid;
    const uint64_t lanes = b.one_pass ? kBothLanes : kOrderedLanes;
    if (!grid_for((bytes + lanes * 16 - 1) / (lanes * 16), &grid)) return hipErrorInvalidValue;
    if (b.one_pass)
        hipLaunchKernelGGL(bounded_both_kernel, grid, dim3(kBothLanes), 0, s, b.op_src, b.op_lin, b.op_dst,
                           &b.plan->bounded_overflow, q_begin, q_end, tile_shift);
    else if (gather)
        hipLaunchKernelGGL(bounded_copy_kernel<true>, grid, dim3(kOrderedLanes), 0, s, b.ga_src, b.ga_lin,
                           &b.plan->bounded_overflow, q_begin, q_end, tile_shift);
    else
        hipLaunchKernelGGL(bounded_copy_kernel<false>, grid, dim3(kOrderedLanes), 0, s, b.ga_dst, b.ga_lin,
                           &b.plan->bounded_overflow, q_begin, q_end, tile_shift);
    return hipGetLastError();
}

hipError_t launch_mark_done_bounded(const BatchDev& b, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(mark_done_bounded_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b);
    return hipGetLastError();
}

}  // namespace tent
