// Slice bytes between paged extents and per-rail staging regions.
//
// Every slice's bytes are read from the transfer's source extents and written contiguously at the slice's staging
// address (the staging hop of Section 4.1 of the paper) and to the destination extents at the slice's absolute offset
// inside the transfer (direct-to-offset writes, Section 4.4), so the result does not depend on the order in which slices
// are moved.  Two forms of that:
//   one pass    (second half of this file) where no destination byte is a source byte of the batch and the arena
//               lies outside the segments: every source byte is read once and stored to both places;
//   two passes  for every other batch: gather (source -> staging), then scatter (staging -> destination), a launch each.
//
// Two passes:
// Work decomposition: one 256-lane workgroup per 4 KiB block of a slice, one 16-byte vector per
// lane, and the workgroup ends after its store.  Consecutive workgroups touch consecutive staging
// addresses, so the set of DRAM pages open at any time stays small; on MI355X this one-shot shape
// sustains more bandwidth than persistent workgroups that loop over larger chunks.  The paged-side
// address comes from the tile table built by the splitter (one 8-byte entry per tile of 1-4 KiB),
// looked up per lane, so extent boundaries inside a block cost nothing as long as they fall on
// tile boundaries, at any address alignment.  A wavefront that meets a flagged tile (extent
// boundary inside the tile) or a slice that ends inside a lane's vector takes the
// generic path, which walks the extent list, aligns its stores and loads at any alignment.
#include "copy_generic.h"

namespace tent {

// One workgroup moves kLanes*16 bytes of one slice; every wavefront is independent of the others
// (no barrier): it moves 1 KiB with one 16-byte vector per lane.  The slice record (scalar load)
// and the tile entry (one load per lane) are fetched together before the first branch, so a
// wavefront sees two memory round trips before its data load: kernel arguments, then metadata.
template <bool kGather, int kLanes>
__global__ void __launch_bounds__(kLanes) copy_kernel(const SliceRec* __restrict__ rec, const uint64_t* __restrict__ tab,
                                                      uint64_t n_slices, uint32_t bps, uint32_t bps_shift,
                                                      uint32_t tiles_per_slice, uint32_t tile_shift,
                                                      const BatchDev* __restrict__ batch)
{
    constexpr uint32_t kBlockBytes = kLanes * 16;
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t i = bps_shift != 0xFFFFFFFFu ? (w >> bps_shift)
                       : (w >> 32) == 0 ? (uint64_t)((uint32_t)w / bps) : w / bps;
    if (i >= n_slices) return;
    const uint32_t c = (uint32_t)(w - i * bps);
    const uint32_t x = c * kBlockBytes + threadIdx.x * 16;   // this lane's byte offset inside the slice
    uint32_t t = x >> tile_shift;
    if (t >= tiles_per_slice) t = tiles_per_slice - 1;
    const uint64_t entry = tab[i * tiles_per_slice + t];
    const SliceRec r = rec[i];
    const bool in_range = x + 16 <= r.len;
    const bool ragged = x < r.len && !in_range;              // slice ends inside this lane's vector
    const bool bad = ragged || (x < r.len && (entry & kTileSlow));
    if (__any(bad)) {
        const uint32_t wave_lo = c * kBlockBytes + (threadIdx.x & ~63u) * 16;
        const uint32_t wave_hi = wave_lo + 1024 < r.len ? wave_lo + 1024 : r.len;
        copy_range_generic<kGather>(*batch, i, wave_lo, wave_hi, (uint8_t*)(r.lin + wave_lo));
        return;
    }
    if (!in_range) return;
    const uint64_t paged = entry + (x & ((1u << tile_shift) - 1));
    const uint64_t mine = r.lin + x;
    if (kGather) {
        vec4u v = __builtin_nontemporal_load((const vec4u_any*)paged);
        __builtin_nontemporal_store(v, (vec4u_any*)mine);
    } else {
        vec4u v = __builtin_nontemporal_load((const vec4u_any*)mine);
        __builtin_nontemporal_store(v, (vec4u_any*)paged);
    }
}

template <bool kGather, int kLanes>
static hipError_t launch_copy_lanes(const BatchDev& b, hipStream_t s)
{
    const uint32_t block_bytes = kLanes * 16;
    const uint32_t bps = (uint32_t)((b.slice_bytes + block_bytes - 1) / block_bytes);
    uint32_t bps_shift = 0xFFFFFFFFu;
    if ((bps & (bps - 1)) == 0) { bps_shift = 0; while ((1u << bps_shift) < bps) ++bps_shift; }
    uint32_t tile_shift = 0;
    while ((1u << tile_shift) < b.tile_bytes) ++tile_shift;
    const uint64_t blocks = b.n_slices * (uint64_t)bps;
    if (blocks == 0) return hipSuccess;
    // 2-D grid so that the block count is not capped by the 1-D limit
    const uint32_t gx = blocks < 65536 ? (uint32_t)blocks : 65536u;
    const uint64_t gy = (blocks + gx - 1) / gx;
    if (gy > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL((copy_kernel<kGather, kLanes>), dim3(gx, (uint32_t)gy), dim3(kLanes), 0, s,
                       b.s_rec, kGather ? b.src_tile : b.dst_tile, b.n_slices, bps, bps_shift,
                       b.tiles_per_slice, tile_shift, b.self);
    return hipGetLastError();
}

// Table-driven copy: workgroup w moves block w (kOrderedLanes x 16 bytes) of an enumeration of the payload in tiles;
// `from` and `to` hold the two addresses of every tile (0 = tile not to be moved).  Gather walks the
// source bytes in declaration order (reads hop between pages, every rail region is written front to
// back); scatter walks the destination bytes in ascending device address (reads hop between the
// rail regions, writes are sequential) -- HBM tolerates scattered reads better than scattered
// writes.  Only used when no tile crosses an extent boundary.  kGather only names the direction
// (the two launches show up separately in a kernel trace); the code is the same.
template <bool kGather>
__global__ void __launch_bounds__(kOrderedLanes) ordered_copy_kernel(const uint64_t* __restrict__ from,
                                                                     const uint64_t* __restrict__ to,
                                                                     uint64_t n_tiles, uint32_t tile_shift)
{
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t at = w * (kOrderedLanes * 16) + (uint64_t)threadIdx.x * 16;   // byte in enumeration order
    // The tile index is the same for all lanes of a wavefront, but the table entries are fetched with
    // ordinary per-lane loads (one cache line per wavefront): scalar loads measured 1 % faster on the
    // KV-migration workload and 2-4 % slower on contiguous tensors and on 2 KiB tiles.
    const uint64_t q = at >> tile_shift;
    if (q >= n_tiles) return;
    const uint64_t src = from[q];
    const uint64_t dst = to[q];
    if (src == 0 || dst == 0) return;
    const uint64_t in_tile = at & ((1ull << tile_shift) - 1);
    vec4u v = __builtin_nontemporal_load((const vec4u_dev*)(src + in_tile));
    __builtin_nontemporal_store(v, (vec4u_dev*)(dst + in_tile));
}

hipError_t launch_copy_ordered(const BatchDev& b, bool gather, hipStream_t s)
{
    uint32_t tile_shift = 0;
    while ((1u << tile_shift) < b.tile_bytes) ++tile_shift;
    const uint64_t bytes = b.n_sc_tiles * (uint64_t)b.tile_bytes;
    const uint64_t block_bytes = kOrderedLanes * 16;
    const uint64_t blocks = (bytes + block_bytes - 1) / block_bytes;
    if (blocks == 0) return hipSuccess;
    const uint32_t gx = blocks < 65536 ? (uint32_t)blocks : 65536u;
    const uint64_t gy = (blocks + gx - 1) / gx;
    if (gy > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid(gx, (uint32_t)gy);
    if (gather)
        hipLaunchKernelGGL(ordered_copy_kernel<true>, grid, dim3(kOrderedLanes), 0, s, b.ga_src, b.ga_lin, b.n_sc_tiles,
                           tile_shift);
    else
        hipLaunchKernelGGL(ordered_copy_kernel<false>, grid, dim3(kOrderedLanes), 0, s, b.sc_lin, b.sc_dst, b.n_sc_tiles,
                           tile_shift);
    return hipGetLastError();
}

// The same copy over a list of tiles (one workgroup per listed tile, tile_bytes / 16 lanes): used when
// few slices of the batch move, so that the launch is sized by what moves.  The grid is an upper
// bound known to the host; workgroups beyond the device-side count leave at once.
template <bool kGather>
__global__ void __launch_bounds__(256) compact_copy_kernel(const uint64_t* __restrict__ from,
                                                           const uint64_t* __restrict__ to,
                                                           const uint64_t* __restrict__ n_act)
{
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (w >= *n_act) return;
    const uint64_t src = from[w];
    const uint64_t dst = to[w];
    const uint64_t in_tile = (uint64_t)threadIdx.x * 16;
    vec4u v = __builtin_nontemporal_load((const vec4u_dev*)(src + in_tile));
    __builtin_nontemporal_store(v, (vec4u_dev*)(dst + in_tile));
}

hipError_t launch_copy_compact(const BatchDev& b, bool gather, uint64_t max_tiles, hipStream_t s)
{
    if (max_tiles > b.act_capacity) max_tiles = b.act_capacity;
    if (max_tiles == 0) return hipSuccess;
    const uint32_t gx = max_tiles < 65536 ? (uint32_t)max_tiles : 65536u;
    const uint64_t gy = (max_tiles + gx - 1) / gx;
    if (gy > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid(gx, (uint32_t)gy), block(b.tile_bytes / 16);
    if (gather)
        hipLaunchKernelGGL(compact_copy_kernel<true>, grid, block, 0, s, b.act_src, b.act_lin, &b.plan->n_act);
    else
        hipLaunchKernelGGL(compact_copy_kernel<false>, grid, block, 0, s, b.act_lin, b.act_dst, &b.plan->n_act);
    return hipGetLastError();
}

// ---- one pass: source -> staging and destination ----------------------------------------------------
// Every source byte is read once and stored twice, so that the scatter's read of the staging region (a quarter of
// the two-pass traffic) falls away.  Allowed where no destination byte is a source byte of the batch (the overlap check
// passed) and the arena lies outside the segments; the two kernels above stay for every other batch.
// HBM-bound.  8 GiB on MI355X, ordinary allocations, two passes -> one pass: 32 KiB pages shuffled on both sides
// 6.02 -> 4.57 ms (5.6 TB/s of the 3 bytes per payload byte it moves), contiguous tensors 5.76 -> 4.00 ms (6.4 TB/s),
// 4.5 GiB of 18 KiB pages in 2 KiB tiles 3.32 -> 2.66 ms.  Order: ascending destination address (declaration order, one
// frontier per rail but scattered destination pages: 2-4 % slower on pages, the same on tensors).  Ordinary
// loads with nontemporal stores: nontemporal loads 5-10 % slower, ordinary stores 4-8 %.  512 lanes: 64, 128,
// 256 and 1024 lanes 1-5 % slower.  A look-up of (slice record, offset) in place of the staging table: 6 % slower.
constexpr int kOnePassLanes = 512;

__device__ __forceinline__ void copy_to_both(const uint64_t* __restrict__ from, const uint64_t* __restrict__ mid,
                                             const uint64_t* __restrict__ to, uint64_t n_tiles, uint32_t tile_shift)
{
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t at = w * (kOnePassLanes * 16) + (uint64_t)threadIdx.x * 16;
    const uint64_t q = at >> tile_shift;
    if (q >= n_tiles) return;
    const uint64_t src = from[q];
    const uint64_t lin = mid[q];
    const uint64_t dst = to[q];
    if (lin == 0) return;
    const uint64_t in_tile = at & ((1ull << tile_shift) - 1);
    const vec4u v = *(const vec4u_dev*)(src + in_tile);
    __builtin_nontemporal_store(v, (vec4u_dev*)(lin + in_tile));
    __builtin_nontemporal_store(v, (vec4u_dev*)(dst + in_tile));
}

__global__ void __launch_bounds__(kOnePassLanes) one_pass_copy_kernel(const uint64_t* __restrict__ from,
                                                                      const uint64_t* __restrict__ mid,
                                                                      const uint64_t* __restrict__ to, uint64_t n_tiles,
                                                                      uint32_t tile_shift)
{
    copy_to_both(from, mid, to, n_tiles, tile_shift);
}

// Over a list of tiles whose length only the device knows; the grid covers the host's bound on it.
__global__ void __launch_bounds__(kOnePassLanes) one_pass_list_copy_kernel(const uint64_t* __restrict__ from,
                                                                           const uint64_t* __restrict__ mid,
                                                                           const uint64_t* __restrict__ to,
                                                                           const uint64_t* __restrict__ n_act,
                                                                           uint32_t tile_shift)
{
    copy_to_both(from, mid, to, *n_act, tile_shift);
}

// Geometry whose tiles cross extent boundaries, slice by slice as copy_kernel: a wavefront whose 1 KiB has one
// address on each side copies straight through registers.  Otherwise its bytes pass through 1 KiB of LDS: the
// side that is cut into several extents is walked piece by piece, the other side and the staging address keep their
// 16-byte accesses.
__global__ void __launch_bounds__(256) one_pass_slice_copy_kernel(const SliceRec* __restrict__ rec,
                                                                  const uint64_t* __restrict__ src_tab,
                                                                  const uint64_t* __restrict__ dst_tab, uint64_t n_slices,
                                                                  uint32_t bps, uint32_t bps_shift, uint32_t tiles_per_slice,
                                                                  uint32_t tile_shift, const BatchDev* __restrict__ batch)
{
    __shared__ vec4u bounce[256];
    const uint64_t w = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t i = bps_shift != 0xFFFFFFFFu ? (w >> bps_shift)
                       : (w >> 32) == 0 ? (uint64_t)((uint32_t)w / bps) : w / bps;
    if (i >= n_slices) return;
    const uint32_t c = (uint32_t)(w - i * bps);
    const uint32_t x = c * 4096u + threadIdx.x * 16;             // this lane's byte offset inside the slice
    uint32_t t = x >> tile_shift;
    if (t >= tiles_per_slice) t = tiles_per_slice - 1;
    const uint64_t from = src_tab[i * tiles_per_slice + t];
    const uint64_t to = dst_tab[i * tiles_per_slice + t];
    const SliceRec r = rec[i];
    const bool in_range = x + 16 <= r.len;
    const bool ragged = x < r.len && !in_range;                  // slice ends inside this lane's vector
    const bool any_ragged = __any(ragged);
    const bool src_cut = any_ragged || __any(x < r.len && (from & kTileSlow));
    const bool dst_cut = any_ragged || __any(x < r.len && (to & kTileSlow));
    const uint32_t in_tile = x & ((1u << tile_shift) - 1);
    vec4u v;
    if (!src_cut && !dst_cut) {
        if (!in_range) return;
        v = *(const vec4u_dev*)(from + in_tile);
        __builtin_nontemporal_store(v, (vec4u_dev*)(r.lin + x));
        __builtin_nontemporal_store(v, (vec4u_dev*)(to + in_tile));
        return;
    }
    const uint32_t wave_lo = c * 4096u + (threadIdx.x & ~63u) * 16;
    const uint32_t wave_hi = wave_lo + 1024 < r.len ? wave_lo + 1024 : r.len;
    if (wave_lo >= wave_hi) return;
    vec4u* mine = &bounce[threadIdx.x & ~63u];                   // this wavefront's 1 KiB
    if (src_cut) {
        walk_cut_side<true>(*batch, i, wave_lo, wave_hi, mine);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        v = bounce[threadIdx.x];                                 // bytes past the slice's end are not used
    } else if (in_range) {
        v = *(const vec4u_dev*)(from + in_tile);
        bounce[threadIdx.x] = v;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    if (in_range) __builtin_nontemporal_store(v, (vec4u_dev*)(r.lin + x));
    if (any_ragged) {                                            // the bytes of the slice's last, partial vector
        const uint32_t whole = (wave_hi - wave_lo) & ~15u, at = whole + (threadIdx.x & 63u);
        if (at < wave_hi - wave_lo) *(byte_dev*)(r.lin + wave_lo + at) = ((const uint8_t*)mine)[at];
    }
    if (dst_cut) walk_cut_side<false>(*batch, i, wave_lo, wave_hi, mine);
    else if (in_range) __builtin_nontemporal_store(v, (vec4u_dev*)(to + in_tile));
}

// 2-D grid so that the block count is not capped by the 1-D limit.
static bool copy_grid(uint64_t blocks, dim3* grid)
{
    const uint32_t gx = blocks < 65536 ? (uint32_t)blocks : 65536u;
    const uint64_t gy = (blocks + gx - 1) / gx;
    if (gy > 0x7FFFFFFFull) return false;
    *grid = dim3(gx, (uint32_t)gy);
    return true;
}

hipError_t launch_copy_one_pass(const BatchDev& b, bool compact, uint64_t max_tiles, hipStream_t s)
{
    uint32_t tile_shift = 0;
    while ((1u << tile_shift) < b.tile_bytes) ++tile_shift;
    dim3 grid;
    if (b.n_sc_tiles == 0) {
        const uint32_t bps = (uint32_t)((b.slice_bytes + 4095) / 4096);
        uint32_t bps_shift = 0xFFFFFFFFu;
        if ((bps & (bps - 1)) == 0) { bps_shift = 0; while ((1u << bps_shift) < bps) ++bps_shift; }
        if (!copy_grid(b.n_slices * (uint64_t)bps, &grid)) return hipErrorInvalidValue;
        hipLaunchKernelGGL(one_pass_slice_copy_kernel, grid, dim3(256), 0, s, b.s_rec, b.src_tile, b.dst_tile, b.n_slices, bps,
                           bps_shift, b.tiles_per_slice, tile_shift, b.self);
        return hipGetLastError();
    }
    const uint64_t tiles = !compact ? b.n_sc_tiles : max_tiles < b.act_capacity ? max_tiles : b.act_capacity;
    if (tiles == 0) return hipSuccess;
    const uint64_t per_block = kOnePassLanes * 16;
    if (!copy_grid(((tiles << tile_shift) + per_block - 1) / per_block, &grid)) return hipErrorInvalidValue;
    if (compact)
        hipLaunchKernelGGL(one_pass_list_copy_kernel, grid, dim3(kOnePassLanes), 0, s, b.act_src, b.act_lin, b.act_dst,
                           &b.plan->n_act, tile_shift);
    else
        hipLaunchKernelGGL(one_pass_copy_kernel, grid, dim3(kOnePassLanes), 0, s, b.op_src, b.op_lin, b.op_dst, b.n_sc_tiles,
                           tile_shift);
    return hipGetLastError();
}

hipError_t launch_copy(const BatchDev& b, bool gather, hipStream_t s)
{
    // 256 lanes (4 KiB per workgroup) measured best among 64/128/256/512 on MI355X
    return gather ? launch_copy_lanes<true, 256>(b, s) : launch_copy_lanes<false, 256>(b, s);
}

}  // namespace tent
