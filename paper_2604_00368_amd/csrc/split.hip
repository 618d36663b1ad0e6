// Slice splitter: prefix sums over extent lengths, per-transfer slice counts and their
// exclusive scan, slice-table expansion, and the pending-list compaction used when a
// batch is re-planned.  Follows the paper's slice decomposition (Section 4.2): a
// transfer of len bytes becomes ceil(len / S) slices; slice k covers [k*S, min((k+1)*S, len))
// and keeps that absolute offset so it can be written straight to its destination.
#include "finish.h"
#include "scan.h"
#include "slices.h"

namespace tent {

uint64_t scan_partials_capacity(uint64_t n) { return (n + kScanTile - 1) / kScanTile + 2; }

// ---- S1: exclusive prefixes of extent lengths over the whole batch ----------------------------
struct ExtentLen {
    const tent_extent* ext;
    __device__ uint64_t operator()(uint64_t e) const { return ext[e].len; }
};
// destination extents in ascending address order (for the tile tables that go by destination address)
struct OrderedLen {
    const tent_extent* ext;
    const uint32_t* order;
    __device__ uint64_t operator()(uint64_t r) const { return ext[order[r]].len; }
};

// all prefixes the batch needs, in the same launches
hipError_t launch_extent_scans(const BatchDev& b, hipStream_t s)
{
    const auto src = scan_job(ExtentLen{b.src_ext}, b.n_src_ext, b.src_pre, b.scan_partials);
    const auto dst = scan_job(ExtentLen{b.dst_ext}, b.n_dst_ext, b.dst_pre, b.scan_partials2);
    if (!b.ord_pre) return run_scans(s, src, dst);
    return run_scans(s, src, dst, scan_job(OrderedLen{b.dst_ext, b.dst_order}, b.n_dst_ext, b.ord_pre, b.scan_partials3));
}

// ---- S2: slices and runs per transfer -----------------------------------------------------------
// (TransferShape in slices.h.)  One scan over the transfers yields the first slice of every transfer (low half of the
// scanned word) and the runs that start before it (high half).
struct StoreCounts {
    uint64_t* first;
    uint32_t* runs;
    __device__ void operator()(uint64_t j, uint64_t v) const
    {
        first[j] = v & 0xFFFFFFFFu;
        runs[j] = (uint32_t)(v >> 32);
    }
};

hipError_t launch_slice_scan(const BatchDev& b, hipStream_t s)
{
    return run_scans(s, ScanJob<TransferCounts, ScanSum, StoreCounts>{TransferCounts{b.src_ptr, b.src_pre, SliceDiv(b.slice_bytes)}, ScanSum{},
                                                                      StoreCounts{b.first, b.runs_before}, b.n_desc, b.scan_partials});
}

// ---- S3: slice table expansion ---------------------------------------------------------------
// A workgroup's 256 slices belong to at most 256 transfers one behind the other (every transfer has a slice): the first of them is found
// by the whole wavefront, 64 places at a time, and their first slices then lie in LDS.  What bounds it is loads that wait for one
// another (MI355X, two requests' 5,000 slices of 128 transfers 12 -> 4.7 us, 1,000,000 slices of 24,576 33 -> 20).
__global__ void __launch_bounds__(256) expand_kernel(BatchDev b)
{
    __shared__ uint32_t first[256];
    const SliceDiv div(b.slice_bytes);
    const uint64_t n = b.n_slices;
    const uint32_t D = b.n_desc, lane = threadIdx.x & 63u;
    for (uint64_t i0 = (uint64_t)blockIdx.x * 256; i0 < n; i0 += (uint64_t)gridDim.x * 256) {
        uint32_t lo = 0, hi = D;                             // the transfer of slice i0 lies in [lo, hi)
        while (hi - lo > 1) {
            const uint32_t step = (hi - lo + 63) >> 6, place = lo + lane * step;
            const uint64_t not_above = __ballot(place < hi && b.first[place < hi ? place : lo] <= i0);
            const uint32_t k = 63u - (uint32_t)__clzll((long long)not_above);       // (place 0 is never above)
            lo += k * step;
            if (hi - lo > step) hi = lo + step;
        }
        __syncthreads();                                     // the round before has been read
        first[threadIdx.x] = lo + threadIdx.x < D ? (uint32_t)b.first[lo + threadIdx.x] : 0xFFFFFFFFu;
        __syncthreads();
        const uint64_t i = i0 + threadIdx.x;
        if (i >= n) continue;
        uint32_t at = 0;                                     // last one that starts at or before slice i
#pragma unroll
        for (uint32_t step = 128; step > 0; step >>= 1)
            if (first[at + step] <= (uint32_t)i) at += step;
        write_slice(b, div, i, lo + at, first[at], b.runs_before[lo + at], b.src_pre, b.dst_pre);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint32_t n_runs = b.runs_before[b.n_desc];
        b.run_start[n_runs] = (uint32_t)n;
        b.plan->n_runs = n_runs;
        b.plan->n_pending = n;
    }
}

hipError_t launch_expand(const BatchDev& b, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(expand_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b);
    return hipGetLastError();
}

// ---- S3b: tile tables ------------------------------------------------------------------------
// The builders are in tile_tables.h.
__global__ void __launch_bounds__(256) tile_tables_kernel(BatchDev b) { build_tile_tables_in(b, blockIdx.x, gridDim.x); }

hipError_t launch_tile_tables(const BatchDev& b, hipStream_t s)
{
    hipLaunchKernelGGL(tile_tables_kernel, dim3(tile_table_blocks(b)), dim3(256), 0, s, b);
    return hipGetLastError();
}

// Copy records: staging address (arena + region base of the rail + offset inside the region) and
// length of every BOUND slice; slices in any other state get length 0 and are skipped by the copy.
// With `mark` the BOUND slices become DONE on the way (nothing behind this kernel reads the state).
__global__ void __launch_bounds__(256) finalize_kernel(BatchDev b, uint8_t* arena, int mark)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride) {
        SliceRec r{0, 0, 0};
        if (b.s_state[i] == TENT_SLICE_BOUND) {
            r.lin = (uint64_t)arena + b.plan->base[b.s_rail[i]] + b.s_stage_off[i];
            r.len = b.s_len[i];
            if (mark) b.s_state[i] = TENT_SLICE_DONE;
        }
        b.s_rec[i] = r;
    }
}

// Staging address of every source-ordered and destination-ordered tile whose slice is about to
// move (0 otherwise).
__global__ void __launch_bounds__(256) finalize_tiles_kernel(BatchDev b)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < b.n_sc_tiles; q += stride) {
        const SliceRec g = b.s_rec[b.ga_slice[q]];
        b.ga_lin[q] = g.len ? g.lin + b.ga_x[q] : 0;
        const SliceRec r = b.s_rec[b.sc_slice[q]];
        b.sc_lin[q] = r.len ? r.lin + b.sc_x[q] : 0;
    }
}

// When only a small part of the batch moves (re-planning epochs), the copy launches should not pay for
// every tile of the batch.  The tiles of the BOUND slices are listed instead: a scan over the slices
// gives each BOUND slice the position of its first tile in the list, and one wavefront per BOUND slice
// resolves the three addresses of each of its tiles (source, staging, destination) from the slice
// table and the extent lists.  The work is proportional to what moves, not to the batch.
struct BoundTiles {
    const SliceRec* rec;
    uint32_t tile_shift;
    __device__ uint64_t operator()(uint64_t i) const { return rec[i].len >> tile_shift; }   // 0 unless BOUND
};

__global__ void __launch_bounds__(256) tile_list_kernel(BatchDev b, uint32_t tile_shift, uint64_t max_tiles)
{
    const uint64_t i = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);      // one wavefront per slice
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint64_t n_act = b.tile_scan[b.n_slices];
        b.plan->n_act = n_act < b.act_capacity ? n_act : b.act_capacity;
        // the copy launches are sized by the host's bound on the BOUND slices; should more tiles move than
        // that (or than the list holds), the copies would be incomplete, so nothing may be marked DONE
        b.plan->compact_overflow = (n_act > max_tiles || n_act > b.act_capacity) ? 1 : 0;
    }
    if (i >= b.n_slices) return;
    const SliceRec r = b.s_rec[i];
    const uint32_t n_t = r.len >> tile_shift;
    if (n_t == 0) return;
    const uint64_t at = b.tile_scan[i];
    const uint32_t j = b.s_desc[i];
    const uint64_t off = b.s_off[i];
    const uint32_t s_hi = b.src_ptr[j + 1], d_hi = b.dst_ptr[j + 1];
    const uint64_t s_pos0 = b.src_pre[b.src_ptr[j]] + off, d_pos0 = b.dst_pre[b.dst_ptr[j]] + off;
    const uint32_t s_e0 = b.s_src_e0[i], d_e0 = b.s_dst_e0[i];
    for (uint32_t t = threadIdx.x & 63; t < n_t; t += 64) {
        const uint64_t p = at + t;
        if (p >= b.act_capacity) break;
        const uint64_t x = (uint64_t)t << tile_shift;
        const uint64_t se = last_not_above(b.src_pre, s_e0, s_hi, s_pos0 + x);
        const tent_extent sx = b.src_ext[se];
        const uint64_t de = last_not_above(b.dst_pre, d_e0, d_hi, d_pos0 + x);
        const tent_extent dx = b.dst_ext[de];
        b.act_src[p] = b.seg_base[sx.seg] + sx.off + (s_pos0 + x - b.src_pre[se]);
        b.act_lin[p] = r.lin + x;
        b.act_dst[p] = b.seg_base[dx.seg] + dx.off + (d_pos0 + x - b.dst_pre[de]);
    }
}

hipError_t launch_finalize(const BatchDev& b, uint8_t* arena, bool compact, uint64_t max_tiles, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(finalize_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, arena, 0);
    if (b.n_sc_tiles && compact) {
        uint32_t tile_shift = 0;
        while ((1u << tile_shift) < b.tile_bytes) ++tile_shift;
        hipError_t e = exclusive_scan(BoundTiles{b.s_rec, tile_shift}, b.n_slices, b.tile_scan, b.tile_partials, s);
        if (e != hipSuccess) return e;
        const uint64_t lists = (b.n_slices + 3) / 4;
        if (lists > 0x7FFFFFFFull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(tile_list_kernel, dim3((uint32_t)lists), dim3(256), 0, s, b, tile_shift, max_tiles);
    } else if (b.n_sc_tiles) {
        blocks = (b.n_sc_tiles + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(finalize_tiles_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b);
    }
    return hipGetLastError();
}

// ---- bookkeeping of the one-pass copies ---------------------------------------------------------
constexpr uint32_t kTilesPerWave = 1024;

// One launch resolves the staging address of every tile that moves and marks its slice DONE: a group of
// lanes (a power of two, up to a wavefront) takes one slice, reads its state, writes the addresses of the slice's
// tiles at their places in the copy's order, and its first lane then changes the state that only this
// group reads.  It was three launches (slice records, tile addresses, marks) and 16 bytes of table per tile more:
// what bounds it is one launch (about 5 us) up to some 10^5 tiles, then 4 bytes read and 8 written per tile.
// Slices of more than kTilesPerWave tiles are shared by `parts` wavefronts, and a launch of its own marks them.
__global__ void __launch_bounds__(256) stage_tiles_kernel(BatchDev b, uint8_t* arena, uint32_t group_shift, uint32_t tile_shift,
                                                          uint32_t parts)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t i = at >> group_shift;
    uint32_t group = 1u << group_shift;
    uint32_t t0 = (uint32_t)at & (group - 1);
    if (parts > 1) {                                                // group = wavefront here
        t0 += 64u * (uint32_t)(i % parts);
        i /= parts;
        group *= parts;
    }
    if (i >= b.n_slices) return;
    const uint32_t n_t = b.s_len[i] >> tile_shift;
    const uint64_t q0 = b.s_pos[i] >> tile_shift;
    const bool bound = b.s_state[i] == TENT_SLICE_BOUND;
    uint64_t lin = 0;
    if (bound) lin = (uint64_t)arena + b.plan->base[b.s_rail[i]] + b.s_stage_off[i];
    for (uint32_t t = t0; t < n_t; t += group) {
        const uint64_t p = b.tile_pos ? b.tile_pos[q0 + t] : q0 + t;
        b.op_lin[p] = bound ? lin + ((uint64_t)t << tile_shift) : 0;
    }
    if (bound && t0 == 0 && parts == 1) b.s_state[i] = TENT_SLICE_DONE;
}

// The same when few slices move: the tiles of the BOUND slices are listed with their three addresses, in any
// order (the copy's result does not depend on it).  A workgroup looks at 16 slices, places those that are BOUND one behind
// the other and takes room for all of them with one atomic add (over 20,000 slices of which 1,200 move: an add per slice
// 32 us; 64 slices to a workgroup 22 us, because BOUND slices lie together and few workgroups then have all the work);
// groups of lanes then write the entries.  A workgroup whose tiles do not fit the list, or the host's bound that sizes the
// copy, leaves its slices BOUND and lists nothing; the others occupy the list without gaps, because the first that does
// not fit moves the counter past the bound.  (The list of the two-pass copies marks nothing DONE in that case.  It takes an
// execute that was recorded into a graph and is replayed over more BOUND slices than it was recorded for.)
constexpr uint32_t kListSlices = 16;
__global__ void __launch_bounds__(256) list_tiles_kernel(BatchDev b, uint8_t* arena, uint32_t group_shift, uint32_t tile_shift,
                                                         uint64_t max_tiles)
{
    __shared__ uint64_t sh_at[kListSlices], sh_lin[kListSlices], sh_q0[kListSlices];
    __shared__ uint32_t sh_n[kListSlices];
    const uint64_t first = (uint64_t)blockIdx.x * kListSlices;
    if (threadIdx.x < kListSlices) {
        const uint64_t i = first + threadIdx.x;
        const bool bound = i < b.n_slices && b.s_state[i] == TENT_SLICE_BOUND;
        uint32_t n_t = 0;
        if (bound) {
            n_t = b.s_len[i] >> tile_shift;
            sh_lin[threadIdx.x] = (uint64_t)arena + b.plan->base[b.s_rail[i]] + b.s_stage_off[i];
            sh_q0[threadIdx.x] = b.s_pos[i] >> tile_shift;
        }
        const uint64_t up_to = wave_inclusive_scan((uint64_t)n_t);
        const uint64_t all = __shfl((unsigned long long)up_to, kListSlices - 1, 64);
        uint64_t from = 0;
        if (threadIdx.x == 0 && all != 0) {
            from = atomicAdd((unsigned long long*)&b.plan->n_act_asked, (unsigned long long)all);
            if (from + all <= max_tiles) atomicAdd((unsigned long long*)&b.plan->n_act, (unsigned long long)all);
        }
        from = __shfl((unsigned long long)from, 0, 64);
        const bool fits = from + all <= max_tiles;
        sh_at[threadIdx.x] = from + up_to - n_t;
        sh_n[threadIdx.x] = fits ? n_t : 0;
        if (bound && fits) b.s_state[i] = TENT_SLICE_DONE;
    }
    __syncthreads();
    const uint32_t group = 1u << group_shift, groups = 256u >> group_shift;
    const uint32_t t0 = threadIdx.x & (group - 1);
    for (uint32_t k = threadIdx.x >> group_shift; k < kListSlices; k += groups) {
        const uint32_t n_t = sh_n[k];
        for (uint32_t t = t0; t < n_t; t += group) {
            const uint64_t q = sh_q0[k] + t, at = sh_at[k] + t;
            const uint64_t p = b.tile_pos ? b.tile_pos[q] : q;
            b.act_src[at] = b.op_src[p];
            b.act_lin[at] = sh_lin[k] + ((uint64_t)t << tile_shift);
            b.act_dst[at] = b.op_dst[p];
        }
    }
}

__global__ void clear_list_kernel(BatchDev b)
{
    b.plan->n_act = 0;
    b.plan->n_act_asked = 0;
}

hipError_t launch_stage_and_mark(const BatchDev& b, uint8_t* arena, bool compact, uint64_t max_tiles, hipStream_t s)
{
    if (b.n_sc_tiles == 0) {
        uint64_t blocks = (b.n_slices + 255) / 256;
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL(finalize_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, arena, 1);
        return hipGetLastError();
    }
    uint32_t tile_shift = 0, group_shift = 0;
    while ((1u << tile_shift) < b.tile_bytes) ++tile_shift;
    while (group_shift < 6 && (1u << group_shift) < b.tiles_per_slice) ++group_shift;
    const uint32_t parts = compact ? 1u : (b.tiles_per_slice + kTilesPerWave - 1) / kTilesPerWave;
    const uint64_t blocks = (((b.n_slices * parts) << group_shift) + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (compact) {
        if (max_tiles > b.act_capacity) max_tiles = b.act_capacity;
        hipLaunchKernelGGL(clear_list_kernel, dim3(1), dim3(1), 0, s, b);
        hipLaunchKernelGGL(list_tiles_kernel, dim3((uint32_t)((b.n_slices + kListSlices - 1) / kListSlices)), dim3(256), 0, s, b, arena,
                           group_shift, tile_shift, max_tiles);
    } else {
        hipLaunchKernelGGL(stage_tiles_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, arena, group_shift, tile_shift, parts);
        if (parts > 1) return launch_mark_done(b, false, s);
    }
    return hipGetLastError();
}

// ---- E1: what a re-plan starts from ------------------------------------------------------------
// Ascending lists of the slices that are not DONE -- those that never failed (bound by predicted cost) and those with a retry
// count (bound by rotation) -- and of the former the bytes before every position and the maximal runs of equal length
// (bind_runs.hip).  A scan in two launches, as in scan.h: what each tile of the slice table holds, then every workgroup
// combines the tiles before its own and writes its part.  A run starts where a pending slice's length differs from that of the
// pending slice before it, which may lie any number of tiles back: a maximum over (place + 1, length) finds it.
// What bounds it is launches: 20,000 slices took six (two scans of two, the lists, the run table) and 30 us on MI355X, and take two and
// 11.  Every workgroup reads 32 bytes of every tile before its own, which up to kSelfSpine tiles (4.2 million slices, 78 us) costs no
// more than a launch; beyond them one workgroup combines them in between: 16.8 million slices 437 -> 260 us, 67 million 5281 -> 982.
struct TileShare {                     // of scan_partials, scan_partials2, scan_partials3 and scan_tmp, an entry per tile
    uint64_t counts;                   // pending | retried << 20 | runs that start inside << 40 (the first pending slice left out)
    uint64_t bytes;                    // of the pending slices
    uint64_t last;                     // (tile + 1) << 32 | length of the last pending slice, 0 if there is none
    uint64_t first_len;                // length of the first pending slice
};

// A thread's kScanItems slices.
struct PendingItems {
    uint32_t len[kScanItems];
    uint32_t pending = 0, retried = 0;                       // a bit per slice
    __device__ PendingItems(const BatchDev& b, uint64_t base)
    {
        static_assert(kScanItems == 8, "a thread's slices are read as two words of states and retries and two of four lengths");
        uint64_t state = 0, retry = 0;
        if (base + kScanItems <= b.n_slices) {               // (the arrays start at multiples of 256 bytes)
            state = *reinterpret_cast<const uint64_t*>(b.s_state + base);
            retry = *reinterpret_cast<const uint64_t*>(b.s_retry + base);
            const uint4 low = *reinterpret_cast<const uint4*>(b.s_len + base), high = *reinterpret_cast<const uint4*>(b.s_len + base + 4);
            len[0] = low.x, len[1] = low.y, len[2] = low.z, len[3] = low.w;
            len[4] = high.x, len[5] = high.y, len[6] = high.z, len[7] = high.w;
        } else {
#pragma unroll
            for (uint32_t k = 0; k < kScanItems; ++k) {
                const bool there = base + k < b.n_slices;
                state |= (uint64_t)(there ? b.s_state[base + k] : TENT_SLICE_DONE) << (8 * k);
                retry |= (uint64_t)(there ? b.s_retry[base + k] : 0) << (8 * k);
                len[k] = there ? b.s_len[base + k] : 0;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kScanItems; ++k) {
            if ((uint8_t)(state >> (8 * k)) == TENT_SLICE_DONE) continue;
            if ((uint8_t)(retry >> (8 * k))) retried |= 1u << k; else pending |= 1u << k;
        }
    }
    // length of the last pending slice, behind one of length `before` (0: none)
    __device__ uint32_t last(uint32_t before) const
    {
#pragma unroll
        for (uint32_t k = 0; k < kScanItems; ++k) if ((pending >> k) & 1) before = len[k];
        return before;
    }
    __device__ uint64_t bytes() const
    {
        uint64_t sum = 0;
#pragma unroll
        for (uint32_t k = 0; k < kScanItems; ++k) if ((pending >> k) & 1) sum += len[k];
        return sum;
    }
    // a bit per slice that starts a run, behind a pending slice of length `before`
    __device__ uint32_t heads(uint32_t before) const
    {
        uint32_t h = 0;
#pragma unroll
        for (uint32_t k = 0; k < kScanItems; ++k) {
            if (!((pending >> k) & 1)) continue;
            if (len[k] != before) h |= 1u << k;
            before = len[k];
        }
        return h;
    }
};
// (place of the thread + 1, length of its last pending slice), 0 if it has none
__device__ __forceinline__ uint64_t last_of(const PendingItems& it)
{
    return it.pending ? ((uint64_t)(threadIdx.x + 1) << 32) | it.last(0) : 0;
}

__global__ void __launch_bounds__(kScanBlock) pending_share_kernel(BatchDev b)
{
    const PendingItems it(b, (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems);
    uint64_t last, counts, bytes;
    const uint64_t before = block_exclusive_scan(last_of(it), &last, ScanMax{});
    uint32_t heads = it.heads((uint32_t)before);
    if (it.pending && before == 0) {                         // the tile's first pending slice: seen by the next kernel
        const uint32_t k = (uint32_t)__ffs((int)it.pending) - 1;
        heads &= ~(1u << k);
        uint32_t first = 0;
#pragma unroll
        for (uint32_t e = 0; e < kScanItems; ++e) first = e == k ? it.len[e] : first;
        b.scan_tmp[blockIdx.x] = first;
    }
    block_exclusive_scan((uint64_t)__popc(it.pending) | ((uint64_t)__popc(it.retried) << 20) | ((uint64_t)__popc(heads) << 40), &counts,
                         ScanSum{});
    block_exclusive_scan(it.bytes(), &bytes, ScanSum{});
    if (threadIdx.x != 0) return;
    b.scan_partials[blockIdx.x] = counts;
    b.scan_partials2[blockIdx.x] = bytes;
    b.scan_partials3[blockIdx.x] = last ? ((uint64_t)(blockIdx.x + 1) << 32) | (uint32_t)last : 0;
}

// What a stretch of tiles holds.
struct TilesHold {
    uint64_t lists = 0;                // pending | retried << 32
    uint64_t runs = 0;
    uint64_t bytes = 0;
    uint64_t last = 0;                 // as in TileShare
};
// The tiles [lo, end), at most kScanBlock of them, a thread each, by a whole workgroup: adds them to `all`, which holds those before lo;
// returns those before the thread's own.
__device__ __forceinline__ TilesHold add_tiles(const BatchDev& b, uint32_t lo, uint32_t end, TilesHold& all)
{
    const uint32_t u = lo + threadIdx.x;
    TileShare s{0, 0, 0, 0};
    if (u < end) s = TileShare{b.scan_partials[u], b.scan_partials2[u], b.scan_partials3[u], b.scan_tmp[u]};
    TilesHold row, own;
    own.last = block_exclusive_scan(s.last, &row.last, ScanMax{});
    own.last = own.last ? own.last : all.last;
    const uint32_t starts = s.last != 0 && (uint32_t)s.first_len != (uint32_t)own.last ? 1u : 0u;
    own.lists = all.lists + block_exclusive_scan((s.counts & 0xFFFFFu) | (((s.counts >> 20) & 0xFFFFFu) << 32), &row.lists, ScanSum{});
    own.runs = all.runs + block_exclusive_scan((s.counts >> 40) + starts, &row.runs, ScanSum{});
    own.bytes = all.bytes + block_exclusive_scan(s.bytes, &row.bytes, ScanSum{});
    all.lists += row.lists;
    all.runs += row.runs;
    all.bytes += row.bytes;
    all.last = row.last ? row.last : all.last;
    return own;
}

// One workgroup: every tile's share -> what the tiles before it hold, in the same words (`runs` where the first length was).
__global__ void __launch_bounds__(kScanBlock) pending_spine_kernel(BatchDev b, uint32_t tiles)
{
    TilesHold all;
    for (uint32_t lo = 0; lo < tiles; lo += kScanBlock) {
        const TilesHold own = add_tiles(b, lo, tiles, all);
        const uint32_t u = lo + threadIdx.x;
        if (u >= tiles) continue;
        b.scan_partials[u] = own.lists;
        b.scan_partials2[u] = own.bytes;
        b.scan_partials3[u] = own.last;
        b.scan_tmp[u] = own.runs;
    }
}

__global__ void __launch_bounds__(kScanBlock) pending_lists_kernel(BatchDev b, int spined)
{
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    const PendingItems it(b, base);
    TilesHold before;
    if (spined) {
        before.lists = b.scan_partials[blockIdx.x];
        before.bytes = b.scan_partials2[blockIdx.x];
        before.last = b.scan_partials3[blockIdx.x];
        before.runs = b.scan_tmp[blockIdx.x];
    } else {
        for (uint32_t lo = 0; lo < blockIdx.x; lo += kScanBlock) add_tiles(b, lo, blockIdx.x, before);
    }
    const uint64_t lists = before.lists, runs = before.runs, last = before.last;
    uint64_t bytes = before.bytes;
    uint64_t total, all_bytes;
    const uint64_t in_tile = block_exclusive_scan(last_of(it), &total, ScanMax{});
    const uint32_t heads = it.heads((uint32_t)(in_tile ? in_tile : last));
    const uint64_t at = block_exclusive_scan(
        (uint64_t)__popc(it.pending) | ((uint64_t)__popc(it.retried) << 20) | ((uint64_t)__popc(heads) << 40), &total, ScanSum{});
    bytes += block_exclusive_scan(it.bytes(), &all_bytes, ScanSum{});
    uint32_t q = (uint32_t)lists + (uint32_t)(at & 0xFFFFFu), r = (uint32_t)(lists >> 32) + (uint32_t)((at >> 20) & 0xFFFFFu);
    uint64_t run = runs + (at >> 40);                        // runs that start before the slice
#pragma unroll
    for (uint32_t k = 0; k < kScanItems; ++k) {
        if ((it.retried >> k) & 1) b.retry_ids[r++] = (uint32_t)(base + k);
        if (!((it.pending >> k) & 1)) continue;
        // a transfer contributes at most two runs, so the capacity of 2 * n_desc always suffices
        if ((heads >> k) & 1) {
            if (run < b.run_capacity) b.run_start[run] = q;
            ++run;
        }
        b.pending[q] = (uint32_t)(base + k);
        b.s_run[q] = (uint32_t)(run - 1);
        b.len_pre[q] = bytes;
        bytes += it.len[k];
        ++q;
    }
    if (blockIdx.x != gridDim.x - 1 || threadIdx.x != 0) return;
    const uint64_t n_pending = (lists & 0xFFFFFFFFu) + (total & 0xFFFFFu);
    uint64_t n_runs = runs + (total >> 40);
    if (n_runs > b.run_capacity) n_runs = b.run_capacity;
    b.plan->n_pending = n_pending;
    b.plan->n_retry = (lists >> 32) + ((total >> 20) & 0xFFFFFu);
    b.plan->n_runs = n_runs;
    b.run_start[n_runs] = (uint32_t)n_pending;
}

hipError_t launch_compact(const BatchDev& b, hipStream_t s)
{
    const uint64_t tiles = scan_tiles(b.n_slices);
    if (tiles == 0 || tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
    // (one tile alone needs no other's share)
    if (tiles > 1) hipLaunchKernelGGL(pending_share_kernel, dim3((uint32_t)tiles), dim3(kScanBlock), 0, s, b);
    const bool spined = tiles > kSelfSpine;
    if (spined) hipLaunchKernelGGL(pending_spine_kernel, dim3(1), dim3(kScanBlock), 0, s, b, (uint32_t)tiles);
    hipLaunchKernelGGL(pending_lists_kernel, dim3((uint32_t)tiles), dim3(kScanBlock), 0, s, b, spined ? 1 : 0);
    return hipGetLastError();
}

// ---- slice state bookkeeping ------------------------------------------------------------------
__global__ void __launch_bounds__(256) mark_done_kernel(BatchDev b, int compact)
{
    if (compact && b.plan->compact_overflow != 0) return;       // incomplete copies: the slices stay BOUND
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride)
        if (b.s_state[i] == TENT_SLICE_BOUND) b.s_state[i] = TENT_SLICE_DONE;
}

hipError_t launch_mark_done(const BatchDev& b, bool compact, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(mark_done_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, compact ? 1 : 0);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256) reset_kernel(BatchDev b)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride) {
        b.s_state[i] = TENT_SLICE_PENDING;
        b.s_retry[i] = 0;
    }
}

hipError_t launch_reset(const BatchDev& b, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(reset_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b);
    return hipGetLastError();
}

// Rail simulator: a bound slice completes iff the rail's byte budget covers the bytes queued
// ahead of the plan, the slices staged before it, and the slice itself; otherwise it returns to
// the pending set.  The count of completed slices is an integer sum, so its value does not
// depend on the order of the atomic adds.
__global__ void __launch_bounds__(256) retire_kernel(BatchDev b, BudgetParams bp, Report told)
{
    __shared__ unsigned long long block_done;
    if (threadIdx.x == 0) block_done = 0;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    unsigned long long mine = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride) {
        if (b.s_state[i] != TENT_SLICE_BOUND) continue;
        const uint32_t d = b.s_rail[i];
        const uint64_t last = bp.queued[d] + b.s_stage_off[i] + b.s_len[i];
        const bool fits = last >= bp.queued[d] && last <= bp.budget[d];
        if (fits) ++mine; else b.s_state[i] = TENT_SLICE_PENDING;
    }
    if (mine) atomicAdd(&block_done, mine);
    __syncthreads();
    unsigned long long added = 0;
    if (threadIdx.x == 0 && block_done) added = atomicAdd((unsigned long long*)&b.plan->n_done, block_done);
    if (!finishes_last(b.plan, kTicketRetire, added) || threadIdx.x != 0) return;
    const unsigned long long total = take_counter(&b.plan->n_done);
    if (!told.to) return;
    tell(&told.to->n_done, (uint64_t)total);
    tell_done(told);
}

hipError_t launch_retire(const BatchDev& b, const BudgetParams& bp, Report told, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(retire_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, bp, told);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256) count_remaining_kernel(BatchDev b, Report told)
{
    __shared__ unsigned long long block_cnt;
    if (threadIdx.x == 0) block_cnt = 0;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    unsigned long long mine = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride)
        mine += b.s_state[i] != TENT_SLICE_DONE;
    if (mine) atomicAdd(&block_cnt, mine);
    __syncthreads();
    unsigned long long added = 0;
    if (threadIdx.x == 0 && block_cnt) added = atomicAdd((unsigned long long*)&b.plan->n_remaining, block_cnt);
    if (!finishes_last(b.plan, kTicketRemaining, added) || threadIdx.x != 0) return;
    tell(&told.to->n_remaining, (uint64_t)take_counter(&b.plan->n_remaining));
    tell_done(told);
}

hipError_t launch_count_remaining(const BatchDev& b, Report told, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 1023) / 1024;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(count_remaining_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, told);
    return hipGetLastError();
}

}  // namespace tent
