// Device side of tent_declare: destination extents in ascending device address (the order in which
// the scatter kernel walks them) and the overlap check between extents.
//
// All extents get a 64-bit key (device address of their first byte) and are sorted with rocPRIM's
// radix sort (the one library primitive of the build).  Over the sorted order, "furthest end seen so
// far" is an exclusive max-scan; a destination extent overlaps something iff it starts before the
// furthest end of everything before it, a source extent overlaps a destination iff it starts before
// the furthest end of the destinations before it.  The scans are the engine's own (scan.h).
//
// Only the address bits in which the extents differ are sorted: KV pages of 32 KiB in a pool of 20 GiB differ in 20 of 64.
// Declarations of up to kSmallOrder extents do all of it in one workgroup (a bitonic sort in LDS), because there the dozen
// launches cost more than the work: 626 extents on either side 115 -> 25 us from the first kernel to the last.
//
// Nothing here allocates, copies to the host or waits: the caller hands in a workspace and a word of host memory
// for the verdict, and reads it when the stream has got that far.
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "scan.h"

namespace tent {

namespace {

// What must start at zero in a batch's tables: retry counts, request modes, the result block.
__device__ __forceinline__ void clear_tables(const BatchDev& b, uint64_t at, uint64_t stride)
{
    for (uint64_t i = at; i < b.n_slices; i += stride) b.s_retry[i] = 0;
    for (uint64_t i = at; i < b.n_desc; i += stride) b.req_mode[i] = 0;
    uint64_t* plan = reinterpret_cast<uint64_t*>(b.plan);
    static_assert(sizeof(PlanState) % 8 == 0, "the result block is cleared in words of 8 bytes");
    for (uint64_t i = at; i < sizeof(PlanState) / 8; i += stride) plan[i] = 0;
}

__global__ void __launch_bounds__(256) declare_clear_kernel(BatchDev b)
{
    clear_tables(b, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, (uint64_t)gridDim.x * blockDim.x);
}

// value = index into [destinations | sources]: v < n_dst is destination extent v
__global__ void __launch_bounds__(256) declare_keys_kernel(BatchDev b, uint64_t n, uint64_t* keys, uint32_t* vals)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    clear_tables(b, at, stride);
    for (uint64_t v = at; v < n; v += stride) {
        const tent_extent x = v < b.n_dst_ext ? b.dst_ext[v] : b.src_ext[v - b.n_dst_ext];
        keys[v] = b.seg_base[x.seg] + x.off;
        vals[v] = (uint32_t)v;
    }
}

// End of the extent at sorted position p (all extents / destinations only).
struct EndAny {
    const tent_extent* dst_ext; const tent_extent* src_ext; uint64_t n_dst;
    const uint64_t* keys; const uint32_t* vals;
    __device__ uint64_t operator()(uint64_t p) const
    {
        const uint32_t v = vals[p];
        return keys[p] + (v < n_dst ? dst_ext[v].len : src_ext[v - n_dst].len);
    }
};
struct EndDst {
    const tent_extent* dst_ext; uint64_t n_dst;
    const uint64_t* keys; const uint32_t* vals;
    __device__ uint64_t operator()(uint64_t p) const
    {
        const uint32_t v = vals[p];
        return v < n_dst ? keys[p] + dst_ext[v].len : 0;
    }
};
struct IsDst {
    const uint32_t* vals; uint64_t n_dst;
    __device__ uint64_t operator()(uint64_t p) const { return vals[p] < n_dst; }
};

// The overlap check, and the destinations in sorted order (a stable compaction of the sorted values).  `told` is host
// memory; every thread that writes it writes the same.
__global__ void __launch_bounds__(256) declare_verdict_kernel(uint64_t n_dst, uint64_t n, const uint64_t* keys, const uint32_t* vals,
                                                              const uint64_t* far_any, const uint64_t* far_dst,
                                                              const uint64_t* pos, uint32_t* order, uint32_t* rank, uint32_t* told)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const uint32_t v = vals[p];
        const bool is_dst = v < n_dst;
        if (far_any) bad |= keys[p] < (is_dst ? far_any[p] : far_dst[p]);
        if (is_dst) {
            order[pos[p]] = v;
            rank[v] = (uint32_t)pos[p];                      // the inverse: position of every extent in address order
        }
    }
    if (bad) *told = 1;
}

constexpr uint32_t kSmallOrder = 4096;           // extents one workgroup puts in order

// ---- all of it in one workgroup ------------------------------------------------------------------
constexpr uint32_t kSmallThreads = 1024;
constexpr uint32_t kSmallBits = 13;              // a sorted word is (differing address bits) << kSmallBits | value

// Exclusive scan of one value per thread over the workgroup.
template <class Op>
__device__ __forceinline__ uint64_t small_scan(uint64_t v, uint64_t* wave_out, Op op)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t inc = wave_inclusive_scan(v, op);
    __syncthreads();
    if (lane == 63) wave_out[wave] = inc;
    __syncthreads();
    uint64_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before = op(before, wave_out[w]);
    const uint64_t below = __shfl_up((unsigned long long)inc, 1, 64);
    return lane == 0 ? before : op(before, below);
}

// Bitonic sort of kItems * kSmallThreads words, of which the first n_pow2 count; thread t holds the words t, t +
// kSmallThreads, ...  Partners up to 32 apart are lanes of one wavefront and those kSmallThreads and more apart are the thread's own,
// so that only one step in four needs LDS and barriers (all steps through LDS: 27 instead of 25 us for the whole kernel
// at 1252 extents).  The sorted words end in LDS.
template <uint32_t kItems>
__device__ __forceinline__ void small_sort(uint64_t (&w)[kItems], uint32_t n_pow2, uint64_t* word)
{
    const uint32_t t = threadIdx.x;
    for (uint32_t k = 2; k <= n_pow2; k <<= 1)
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            uint64_t other[kItems];
            if (j >= kSmallThreads) {
#pragma unroll
                for (uint32_t e = 0; e < kItems; ++e)
                    other[e] = (j / kSmallThreads) == 1 ? w[(e ^ 1) % kItems] : w[(e ^ 2) % kItems];
            } else if (j >= 64) {
#pragma unroll
                for (uint32_t e = 0; e < kItems; ++e) word[e * kSmallThreads + t] = w[e];
                __syncthreads();
#pragma unroll
                for (uint32_t e = 0; e < kItems; ++e) other[e] = word[e * kSmallThreads + (t ^ j)];
                __syncthreads();
            } else {
#pragma unroll
                for (uint32_t e = 0; e < kItems; ++e) other[e] = __shfl_xor((unsigned long long)w[e], (int)j, 64);
            }
#pragma unroll
            for (uint32_t e = 0; e < kItems; ++e) {
                const uint32_t p = e * kSmallThreads + t;
                const bool take_least = ((p & j) == 0) == ((p & k) == 0);
                const uint64_t least = w[e] < other[e] ? w[e] : other[e], most = w[e] < other[e] ? other[e] : w[e];
                w[e] = take_least ? least : most;
            }
        }
#pragma unroll
    for (uint32_t e = 0; e < kItems; ++e) word[e * kSmallThreads + t] = w[e];
    __syncthreads();
}

template <uint32_t kItems>
__global__ void __launch_bounds__(kSmallThreads) declare_small_kernel(BatchDev b, uint32_t n, uint32_t n_pow2, int check, KeyBits bits,
                                                                      uint32_t* order, uint32_t* rank, uint32_t* told)
{
    __shared__ uint64_t word[kItems * kSmallThreads];
    __shared__ uint64_t wave_out[kSmallThreads / 64];
    const uint32_t t = threadIdx.x;
    clear_tables(b, t, kSmallThreads);
    const uint32_t n_dst = (uint32_t)b.n_dst_ext;
    const uint64_t mask = (1ull << (bits.end - bits.begin)) - 1;
    uint64_t w[kItems];
#pragma unroll
    for (uint32_t e = 0; e < kItems; ++e) {
        const uint32_t v = e * kSmallThreads + t;
        w[e] = ~0ull;                                        // behind every extent
        if (v < n) {
            const tent_extent x = v < n_dst ? b.dst_ext[v] : b.src_ext[v - n_dst];
            w[e] = (((b.seg_base[x.seg] + x.off) >> bits.begin & mask) << kSmallBits) | v;
        }
    }
    small_sort<kItems>(w, n_pow2, word);
    // kItems consecutive sorted extents per thread
    uint64_t begin[kItems], end_any[kItems], end_dst[kItems];
    uint32_t value[kItems];
    uint64_t far_any = 0, far_dst = 0, dsts = 0;
#pragma unroll
    for (uint32_t i = 0; i < kItems; ++i) {
        const uint32_t p = t * kItems + i;
        value[i] = 0xFFFFFFFFu;
        begin[i] = end_any[i] = end_dst[i] = 0;
        if (p < n) {
            const uint32_t v = (uint32_t)word[p] & ((1u << kSmallBits) - 1);
            const bool is_dst = v < n_dst;
            const tent_extent x = is_dst ? b.dst_ext[v] : b.src_ext[v - n_dst];
            value[i] = v;
            begin[i] = b.seg_base[x.seg] + x.off;
            end_any[i] = begin[i] + x.len;
            end_dst[i] = is_dst ? end_any[i] : 0;
            dsts += is_dst ? 1 : 0;
        }
        far_any = end_any[i] > far_any ? end_any[i] : far_any;
        far_dst = end_dst[i] > far_dst ? end_dst[i] : far_dst;
    }
    far_any = small_scan(far_any, wave_out, ScanMax{});
    far_dst = small_scan(far_dst, wave_out, ScanMax{});
    uint64_t pos = small_scan(dsts, wave_out, ScanSum{});
    bool bad = false;
#pragma unroll
    for (uint32_t i = 0; i < kItems; ++i) {
        if (value[i] == 0xFFFFFFFFu) continue;
        const bool is_dst = value[i] < n_dst;
        bad |= begin[i] < (is_dst ? far_any : far_dst);
        if (is_dst) {
            order[pos] = value[i];
            rank[value[i]] = (uint32_t)pos;
            ++pos;
        }
        far_any = end_any[i] > far_any ? end_any[i] : far_any;
        far_dst = end_dst[i] > far_dst ? end_dst[i] : far_dst;
    }
    if (bad && check) *told = 1;
}

uint32_t grid_for(uint64_t n)
{
    uint64_t blocks = (n + 255) / 256;
    return (uint32_t)(blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks));
}

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Carves the workspace: two key arrays, two value arrays, three scan outputs, scan partials, the
// sort's own temporary storage.
struct OrderWorkspace {
    uint64_t *keys_in, *keys, *far_any, *far_dst, *pos, *partials, *partials2, *partials3;
    uint32_t *vals_in, *vals;
    void* sort_tmp;
    size_t sort_bytes, total;
};

hipError_t layout(uint64_t n, KeyBits bits, uint8_t* base, OrderWorkspace* w)
{
    size_t sort_bytes = 0;
    hipError_t e = rocprim::radix_sort_pairs(nullptr, sort_bytes, (uint64_t*)nullptr, (uint64_t*)nullptr,
                                             (uint32_t*)nullptr, (uint32_t*)nullptr, n, bits.begin, bits.end, nullptr);
    if (e != hipSuccess) return e;
    const size_t n8 = up256((size_t)(n + 1) * 8), n4 = up256((size_t)n * 4);
    size_t at = 0;
    auto take = [&](size_t bytes) { uint8_t* p = base ? base + at : nullptr; at += up256(bytes); return p; };
    w->keys_in = (uint64_t*)take(n8);
    w->keys = (uint64_t*)take(n8);
    w->far_any = (uint64_t*)take(n8);
    w->far_dst = (uint64_t*)take(n8);
    w->pos = (uint64_t*)take(n8);
    w->partials = (uint64_t*)take(scan_partials_capacity(n) * 8);
    w->partials2 = (uint64_t*)take(scan_partials_capacity(n) * 8);
    w->partials3 = (uint64_t*)take(scan_partials_capacity(n) * 8);
    w->vals_in = (uint32_t*)take(n4);
    w->vals = (uint32_t*)take(n4);
    w->sort_tmp = take(sort_bytes);
    w->sort_bytes = sort_bytes;
    w->total = at;
    return hipSuccess;
}

}  // namespace

static bool is_small(uint64_t n, KeyBits bits) { return n <= kSmallOrder && bits.end - bits.begin + kSmallBits < 64; }

// Bytes of workspace launch_declare needs for n_dst destination and n_src source extents.
hipError_t order_workspace_bytes(uint64_t n_dst, uint64_t n_src, bool check, KeyBits bits, uint64_t* bytes_out)
{
    const uint64_t n = n_dst + (check ? n_src : 0);
    *bytes_out = 0;
    if (is_small(n, bits)) return hipSuccess;
    OrderWorkspace w;
    hipError_t e = layout(n, bits, nullptr, &w);
    *bytes_out = w.total;
    return e;
}

// What the address order counts against the limit of tent_declare_static: the workspace of a sort over all address
// bits with one array of scan partials, whatever order_workspace_bytes() comes to.
hipError_t order_measure(uint64_t n_dst, uint64_t n_src, bool check, uint64_t* bytes_out)
{
    const uint64_t n = n_dst + (check ? n_src : 0);
    OrderWorkspace w;
    hipError_t e = layout(n, KeyBits{0, 64}, nullptr, &w);
    if (e != hipSuccess) return e;
    *bytes_out = w.total - 2 * up256(scan_partials_capacity(n) * 8);
    return hipSuccess;
}

// The device work of a declaration whose descriptors lie in the batch's tables.  Clears what must start at zero; with
// `order` fills order_out[n_dst] with destination extent indices in ascending address and rank_out[n_dst] with the
// inverse (position of every extent in that order); with `check` sets *overlap_told (host memory, 0 before) if a
// destination extent overlaps another destination or any source extent.  Only enqueues on `s`; `workspace`
// (device, order_workspace_bytes() bytes, 256-byte aligned) is in use until the stream has passed this work.
hipError_t launch_declare(const BatchDev& b, bool order, bool check, KeyBits bits, uint32_t* order_out, uint32_t* rank_out,
                          uint32_t* overlap_told, void* workspace, hipStream_t s)
{
    const uint64_t n = b.n_dst_ext + (check ? b.n_src_ext : 0);
    if (!order) {
        hipLaunchKernelGGL(declare_clear_kernel, dim3(grid_for(b.n_slices)), dim3(256), 0, s, b);
        return hipGetLastError();
    }
    if (is_small(n, bits)) {
        uint32_t n_pow2 = 2;
        while (n_pow2 < n) n_pow2 <<= 1;
        const dim3 one(1), block(kSmallThreads);
        const int test = check ? 1 : 0;
        if (n <= kSmallThreads)
            hipLaunchKernelGGL(declare_small_kernel<1>, one, block, 0, s, b, (uint32_t)n, n_pow2, test, bits, order_out, rank_out, overlap_told);
        else if (n <= 2 * kSmallThreads)
            hipLaunchKernelGGL(declare_small_kernel<2>, one, block, 0, s, b, (uint32_t)n, n_pow2, test, bits, order_out, rank_out, overlap_told);
        else
            hipLaunchKernelGGL(declare_small_kernel<4>, one, block, 0, s, b, (uint32_t)n, n_pow2, test, bits, order_out, rank_out, overlap_told);
        return hipGetLastError();
    }
    OrderWorkspace w;
    hipError_t e = layout(n, bits, static_cast<uint8_t*>(workspace), &w);
    if (e != hipSuccess) return e;
    const uint32_t g = grid_for(n);
    hipLaunchKernelGGL(declare_keys_kernel, dim3(g), dim3(256), 0, s, b, n, w.keys_in, w.vals_in);
    size_t bytes = w.sort_bytes;
    e = rocprim::radix_sort_pairs(w.sort_tmp, bytes, w.keys_in, w.keys, w.vals_in, w.vals, n, bits.begin, bits.end, s);
    if (e != hipSuccess) return e;
    const auto pos = scan_job(IsDst{w.vals, b.n_dst_ext}, n, w.pos, w.partials3);
    if (check) {
        e = run_scans(s, scan_job(EndAny{b.dst_ext, b.src_ext, b.n_dst_ext, w.keys, w.vals}, n, w.far_any, w.partials, ScanMax{}),
                      scan_job(EndDst{b.dst_ext, b.n_dst_ext, w.keys, w.vals}, n, w.far_dst, w.partials2, ScanMax{}), pos);
    } else {
        e = run_scans(s, pos);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(declare_verdict_kernel, dim3(g), dim3(256), 0, s, b.n_dst_ext, n, w.keys, w.vals, check ? w.far_any : nullptr,
                       w.far_dst, w.pos, order_out, rank_out, overlap_told);
    return hipGetLastError();
}

}  // namespace tent
