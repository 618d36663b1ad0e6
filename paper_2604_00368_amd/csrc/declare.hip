// Device side of tent_declare: destination extents in ascending device address (the order in which the copies walk them) and the
// overlap check between extents.
//
// Only destinations are put in order.  Two of them overlap iff some extent reaches beyond the start of the next one; a source
// overlaps a destination iff the last destination that starts before the source's end reaches beyond its start (where
// destinations overlap each other the batch is refused anyway).
//
// Three ways to the order, by how many extents there are and in how many address bits the destinations differ (all other bits are
// the same, and KV pages of 32 KiB in a pool of 20 GiB differ in 20 of 64):
//   one workgroup   up to kSmallOrder extents a side, where launches cost more than the work;
//   by slots        where the differing bits number at most kSlotsPerExtent places per destination: every destination is put at
//                   its place in a table and a scan over the table counts the destinations before each place.  Paged pools, whose pages
//                   lie at multiples of a power of two, nearly fill such a table;
//   by sorting      everything else (byte ranges at any address): rocPRIM's radix sort of (address, index) pairs, the one library
//                   primitive of the build.
// MI355X: 41,000 pages of 32 KiB a side in 14 launches and 165 us when both sides were sorted and scanned, in 5 and 50 us by slots;
// 626 pages a side in one workgroup 24.5 -> 4.6 us (by sorting, where the addresses differ in more bits, 18).
//
// Nothing here allocates, copies to the host or waits: the caller hands in a workspace and a word of host memory
// for the verdict, and reads it when the stream has got that far.  A batch whose destinations overlap still gets a sound order
// (a permutation), because it may be planned before the verdict is read.
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

__device__ __forceinline__ uint64_t begin_of(const BatchDev& b, const tent_extent& x) { return b.seg_base[x.seg] + x.off; }

constexpr uint32_t kSmallOrder = 4096;           // extents a side that one workgroup puts in order
constexpr uint64_t kSlotsPerExtent = 16;         // beyond this the table costs more than the sort (both are bound by memory then)

// ---- all of it in one workgroup ------------------------------------------------------------------
constexpr uint32_t kSmallThreads = 1024;
constexpr uint32_t kSmallSlots = 8192;           // places of a table in LDS
constexpr uint32_t kSmallBits = 12;              // a sorted word is (differing address bits) << kSmallBits | index

// Exclusive prefix sum of one value per thread over the workgroup.
__device__ __forceinline__ uint32_t small_prefix(uint32_t v, uint32_t* wave_out)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = __shfl_up(inc, d, 64);
        if ((int)lane >= d) inc += up;
    }
    if (lane == 63) wave_out[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before += wave_out[w];
    return before + inc - v;
}

// Bitonic sort of kItems * kSmallThreads words, of which the first n_pow2 count; thread t holds the words t, t +
// kSmallThreads, ...  Partners up to 32 apart are lanes of one wavefront and those kSmallThreads and more apart are the thread's own,
// so that only one step in four needs LDS and barriers.  The sorted words end in LDS.
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

// kItems extents a side per thread; kSlots: the destinations' places lie in LDS, else they are sorted there.
template <uint32_t kItems, bool kSlots>
__global__ void __launch_bounds__(kSmallThreads) declare_small_kernel(BatchDev b, uint32_t n_src, uint32_t n_pow2, int check,
                                                                      AddressSlots map, uint32_t* order, uint32_t* rank, uint32_t* told)
{
    struct Table {
        uint32_t who[kSmallSlots];               // 1 + destination at the place, 0: none
        uint16_t before[kSmallSlots + 1];        // destinations at lower places
        uint16_t order[kSmallOrder];
        uint32_t doubles;
    };
    union Lds {
        uint64_t word[kItems * kSmallThreads];
        Table table;
        __device__ Lds() {}
    };
    __shared__ Lds sh;
    __shared__ uint32_t wave_out[kSmallThreads / 64];
    const uint32_t t = threadIdx.x;
    const uint32_t n_dst = (uint32_t)b.n_dst_ext;
    uint64_t begin[kItems], end[kItems], src_begin[kItems], src_end[kItems];
#pragma unroll
    for (uint32_t e = 0; e < kItems; ++e) {
        const uint32_t v = e * kSmallThreads + t;
        begin[e] = end[e] = src_begin[e] = src_end[e] = 0;
        if (v < n_dst) {
            const tent_extent x = b.dst_ext[v];
            begin[e] = begin_of(b, x);
            end[e] = begin[e] + x.len;
        }
        if (v < n_src) {
            const tent_extent x = b.src_ext[v];
            src_begin[e] = begin_of(b, x);
            src_end[e] = src_begin[e] + x.len;
        }
    }
    clear_tables(b, t, kSmallThreads);
    bool bad = false;
    if constexpr (kSlots) {
        Table& tab = sh.table;
        const uint32_t n_slots = (uint32_t)map.n_slots;
        for (uint32_t i = t; i < n_slots; i += kSmallThreads) tab.who[i] = 0;
        if (t == 0) tab.doubles = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < kItems; ++e) {
            const uint32_t v = e * kSmallThreads + t;
            if (v >= n_dst) continue;
            if (atomicCAS(&tab.who[map.slot(begin[e])], 0u, v + 1) != 0) {       // two at one place: behind all others
                const uint32_t p = n_dst - 1 - atomicAdd(&tab.doubles, 1u);
                order[p] = v;
                rank[v] = p;
                tab.order[p] = (uint16_t)v;
                bad = true;
            }
        }
        __syncthreads();
        const uint32_t each = n_slots > kSmallThreads ? n_slots / kSmallThreads : 1, first = t * each;
        uint32_t here = 0;
        if (first < n_slots)
            for (uint32_t i = first; i < first + each; ++i) here += tab.who[i] != 0 ? 1u : 0u;
        uint32_t p = small_prefix(here, wave_out);
        if (first < n_slots) {
            for (uint32_t i = first; i < first + each; ++i) {
                tab.before[i] = (uint16_t)p;
                const uint32_t v = tab.who[i];
                if (v == 0) continue;
                order[p] = v - 1;
                rank[v - 1] = p;
                tab.order[p] = (uint16_t)(v - 1);
                ++p;
            }
            if (first + each == n_slots) tab.before[n_slots] = (uint16_t)p;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < kItems; ++e) {
            const uint32_t v = e * kSmallThreads + t;
            if (v < n_dst) bad |= tab.before[map.starts_before(end[e])] != tab.before[map.slot(begin[e]) + 1];
            if (v < n_src) {
                const uint32_t last = tab.before[map.starts_before(src_end[e])];
                if (last != 0) {
                    const tent_extent x = b.dst_ext[tab.order[last - 1]];
                    bad |= begin_of(b, x) + x.len > src_begin[e];
                }
            }
        }
    } else {
        uint64_t w[kItems];
#pragma unroll
        for (uint32_t e = 0; e < kItems; ++e) {
            const uint32_t v = e * kSmallThreads + t;
            w[e] = v < n_dst ? (map.slot(begin[e]) << kSmallBits) | v : ~0ull;    // the others behind every extent
        }
        small_sort<kItems>(w, n_pow2, sh.word);
        auto start = [&](uint32_t p) { return map.base + ((sh.word[p] >> kSmallBits) << map.shift); };
#pragma unroll
        for (uint32_t e = 0; e < kItems; ++e) {
            const uint32_t p = e * kSmallThreads + t;
            if (p < n_dst) {
                const uint32_t v = (uint32_t)sh.word[p] & ((1u << kSmallBits) - 1);
                order[p] = v;
                rank[v] = p;
                if (p + 1 < n_dst) bad |= start(p) + b.dst_ext[v].len > start(p + 1);
            }
            if (p < n_src) {
                uint32_t lo = 0, hi = n_dst;                          // destinations that start before the source's end
                while (lo < hi) {
                    const uint32_t mid = lo + ((hi - lo) >> 1);
                    if (start(mid) < src_end[e]) lo = mid + 1; else hi = mid;
                }
                if (lo != 0) {
                    const tent_extent x = b.dst_ext[(uint32_t)sh.word[lo - 1] & ((1u << kSmallBits) - 1)];
                    bad |= begin_of(b, x) + x.len > src_begin[e];
                }
            }
        }
    }
    if (bad && check) *told = 1;
}

// ---- by slots --------------------------------------------------------------------------------------
struct SlotTable {
    uint32_t* who;               // [n_slots] 1 + destination at the place, 0: none
    uint32_t* before;            // [n_slots + 1] destinations at lower places
    uint32_t* doubles;           // [n_dst] destinations whose place was taken
    uint32_t* n_doubles;
};

__global__ void __launch_bounds__(256) slots_clear_kernel(BatchDev b, SlotTable tab, uint64_t n_slots)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    clear_tables(b, at, stride);
    for (uint64_t i = at; i < n_slots; i += stride) tab.who[i] = 0;
    if (at == 0) *tab.n_doubles = 0;
}

__global__ void __launch_bounds__(256) slots_fill_kernel(BatchDev b, SlotTable tab, AddressSlots map, uint32_t* told)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < b.n_dst_ext; v += stride) {
        if (atomicCAS(&tab.who[map.slot(begin_of(b, b.dst_ext[v]))], 0u, (uint32_t)v + 1) == 0) continue;
        tab.doubles[atomicAdd(tab.n_doubles, 1u)] = (uint32_t)v;
        *told = 1;
    }
}

struct Occupied {
    const uint32_t* who;
    __device__ uint64_t operator()(uint64_t i) const { return who[i] != 0; }
};
struct StoreOrder {
    SlotTable tab;
    uint64_t n_slots;
    uint32_t *order, *rank;
    __device__ void operator()(uint64_t i, uint64_t p) const
    {
        tab.before[i] = (uint32_t)p;
        const uint32_t v = i < n_slots ? tab.who[i] : 0;
        if (v == 0) return;
        order[p] = v - 1;
        rank[v - 1] = (uint32_t)p;
    }
};

// `told` is host memory; every thread that writes it writes the same.
__global__ void __launch_bounds__(256) slots_verdict_kernel(BatchDev b, SlotTable tab, AddressSlots map, uint32_t* order, uint32_t* rank,
                                                            uint32_t* told)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (uint64_t v = at; v < b.n_dst_ext; v += stride) {
        const tent_extent x = b.dst_ext[v];
        const uint64_t begin = begin_of(b, x);
        bad |= tab.before[map.starts_before(begin + x.len)] != tab.before[map.slot(begin) + 1];
    }
    for (uint64_t v = at; v < b.n_src_ext; v += stride) {
        const tent_extent x = b.src_ext[v];
        const uint64_t begin = begin_of(b, x);
        const uint32_t last = tab.before[map.starts_before(begin + x.len)];
        if (last == 0) continue;
        const tent_extent d = b.dst_ext[order[last - 1]];
        bad |= begin_of(b, d) + d.len > begin;
    }
    const uint32_t doubles = *tab.n_doubles;                             // behind all others: the order stays a permutation
    for (uint64_t k = at; k < doubles; k += stride) {
        const uint32_t v = tab.doubles[k], p = (uint32_t)(b.n_dst_ext - 1 - k);
        order[p] = v;
        rank[v] = p;
    }
    if (bad) *told = 1;
}

// ---- by sorting ------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) declare_keys_kernel(BatchDev b, uint64_t* keys, uint32_t* vals)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    clear_tables(b, at, stride);
    for (uint64_t v = at; v < b.n_dst_ext; v += stride) {
        keys[v] = begin_of(b, b.dst_ext[v]);
        vals[v] = (uint32_t)v;
    }
}

__global__ void __launch_bounds__(256) sorted_verdict_kernel(BatchDev b, int check, const uint64_t* keys, const uint32_t* vals,
                                                             uint32_t* order, uint32_t* rank, uint32_t* told)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (uint64_t p = at; p < b.n_dst_ext; p += stride) {
        const uint32_t v = vals[p];
        order[p] = v;
        rank[v] = (uint32_t)p;                                           // the inverse: position of every extent in address order
        if (check && p + 1 < b.n_dst_ext) bad |= keys[p] + b.dst_ext[v].len > keys[p + 1];
    }
    if (check)
        for (uint64_t v = at; v < b.n_src_ext; v += stride) {
            const tent_extent x = b.src_ext[v];
            const uint64_t begin = begin_of(b, x), end = begin + x.len;
            uint64_t lo = 0, hi = b.n_dst_ext;                           // destinations that start before the source's end
            while (lo < hi) {
                const uint64_t mid = lo + ((hi - lo) >> 1);
                if (keys[mid] < end) lo = mid + 1; else hi = mid;
            }
            if (lo != 0) bad |= keys[lo - 1] + b.dst_ext[vals[lo - 1]].len > begin;
        }
    if (bad) *told = 1;
}

uint32_t grid_for(uint64_t n)
{
    uint64_t blocks = (n + 255) / 256;
    return (uint32_t)(blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks));
}

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Hands out pieces of the workspace, or (without one) adds up what they come to.
struct Pieces {
    uint8_t* base;
    size_t at = 0;
    explicit Pieces(void* ws) : base(static_cast<uint8_t*>(ws)) {}
    template <class T>
    void take(T** out, size_t count)
    {
        *out = base ? reinterpret_cast<T*>(base + at) : nullptr;
        at += up256(count * sizeof(T));
    }
};

hipError_t sort_bytes(uint64_t n, uint32_t first_bit, uint32_t last_bit, size_t* bytes)
{
    *bytes = 0;
    return rocprim::radix_sort_pairs(nullptr, *bytes, (uint64_t*)nullptr, (uint64_t*)nullptr, (uint32_t*)nullptr, (uint32_t*)nullptr, n,
                                     first_bit, last_bit, nullptr);
}

struct SortWorkspace {
    uint64_t *keys_in, *keys;
    uint32_t *vals_in, *vals;
    uint8_t* tmp;
    SortWorkspace(Pieces& p, uint64_t n, size_t tmp_bytes)
    {
        p.take(&keys_in, n);
        p.take(&keys, n);
        p.take(&vals_in, n);
        p.take(&vals, n);
        p.take(&tmp, tmp_bytes);
    }
};

struct SlotWorkspace {
    SlotTable tab;
    uint64_t* partials;
    SlotWorkspace(Pieces& p, uint64_t n_dst, uint64_t n_slots)
    {
        p.take(&tab.who, n_slots);
        p.take(&tab.before, n_slots + 1);
        p.take(&tab.doubles, n_dst);
        p.take(&tab.n_doubles, 1);
        p.take(&partials, scan_partials_capacity(n_slots));
    }
};

}  // namespace

// How the destinations of a declaration are put in order, and the bytes of workspace launch_declare needs for it; at most
// `most` bytes where there is a choice.  Without the check the order of destinations at one place is that of the list, as a
// stable sort leaves it.
hipError_t plan_order(uint64_t n_dst, uint64_t n_src, bool check, KeyBits bits, uint64_t origin, uint64_t most, OrderPlan* out)
{
    const uint32_t differing = bits.end - bits.begin;
    const uint64_t same = differing < 64 ? ~(((1ull << differing) - 1) << bits.begin) : 0;
    out->bits = bits;
    out->map = AddressSlots{origin & same, differing < 63 ? 1ull << differing : 1ull << 63, bits.begin};
    out->bytes = 0;
    const uint64_t n = check ? (n_src > n_dst ? n_src : n_dst) : n_dst;
    if (n <= kSmallOrder && (differing + kSmallBits < 64 || out->map.n_slots <= kSmallSlots)) {
        out->way = check && out->map.n_slots <= kSmallSlots ? OrderPlan::kSmallSlots : OrderPlan::kSmallSort;
        return hipSuccess;
    }
    if (check && differing < 32 && out->map.n_slots <= kSlotsPerExtent * n_dst) {
        Pieces p(nullptr);
        SlotWorkspace(p, n_dst, out->map.n_slots);
        if (p.at <= most) {
            out->way = OrderPlan::kSlots;
            out->bytes = p.at;
            return hipSuccess;
        }
    }
    out->way = OrderPlan::kSort;
    size_t tmp = 0;
    const hipError_t e = sort_bytes(n_dst, bits.begin, bits.end, &tmp);
    Pieces p(nullptr);
    SortWorkspace(p, n_dst, tmp);
    out->bytes = p.at;
    return e;
}

// What the address order counts against the limit of tent_declare_static: five arrays of 8 bytes and two of 4 per extent that the
// check looks at, one array of scan partials and the storage of a sort over all address bits -- the limit's definition, whatever
// plan_order() comes to (which is never more).
hipError_t order_measure(uint64_t n_dst, uint64_t n_src, bool check, uint64_t* bytes_out)
{
    const uint64_t n = n_dst + (check ? n_src : 0);
    size_t tmp = 0;
    const hipError_t e = sort_bytes(n, 0, 64, &tmp);
    *bytes_out = 5 * up256((n + 1) * 8) + up256(scan_partials_capacity(n) * 8) + 2 * up256(n * 4) + up256(tmp);
    return e;
}

// The device work of a declaration whose descriptors lie in the batch's tables.  Clears what must start at zero; with
// `order` fills order_out[n_dst] with destination extent indices in ascending address and rank_out[n_dst] with the
// inverse (position of every extent in that order); with `check` sets *overlap_told (host memory, 0 before) if a
// destination extent overlaps another destination or any source extent.  Only enqueues on `s`; `workspace`
// (device, plan.bytes, 256-byte aligned) is in use until the stream has passed this work.
hipError_t launch_declare(const BatchDev& b, bool order, bool check, const OrderPlan& plan, uint32_t* order_out, uint32_t* rank_out,
                          uint32_t* overlap_told, void* workspace, hipStream_t s)
{
    if (!order) {
        hipLaunchKernelGGL(declare_clear_kernel, dim3(grid_for(b.n_slices)), dim3(256), 0, s, b);
        return hipGetLastError();
    }
    const uint64_t n_src = check ? b.n_src_ext : 0, n = n_src > b.n_dst_ext ? n_src : b.n_dst_ext;
    const dim3 grid(grid_for(n)), block(256);
    switch (plan.way) {
    case OrderPlan::kSmallSlots:
    case OrderPlan::kSmallSort: {
        uint32_t n_pow2 = 2;
        while (n_pow2 < b.n_dst_ext) n_pow2 <<= 1;
        const auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), 0, s, b, (uint32_t)n_src, n_pow2, check ? 1 : 0, plan.map, order_out,
                               rank_out, overlap_told);
        };
        const bool slots = plan.way == OrderPlan::kSmallSlots;
        if (n <= kSmallThreads)          slots ? launch(declare_small_kernel<1, true>) : launch(declare_small_kernel<1, false>);
        else if (n <= 2 * kSmallThreads) slots ? launch(declare_small_kernel<2, true>) : launch(declare_small_kernel<2, false>);
        else                             slots ? launch(declare_small_kernel<4, true>) : launch(declare_small_kernel<4, false>);
        return hipGetLastError();
    }
    case OrderPlan::kSlots: {
        Pieces p(workspace);
        const SlotWorkspace w(p, b.n_dst_ext, plan.map.n_slots);
        hipLaunchKernelGGL(slots_clear_kernel, dim3(grid_for(plan.map.n_slots)), block, 0, s, b, w.tab, plan.map.n_slots);
        hipLaunchKernelGGL(slots_fill_kernel, dim3(grid_for(b.n_dst_ext)), block, 0, s, b, w.tab, plan.map, overlap_told);
        const hipError_t e = run_scans(s, ScanJob<Occupied, ScanSum, StoreOrder>{
            Occupied{w.tab.who}, ScanSum{}, StoreOrder{w.tab, plan.map.n_slots, order_out, rank_out}, plan.map.n_slots, w.partials});
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(slots_verdict_kernel, grid, block, 0, s, b, w.tab, plan.map, order_out, rank_out, overlap_told);
        return hipGetLastError();
    }
    default: break;
    }
    size_t tmp = 0;
    hipError_t e = sort_bytes(b.n_dst_ext, plan.bits.begin, plan.bits.end, &tmp);
    if (e != hipSuccess) return e;
    Pieces p(workspace);
    const SortWorkspace w(p, b.n_dst_ext, tmp);
    hipLaunchKernelGGL(declare_keys_kernel, dim3(grid_for(b.n_dst_ext)), block, 0, s, b, w.keys_in, w.vals_in);
    e = rocprim::radix_sort_pairs(w.tmp, tmp, w.keys_in, w.keys, w.vals_in, w.vals, b.n_dst_ext, plan.bits.begin, plan.bits.end, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sorted_verdict_kernel, grid, block, 0, s, b, check ? 1 : 0, w.keys, w.vals, order_out, rank_out, overlap_told);
    return hipGetLastError();
}

}  // namespace tent
