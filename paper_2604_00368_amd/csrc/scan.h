// Device-wide exclusive prefix scan over 64-bit integers for gfx950.
//
// Two launches: (1) every workgroup reduces its tile, (2) every workgroup combines the results of the tiles
// before its own and scans its tile behind them.  One launch when everything fits one tile, three (the
// tile results scanned by one workgroup in between) from kSelfSpine tiles on, where reading them all in every
// workgroup would cost more than the launch.  Inside a workgroup each lane owns kScanItems consecutive elements; lane
// totals are combined with a 64-wide wavefront scan and the wavefront totals are carried through LDS.
// The operator is any associative, commutative integer operation with identity 0 (sum by default,
// maximum for "furthest end seen so far").  The result does not depend on scheduling (a fixed
// tree of integer operations), and no workgroup ever waits on another one.
//
// What bounds a scan here is the launches (4.6 us each on MI355X even when they do next to nothing), so scans that do not
// depend on each other are jobs of one call and share theirs, one row of workgroups per job.
#pragma once

#include "tent_internal.h"

namespace tent {

struct ScanSum { __device__ __forceinline__ uint64_t operator()(uint64_t a, uint64_t b) const { return a + b; } };
struct ScanMax { __device__ __forceinline__ uint64_t operator()(uint64_t a, uint64_t b) const { return a > b ? a : b; } };

template <class Op>
__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t v, Op op)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t up = __shfl_up((unsigned long long)v, d, 64);
        if (lane >= d) v = op(up, v);
    }
    return v;
}
__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t v) { return wave_inclusive_scan(v, ScanSum{}); }

// Exclusive scan of one value per lane across a workgroup of kScanBlock lanes.
// Returns the lane's exclusive prefix; *block_total receives the result over the workgroup.
template <class Op>
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t* block_total, Op op)
{
    constexpr int kWaves = kScanBlock / 64;
    __shared__ uint64_t wave_sum[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t inc = wave_inclusive_scan(v, op);
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    uint64_t carry = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        uint64_t s = wave_sum[w];
        if (w < wave) carry = op(carry, s);
        total = op(total, s);
    }
    __syncthreads();
    *block_total = total;
    const uint64_t before = __shfl_up((unsigned long long)inc, 1, 64);   // inclusive result of the lane below
    return lane == 0 ? carry : op(carry, before);
}

// Where a scan's results go: out(i, f(0) op ... op f(i - 1)) is called for every i in [0, n].
struct StoreTo {
    uint64_t* out;
    __device__ __forceinline__ void operator()(uint64_t i, uint64_t v) const { out[i] = v; }
};

// One scan of n > 0 values f(0) .. f(n - 1); partials needs scan_partials_capacity(n) entries.
template <class F, class Op, class Out>
struct ScanJob {
    F f;
    Op op;
    Out out;
    uint64_t n;
    uint64_t* partials;
};
template <class F, class Op = ScanSum>
ScanJob<F, Op, StoreTo> scan_job(F f, uint64_t n, uint64_t* out, uint64_t* partials, Op op = Op{})
{
    return {f, op, StoreTo{out}, n, partials};
}

constexpr uint64_t kSelfSpine = 2048;

inline uint64_t scan_tiles(uint64_t n) { return (n + kScanTile - 1) / kScanTile; }

// (everything below has internal linkage: the same instantiation may exist in several translation units, each
// with its own code object)
// A lane's items, 0 behind the last one.  Without a branch around f its loads are all in flight at once; a scan of 128 transfers,
// whose f loads twice, was eight such pairs one after the other (MI355X: 9.3 -> 6.7 us).
template <class J>
static __device__ __forceinline__ void read_items(const J& job, uint64_t base, uint64_t (&v)[kScanItems])
{
#pragma unroll
    for (int k = 0; k < (int)kScanItems; ++k) {
        const uint64_t i = base + k;
        const uint64_t x = job.f(i < job.n ? i : job.n - 1);
        v[k] = i < job.n ? x : 0;
    }
}

template <class J>
static __device__ __forceinline__ void scan_reduce_job(const J& job)
{
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    if ((uint64_t)blockIdx.x * kScanTile >= job.n) return;
    uint64_t v[kScanItems], sum = 0;
    read_items(job, base, v);
#pragma unroll
    for (int k = 0; k < (int)kScanItems; ++k) sum = job.op(sum, v[k]);
    uint64_t total;
    block_exclusive_scan(sum, &total, job.op);
    if (threadIdx.x == 0) job.partials[blockIdx.x] = total;
}

// One workgroup: partials[0..nb) -> exclusive prefix in place.
template <class J>
static __device__ __forceinline__ void scan_spine_job(const J& job)
{
    const uint64_t nb = (job.n + kScanTile - 1) / kScanTile;
    uint64_t carry = 0;
    for (uint64_t lo = 0; lo < nb; lo += kScanBlock) {
        const uint64_t i = lo + threadIdx.x;
        const uint64_t v = i < nb ? job.partials[i] : 0;
        uint64_t total;
        const uint64_t ex = block_exclusive_scan(v, &total, job.op);
        if (i < nb) job.partials[i] = job.op(carry, ex);
        carry = job.op(carry, total);
    }
}

template <class J>
static __device__ __forceinline__ void scan_down_job(const J& job, bool spined)
{
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    if ((uint64_t)blockIdx.x * kScanTile >= job.n) return;
    uint64_t before = 0;                                     // what the tiles before this one hold
    if (spined) {
        before = job.partials[blockIdx.x];
    } else if (blockIdx.x != 0) {
        uint64_t mine = 0;
        for (uint64_t t = threadIdx.x; t < blockIdx.x; t += kScanBlock) mine = job.op(mine, job.partials[t]);
        block_exclusive_scan(mine, &before, job.op);
    }
    uint64_t v[kScanItems], sum = 0;
    read_items(job, base, v);
#pragma unroll
    for (int k = 0; k < (int)kScanItems; ++k) sum = job.op(sum, v[k]);
    uint64_t total;
    uint64_t run = job.op(before, block_exclusive_scan(sum, &total, job.op));
#pragma unroll
    for (int k = 0; k < (int)kScanItems; ++k) {
        if (base + k <= job.n) job.out(base + k, run);       // entry n: the grand total, by the lane that reaches it
        run = job.op(run, v[k]);
    }
    if (base + kScanItems == job.n) job.out(job.n, run);
}

// workgroup row y takes job y
template <class... J>
static __global__ void __launch_bounds__(kScanBlock) scan_reduce_kernel(J... jobs)
{
    uint32_t y = 0;
    ((blockIdx.y == y++ ? scan_reduce_job(jobs) : void()), ...);
}
template <class... J>
static __global__ void __launch_bounds__(kScanBlock) scan_spine_kernel(J... jobs)
{
    uint32_t y = 0;
    ((blockIdx.y == y++ ? scan_spine_job(jobs) : void()), ...);
}
template <class... J>
static __global__ void __launch_bounds__(kScanBlock) scan_down_kernel(bool spined, J... jobs)
{
    uint32_t y = 0;
    ((blockIdx.y == y++ ? scan_down_job(jobs, spined) : void()), ...);
}

template <class... J>
hipError_t run_scans(hipStream_t s, J... jobs)
{
    uint64_t n = 0;
    for (uint64_t each : {jobs.n...}) {
        if (each == 0) return hipErrorInvalidValue;
        n = each > n ? each : n;
    }
    const uint64_t nb = scan_tiles(n);
    if (nb > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)nb, (uint32_t)sizeof...(J)), block(kScanBlock);
    const bool spined = nb > kSelfSpine;
    if (nb > 1) hipLaunchKernelGGL((scan_reduce_kernel<J...>), grid, block, 0, s, jobs...);
    if (spined) hipLaunchKernelGGL((scan_spine_kernel<J...>), dim3(1, grid.y), block, 0, s, jobs...);
    hipLaunchKernelGGL((scan_down_kernel<J...>), grid, block, 0, s, spined, jobs...);
    return hipGetLastError();
}

// out[i] = op over f(0..i-1) for i in [0, n] (out has n + 1 entries).
template <class F, class Op = ScanSum>
hipError_t exclusive_scan(F f, uint64_t n, uint64_t* out, uint64_t* partials, hipStream_t s, Op op = Op{})
{
    return run_scans(s, scan_job(f, n, out, partials, op));
}

}  // namespace tent
