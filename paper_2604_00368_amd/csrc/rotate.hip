// Retry rotation (Section 4.3, "Link-Level Resilience") and failure marking of the rail simulator.
//
// A slice that failed on a rail is not bound by predicted cost again: slice i on its k-th retry
// takes candidate number (i + k) mod |candidates| of the rotation order the host derived from the
// rails' health, the retried slices are issued ahead of everything else in ascending slice index,
// and their bytes count in the queue statistics the cost model then starts from.  The rail of a
// retried slice is therefore a pure function of (i, k); what needs work is its staging offset, the
// bytes of the earlier retried slices on the same rail -- one prefix sum per rail over the retry
// list.  Three launches: per-chunk byte and slice counts per rail, an exclusive scan of those
// over the chunks (one lane per rail), and the in-order walk of every chunk by one wavefront; one for a small batch.
#include "finish.h"

namespace tent {
namespace {

__device__ __forceinline__ uint64_t lane_read64(uint64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t rotation_rail(const RotateParams& rot, uint32_t id, uint32_t retry)
{
    return rot.cand[((uint64_t)id + retry) % rot.n_cand];
}

// Step 1: bytes and slices per (chunk, rail).  Integer sums: the order of the atomics is immaterial.
__global__ void __launch_bounds__(64) rotate_count_kernel(BatchDev b, RotateParams rot)
{
    __shared__ unsigned long long bytes[TENT_MAX_RAILS];
    __shared__ uint32_t cnt[TENT_MAX_RAILS];
    const uint64_t n = b.plan->n_retry;
    const uint64_t begin = (uint64_t)blockIdx.x * kRotChunk;
    if (begin >= n) return;
    bytes[threadIdx.x] = 0;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t end = begin + kRotChunk < n ? begin + kRotChunk : n;
    for (uint64_t q = begin + threadIdx.x; q < end; q += 64) {
        const uint32_t id = b.retry_ids[q];
        const uint32_t d = rotation_rail(rot, id, b.s_retry[id]);
        atomicAdd(&bytes[d], (unsigned long long)b.s_len[id]);
        atomicAdd(&cnt[d], 1u);
    }
    __syncthreads();
    b.rot_bytes[(uint64_t)blockIdx.x * TENT_MAX_RAILS + threadIdx.x] = bytes[threadIdx.x];
    b.rot_cnt[(uint64_t)blockIdx.x * TENT_MAX_RAILS + threadIdx.x] = cnt[threadIdx.x];
}

// Step 2: lane d turns rail d's per-chunk byte counts into their exclusive prefix and publishes
// the totals of the rotation pass.
__global__ void __launch_bounds__(64) rotate_spine_kernel(BatchDev b)
{
    const uint64_t n = b.plan->n_retry;
    const uint64_t chunks = (n + kRotChunk - 1) / kRotChunk;
    uint64_t run = 0, slices = 0;
    constexpr int kAhead = 8;                                    // loads in flight per lane
    for (uint64_t c0 = 0; c0 < chunks; c0 += kAhead) {
        uint64_t bytes[kAhead];
        uint32_t count[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const uint64_t at = (c0 + k) * TENT_MAX_RAILS + threadIdx.x;
            bytes[k] = c0 + k < chunks ? b.rot_bytes[at] : 0;
            count[k] = c0 + k < chunks ? b.rot_cnt[at] : 0;
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (c0 + k < chunks) b.rot_bytes[(c0 + k) * TENT_MAX_RAILS + threadIdx.x] = run;
            run += bytes[k];
            slices += count[k];
        }
    }
    b.plan->Tr[threadIdx.x] = run;
    b.plan->cr[threadIdx.x] = slices;
}

// Step 3: one wavefront walks its chunk in order, 64 retried slices at a time.  Lane d keeps the
// running byte count of rail d; for every rail present among the 64 slices a wave-wide inclusive
// scan over the lengths of that rail's slices gives each its offset.
__device__ __forceinline__ void bind_retried(const BatchDev& b, const RotateParams& rot, uint64_t begin, uint64_t end, uint64_t my_base)
{
    const int lane = threadIdx.x & 63;
    for (uint64_t blk = begin; blk < end; blk += 64) {
        const uint64_t q = blk + lane;
        const bool valid = q < end;
        uint32_t id = 0, len = 0, d = 0;
        if (valid) {
            id = b.retry_ids[q];
            len = b.s_len[id];
            d = rotation_rail(rot, id, b.s_retry[id]);
        }
        uint64_t off = 0;
        uint64_t todo = __ballot(valid);
        while (todo) {                                           // one round per rail present in the block
            const int leader = __ffsll((long long)todo) - 1;
            const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)d, leader);
            const bool mine = valid && d == r;
            uint64_t incl = mine ? len : 0;
#pragma unroll
            for (int step = 1; step < 64; step <<= 1) {
                const uint64_t up = (uint64_t)__shfl_up((unsigned long long)incl, step, 64);
                if (lane >= step) incl += up;
            }
            const uint64_t base_r = lane_read64(my_base, (int)r);
            if (mine) off = base_r + incl - len;
            const uint64_t total = lane_read64(incl, 63);
            if (lane == (int)r) my_base += total;
            todo &= ~__ballot(mine);
        }
        if (valid) {
            b.s_rail[id] = d;
            b.s_stage_off[id] = off;
            b.s_state[id] = TENT_SLICE_BOUND;
        }
    }
}

__global__ void __launch_bounds__(64) rotate_emit_kernel(BatchDev b, RotateParams rot)
{
    const uint64_t n = b.plan->n_retry;
    const uint64_t begin = (uint64_t)blockIdx.x * kRotChunk;
    if (begin >= n) return;
    bind_retried(b, rot, begin, begin + kRotChunk < n ? begin + kRotChunk : n, b.rot_bytes[(uint64_t)blockIdx.x * TENT_MAX_RAILS + threadIdx.x]);
}

// The three steps in one launch, by one workgroup of a wavefront per chunk, for batches of up to kRotateSmall slices: there launches cost
// more than the work.  MI355X, lists, rotation and chain of 2,000 slices on 9 rails with what one of them had failed 60.6 -> 53.0 us, with
// all of it failed 41.6 -> 34.8, on 64 rails 106.3 -> 105.9; 20,000 slices in rounds of 4,096 would take 129.9 us for 133.0, but 141 for
// 64 where all have failed.
constexpr uint32_t kRotateWaves = 8;
constexpr uint64_t kRotateSmall = (uint64_t)kRotateWaves * kRotChunk;

__global__ void __launch_bounds__(64 * kRotateWaves) rotate_small_kernel(BatchDev b, RotateParams rot)
{
    __shared__ unsigned long long bytes[kRotateWaves][TENT_MAX_RAILS];
    __shared__ uint32_t cnt[kRotateWaves][TENT_MAX_RAILS];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint64_t n = b.plan->n_retry;                          // at most n_slices
    const uint64_t begin = (uint64_t)wave * kRotChunk, end = begin + kRotChunk < n ? begin + kRotChunk : n;
    bytes[wave][lane] = 0;
    cnt[wave][lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (uint64_t q = begin + lane; q < end; q += 64) {
        const uint32_t id = b.retry_ids[q];
        const uint32_t d = rotation_rail(rot, id, b.s_retry[id]);
        atomicAdd(&bytes[wave][d], (unsigned long long)b.s_len[id]);
        atomicAdd(&cnt[wave][d], 1u);
    }
    __syncthreads();
    uint64_t before = 0, all = 0, slices = 0;                    // lane = rail
    for (uint32_t w = 0; w < kRotateWaves; ++w) {
        if (w == wave) before = all;
        all += bytes[w][lane];
        slices += cnt[w][lane];
    }
    if (begin < n) bind_retried(b, rot, begin, end, before);
    if (wave != 0) return;
    b.plan->Tr[lane] = all;
    b.plan->cr[lane] = slices;
}

// Rail simulator: every BOUND slice on a failed rail returns to the pending set with one more retry.
__global__ void __launch_bounds__(256) fail_kernel(BatchDev b, FailParams fp, Report told)
{
    __shared__ uint32_t cnt[TENT_MAX_RAILS];
    if (threadIdx.x < TENT_MAX_RAILS) cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride) {
        if (b.s_state[i] != TENT_SLICE_BOUND) continue;
        const uint32_t d = b.s_rail[i];
        if (d >= TENT_MAX_RAILS || !fp.failed[d]) continue;
        b.s_state[i] = TENT_SLICE_PENDING;
        const uint8_t k = b.s_retry[i];
        if (k < 255) b.s_retry[i] = (uint8_t)(k + 1);
        atomicAdd(&cnt[d], 1u);
    }
    __syncthreads();
    unsigned long long added = 0;
    if (threadIdx.x < TENT_MAX_RAILS && cnt[threadIdx.x])
        added = atomicAdd((unsigned long long*)&b.plan->fail_cnt[threadIdx.x], (unsigned long long)cnt[threadIdx.x]);
    if (!finishes_last(b.plan, kTicketFail, added) || threadIdx.x >= TENT_MAX_RAILS) return;
    const unsigned long long total = take_counter(&b.plan->fail_cnt[threadIdx.x]);
    if (!told.to) return;
    tell(&told.to->fail_cnt[threadIdx.x], (uint64_t)total);
    if (threadIdx.x == 0) tell_done(told);
}

}  // namespace

hipError_t launch_rotate(const BatchDev& b, const RotateParams& rot, hipStream_t s)
{
    if (rot.n_cand == 0 || rot.n_cand > TENT_MAX_RAILS) return hipErrorInvalidValue;
    const uint64_t chunks = (b.n_slices + kRotChunk - 1) / kRotChunk;          // upper bound; idle chunks exit at once
    if (chunks == 0 || chunks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (b.n_slices <= kRotateSmall) {
        hipLaunchKernelGGL(rotate_small_kernel, dim3(1), dim3(64 * kRotateWaves), 0, s, b, rot);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(rotate_count_kernel, dim3((uint32_t)chunks), dim3(64), 0, s, b, rot);
    hipLaunchKernelGGL(rotate_spine_kernel, dim3(1), dim3(64), 0, s, b);
    hipLaunchKernelGGL(rotate_emit_kernel, dim3((uint32_t)chunks), dim3(64), 0, s, b, rot);
    return hipGetLastError();
}

hipError_t launch_fail(const BatchDev& b, const FailParams& fp, Report told, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(fail_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b, fp, told);
    return hipGetLastError();
}

}  // namespace tent
