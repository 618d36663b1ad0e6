// Counting kernels that end in one launch: every workgroup adds its share to counters in device memory, the last one
// to finish reads the sums, hands them on and leaves the counters at zero for the next launch.  Against a launch
// that clears the counters, the count, and a copy of the result block to the host this saves two launches (about 5 us each on
// MI355X, 10 us with the copy engine's share); no workgroup waits on another.
#pragma once

#include "report.h"

namespace tent {

enum : int { kTicketRetire = 0, kTicketRemaining = 1, kTicketFail = 2, kTicketProbe = 3 };

// True in every thread of the workgroup that finishes last (and has then seen what all others added).  `added` is what this
// thread's own atomic add or maximum returned (0 if it made none): once the old value is back the addition has
// happened where every workgroup's atomics happen, which is all the order the counters need -- a device-wide fence would
// write the caches back and cost 6 us more.  It orders nothing else: what other workgroups have written with plain stores
// must not be read behind it, and the counters only with atomics (take_counter).
__device__ __forceinline__ bool finishes_last(PlanState* plan, int kind, unsigned long long added)
{
    __shared__ uint32_t is_last;
    asm volatile("" : : "v"((uint32_t)added), "v"((uint32_t)(added >> 32)) : "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        is_last = atomicAdd(&plan->ticket[kind], 1u) == gridDim.x - 1 ? 1u : 0u;
        if (is_last) atomicExch(&plan->ticket[kind], 0u);
    }
    __syncthreads();
    return is_last != 0;
}

// A counter other workgroups have added to, read where its atomics happen and set back to zero.
__device__ __forceinline__ unsigned long long take_counter(uint64_t* p)
{
    return atomicExch((unsigned long long*)p, 0ull);
}

}  // namespace tent
