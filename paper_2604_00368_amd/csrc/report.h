// Figures for the host.  A kernel stores them, and behind them the number of the call, straight to host memory; the host looks for
// the number (await_report in tent_api.hip).  Waiting for the stream costs a packet behind the kernel that releases the caches to
// the whole system, and a plan's figures are there before its last kernel has ended.  MI355X, waiting -> looking: the serving
// call of 64 short transfers, which asks twice, 119 -> 112 us; two requests' 82,000 pages, twice, 840 -> 829; sixteen telemetry
// windows, 35 times, 6260 -> 6070.  Figures are all that is there then: a poll that reports complete waits for the copies' release too.
#pragma once

#include "tent_internal.h"

namespace tent {

// The result block lies in coherent host memory, which a store of system scope reaches without any cache keeping it.
template <class T>
__device__ __forceinline__ void tell(T* where, T value)
{
    __hip_atomic_store(where, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// By one lane of the only wavefront that has told something: its stores have arrived before the number goes out.  (A release
// would say the same and write back the whole L2, whose contents the figures do not depend on.)
__device__ __forceinline__ void tell_done(Report told)
{
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    tell(&told.to->call, told.call);
}

}  // namespace tent
