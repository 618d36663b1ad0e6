// The slice table, one row at a time (slice decomposition of Section 4.2): shared by the kernels that build it for batches
// of any size and the workgroup that plans a small batch alone.
#pragma once

#include "tile_tables.h"

namespace tent {

// A transfer of len bytes has ceil(len / S) slices, all of S bytes but the last.  Maximal runs of equal-length
// slices (bind_runs.hip) therefore start in at most two places per transfer: at its first slice, unless that is as long as the
// slice before it, and at its last one, if that is short and not also the first.
struct TransferShape {
    uint64_t slices, last;         // slices; length of the last one
    bool new_run, short_tail;      // runs that start at the first slice, at the last one
    __device__ TransferShape(const uint32_t* ptr, const uint64_t* pre, uint64_t S, uint64_t j)
    {
        const uint64_t at = pre[ptr[j]], len = pre[ptr[j + 1]] - at;
        slices = (len + S - 1) / S;
        last = len - (slices - 1) * S;
        short_tail = slices > 1 && last != S;
        new_run = true;
        if (j > 0) {
            const uint64_t len_before = at - pre[ptr[j - 1]];
            const uint64_t last_before = len_before - ((len_before + S - 1) / S - 1) * S;
            new_run = last_before != (len < S ? len : S);
        }
    }
};
struct TransferCounts {
    const uint32_t* ptr;
    const uint64_t* pre;
    uint64_t S;
    __device__ uint64_t operator()(uint64_t j) const
    {
        const TransferShape t(ptr, pre, S, j);
        return ((uint64_t)((t.new_run ? 1u : 0u) + (t.short_tail ? 1u : 0u)) << 32) | t.slices;
    }
};

// Row i of the slice table, a slice of transfer j whose first slice is `first` and before which `runs_before` runs start;
// a slice that starts a run enters it in the run table.  The extent prefixes may lie in LDS.
template <class Pre>
__device__ __forceinline__ void write_slice(const BatchDev& b, uint64_t i, uint32_t j, uint64_t first, uint32_t runs_before,
                                            const Pre& src_pre, const Pre& dst_pre)
{
    const uint32_t slo = b.src_ptr[j], shi = b.src_ptr[j + 1];
    const uint32_t dlo = b.dst_ptr[j], dhi = b.dst_ptr[j + 1];
    const uint64_t len_j = src_pre[shi] - src_pre[slo];
    const uint64_t off = (i - first) * b.slice_bytes;
    const uint64_t rest = len_j - off;
    b.s_desc[i] = j;
    b.s_off[i] = off;
    b.s_pos[i] = src_pre[slo] + off;
    b.s_len[i] = (uint32_t)(rest < b.slice_bytes ? rest : b.slice_bytes);
    b.s_src_e0[i] = (uint32_t)last_not_above(src_pre, slo, shi, src_pre[slo] + off);
    b.s_dst_e0[i] = (uint32_t)last_not_above(dst_pre, dlo, dhi, dst_pre[dlo] + off);
    b.s_rail[i] = 0xFFFFFFFFu;
    b.s_stage_off[i] = 0;
    b.s_state[i] = TENT_SLICE_PENDING;
    // the run table: every run is entered by the slice it starts at
    const TransferShape t(b.src_ptr, src_pre, b.slice_bytes, j);
    const uint32_t run = runs_before + (t.new_run ? 1u : 0u) - 1u;      // of the transfer's first slice
    const bool tail = t.short_tail && rest <= b.slice_bytes;
    b.s_run[i] = run + (tail ? 1u : 0u);
    if ((off == 0 && t.new_run) || tail) b.run_start[run + (tail ? 1u : 0u)] = (uint32_t)i;
}

}  // namespace tent
