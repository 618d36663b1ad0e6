// The slice table, one row at a time (slice decomposition of Section 4.2): shared by the kernels that build it for batches
// of any size and the workgroup that plans a small batch alone.
#pragma once

#include "tile_tables.h"

namespace tent {

// Division by the slice size.  Below 2^53 (a plan refuses a payload from there on) the double quotient is off by at most one, which
// the remainder shows; a 64-bit division takes about six times the instructions.
struct SliceDiv {
    uint64_t S;
    double inv;
    __host__ __device__ explicit SliceDiv(uint64_t slice_bytes) : S(slice_bytes), inv(1.0 / (double)slice_bytes) {}
    // slices of a transfer of len > 0 bytes, and the length of the last one
    __device__ __forceinline__ uint64_t slices(uint64_t len, uint64_t* last) const
    {
        uint64_t q = (uint64_t)((double)len * inv);
        int64_t rest = (int64_t)(len - q * S);
        if (rest > (int64_t)S) { ++q; rest -= (int64_t)S; }
        if (rest <= 0) { --q; rest += (int64_t)S; }
        if (rest <= 0) { --q; rest += (int64_t)S; }
        *last = (uint64_t)rest;
        return q + 1;
    }
};

// A transfer of len bytes has ceil(len / S) slices, all of S bytes but the last.  Maximal runs of equal-length
// slices (bind_runs.hip) therefore start in at most two places per transfer: at its first slice, unless that is as long as the
// slice before it, and at its last one, if that is short and not also the first.
struct TransferShape {
    uint64_t slices, last;         // slices; length of the last one
    bool new_run, short_tail;      // runs that start at the first slice, at the last one
    template <class Pre>
    __device__ __forceinline__ TransferShape(const uint32_t* ptr, const Pre& pre, const SliceDiv& div, uint64_t j)
    {
        const uint64_t at = pre[ptr[j]], len = pre[ptr[j + 1]] - at, before = pre[ptr[j > 0 ? j - 1 : 0]];
        slices = div.slices(len, &last);
        short_tail = slices > 1 && last != div.S;
        uint64_t last_before;
        div.slices(j > 0 ? at - before : 1, &last_before);
        new_run = j == 0 || last_before != (len < div.S ? len : div.S);
    }
};
struct TransferCounts {
    const uint32_t* ptr;
    const uint64_t* pre;
    SliceDiv div;
    __device__ __forceinline__ uint64_t operator()(uint64_t j) const
    {
        const TransferShape t(ptr, pre, div, j);
        return ((uint64_t)((t.new_run ? 1u : 0u) + (t.short_tail ? 1u : 0u)) << 32) | t.slices;
    }
};

// The extents in [lo, hi) of either side that hold byte `off` of a transfer of `len` bytes.  Both sides are looked up side by side,
// first where the byte would lie if all extents were as long as their mean: pages are, and the search ends there.
template <class Pre>
__device__ __forceinline__ void extents_at(const Pre& src_pre, uint32_t slo, uint32_t shi, const Pre& dst_pre, uint32_t dlo, uint32_t dhi,
                                           uint64_t off, uint64_t len, uint32_t* src_e, uint32_t* dst_e)
{
    const uint64_t src_key = src_pre[slo] + off, dst_key = dst_pre[dlo] + off;
    const double share = (double)off / (double)len;
    auto guess = [&](uint32_t lo, uint32_t hi) {
        const uint32_t e = lo + (uint32_t)(share * (double)(hi - lo) + 1.0 / 1024.0);
        return e < hi ? e : hi - 1;
    };
    const uint32_t gs = guess(slo, shi), gd = guess(dlo, dhi);
    const uint64_t s0 = src_pre[gs], s1 = src_pre[gs + 1], d0 = dst_pre[gd], d1 = dst_pre[gd + 1];
    auto narrow = [](uint32_t& lo, uint32_t& hi, uint32_t g, uint64_t g0, uint64_t g1, uint64_t key) {
        if (key < g0) hi = g;
        else if (key >= g1) lo = g + 1;
        else { lo = g; hi = g + 1; }
    };
    narrow(slo, shi, gs, s0, s1, src_key);
    narrow(dlo, dhi, gd, d0, d1, dst_key);
    while (shi - slo > 1 || dhi - dlo > 1) {
        const uint32_t ms = slo + ((shi - slo) >> 1), md = dlo + ((dhi - dlo) >> 1);
        const uint64_t vs = src_pre[ms], vd = dst_pre[md];
        if (vs <= src_key) slo = ms; else shi = ms;
        if (vd <= dst_key) dlo = md; else dhi = md;
    }
    *src_e = slo;
    *dst_e = dlo;
}

// Row i of the slice table, a slice of transfer j whose first slice is `first` and before which `runs_before` runs start;
// a slice that starts a run enters it in the run table.  The extent prefixes may lie in LDS.
template <class Pre>
__device__ __forceinline__ void write_slice(const BatchDev& b, const SliceDiv& div, uint64_t i, uint32_t j, uint64_t first,
                                            uint32_t runs_before, const Pre& src_pre, const Pre& dst_pre)
{
    const uint32_t slo = b.src_ptr[j], shi = b.src_ptr[j + 1];
    const uint32_t dlo = b.dst_ptr[j], dhi = b.dst_ptr[j + 1];
    const TransferShape t(b.src_ptr, src_pre, div, j);
    const uint64_t at = src_pre[slo], len_j = src_pre[shi] - at;
    const uint64_t off = (i - first) * b.slice_bytes;
    const uint64_t rest = len_j - off;
    uint32_t src_e, dst_e;
    extents_at(src_pre, slo, shi, dst_pre, dlo, dhi, off, len_j, &src_e, &dst_e);
    b.s_desc[i] = j;
    b.s_off[i] = off;
    b.s_pos[i] = at + off;
    b.s_len[i] = (uint32_t)(rest < b.slice_bytes ? rest : b.slice_bytes);
    b.s_src_e0[i] = src_e;
    b.s_dst_e0[i] = dst_e;
    b.s_rail[i] = 0xFFFFFFFFu;
    b.s_stage_off[i] = 0;
    b.s_state[i] = TENT_SLICE_PENDING;
    // the run table: every run is entered by the slice it starts at
    const uint32_t run = runs_before + (t.new_run ? 1u : 0u) - 1u;      // of the transfer's first slice
    const bool tail = t.short_tail && rest <= b.slice_bytes;
    b.s_run[i] = run + (tail ? 1u : 0u);
    if ((off == 0 && t.new_run) || tail) b.run_start[run + (tail ? 1u : 0u)] = (uint32_t)i;
}

}  // namespace tent
