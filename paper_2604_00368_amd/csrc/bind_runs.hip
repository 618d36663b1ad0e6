// Run-parallel rail assignment.  Produces exactly the binding of the slice-by-slice rule
// (Algorithm 1 Stage 2 of the paper with per-slice earliest completion, Section 4.2; ties to the
// lowest rail; in-flight bytes A_d grow with every bound slice), but only the chain over *runs* of
// equal-length slices is sequential.
//
// Why this is exact.  Inside a run of m slices of equal length l, rail d's successive candidate costs
//     f_d(k) = c0_d + (((A_d + (k+1) l) c1_d) >> 16),   k = 0, 1, ...
// are nondecreasing in k, so picking the cheapest rail m times is a merge of R sorted sequences: the
// run takes the m smallest triples (f_d(k), d, k) in lexicographic order, and the slice at position
// p of the run gets the triple of rank p.  Three steps follow from that:
//   1. run table     maximal runs of equal-length pending slices: on a first plan written with the slice table, on a
//                    re-plan with the list of pending slices (split.hip);
//   2. chain         one wavefront, lane = rail, walks the runs in order and finds, per run, how many
//                    slots k_d each rail takes.  A second wavefront, the feeder, goes ahead of it and hands it one record
//                    per run with everything that does not depend on the rails' state, among it the cost level at
//                    which the run will end according to a floating-point water-filling model.  The split is found
//                    from that level (slots at or below it, per rail) and repaired one slot at a time (add the
//                    cheapest free slot / drop the dearest taken slot) until exactly m slots are taken; where
//                    the level does not serve, count_d(v) = #{k : f_d(k) <= v} (closed form, two integer
//                    divisions) is evaluated at bracketed levels instead.  The level only steers the guess; the
//                    counts and repairs are exact.  Runs of one slice (tails) are a plain argmin.  With up to 16
//                    rails all slots a guess lacks are added at once, by rank, and a third wavefront, the drainer, turns
//                    what the chain finds into the rows of the run table (bind_chain16).
//   3. emit          one lane per slot (d, k): its rank in the run is
//                    k + sum_{d' < d} count_d'(f) + sum_{d' > d} count_d'(f - 1),  f = f_d(k),
//                    which gives the slice it belongs to; staging offset = T_d at run start + k l.
#include <type_traits>

#include "scan.h"
#include "slices.h"
#include "wave.h"

namespace tent {

namespace {

constexpr int kTol = 4;                    // repair at most this many slots one by one
constexpr uint64_t kCostCap = 1ull << 47;  // every feasible (X * c1) >> 16 is below this (host precondition)

// floor(a / b) for 1 <= b < 2^32 with inv = 1.0 / b.  The floating-point quotient is only an
// estimate; the remainder check makes the result exact for every a.
__device__ __forceinline__ uint64_t div_exact(uint64_t a, uint32_t b, double inv)
{
    if (a >> 50) return a / b;
    uint64_t q = (uint64_t)((double)a * inv);
    int64_t r = (int64_t)(a - q * b);
#pragma clang loop unroll(disable)
    while (r < 0) { --q; r += b; }
#pragma clang loop unroll(disable)
    while (r >= (int64_t)b) { ++q; r -= b; }
    return q;
}

// Per-rail constants of one plan.
struct Rail {
    uint64_t c0;
    uint32_t c1;        // >= 1
    double inv_c1;
};

// Cost of the rail's slot k (0-based) of a run of l-byte slices when A bytes are already queued.
// k + 1 <= 2^32 - 1 because a batch holds fewer than 2^32 - 1 slices.
__device__ __forceinline__ uint64_t slot_cost(const Rail& r, uint64_t A, uint32_t l, uint32_t k)
{
    const uint64_t x = A + (uint64_t)(k + 1u) * l;
    return r.c0 + ((x * (uint64_t)r.c1) >> 16);
}

// #{k >= 0 : slot_cost(k) <= v}, clamped to m.  v may be negative.
__device__ __forceinline__ uint32_t slots_upto(const Rail& r, uint64_t A, uint32_t l, double inv_l, int64_t v, uint32_t m)
{
    if (v < 0 || (uint64_t)v < r.c0) return 0;
    uint64_t w1 = (uint64_t)v - r.c0 + 1;
    if (w1 > kCostCap) w1 = kCostCap;
    // largest X with (X * c1) >> 16 <= w1 - 1, i.e. floor((w1 * 65536 - 1) / c1), without overflow
    const uint64_t q1 = div_exact(w1, r.c1, r.inv_c1);
    const uint64_t r1 = w1 - q1 * r.c1;
    const uint64_t xmax = r1 == 0 ? (q1 << 16) - 1 : (q1 << 16) + div_exact((r1 << 16) - 1, r.c1, r.inv_c1);
    if (xmax < A + l) return 0;
    uint64_t room = xmax - A;
    const uint64_t want = (uint64_t)m * l;
    if (room > want) room = want;
    const uint64_t k = div_exact(room, l, inv_l);
    return (uint32_t)(k < m ? k : m);
}

// ---- step 2: chain over runs: exact slot counts -----------------------------------------------
// Same value as slots_upto, reached from a floating-point estimate that is then checked against
// the integer cost of the neighbouring slots; falls back to the closed form when the estimate
// cannot be trusted to be within a few slots.
__device__ __forceinline__ uint32_t slots_upto_fast(const Rail& r, uint64_t A, uint32_t l, double inv_l, int64_t v, uint32_t m)
{
    if (v < 0 || (uint64_t)v < r.c0) return 0;
    const uint64_t w1 = (uint64_t)v - r.c0 + 1;
    if ((w1 >> 36) || (A >> 52)) return slots_upto(r, A, l, inv_l, v, m);
    const double x = (double)(w1 << 16) * r.inv_c1;            // bytes the rail may hold at cost v
    double kf = (x - (double)A) * inv_l;
    kf = kf < 0.0 ? 0.0 : (kf > (double)m ? (double)m : kf);
    uint32_t k = (uint32_t)kf;
    // the estimate is almost always exact: two cost evaluations confirm it
    const bool low = k < m && slot_cost(r, A, l, k) <= (uint64_t)v;
    const bool high = k > 0 && slot_cost(r, A, l, k - 1) > (uint64_t)v;
    if (low) {
        ++k;
#pragma clang loop unroll(disable)
        while (k < m && slot_cost(r, A, l, k) <= (uint64_t)v) ++k;
    } else if (high) {
        --k;
#pragma clang loop unroll(disable)
        while (k > 0 && slot_cost(r, A, l, k - 1) > (uint64_t)v) --k;
    }
    return k;
}

// ---- the feeder: one record per run ------------------------------------------------------------
// Cost level at which a run ends, from the water-filling model: the rails that take part end a run at a common cost
// level, level(bytes) = (bytes + sum_d h_d G_d) / sum_d G_d over those rails, with G_d = 65536 / c1_d bytes per picosecond and
// h_d the rail's head cost; a rail takes part once the level has passed its head cost.  The bytes bound
// before a run are known in advance (a prefix sum of the pending lengths), so the level after every run is too.
struct LevelModel {
    // admitted rails in ascending order of their head cost h_d = c0_d + A_d c1_d / 65536 (what the rail's next byte
    // would cost): h[j] the j-th smallest, G[j] and hG[j] the sums of G_d and of h_d G_d over the first j + 1, inv_G[j] = 1 / G[j]
    double h[TENT_MAX_RAILS], G[TENT_MAX_RAILS], hG[TENT_MAX_RAILS], inv_G[TENT_MAX_RAILS];
    uint32_t live;
    double max_c1, min_c1;
    double short_by;               // slots by which the first guess of a run's split is meant to fall short
};

__device__ __forceinline__ double from_lane(double x, int at) { return __shfl(x, at, 64); }
__device__ __forceinline__ double uniform_from(double x, int at)       // `at` the same in all lanes
{
    return __longlong_as_double((long long)read_lane64((uint64_t)__double_as_longlong(x), at));
}

// By a whole workgroup (at least 64 threads), with barriers; the first wavefront does the work, lane = rail.
template <int kWide>
__device__ __forceinline__ void build_level_model(LevelModel& lm, const BatchDev& b, const RailParams& rp, int mode)
{
    const uint32_t t = threadIdx.x;
    if (t < 64) {
        const uint64_t live_mask = rp.n_rails < 64 ? rp.admitted & ((1ull << rp.n_rails) - 1) : rp.admitted;
        const bool live = (live_mask >> t) & 1;
        const uint32_t n_live = (uint32_t)__popcll(live_mask);
        const double c1 = live ? (double)(uint32_t)rp.c1[t] : 1.0;                 // c1 >= 1 on this path
        const double G = 65536.0 / c1;
        const uint64_t A = rp.A[t] + ((mode & kBindAfterRotation) ? b.plan->Tr[t] : 0);
        const double h = (double)rp.c0[t] + (double)A * c1 * (1.0 / 65536.0);
        uint32_t rank = 0;
        double max_c1 = 0.0, min_c1 = 4294967296.0, sum_G = 0.0;
        for (uint32_t d = 0; d < rp.n_rails; ++d) {
            if (!((live_mask >> d) & 1)) continue;
            const double hd = uniform_from(h, (int)d), c1_d = uniform_from(c1, (int)d);
            max_c1 = c1_d > max_c1 ? c1_d : max_c1;
            min_c1 = c1_d < min_c1 ? c1_d : min_c1;
            sum_G += uniform_from(G, (int)d);
            rank += (hd < h || (hd == h && d < t)) ? 1u : 0u;
        }
        if (live) { lm.h[rank] = h; lm.G[rank] = G; lm.hG[rank] = h * G; }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        double g = t < n_live ? lm.G[t] : 0.0, hg = t < n_live ? lm.hG[t] : 0.0;
        for (int step = 1; step < (int)n_live; step <<= 1) {
            const double g_up = __shfl_up(g, step, 64), hg_up = __shfl_up(hg, step, 64);
            if ((int)t >= step) { g += g_up; hg += hg_up; }
        }
        if (t < n_live) { lm.G[t] = g; lm.hG[t] = hg; lm.inv_G[t] = 1.0 / g; }
        if (t == 0) {
            lm.live = n_live;
            lm.max_c1 = max_c1;
            lm.min_c1 = min_c1;
            // What rounding takes off the slot counts is a sum of n_live fractions, n_live / 2 with a deviation of
            // sqrt(n_live / 12).  Three deviations leave next to no guess too high; half the slots that all rails take while the
            // fastest takes one, if that is less, so that seldom a rail is short of two.  Of 24,000 runs of 8 - 72 slices (counted with
            // this arithmetic redone on the CPU) 0.03 % are too high and none short of two on 16 rails in two speeds, 0.05 % each
            // on 8 rails of 12.5 - 100 GB/s, 6 % each on 8 equal rails and one of eight times their speed.
            const double spread = sqrt(0.75 * (double)n_live), room = 0.5 * sum_G * min_c1 * (1.0 / 65536.0);
            lm.short_by = kWide > 16 ? 0.0 : spread < room ? spread : room;
        }
    }
    __syncthreads();
}

// Half a slice per participating rail comes on top of the bytes, because the slot counts are rounded down, less what the
// guess is meant to fall short by.  Nearly always all rails take part.
__device__ __forceinline__ double level_at(const LevelModel& lm, double bytes, double half_slice)
{
    const uint32_t last = lm.live - 1;
    bytes -= 2.0 * half_slice * lm.short_by;
    double v = (bytes + half_slice * (double)lm.live + lm.hG[last]) * lm.inv_G[last];
    if (!(v > lm.h[last]))
        for (uint32_t j = 0; j < last; ++j) {
            v = (bytes + half_slice * (double)(j + 1) + lm.hG[j]) * lm.inv_G[j];
            if (v <= lm.h[j + 1]) break;
        }
    return v;
}

// What a record holds: the slices m of the run (0: a single slice that does not stand behind a longer run, with no run
// before it), the shift from the level of the record before to this one's, the level, the slice length l and 1 / l, the length
// of the single slice behind the run, the run's index, and flags:
typedef uint32_t Quad __attribute__((ext_vector_type(4)));
constexpr uint32_t kRecTail = 1u;          // a single slice follows the run and is bound with it
constexpr uint32_t kRecSingle = 2u;        // there is no run, only a single slice
constexpr uint32_t kRecNoLevel = 4u;       // the level does not serve: general path
constexpr uint32_t kRecRebase = 8u;        // the chain takes its relative state afresh from the integers first
constexpr uint32_t kRecSame = 16u;         // the run's slices are as long as those of the run before
constexpr uint32_t kRecEnd = 32u;          // behind the last run
constexpr uint32_t kRecShort = kRecTail | kRecSame;   // what nearly every record of a long batch is: the short path
// up to 16 rails: how the chain may take the record, and how many from it on it may take in the same way
constexpr uint32_t kTakeOdd = 0u, kTakeSame = 1u, kTakeRun = 2u, kTakeSingle = 3u;
constexpr uint32_t kRecTake = 6, kRecCount = 8;        // first bits of the two
constexpr uint32_t kFeedBlock = 64;        // runs the feeder looks at a time, one per lane
constexpr uint32_t kRingRecords = 256;     // ring of more than 16 rails, in records
constexpr uint32_t kRingBlocks = 3;        // ring of up to 16 rails, in blocks of kFeedBlock records: one fed, one walked, one drained
                                           // (4,096 transfers 553 us; with two 551, with four 543 and 8 KB more of LDS)

// The chain keeps costs relative to the level in units of 2^-16 ps, as doubles that hold whole numbers below 2^53
// exactly.  A rail 2^kFarBits ps or more above the level counts as infinitely far until the state is rebased, which
// happens at least once while the level rises by 2^kStepBits ps; a run that lifts the level by more than that, or whose single
// slot costs more, goes the general way.
constexpr int kFarBits = 36, kStepBits = 34;
constexpr double kMaxLevel = 4.0e15;       // ps; levels are whole numbers, exact as doubles
constexpr uint32_t kLevelRunMax = 1u << 25;   // slices: slot counts of up to 64 rails are summed in 32 bits
constexpr double kUnit = 65536.0;

// The same for up to 16 rails, whose chain keeps them in units of 2^-4 ps (whole multiples of 2^-12) above a floor that lies kBias
// below the level, so that a 32-bit key (whole ps << 4 | rail) is one conversion away: keys cover 134 us on either side of the
// level.  The short path takes runs whose slice costs at most kMaxStep on the slowest and the fastest rail together, which is what
// keeps every key it looks at inside that window, and whose level and record before lie less than kMaxShift apart.
constexpr double kBias = 2147483648.0;         // 2^31; a slot costs no more than the level iff it ends below kBias + 16
constexpr double kFineUnit = 4096.0;           // units of 2^-16 ps in one of these
constexpr double kGuessAt = kBias + 16.0 - 1.0 / 8192.0;   // half a unit below that bound
constexpr double kDownFrom = 2.0 * kBias + 32.0 - 1.0 / kFineUnit;   // less where a taken slot ends: kBias + (1 - floor(ps)) * 16 and a rest
constexpr double kMaxStep = 2147483584.0;      // 2^31 - 64
constexpr double kMaxShift = 68719476736.0;    // 2^36
constexpr double kMaxSlots = 67108864.0;       // 2^26: slots a level may lie above a rail's head; 16 rails' sums stay below 2^32
constexpr uint32_t kFarKey16 = 0xFFFFFFF0u;
constexpr uint32_t kLastBlock = 0x80000000u, kSteepBlock = 0x40000000u;
constexpr uint32_t kStepped = ~0u;         // StepRing::Record::single of a record that stepped
constexpr uint32_t kWalkLast = 24;         // records of the last block the chain takes between two reports to the drainer
constexpr uint32_t kBitsOfSlots = 28;      // of a word in found
// A record whose guess does not hold costs a stretch of walk_same about what kMissWorth of its records save against walk_runs: where
// more of them miss, kMissFew at least, the rest of the block goes through walk_runs.  MI355X, chain and emit: 448 records of
// which a third miss 257 us without this and 171 with it (at two misses 158, at three 165), 1,792 of which 6 % miss 403 and 380 (372,
// 376), 512 of which 6 % miss 133 either way.
constexpr uint32_t kMissFew = 4, kMissWorth = 8;

constexpr uint32_t kLeastStretch = 6;       // records of equal slice lengths that go by ranks

struct RecordRing {                        // more than 16 rails
    // {m, flags, shift} {length of the single slice as a double, run} {level, l, that length} {1 / l}
    Quad rec[kRingRecords][4];
    uint32_t filled;                       // records written
    uint32_t taken;                        // records read
};

// Up to 16 rails: records in blocks that start at multiples of kFeedBlock, and what the chain finds for each of them.
struct StepRing {
    struct Record {
        Quad step;                         // {shift, length of the single slice less the run's l as a signed word, m}
        Quad run;                          // {1 / l, l, near_key (see bind_chain16)}
        Quad level;                        // {level, length of the single slice or 0, index of the run}
        uint32_t flags;
        uint32_t single;                   // key of the single slice (low four bits: its rail); kStepped: stands in found
        uint32_t pad[2];
    };
    Record rec[kRingBlocks * kFeedBlock + 8];          // (the chain reads up to eight records ahead)
    // per rail the slots of the run; a record that steps has fewer than 2^28, and the single slice's rail in the bits above
    uint32_t found[kRingBlocks * kFeedBlock][16];
    uint32_t count[kRingBlocks];           // records in the block; kLastBlock marks the last one
    uint32_t filled;                       // blocks written by the feeder
    uint32_t walked;                       // records the chain is through with, as block * kFeedBlock + record
    uint32_t drained;                      // blocks whose rows have been written
};

__device__ __forceinline__ double join_f64(uint32_t lo, uint32_t hi) { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); }
__device__ __forceinline__ uint32_t low_f64(double x) { return (uint32_t)(uint64_t)__double_as_longlong(x); }
__device__ __forceinline__ uint32_t high_f64(double x) { return (uint32_t)((uint64_t)__double_as_longlong(x) >> 32); }

// v_cvt_u32_f64: truncates; values below zero, minus infinity and not-a-number give 0, above 2^32 - 1 saturate.
__device__ __forceinline__ uint32_t saturating_u32(double x)
{
    uint32_t r;
    asm("v_cvt_u32_f64_e32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// The same with the low four bits replaced by the rail.
__device__ __forceinline__ uint32_t tagged_key(double x, uint32_t who)
{
    uint32_t r;
    asm("v_cvt_u32_f64_e32 %0, %1\n\tv_and_or_b32 %0, %0, -16, %2" : "=&v"(r) : "v"(x), "v"(who));
    return r;
}

// The records of `written` around the lane's own that are `alike`, up to the next ones that are not.
__device__ __forceinline__ uint64_t stretch_of(uint64_t written, bool alike, uint32_t lane)
{
    const uint64_t others = written & ~__ballot(alike), below = (1ull << lane) - 1;
    const uint64_t before = others & below, behind = others & ~below;
    return written & (before ? ~((2ull << (63 - __clzll((long long)before))) - 1) : ~0ull) &
           (behind ? (1ull << (__ffsll((long long)behind) - 1)) - 1 : ~0ull);
}

// Run records reach the chain through a ring in LDS.  A load that the chain issued itself would have to be
// awaited at full memory latency, which is long while another batch's copies saturate the memory.  The feeder goes ahead of
// the chain, as far as the ring allows.  None of the waits depends on the waiting wavefront itself: the feeder waits for room,
// which the chain (more than 16 rails) or the drainer (up to 16) makes for records that are written, the chain for records
// that are not, the drainer for the chain; and all loops end with the run table.
template <int kWide, class Ring>
__device__ __forceinline__ void feed_records(const BatchDev& b, int mode, const LevelModel& lm, Ring& ring, uint32_t lane)
{
    const uint32_t n_runs = (uint32_t)b.plan->n_runs;
    const bool pending = (mode & kBindUsePending) != 0;
    const double step = (double)(1ull << kStepBits);
    uint32_t written = 0, block = 0;
    // of the last record written: its level, whether it served, and the slice length of the last run of several slices
    double last_level = 0.0;
    bool last_served = false;
    uint32_t last_len = 0;
    double last_run_level = 0.0;           // and the level of that run
    auto wait_for_room = [&](uint32_t count) {
        if constexpr (kWide > 16) {
            while (written + count - __hip_atomic_load(&ring.taken, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) > kRingRecords)
                __builtin_amdgcn_s_sleep(4);
        } else {
            while (block - __hip_atomic_load(&ring.drained, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= kRingBlocks)
                __builtin_amdgcn_s_sleep(2);
        }
    };
    // what the run table says about the lane's run: read a block ahead, two levels of loads
    struct Run { uint32_t before, start, end, after, len, len_after; uint64_t bytes; };
    auto places = [&](uint32_t at, Run& v) {
        const uint32_t r = at + lane < n_runs ? at + lane : n_runs - 1;
        v.start = b.run_start[r];
        v.end = b.run_start[r + 1];
        v.after = r + 1 < n_runs ? b.run_start[r + 2] : v.end;
        v.before = r > 0 ? b.run_start[r - 1] : v.start;
    };
    auto lengths = [&](Run& v) {
        v.len = b.s_len[pending ? b.pending[v.start] : v.start];
        v.len_after = v.after > v.end ? b.s_len[pending ? b.pending[v.end] : v.end] : 0;
        v.bytes = pending ? b.len_pre[v.start] : b.s_pos[v.start];
    };
    Run now, next;
    if (n_runs > 0) {
        places(0, now);
        lengths(now);
        places(kFeedBlock, next);
    }
    for (uint32_t at = 0; at < n_runs; at += kFeedBlock) {
        const bool here = at + lane < n_runs;
        const uint32_t r = here ? at + lane : n_runs - 1;
        const Run run = now;
        if (at + kFeedBlock < n_runs) {
            now = next;
            lengths(now);
            places(at + 2 * kFeedBlock, next);
        }
        const uint32_t m = run.end - run.start;
        const bool single = m == 1;
        const bool joined = single && run.start - run.before > 1;    // bound together with the run before it
        const bool has_tail = !single && run.after - run.end == 1;
        const uint32_t tail = single ? run.len : has_tail ? run.len_after : 0;
        const double l_f = (double)run.len;
        const double bytes = (double)run.bytes;
        const double v = level_at(lm, bytes + (double)m * l_f, 0.5 * l_f), v_before = level_at(lm, bytes, 0.0);
        const bool valid = v >= 0.0 && v < kMaxLevel;
        const bool serves = valid && v - v_before < step && m < kLevelRunMax && l_f * lm.max_c1 < step * kUnit;
        double level = valid ? __builtin_floor(v) : 0.0;
        // the records written before this one: the lane below among those that are written, or the last block's last
        const uint64_t written_mask = __ballot(here && !joined), run_mask = __ballot(here && !single);
        const uint64_t served_mask = __ballot(serves);
        const uint64_t below = (1ull << lane) - 1;
        const uint64_t prev_mask = written_mask & below, prev_run_mask = run_mask & below;
        const int prev = prev_mask ? 63 - __clzll((long long)prev_mask) : -1;
        const int prev_run = prev_run_mask ? 63 - __clzll((long long)prev_run_mask) : -1;
        const uint32_t len_there = __shfl(run.len, prev_run < 0 ? 0 : prev_run, 64);
        const bool prev_served = prev < 0 ? last_served : ((served_mask >> (prev < 0 ? 0 : prev)) & 1) != 0;
        const uint32_t prev_len = prev_run < 0 ? last_len : len_there;
        // Up to 16 rails a single slice can go as a run of no slices behind the last run: at that run's level, below which no slot
        // is free any more, as long as the slice's cost is not too far above it.  That costs twice what walk_singles takes for a
        // slice, but saves a change from runs to single slices and back, so it is for up to six in a row, in a stretch that goes by
        // ranks.  MI355X, plans of about 4,000 transfers with as many short ones behind every few long ones: one 1109 -> 624 us,
        // two 982 -> 623, four 834 -> 619, six 743 -> 610; rows of eight and ten take 704 and 646 the other way and would take
        // 611 and 608 as runs of none, but 4,096 transfers of which most are single slices 502 -> 518 and 534.
        // That no slot is free below the run's level holds only as long as the heads lie a few of its slices apart, not behind
        // single slices of many times their length, nor behind the first run of a length, where the longer slices before it still tell.
        // There the records miss the ranks' check one by one.  Plans of 72 transfers of 2 to 35 bytes, two of 2 in every nine, 75 us
        // without these two conditions and 45 with them, of 294 with runs of short slices among long ones 127 and 90.
        bool no_run = false;
        if constexpr (kWide == 16) {
            const uint64_t runs_behind = run_mask & ~below;
            const uint64_t between = written_mask & (prev_run < 0 ? ~0ull : ~((2ull << prev_run) - 1)) &
                                     (runs_behind ? (1ull << (__ffsll((long long)runs_behind) - 1)) - 1 : ~0ull);
            const double level_run = from_lane(level, prev_run < 0 ? 0 : prev_run);
            const double at_run = prev_run < 0 ? last_run_level : level_run;
            no_run = single && __popcll(between) <= 6 && tail <= 2 * (uint64_t)prev_len && serves && prev_served && prev_len != 0 &&
                     (v - at_run) * (kUnit / kFineUnit) <= 0.5 * kMaxStep && (double)tail * lm.max_c1 <= 0.25 * kMaxStep * kFineUnit &&
                     (double)prev_len * (lm.max_c1 + lm.min_c1) <= kMaxStep * kFineUnit;
            if (run_mask) last_run_level = from_lane(level, 63 - __clzll((long long)run_mask));
            // only in a stretch that is likely to be long enough to go by ranks, see below
            const bool run_alike = has_tail && serves && prev_len == run.len;
            const uint64_t likely = stretch_of(written_mask, no_run || run_alike, lane), runs_alike = __ballot(run_alike);
            no_run = no_run && __popcll(likely) >= (int)kLeastStretch && (likely & runs_alike) != 0;
            level = no_run ? at_run : level;
        }
        const double level_there = from_lane(level, prev < 0 ? 0 : prev);
        const double prev_level = prev < 0 ? last_level : level_there;
        // a block over which the level rises far is rebased record by record, any other at its start
        const double v_first = from_lane(v_before, 0), v_last = from_lane(v, 63);
        uint32_t flags = (single ? kRecSingle : 0u) | (has_tail ? kRecTail : 0u) | (serves ? 0u : kRecNoLevel);
        if (!single && prev_len == run.len) flags |= kRecSame;
        const uint32_t place = (uint32_t)__popcll(prev_mask);
        const double inv = 1.0 / l_f;
        if constexpr (kWide > 16) {
            if (prev < 0 || !prev_served || !(v_last - v_first < step)) flags |= kRecRebase;
            const double shift = (prev_level - level) * kUnit, tail_f = (double)tail;
            wait_for_room(kFeedBlock);
            if (here && !joined) {
                Quad* out = ring.rec[(written + place) % kRingRecords];
                out[0] = Quad{single ? 0u : m, flags, low_f64(shift), high_f64(shift)};
                out[1] = Quad{low_f64(tail_f), high_f64(tail_f), r, 0u};
                out[2] = Quad{low_f64(level), high_f64(level), run.len, tail};
                out[3] = Quad{low_f64(inv), high_f64(inv), 0u, 0u};
            }
            written += (uint32_t)__popcll(written_mask);
            __hip_atomic_store(&ring.filled, written, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
            const double shift = (prev_level - level) * (kUnit / kFineUnit);
            const double longest = (double)(tail > run.len ? tail : run.len);
            const double rise = shift < 0.0 ? -shift : shift;
            // (a rail that lies far above the level makes the chain rebase at the start of a block, or for every record of one over
            // which the level rises far)
            if (!prev_served || !(rise < step * (kUnit / kFineUnit))) flags |= kRecRebase;
            const bool follows = serves && prev_served && !(flags & kRecRebase);
            const bool run_fits = longest * (lm.max_c1 + lm.min_c1) <= kMaxStep * kFineUnit && rise < kMaxShift;
            const bool same_fits = rise * kFineUnit < l_f * lm.min_c1 * kMaxSlots;
            uint32_t take = !follows ? kTakeOdd : no_run ? kTakeSame : single ? kTakeSingle : !run_fits ? kTakeOdd
                                : flags == kRecShort && same_fits ? kTakeSame : kTakeRun;
            // a stretch of few records goes with the runs around it: a change of the way costs as much as a record.  MI355X, plans of
            // 4,096 transfers in stretches of four equal slice lengths 1128 us by walk_same, 952 by walk_runs; of five 1025 and 970, of
            // six 947 and 942, of eight 942 and 964
            const uint64_t stretch = stretch_of(written_mask, take == kTakeSame, lane);
            if (take == kTakeSame && __popcll(stretch) < (int)kLeastStretch) take = kTakeRun;
            // how many records from here on may be taken the same way
            const uint64_t same = __ballot(take == kTakeSame), runs = __ballot(take == kTakeRun), singles = __ballot(take == kTakeSingle);
            const uint64_t alike = take == kTakeSame ? same : take == kTakeRun ? runs : take == kTakeSingle ? singles : 0;
            const uint64_t stops = written_mask & ~alike & ~below;
            const uint64_t until = stops ? (1ull << (__ffsll((long long)stops) - 1)) - 1 : ~0ull;
            flags |= (take << kRecTake) | ((uint32_t)__popcll(written_mask & ~below & until) << kRecCount);
            wait_for_room(0);
            const uint32_t slot = block % kRingBlocks;
            if (here && !joined) {
                StepRing::Record& out = ring.rec[slot * kFeedBlock + place];
                // (a single slice that goes as a run of none has the last run's slice length)
                const uint32_t l_step = no_run ? prev_len : take == kTakeSingle ? 0u : run.len, l_run = no_run ? prev_len : run.len;
                const double inv_l = no_run ? 1.0 / (double)prev_len : inv;
                const uint32_t near_key = saturating_u32(fma((double)l_run * lm.min_c1, 1.0 / kFineUnit, kBias + 16.0)) & ~15u;
                out.step = Quad{low_f64(shift), high_f64(shift), tail - l_step, single ? 0u : m};
                out.run = Quad{low_f64(inv_l), high_f64(inv_l), l_run, near_key};
                out.level = Quad{low_f64(level), high_f64(level), tail, r};
                out.flags = flags;
                out.single = kStepped;
            }
            ring.count[slot] = (uint32_t)__popcll(written_mask) | (at + kFeedBlock < n_runs ? 0u : kLastBlock) |
                               (v_last - v_first < step ? 0u : kSteepBlock);
            ++block;
            __hip_atomic_store(&ring.filled, block, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (written_mask) {
            const int last = 63 - __clzll((long long)written_mask);
            last_level = from_lane(level, last);
            last_served = ((served_mask >> last) & 1) != 0;
        }
        if (run_mask) last_len = __shfl(run.len, 63 - __clzll((long long)run_mask), 64);
    }
    if constexpr (kWide > 16) {
        wait_for_room(1);
        if (lane == 0) {
            Quad* out = ring.rec[written % kRingRecords];
            out[0] = Quad{0u, kRecEnd, 0u, 0u};
            out[1] = out[2] = out[3] = Quad{0u, 0u, 0u, 0u};
        }
        __hip_atomic_store(&ring.filled, written + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else if (n_runs == 0) {
        ring.count[0] = kLastBlock;
        __hip_atomic_store(&ring.filled, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// ---- the chain ---------------------------------------------------------------------------------
// A run of m slices of l bytes from any state and with any (or no) level estimate: the level is searched
// with exact slot counts (bracket, interpolation, bisection) and the split repaired slot by slot.  Kept
// out of line: the chain's loop calls it only where its short path does not apply.  Returns the lane's slot count.
template <int kWide>
__device__ __attribute__((noinline)) uint32_t bind_run_general(uint64_t T, uint32_t cnt, Rail rail, bool live, uint64_t A_less_T,
                                                               int lane, uint32_t l, uint32_t m, bool has_level, double level_f,
                                                               double inv_l)
{
    constexpr int R = kWide;
    const uint64_t live_mask = __ballot(live);
    const double G = live ? 65536.0 * rail.inv_c1 : 0.0;      // bytes the rail absorbs per picosecond
    const double g = (double)rail.c0 * G;                     // its fixed latency expressed in bytes
    uint32_t k = 0, taken = 0;
    const uint64_t A = A_less_T + T;
    const bool all_proven = __ballot(live && cnt > 0) == live_mask;   // every admitted rail has received a slot
    if (m > (uint32_t)kTol) {
        double v;
        if (has_level && all_proven) {
            v = level_f;
        } else {
            // rails whose next slot already costs more than the level stay out of the pool
            const uint64_t head = live ? slot_cost(rail, A, l, 0) : ~0ull;
            bool wet = live;
            v = 0.0;
            for (int pass = 0; pass < 64; ++pass) {
                const uint64_t wet_mask = __ballot(wet);
                const double sumG = wave_sum_f64(wet ? G : 0.0, R);
                const double sumB = wave_sum_f64(wet ? g + (double)A : 0.0, R);
                const double need = ((double)m + 0.5 * (double)__popcll(wet_mask)) * (double)l;
                v = __longlong_as_double((long long)uniform64((uint64_t)__double_as_longlong((need + sumB) / sumG)));
                const bool still = wet && (cnt > 0 || (double)head <= v);
                const uint64_t still_mask = __ballot(still);
                if (still_mask == wet_mask || still_mask == 0) break;
                wet = still;
            }
        }
        // bracket (computed only if the first guess misses):
        // slots summed over rails stay below m at `lo` and reach at least m at `hi`
        bool bracketed = false;
        int64_t lo = 0, hi = 0;
        for (int iter = 0;; ++iter) {
            int64_t vg = (v >= 0.0 && v < 9.0e18) ? (int64_t)v : -1;
            if (!bracketed && vg < 0) {
                const uint64_t head = live ? slot_cost(rail, A, l, 0) : ~0ull;
                const uint64_t alone = live ? slot_cost(rail, A, l, m - 1) : ~0ull;
                lo = (int64_t)uniform64(wave_reduce64(head, R, OpMin{})) - 1;
                hi = (int64_t)uniform64(wave_reduce64(alone, R, OpMin{}));
                bracketed = true;
            }
            if (bracketed && (iter >= 8 || vg <= lo || vg >= hi)) {   // guess unusable: bisect
                vg = lo + (hi - lo) / 2;
                if (vg <= lo) vg = hi;
            }
            const uint32_t kk = live ? slots_upto_fast(rail, A, l, inv_l, vg, m) : 0;
            const uint64_t tt = uniform64(wave_reduce64(kk, R, OpAdd{}));
            const int64_t miss = (int64_t)m - (int64_t)tt;
            if (miss <= kTol && miss >= -kTol) { k = kk; taken = (uint32_t)tt; break; }
            if (!bracketed) {
                const uint64_t head = live ? slot_cost(rail, A, l, 0) : ~0ull;
                const uint64_t alone = live ? slot_cost(rail, A, l, m - 1) : ~0ull;
                lo = (int64_t)uniform64(wave_reduce64(head, R, OpMin{})) - 1;
                hi = (int64_t)uniform64(wave_reduce64(alone, R, OpMin{}));
                bracketed = true;
            }
            if (miss > 0) { if (vg > lo) lo = vg; } else { if (vg < hi) hi = vg; }
            if (hi - lo == 1) {
                // the whole deficit sits at cost `hi`: hand it out in rail order
                const uint32_t k_lo = live ? slots_upto(rail, A, l, inv_l, lo, m) : 0;
                const uint32_t k_hi = live ? slots_upto(rail, A, l, inv_l, hi, m) : 0;
                const uint64_t below = uniform64(wave_reduce64(k_lo, R, OpAdd{}));
                uint64_t tie = k_hi - k_lo, inc = tie;
#pragma unroll
                for (int d = 1; d < kWide; d <<= 1) {
                    uint64_t up = (uint64_t)__shfl_up((unsigned long long)inc, d, 64);
                    if (lane >= d) inc += up;
                }
                const uint64_t before = inc - tie;                 // ties on lower rails
                const uint64_t rem = (uint64_t)m - below;
                const uint64_t take = before >= rem ? 0 : (rem - before < tie ? rem - before : tie);
                k = k_lo + (uint32_t)take;
                taken = m;
                break;
            }
            const bool near = live && (kk > 0 || slot_cost(rail, A, l, 0) <= (uint64_t)(vg < 0 ? 0 : vg) + 1);
            double rate = wave_sum_f64(near ? G : 0.0, R);
            if (!(rate > 0.0)) rate = wave_sum_f64(G, R);
            v = __longlong_as_double((long long)uniform64(
                (uint64_t)__double_as_longlong((double)vg + (double)miss * (double)l / rate)));
        }
    }
    // repair: add the cheapest free slot / drop the dearest taken slot
    while (taken < m) {
        const int win = argmin_cost(slot_cost(rail, A, l, k), live && k < m, lane, R);
        k += lane == win;
        ++taken;
    }
    while (taken > m) {
        const int win = argmax_cost(slot_cost(rail, A, l, k > 0 ? k - 1 : 0), live && k > 0, lane, R);
        k -= lane == win;
        --taken;
    }
    return k;
}

// Keys of the chain's 32-bit reductions: (cost relative to the level, in ps) << 6 | lane, made from the cost in units of
// 2^-10 ps with the lane over its low bits.  The conversion saturates: a cost 2^26 ps or more away has a key from
// kFarKey on (no near candidate); one that would have to lie on the other side of the level comes out below 64.
constexpr uint32_t kFarKey = 0xFFFFFFC0u;
constexpr double kKeyUnit = 1.0 / 1024.0;
constexpr double kSingleBias = (double)(1ull << 31);   // single slices: the window reaches 2^25 ps to either side of the level
constexpr int kRepairMax = 8;              // slots added or dropped one by one before the general path takes over

// What the next byte of a rail with A bytes queued would cost, relative to the level, in units of 2^-16 ps, exactly (A c1 is,
// by the plan's precondition); infinity for a rail that is far above the level or takes no slices, not-a-number for
// one far below it (every key made from it then comes out below 64, which sends the run or slice to the integers).
__device__ __forceinline__ double relative_cost(const Rail& rail, bool live, uint64_t A, double level)
{
    const uint64_t P = A * (uint64_t)rail.c1;
    const int64_t ps = (int64_t)(rail.c0 + (P >> 16) - (uint64_t)level);
    double x = (double)ps * kUnit + (double)(uint32_t)(P & 65535u);
    if (ps < -(1ll << kFarBits)) x = __builtin_nan("");
    if (!live || ps >= (1ll << kFarBits)) x = __builtin_inf();
    return x;
}

// First guess of a run's split for one rail: the slots at or below the level.  Slot j is iff X + (j + 1) lc1 < 65536,
// so the count is trunc((65535.5 - X) / lc1); half a unit keeps the quotient off the whole numbers by more than it can be
// rounded.  A wrong count would show: its last slot above the level, or its first free one not, gives a key below 64.
struct SplitGuess {
    double p, p_next;                      // where the last slot taken and the first free one end, relative to the level
    uint32_t kk;                           // slots taken
    __device__ __forceinline__ SplitGuess(double X, double lc1, double inv, double kf0)
    {
        kk = saturating_u32(fma(-X, inv, kf0));
        kk = kk < kLevelRunMax ? kk : kLevelRunMax;
        p = fma((double)kk, lc1, X);
        p_next = p + lc1;
    }
    // cheapest free slot: floor(p_next / 65536) >= 1; dearest taken slot: 1 - floor(p / 65536) >= 1
    // (ties: the free slot of the lowest rail is next, the taken slot of the highest rail is last)
    __device__ __forceinline__ uint32_t up_key(uint32_t who) const { return (saturating_u32(p_next * kKeyUnit) & ~63u) | who; }
    __device__ __forceinline__ uint32_t down_key(uint32_t who, double unit, double bias) const
    {
        const uint32_t key = (saturating_u32(fma(p, -unit, bias)) & ~63u) | who;
        return kk != 0 ? key : ~0u;
    }
};

struct SplitResult {
    double X;
    uint32_t kk;
};

// A run whose guess does not hold, by the general path.  Out of line, like everything the chain's loop seldom needs.
template <int kWide>
__device__ __attribute__((noinline)) SplitResult split_odd_run(uint32_t m, bool serves, double T, uint32_t cnt, Rail rail,
                                                               bool live, uint64_t A_less_T, int lane, const Quad* rec)
{
    const Quad q2 = rec[2], q3 = rec[3];
    const double level = join_f64(q2.x, q2.y);
    const uint32_t kk = bind_run_general<kWide>((uint64_t)T, cnt, rail, live, A_less_T, lane, q2.z, m, serves, level, join_f64(q3.x, q3.y));
    return SplitResult{relative_cost(rail, live, A_less_T + (uint64_t)T + (uint64_t)kk * q2.z, level), kk};
}

// The rail of one slice that leaves `end` bytes queued on the rail, from the whole costs.
template <int kWide>
__device__ __attribute__((noinline)) uint32_t odd_single(Rail rail, uint64_t end, bool live, int lane)
{
    return (uint32_t)argmin_cost(rail.c0 + ((end * (uint64_t)rail.c1) >> 16), live, lane, kWide);
}

// Per-rail totals and staging region bases (exclusive sum of 256-byte-rounded totals), lane = rail.
template <int kWide>
__device__ __forceinline__ void write_totals(const BatchDev& b, int lane, uint64_t queued, uint64_t bound, uint32_t cnt,
                                             uint64_t n_bound)
{
    const uint64_t rounded = (bound + 255) & ~255ull;
    uint64_t inc = rounded;
#pragma unroll
    for (int d = 1; d < kWide; d <<= 1) {
        uint64_t up = (uint64_t)__shfl_up((unsigned long long)inc, d, 64);
        if (lane >= d) inc += up;
    }
    PlanState* ps = b.plan;
    ps->T[lane] = bound;
    ps->cnt[lane] = cnt;
    ps->A_after[lane] = queued + bound;
    ps->base[lane] = inc - rounded;
    if (lane == 0) ps->n_bound = n_bound;
}

// More than 16 rails (kWide = 32 or 64: lanes that can hold a rail; up to 16 go through bind_chain16 below, whose ranks and
// replicated state need the rails in one row of 16 lanes).
// Runs in lanes 0 .. kWide-1 of the first wavefront of a workgroup; the other lanes leave at once.
//
// The loop is a chain of dependent instructions on one wavefront that leaves the device idle, so what bounds a plan
// of many transfers is how many instructions it issues per transfer (4-5 cycles each, 8 when the next depends on
// it, 16 for a cross-lane step, 25 and more for a branch taken).  Hence: all state as doubles relative to the level, so
// that a slot's cost is one fma and the comparison with the level needs no shift; the checks of the estimate folded into
// the keys that are reduced anyway; the first repair step without a branch; a lane knows that it won a reduction by its own
// key; what depends on the slice length only is kept from run to run; two 16-byte record reads ahead of their use, by all
// lanes at one address; one 16-byte row store per transfer; and everything unusual behind one test of the record's flags.
// Bytes bound (T) are whole numbers below 2^53, which convert_rails sees to, so a double holds them exactly.
// About 110 instructions and 270 ns per transfer of a run and a tail on MI355X (measured with 16 rails when those came this way),
// from 190 and 510 ns when the state was kept in 64-bit integers and every single slice had a record and a row of its own.
template <int kWide>
__device__ __forceinline__ void bind_chain(const BatchDev& b, const RailParams& rp, int mode, RecordRing& ring)
{
    const int lane = threadIdx.x;
    if (lane >= kWide) return;
    constexpr int R = kWide;                                  // reduction width
    const bool live = lane < (int)rp.n_rails && ((rp.admitted >> lane) & 1);
    Rail rail;
    rail.c0 = rp.c0[lane];
    rail.c1 = live ? (uint32_t)rp.c1[lane] : 1u;
    rail.inv_c1 = 1.0 / (double)rail.c1;
    const double c1_f = (double)rail.c1;
    double T = 0.0;                                           // bytes bound so far, a whole number
    uint32_t cnt = 0;                                         // a batch holds fewer than 2^32 - 1 slices
    uint64_t n_before = 0;
    if (mode & kBindAfterRotation) {          // the rotation pass went first: its bytes are queued and staged ahead
        T = (double)b.plan->Tr[lane];
        cnt = (uint32_t)b.plan->cr[lane];
        n_before = b.plan->n_retry;
    }
    const uint64_t A_less_T = rp.A[lane];                     // A = A_less_T + T at any time
    const uint32_t lane_up = (uint32_t)lane, lane_down = 63u - (uint32_t)lane;

    double X = 0.0;                                           // see relative_cost
    // what depends on the slice length of the current run only
    double l_f = 0.0, lc1 = 0.0, inv = 0.0, kf0 = 0.0;
    uint32_t at = 0;                                          // record in hand
    // constants that have to stay in registers (as literals they would cost two moves at every use)
    double down_bias = 131071.0 * kKeyUnit, single_bias = kSingleBias, key_unit = kKeyUnit;
    asm("" : "+v"(down_bias), "+v"(single_bias), "+s"(key_unit));

    // Split a run of m slices: returns the slots this rail takes and moves X.
    auto split_run = [&](uint32_t m, bool serves) -> uint32_t {
        SplitGuess g(X, lc1, inv, kf0);
        // three reductions side by side: slots taken, cheapest free slot, dearest taken slot
        uint32_t my_up = g.up_key(lane_up), my_down = g.down_key(lane_down, key_unit, down_bias);
        const uint32_t sum = wave_reduce32(g.kk, R, Add32{});
        uint32_t up = wave_reduce32(my_up, R, Min32{});
        uint32_t down = wave_reduce32(my_down, R, Min32{});
        int miss = (int)(m - sum);
        const uint32_t nearest = up < down ? up : down;
        uint32_t dearest = 0;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64((uint32_t)(miss + 1) > 2u) != 0, 0)) {
            // all but the last slot to add or drop (with 16 rails one run in four needs this, with 9 one in eight)
            int left = __builtin_amdgcn_readfirstlane(miss);
            if (left > 1 && left <= kRepairMax) {
                do {
                    dearest = up > dearest ? up : dearest;
                    if (my_up == up) { ++g.kk; g.p = g.p_next; g.p_next += lc1; my_up = g.up_key(lane_up); }
                    up = wave_reduce32(my_up, R, Min32{});
                } while (--left > 1);
            } else if (left < -1 && left >= -kRepairMax) {
                do {
                    dearest = down > dearest ? down : dearest;
                    if (my_down == down) { --g.kk; g.p_next = g.p; g.p -= lc1; my_down = g.down_key(lane_down, key_unit, down_bias); }
                    down = wave_reduce32(my_down, R, Min32{});
                } while (++left < -1);
            }
            miss = left;
        }
        const uint32_t used = miss == 1 ? up : down;
        const bool odd = ((uint32_t)(miss + 1) > 2u) | (nearest < 64u) | ((used > dearest ? used : dearest) >= kFarKey);
        // the last slot: add it (miss = 1), drop it (miss = -1) or nothing
        const bool add = (my_up == up) & (miss == 1), drop = (my_down == down) & (miss == -1);
        double X_after = add ? g.p_next : drop ? g.p - lc1 : g.p;
        uint32_t kk = g.kk + (add ? 1u : 0u) - (drop ? 1u : 0u);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) != 0 || !serves, 0)) {
            const SplitResult r = split_odd_run<kWide>(m, serves, T, cnt, rail, live, A_less_T, lane,
                                                       &ring.rec[at % kRingRecords][0]);
            X_after = r.X;
            kk = r.kk;
        }
        X = X_after;
        return kk;
    };

    // One slice of t bytes: plain argmin.  Returns a word whose low six bits name the rail.
    auto bind_single = [&](double t, bool serves) -> uint32_t {
        const double p = fma(t, c1_f, X);
        uint32_t mine = (saturating_u32(fma(p, key_unit, single_bias)) & ~63u) | lane_up;
        uint32_t best = wave_reduce32(mine, R, Min32{});
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(best - 64u >= kFarKey - 64u) != 0 || !serves, 0)) {
            // outside the window: compare whole costs
            best = odd_single<kWide>(rail, A_less_T + (uint64_t)T + (uint64_t)t, live, lane);
            mine = lane_up;
        }
        const bool won = mine == best;
        X = won ? p : X;
        const double T_more = T + t;
        T = won ? T_more : T;
        cnt += won ? 1u : 0u;
        return best;
    };

    // The records' cells: the rail's bytes before the run, its slots, and the rail of the single slice behind it.
    RunCell* const my_cell = b.run_cell + lane;
    const uint32_t stride = b.run_stride;
    uint32_t block_end = 0;                                   // the chain may read records before this one
    auto next_block = [&]() {
        if (lane == 0) __hip_atomic_store(&ring.taken, at, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        uint32_t filled;
        while ((filled = (uint32_t)__builtin_amdgcn_readfirstlane(
                    (int)__hip_atomic_load(&ring.filled, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP))) <= at)
            __builtin_amdgcn_s_sleep(1);
        block_end = filled < at + kFeedBlock ? filled : at + kFeedBlock;
    };
    next_block();
    Quad q0 = ring.rec[0][0], q1 = ring.rec[0][1];
    auto step_on = [&]() {
        ++at;
        if (__builtin_expect(at == block_end, 0)) next_block();
        q0 = ring.rec[at % kRingRecords][0];
    };
    for (;;) {
        uint32_t flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)q0.y);
        while (flags == kRecShort) {                                  // a loop of its own: nothing to merge with the rest
            const double T_before = T;
            X += join_f64(q0.z, q0.w);                                // from the level of the record before to this one's
            const uint32_t kk = split_run(q0.x, true);
            T = fma((double)kk, l_f, T);
            cnt += kk;
            step_on();
            const uint32_t tail_rail = bind_single(join_f64(q1.x, q1.y), true);
            *(my_cell + (uint64_t)q1.z * stride) = RunCell{T_before, kk, tail_rail};
            q1 = ring.rec[at % kRingRecords][1];
            flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)q0.y);
        }
        if (flags & kRecEnd) break;
        const Quad q2 = ring.rec[at % kRingRecords][2], q3 = ring.rec[at % kRingRecords][3];
        const bool serves = !(flags & kRecNoLevel);
        const double T_before = T;
        uint32_t kk = 0, tail_rail = 0;
        if (flags & kRecRebase) X = relative_cost(rail, live, A_less_T + (uint64_t)T, join_f64(q2.x, q2.y));
        else X += join_f64(q0.z, q0.w);
        if (!(flags & kRecSingle)) {
            l_f = (double)q2.z;
            lc1 = l_f * c1_f;                                         // whole, below 2^53 where the record serves
            inv = join_f64(q3.x, q3.y) * rail.inv_c1;
            kf0 = 65535.5 * inv;
            kk = split_run(q0.x, serves);
            T = fma((double)kk, l_f, T);
            cnt += kk;
        }
        if (flags & (kRecTail | kRecSingle)) tail_rail = bind_single(join_f64(q1.x, q1.y), serves);
        *(my_cell + (uint64_t)q1.z * stride) = RunCell{T_before, kk, tail_rail};
        step_on();
        q1 = ring.rec[at % kRingRecords][1];
    }

    write_totals<kWide>(b, lane, A_less_T, (uint64_t)T, cnt, b.plan->n_pending + n_before);
}

// ---- the chain of up to 16 rails -------------------------------------------------------------------
// All-reduce over rows of 16 lanes.
template <class Op>
__device__ __forceinline__ uint32_t row_reduce32(uint32_t v, Op op) { return wave_reduce32(v, 16, op); }

// The cross-lane part of a step, for a wavefront whose four rows of 16 lanes hold the same state.  From the guess u of the slots
// (below zero: none): kk, the whole slots; p_next = Y0 + kk lc1, where the slot behind them ends, and key, its key; sum, kk
// over the rails; returns how many rails have a smaller key (keys are distinct and less than 2^31 apart).
// Row r compares with the lanes 4 r .. 4 r + 3 further on; a byte of each difference's sign is gathered, and one matrix
// instruction adds up (-1) (-1) over the bytes of all four rows.  One block of assembler, so that the wait states between a
// register's write and its use by a cross-lane (DPP) instruction -- two instructions -- are filled by hand: kk is used four
// instructions behind its conversion, key and turned two behind their last write, sum's steps two and more apart.
typedef int Int4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Int4 rank_next_slots(double u, double lc1, double Y0, uint32_t who, uint32_t& kk, uint32_t& key,
                                                double& p_next, uint32_t& sum)
{
    uint32_t turned, d0, d1, d2, d3, half;
    double kf;
    asm("v_cvt_u32_f64_e32 %[kk], %[u]\n\t"
        "v_cvt_f64_u32_e32 %[kf], %[kk]\n\t"
        "v_fma_f64 %[pn], %[kf], %[lc1], %[Y0]\n\t"
        "v_cvt_u32_f64_e32 %[key], %[pn]\n\t"
        "v_and_or_b32 %[key], %[key], -16, %[who]\n\t"
        "v_add_u32_dpp %[half], %[kk], %[kk] quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b32_e32 %[tu], %[key]\n\t"
        "v_mov_b32_dpp %[tu], %[key] row_ror:4 row_mask:0x2 bank_mask:0xf\n\t"
        "v_mov_b32_dpp %[tu], %[key] row_ror:8 row_mask:0x4 bank_mask:0xf\n\t"
        "v_mov_b32_dpp %[tu], %[key] row_ror:12 row_mask:0x8 bank_mask:0xf\n\t"
        "v_add_u32_dpp %[half], %[half], %[half] quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_sub_u32_e32 %[d0], %[tu], %[key]\n\t"
        "v_sub_u32_dpp %[d1], %[tu], %[key] row_ror:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_sub_u32_dpp %[d2], %[tu], %[key] row_ror:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_sub_u32_dpp %[d3], %[tu], %[key] row_ror:3 row_mask:0xf bank_mask:0xf"
        : [kk] "=&v"(kk), [key] "=&v"(key), [half] "=&v"(half), [tu] "=&v"(turned), [d0] "=&v"(d0), [d1] "=&v"(d1),
          [d2] "=&v"(d2), [d3] "=&v"(d3), [kf] "=&v"(kf), [pn] "=&v"(p_next)
        : [u] "v"(u), [lc1] "v"(lc1), [Y0] "v"(Y0), [who] "v"(who));
    // bytes: 0xFF where a difference is negative, else 0 (selectors 11 and 9: the sign of either operand, 12: zero)
    const uint64_t signs = (uint64_t)__builtin_amdgcn_perm(d0, d1, 0x0C0C0B09u) |
                           ((uint64_t)__builtin_amdgcn_perm(d2, d3, 0x0C0C0B09u) << 32);
    const Int4 none = {0, 0, 0, 0};
    const Int4 rank = __builtin_amdgcn_mfma_i32_16x16x32_i8(-1l, (long)signs, none, 0, 0, 0);
    half += dpp32<0x141>(half);
    sum = half + dpp32<0x140>(half);
    return rank;                           // four times the same
}

// The loop is a chain of dependent instructions on one wavefront that leaves the device idle.  A lone wavefront issues an
// instruction every 4-5 cycles whatever its kind, a wait state of a cross-lane step costs as much, a branch on a fresh comparison 25
// more.  So what bounds a plan of many transfers is the number of instructions between one transfer's state and the
// next one's, and the short path (walk) is made of as few as possible, without a branch but the one that checks it:
//   - the guess is taken at a level that is meant to be a little too low (LevelModel::short_by), so that slots are only ever
//     added; all of them at once, to the rails whose next slots are the cheapest, by rank instead of one by one;
//   - all four rows of the wavefront hold the rails' state, and each compares a quarter of the pairs (rank_next_slots);
//   - the guess is exact by its arithmetic (below), so it needs no check; that no rail lacks two slots is seen from the keys;
//   - whatever the chain finds is left in LDS, and a third wavefront, the drainer, derives the bytes bound from it and writes the
//     rows, so that the state here is one number per rail.
// State: X, the cost of the rail's next byte, in units of 2^-4 ps above kBias below the level, a whole multiple of 2^-12 and held
// exactly (infinity: the rail takes no slices or lies far above the level; the bytes queued are then in A_far).
//   Guess: slot j ends at X + (j + 1) lc1 and costs no more than the level iff that is below kBias + 16, so kk = trunc(Q),
//   Q = (N - X) / lc1 with N half a unit (2^-13) below that.  Q is at least 2^-13 / lc1 off the whole numbers; its computed
//   value is off by less than (|N - X| 2^-51 + 2^-22) / lc1, which is less while |N - X| < 2^37: kMaxShift and the test of
//   `tight` see to that.  (Below zero both give 0.)
//   Taken: the run takes the guessed slots and the m - sum cheapest of the rails' next ones, if no rail takes two of those:
//   its second one costs more than the level by at least the smallest lc1, so keys below near_key are all in order.
//   Single slice: where slots were only added every rail's next slot ends above the level and some rail's last one below near_key,
//   so by kMaxStep no key lies below the window, the least one lies inside it, and it is the cheapest.  Behind dropped slots
//   (walk_runs) and behind another single slice a key may lie below the window too, where all are 0 but for the rail: there
//   a least key from either end of the window sends the record to odd_record.
// MI355X: about 65 instructions and 310 clocks (125 ns) per transfer of a run and a tail, from 110 and 640 with one-by-one
// repairs and the bytes bound kept here: reset, plan and execute of 24,576 transfers on 16 rails 15.5 -> 11.6 ms, of 4,096 2.68
// -> 2.04 ms, of 2,048 shorter by partial pages 1.44 -> 1.06 ms.  What is not a stretch of equal slice lengths goes through
// walk_runs (about 600 clocks a record, 700 with what is added and dropped slot by slot) and walk_singles (180), and only the first
// record, one behind a rebase, and a guess off by more than a few slots through odd_record (1,100); a change of the way costs about
// 250, a plan of 50 runs takes what it took.  With a check and a branch for everything that may not hold, and the records read when
// they were due, walk_runs took 850 and walk_singles 290: plans of 4,096 transfers of a slice 635 -> 502 us, of 4,054 pairs of one
// or two slices of 1 MiB 1065 -> 819.
struct ChainState {
    double X, lc1, inv, kf0;
    uint32_t near_key;
};

// A run or single slice the short path does not take.  Out of line, like everything the loop seldom needs.
struct OddSplit {
    uint32_t kk;
    uint64_t A;
};
__device__ __attribute__((noinline)) OddSplit general_split16(Rail rail, bool live, uint64_t A, int lane, uint32_t l, uint32_t m,
                                                              bool serves, double level, double inv_l)
{
    // (in the first row alone: the general path counts lanes)
    uint32_t kk = 0;
    if (lane < 16) kk = bind_run_general<16>(0, 1u, rail, live, A, lane, l, m, serves, level, inv_l);
    kk = (uint32_t)__shfl((int)kk, lane & 15, 64);
    return OddSplit{kk, A + (uint64_t)kk * l};
}

// Runs in all lanes of the first wavefront of a workgroup: lane % 16 = rail.
__device__ __forceinline__ void bind_chain16(const BatchDev& b, const RailParams& rp, int mode, StepRing& ring)
{
    const int lane = threadIdx.x;
    const uint32_t who = (uint32_t)lane & 15u;
    const bool live = who < rp.n_rails && ((rp.admitted >> who) & 1);
    Rail rail;
    rail.c0 = rp.c0[who];
    rail.c1 = live ? (uint32_t)rp.c1[who] : 1u;
    rail.inv_c1 = 1.0 / (double)rail.c1;
    const double c1 = (double)rail.c1 * (1.0 / kFineUnit);
    uint64_t A_far = rp.A[who];                               // bytes queued on a rail whose X is infinite
    if (mode & kBindAfterRotation) A_far += b.plan->Tr[who];
    ChainState st{__builtin_inf(), 0.0, 0.0, 0.0, 0u};
    double l_f = 0.0;                                         // length of the last run's slices

    // X from the bytes queued, for a level; and the bytes queued from X and the level it refers to.
    auto set_state = [&](uint64_t A, double level) {
        const double x = relative_cost(rail, live, A, level);            // not-a-number: far below the level
        const bool known = x - x == 0.0;
        st.X = known ? fma(x, 1.0 / kFineUnit, kBias) : __builtin_inf();
        A_far = A;
        return __builtin_amdgcn_ballot_w64(x != x) != 0;                  // such a rail: the keys cannot be used
    };
    auto queued = [&](double level) -> uint64_t {
        // A c1 = X / 2^-16 ps + (level - c0) 2^16: exact in 64-bit arithmetic with wrap, and below 2^63
        const double rel = (st.X - kBias) * kFineUnit;
        const uint64_t P = (uint64_t)(int64_t)(st.X < 1.0e300 ? rel : 0.0) + (((uint64_t)level - rail.c0) << 16);
        uint64_t q = (uint64_t)((double)P * rail.inv_c1);                 // off by a few units at most
        const int64_t rest = (int64_t)(P - q * rail.c1);                  // a multiple of c1
        q += (uint64_t)(int64_t)__builtin_rint((double)rest * rail.inv_c1);
        return st.X < 1.0e300 ? q : A_far;
    };

    // One record by the checked way.
    auto odd_record = [&](uint32_t at, bool rebase) {
        const Quad s = ring.rec[at].step, r0 = ring.rec[at].level, r1 = ring.rec[at].run;
        const uint32_t flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)ring.rec[at].flags);
        const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.w);
        const double level = join_f64(r0.x, r0.y), shift = join_f64(s.x, s.y), inv_l = join_f64(r1.x, r1.y);
        const uint32_t l = r1.z, tail = r0.z;
        const bool serves = !(flags & kRecNoLevel);
        bool usable = serves;
        if (rebase || (flags & kRecRebase) || !serves) {
            const uint64_t A = queued(level + shift * (kFineUnit / kUnit));   // (the level of the record before)
            if (set_state(A, level)) usable = false;
            if (!usable) st.X = __builtin_inf();
        } else {
            st.X += shift;
        }
        uint32_t kk = 0, best = 0;
        if (!(flags & kRecSingle)) {
            l_f = (double)l;
            st.lc1 = l_f * c1;                                            // whole multiples of 2^-12, below 2^41 where the record serves
            st.inv = inv_l * rail.inv_c1 * kFineUnit;
            st.kf0 = kGuessAt * st.inv;
            st.near_key = r1.w;
            bool done = false;
            if (usable) {
                // guess, then one slot at a time: the cheapest free one, or the dearest taken one
                uint32_t k = saturating_u32(fma(-st.X, st.inv, st.kf0));
                k = k < kLevelRunMax ? k : kLevelRunMax;
                double p_next = fma((double)k, st.lc1, st.X) + st.lc1;    // where the cheapest free slot ends; the dearest taken one: lc1 before
                auto down_key = [&]() { return k != 0 ? tagged_key(kDownFrom + st.lc1 - p_next, 15u - who) : ~0u; };
                uint32_t my_up = tagged_key(p_next, who), my_down = down_key();
                const uint32_t sum = row_reduce32(k, Add32{}), level_key = (uint32_t)kBias + 16u;
                uint32_t farthest = 0;
                int left = __builtin_amdgcn_readfirstlane((int)(m - sum));
                if (left >= -kRepairMax && left <= kRepairMax && __builtin_amdgcn_ballot_w64(my_up < level_key || my_down < level_key) == 0) {
                    for (; left > 0; --left) {
                        const uint32_t up = row_reduce32(my_up, Min32{});
                        const double beyond = p_next + st.lc1;
                        farthest = up > farthest ? up : farthest;
                        k += my_up == up ? 1u : 0u;
                        p_next = my_up == up ? beyond : p_next;
                        my_up = tagged_key(p_next, who);
                    }
                    for (; left < 0; ++left) {
                        const uint32_t down = row_reduce32(my_down, Min32{});
                        const double before = p_next - st.lc1;
                        farthest = down > farthest ? down : farthest;
                        k -= my_down == down ? 1u : 0u;
                        p_next = my_down == down ? before : p_next;
                        my_down = down_key();
                    }
                    done = __builtin_amdgcn_ballot_w64(farthest >= kFarKey16) == 0;
                }
                if (done) { kk = k; st.X = p_next - st.lc1; }
            }
            if (!done) {
                const OddSplit g = general_split16(rail, live, queued(level), lane, l, m, serves, level, inv_l);
                kk = g.kk;
                usable = !set_state(g.A, level) && serves;
                if (!usable) st.X = __builtin_inf();
            }
        }
        if (tail != 0) {
            const double t = (double)tail, y = fma(t, c1, st.X);
            uint32_t mine = (saturating_u32(y) & ~15u) | who;
            best = row_reduce32(mine, Min32{});
            // outside the window (or a state that does not serve): compare whole costs
            if (!usable || __builtin_amdgcn_ballot_w64(best - 16u >= kFarKey16 - 16u) != 0) {
                const uint64_t A = queued(level);
                best = odd_single<16>(rail, A + tail, live, (int)who);
                mine = who;
                if (mine == best) A_far = A + tail;
            }
            st.X = mine == best ? y : st.X;
        }
        if (!usable) st.X = __builtin_inf();                              // (A_far holds the bytes)
        if (lane < 16) ring.found[at][who] = kk;
        ring.rec[at].single = best;
        return usable;                                                    // if not, the next record rebases
    };
    // Whether the heads lie where a guess is exact and not too large.
    auto is_tight = [&]() {
        const double below = kBias - st.X;
        return l_f != 0.0 && __builtin_amdgcn_ballot_w64(live && !(below < kMaxShift && below < st.lc1 * kMaxSlots)) == 0;
    };

    // Records [at, at + n) of runs with the last one's slice length: returns how many it took, fewer than n if one did not pass
    // its check.  Four records share a check, and each keeps the state it leaves, for the case that a later one does not pass.
    auto walk_same = [&](uint32_t at, uint32_t n) -> uint32_t {
        double Y = st.X + st.lc1;                                          // where the rail's next slot would end
        const double lc1 = st.lc1, inv = st.inv, kf0 = fma(lc1, inv, st.kf0);
        const uint32_t near_key = st.near_key;
        const StepRing::Record* rec = &ring.rec[at];
        uint32_t* found = &ring.found[at][who];
        Quad s = rec->step;
        // One record: the state behind it, what it found, and the lanes that object to it.
        auto one = [&](const StepRing::Record* next, double Y_in, double& Y_out, uint32_t& word) -> uint64_t {
            const double Y0 = Y_in + join_f64(s.x, s.y), less = (double)(int)s.z;
            const uint32_t m = s.w;
            uint32_t kk, key, sum;
            double pn;
            const Int4 rank = rank_next_slots(fma(-Y0, inv, kf0), lc1, Y0, who, kk, key, pn, sum);
            // while the ranks are summed: where the rail stands with the next slot and without, with the single slice and without
            const double pn_more = pn + lc1, y = fma(less, c1, pn), y_more = fma(less, c1, pn_more);
            const uint32_t mine_less = tagged_key(y, who), mine_more = tagged_key(y_more, who);
            const uint32_t lacking = m - sum;
            const bool takes = rank[0] < (int)lacking;
            asm volatile("" : : "v"(rank));                                // (its registers are not reused before: that would wait)
            const uint64_t bad = (__builtin_amdgcn_ballot_w64(takes) & __builtin_amdgcn_ballot_w64(key >= near_key)) |
                                 __builtin_amdgcn_ballot_w64(lacking > 15u);
            const uint32_t mine = takes ? mine_more : mine_less;
            s = next->step;
            double Y1 = takes ? pn_more : pn, won = (takes ? y_more : y) + lc1;
            kk += takes ? 1u : 0u;
            asm volatile("" : "+v"(Y1), "+v"(won), "+v"(kk));              // here, where they fill the wait states of the minimum
            const uint32_t best = row_reduce32(mine, Min32{});
            Y_out = mine == best ? won : Y1;
            word = (best << kBitsOfSlots) | kk;
            return bad | __builtin_amdgcn_ballot_w64(best >= kFarKey16);
        };
        uint32_t left = n;
        // Where the loop lies counts: 4,096 transfers take 540 to 560 us over the sixteen places in a 64-byte line, with the least every
        // 32 bytes.  Left to itself it moves with every change of the code around it.
        asm volatile(".p2align 5\n\t.rept 7\n\ts_nop 0\n\t.endr");
        for (; left >= 4; left -= 4) {
            double Y1, Y2, Y3, Y4;
            uint32_t w1, w2, w3, w4;
            const uint64_t b1 = one(rec + 1, Y, Y1, w1), b2 = one(rec + 2, Y1, Y2, w2);
            found[0] = w1;
            found[16] = w2;
            const uint64_t b3 = one(rec + 3, Y2, Y3, w3), b4 = one(rec + 4, Y3, Y4, w4);
            found[32] = w3;                                                // (written again if the record does not pass)
            found[48] = w4;
            if (__builtin_expect((b1 | b2 | b3 | b4) != 0, 0)) {
                if (b1 == 0) { Y = Y1; --left; if (b2 == 0) { Y = Y2; --left; if (b3 == 0) { Y = Y3; --left; } } }
                st.X = Y - lc1;
                return n - left;
            }
            Y = Y4;
            rec += 4;
            found += 64;
        }
        for (; left != 0; --left) {
            double Y1;
            uint32_t w1;
            const uint64_t b1 = one(rec + 1, Y, Y1, w1);
            found[0] = w1;
            if (b1 != 0) break;
            Y = Y1;
            ++rec;
            found += 16;
        }
        st.X = Y - lc1;
        return n - left;
    };

    // Records of runs of any slice length, with a single slice behind them or not, one by one: by ranks, with one check for all that may
    // not hold, and otherwise slot by slot.  (Without a single slice one of no bytes is bound, which changes nothing; the drainer and the
    // emit step do not look at its rail.)
    auto walk_runs = [&](uint32_t at, uint32_t n) -> uint32_t {
        const StepRing::Record* rec = &ring.rec[at];
        uint32_t* found = &ring.found[at][who];
        const double inv_c1 = rail.inv_c1 * kFineUnit;
        uint32_t left = n;
        Quad s = rec->step, r = rec->run;
        for (; left != 0; --left, found += 16) {
            const uint32_t near_key = r.w, m = s.w;
            const double X0 = st.X + join_f64(s.x, s.y), lc1 = (double)r.z * c1, inv = join_f64(r.x, r.y) * inv_c1, len = (double)r.z;
            const double Y0 = X0 + lc1, kf0 = kGuessAt * inv, tail = (double)(s.z + r.z);
            uint32_t kk, key, sum;
            double pn;
            const Int4 rank = rank_next_slots(fma(-X0, inv, kf0), lc1, Y0, who, kk, key, pn, sum);
            const double held = pn - lc1, y_less = fma(tail, c1, held), y_more = fma(tail, c1, pn);
            const uint32_t mine_less = tagged_key(y_less, who), mine_more = tagged_key(y_more, who);
            ++rec;
            s = rec->step;
            r = rec->run;
            const uint32_t lacking = m - sum;
            const bool takes = rank[0] < (int)lacking;
            asm volatile("" : : "v"(rank));                                // (its registers are not reused before: that would wait)
            uint32_t mine = takes ? mine_more : mine_less;
            double X1 = takes ? pn : held, y = takes ? y_more : y_less;
            uint32_t best = row_reduce32(mine, Min32{});
            // (a rail that does not take slices or lies far above the level has an infinite head)
            const bool odd = (lacking > 15u) | !(kBias - X0 < kMaxShift) | (kk >= (uint32_t)kMaxSlots) | (takes & (key >= near_key)) |
                             (best - 16u >= kFarKey16 - 16u);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) == 0, 1)) {
                kk += takes ? 1u : 0u;
            } else {
                // where some rail lacks two slots they are added one by one, to the cheapest free one each time; where the guess took too
                // many (rails that the last run left far above the level, in terms of this run's shorter slices, make the level too high)
                // the dearest are dropped one by one
                const bool far = (lacking + (uint32_t)kRepairMax > 15u + (uint32_t)kRepairMax) | !(kBias - X0 < kMaxShift) | (kk >= (uint32_t)kMaxSlots);
                if (__builtin_amdgcn_ballot_w64(far) != 0) break;
                uint32_t farthest = 0;                                     // of all keys used
                int more = __builtin_amdgcn_readfirstlane((int)lacking);
                for (; more > 0; --more) {
                    const uint32_t up = row_reduce32(key, Min32{});
                    const double beyond = pn + lc1;
                    farthest = up > farthest ? up : farthest;
                    kk += key == up ? 1u : 0u;
                    pn = key == up ? beyond : pn;
                    key = tagged_key(pn, who);
                }
                // 1 - floor(ps) of the last slot taken, 1 and up.  Where that is beyond the window on every rail with a slot, rails
                // without one are taken for it too, and what follows has any key: the first such step must not be forgotten
                for (; more < 0; ++more) {
                    const uint32_t down = kk != 0 ? tagged_key(kDownFrom + lc1 - pn, 15u - who) : ~0u;
                    const double before = pn - lc1;
                    const uint32_t least = row_reduce32(down, Min32{});
                    farthest = least > farthest ? least : farthest;
                    kk -= down == least ? 1u : 0u;
                    pn = down == least ? before : pn;
                }
                X1 = pn - lc1;
                y = fma(tail, c1, X1);
                mine = tagged_key(y, who);
                best = row_reduce32(mine, Min32{});
                // (without a single slice a least key outside the window means nothing)
                if (__builtin_amdgcn_ballot_w64((farthest >= kFarKey16) | ((tail != 0.0) & (best - 16u >= kFarKey16 - 16u))) != 0) break;
            }
            *found = kk | (best << kBitsOfSlots);
            st = ChainState{mine == best ? y : X1, lc1, inv, kf0, near_key};
            l_f = len;
        }
        return n - left;
    };

    // Single slices, one by one: a plain argmin by keys, unless they lie outside the window.  Four records share a check, and each
    // keeps the state it leaves, for the case that a later one does not pass; the next four are read meanwhile.  The first has a check
    // of its own, because where one lies outside the next is likely to, and three would be bound in vain: plans of slices of
    // milliseconds each took 0.80 us a slice instead of 0.66 (4,186 transfers 5027 us, 4087 with it), 2,048 of which a fifth are outside 589
    // instead of 523; where none is it makes no difference.
    auto walk_singles = [&](uint32_t at, uint32_t n) -> uint32_t {
        const StepRing::Record* rec = &ring.rec[at];
        uint32_t* found = &ring.found[at][who];
        // One record: the state behind it and its key, less the least one inside the window (from kFarKey16 - 16 on: outside).
        auto one = [&](const Quad& s, double X_in, double& X_out, uint32_t* out) -> uint32_t {
            const double X0 = X_in + join_f64(s.x, s.y), y = fma((double)s.z, c1, X0);
            const uint32_t mine = tagged_key(y, who), best = row_reduce32(mine, Min32{});
            X_out = mine == best ? y : X0;
            *out = best << kBitsOfSlots;
            return best - 16u;
        };
        auto outside = [&](uint32_t key) { return __builtin_amdgcn_ballot_w64(key >= kFarKey16 - 16u) != 0; };
        Quad s1 = rec[0].step, s2 = rec[1].step, s3 = rec[2].step, s4 = rec[3].step;
        uint32_t left = n;
        {
            double X1;
            const uint32_t b1 = one(s1, st.X, X1, found);
            if (outside(b1)) return 0u;
            st.X = X1;
            found += 16;
            --left;
            s1 = s2;
            s2 = s3;
            s3 = s4;
            s4 = rec[4].step;
            ++rec;
        }
        for (; left >= 4; left -= 4) {
            const Quad n1 = rec[4].step, n2 = rec[5].step, n3 = rec[6].step, n4 = rec[7].step;
            double X1, X2, X3, X4;
            const uint32_t b1 = one(s1, st.X, X1, found), b2 = one(s2, X1, X2, found + 16);
            const uint32_t b3 = one(s3, X2, X3, found + 32), b4 = one(s4, X3, X4, found + 48);
            const uint32_t b12 = b1 > b2 ? b1 : b2, b34 = b3 > b4 ? b3 : b4;
            if (__builtin_expect(outside(b12 > b34 ? b12 : b34), 0)) {
                if (outside(b1)) return n - left;
                st.X = X1;
                if (outside(b2)) return n - left + 1;
                st.X = X2;
                if (outside(b3)) return n - left + 2;
                st.X = X3;
                return n - left + 3;
            }
            st.X = X4;
            rec += 4;
            found += 64;
            s1 = n1;
            s2 = n2;
            s3 = n3;
            s4 = n4;
        }
        for (; left != 0; --left) {
            double X1;
            const uint32_t b1 = one(s1, st.X, X1, found);
            if (outside(b1)) break;
            st.X = X1;
            found += 16;
            s1 = s2;
            s2 = s3;
        }
        return n - left;
    };

    bool rebase = true, tight = false;
    for (uint32_t block = 0;; ++block) {
        while (__hip_atomic_load(&ring.filled, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= block) __builtin_amdgcn_s_sleep(1);
        const uint32_t slot = block % kRingBlocks, base = slot * kFeedBlock;
        const uint32_t told = (uint32_t)__builtin_amdgcn_readfirstlane((int)ring.count[slot]);
        const uint32_t n = told & ~(kLastBlock | kSteepBlock);
        uint32_t flags = ring.rec[base].flags, missed = 0;
        bool one_by_one = false;                               // the block's stretches of equal slices too
        for (uint32_t i = 0; i < n;) {
            // a rail far above the level counts as infinitely far: look again where it lies
            if (i == 0 || (told & kSteepBlock)) rebase = rebase || __builtin_amdgcn_ballot_w64(live && !(st.X < 1.0e300)) != 0;
            flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)flags);
            const uint32_t take = (flags >> kRecTake) & 3u;
            uint32_t count = rebase || take == kTakeOdd ? 0u : flags >> kRecCount, went = 0;
            if ((told & kLastBlock) && count > kWalkLast) count = kWalkLast;
            if (count != 0) {
                if (take == kTakeSame && !one_by_one && (tight || is_tight())) {
                    flags = ring.rec[base + i + count].flags;            // of the record behind, as a rule the next one to look at
                    went = walk_same(base + i, count);
                    tight = true;
                    if (went < count) {
                        flags = (kTakeRun << kRecTake) | (1u << kRecCount);   // not by ranks: with the repairs of walk_runs
                        i += went;
                        ++missed;
                        one_by_one = missed >= kMissFew && missed * kMissWorth > i;
                        continue;
                    }
                } else if (take == kTakeSingle) {
                    flags = ring.rec[base + i + count].flags;
                    went = walk_singles(base + i, count);
                    tight = false;
                } else {
                    count = take == kTakeSame && !one_by_one ? 1u : count;
                    flags = ring.rec[base + i + count].flags;
                    went = walk_runs(base + i, count);
                    tight = true;
                }
            }
            i += went;
            if (count == 0 || went < count) {                  // this one by the checked way
                rebase = !odd_record(base + i, rebase);
                tight = false;
                ++i;
                flags = ring.rec[base + i].flags;
            }
            if (told & kLastBlock)
                __hip_atomic_store(&ring.walked, block * kFeedBlock + i, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __hip_atomic_store(&ring.walked, (block + 1) * kFeedBlock, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (told & kLastBlock) break;
    }
}

// The drainer: from the slots and single slices of every record the bytes bound to every rail before it, the row that the emit
// step reads, and the plan's totals.  T, whole and below 2^53, is exact as a double.  Lane % 16 = rail; the first row writes.
__device__ __forceinline__ void drain_steps16(const BatchDev& b, const RailParams& rp, int mode, StepRing& ring, uint32_t lane)
{
    const uint32_t who = lane & 15u;
    double T = 0.0;
    uint32_t cnt = 0;
    uint64_t n_before = 0;
    if (mode & kBindAfterRotation) {          // the rotation pass went first: its bytes are queued and staged ahead
        T = (double)b.plan->Tr[who];
        cnt = (uint32_t)b.plan->cr[who];
        n_before = b.plan->n_retry;
    }
    const uint64_t queued = rp.A[who], n_bound = b.plan->n_pending + n_before;
    RunCell* const my_cell = b.run_cell + who;
    const uint32_t stride = b.run_stride;
    for (uint32_t block = 0;; ++block) {
        while (__hip_atomic_load(&ring.filled, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= block) __builtin_amdgcn_s_sleep(1);
        const uint32_t slot = block % kRingBlocks, base = slot * kFeedBlock;
        const uint32_t told = (uint32_t)__builtin_amdgcn_readfirstlane((int)ring.count[slot]);
        const uint32_t n = told & ~(kLastBlock | kSteepBlock);
        for (uint32_t i = 0; i < n;) {
            uint32_t ready;
            while ((ready = (uint32_t)__builtin_amdgcn_readfirstlane(
                        (int)__hip_atomic_load(&ring.walked, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP))) <= block * kFeedBlock + i)
                __builtin_amdgcn_s_sleep(1);
            ready -= block * kFeedBlock;
            if (ready > n) ready = n;
            // four records' reads at a time; the chain hands over few at a time where it changes its way often
            for (; i < ready; i += 4) {
                Quad r0[4];
                uint32_t l[4], word[4], single[4];
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t at = base + (i + k < ready ? i + k : i);
                    r0[k] = ring.rec[at].level;
                    l[k] = ring.rec[at].run.z;
                    single[k] = ring.rec[at].single;
                    word[k] = ring.found[at][who];
                }
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    if (i + k >= ready) break;
                    const uint32_t tail = r0[k].z;
                    const bool stepped = single[k] == kStepped;
                    const uint32_t slots = stepped ? word[k] & ((1u << kBitsOfSlots) - 1) : word[k];
                    const uint32_t rail = stepped ? word[k] >> kBitsOfSlots : single[k] & 15u;
                    if (lane < 16) *(my_cell + (uint64_t)r0[k].w * stride) = RunCell{T, slots, rail};
                    const bool won = rail == who && tail != 0;
                    T = fma((double)slots, (double)l[k], T) + (won ? (double)tail : 0.0);
                    cnt += slots + (won ? 1u : 0u);
                }
            }
            i = ready;
        }
        __hip_atomic_store(&ring.drained, block + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (told & kLastBlock) break;
    }
    if (lane >= 16) return;
    write_totals<16>(b, lane, queued, (uint64_t)T, cnt, n_bound);
}

template <int kWide>
using Ring = std::conditional_t<kWide == 16, StepRing, RecordRing>;
constexpr uint32_t kChainThreads = 192;

// Clears the ring; a barrier follows before anyone uses it.
__device__ __forceinline__ void start_ring(RecordRing& ring) { ring.filled = ring.taken = 0; }
__device__ __forceinline__ void start_ring(StepRing& ring) { ring.filled = ring.walked = ring.drained = 0; }

// Wavefront 0 walks the chain, wavefront 1 feeds it the run records, wavefront 2 drains it (up to 16 rails).
template <int kWide>
__device__ __forceinline__ void chain_waves(const BatchDev& b, const RailParams& rp, int mode, Ring<kWide>& ring, LevelModel& lm)
{
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);                 // other workgroups' or wavefronts' work must not take its issue slots
        if constexpr (kWide == 16) bind_chain16(b, rp, mode, ring);
        else bind_chain<kWide>(b, rp, mode, ring);
    } else if (wave == 1) {
        __builtin_amdgcn_s_setprio(2);
        feed_records<kWide>(b, mode, lm, ring, lane);
    } else if (wave == 2) {
        __builtin_amdgcn_s_setprio(2);
        if constexpr (kWide == 16) drain_steps16(b, rp, mode, ring, lane);
    }
}

template <int kWide>
__device__ __forceinline__ void chain_workgroup(const BatchDev& b, const RailParams& rp, int mode, Ring<kWide>& ring, LevelModel& lm)
{
    if (threadIdx.x == 0) start_ring(ring);
    build_level_model<kWide>(lm, b, rp, mode);                       // (with barriers)
    chain_waves<kWide>(b, rp, mode, ring, lm);
}

template <int kWide>
__global__ void __launch_bounds__(kChainThreads, 2) bind_chain_kernel(BatchDev b, RailParams rp, int mode)
{
    __shared__ Ring<kWide> ring;
    __shared__ LevelModel lm;
    chain_workgroup<kWide>(b, rp, mode, ring, lm);
}

// The chain is one wavefront; the tile tables of the copy kernels depend on the slice table only, not
// on the binding.  On a first plan both go into one launch: workgroup 0 walks the chain, the others
// build the tables, so the tables cost no time of their own.
template <int kWide>
__global__ void __launch_bounds__(256, 2) bind_chain_tables_kernel(BatchDev b, RailParams rp, int mode)
{
    __shared__ Ring<kWide> ring;
    __shared__ LevelModel lm;
    if (blockIdx.x == 0) {
        chain_workgroup<kWide>(b, rp, mode, ring, lm);
        return;
    }
    build_tile_tables_in(b, blockIdx.x - 1, gridDim.x - 1);
}

// ---- step 3: emit -----------------------------------------------------------------------------
// One lane per position q of the pending sequence; inside its run the lane enumerates slot
// t = q - run_start as (rail d, index k) in rail-major order and computes the slot's rank.
// A small plan is bound by the loads of a lane's row one after the other, a large one by the instructions of the counts: the row is
// read kCells rails at a time, the counts come from the checked estimate.  MI355X, against one rail at a time and the closed form:
// 1,000,000 slices on 16 rails 71 -> 45 us, 20,000 on 9 rails 11.5 -> 8.4.  A report's 2 KB take about 3 us to reach the host and
// are told by a workgroup of their own.
struct EmitRails {
    uint64_t c0[TENT_MAX_RAILS];
    uint64_t A[TENT_MAX_RAILS];
    double inv[TENT_MAX_RAILS];
    uint32_t c1[TENT_MAX_RAILS];
    uint64_t admitted;
};
constexpr uint32_t kCells = 4;             // rails of a row read at a time (rows are 16, 32 or 64 long)

// By a whole workgroup (with a barrier), thread `at` of `threads`.
__device__ __forceinline__ void bind_emit(const BatchDev& b, const RailParams& rp, int use_pending, EmitRails& er,
                                          uint64_t at, uint64_t threads)
{
    const uint32_t R = rp.n_rails;
    if (threadIdx.x < TENT_MAX_RAILS) {
        const uint32_t c1 = (uint32_t)rp.c1[threadIdx.x];
        er.c0[threadIdx.x] = rp.c0[threadIdx.x];
        er.A[threadIdx.x] = rp.A[threadIdx.x];
        er.c1[threadIdx.x] = c1 ? c1 : 1u;
        er.inv[threadIdx.x] = 1.0 / (double)(c1 ? c1 : 1u);
        if (threadIdx.x == 0) er.admitted = rp.admitted;
    }
    __syncthreads();
    const uint64_t n = b.plan->n_pending;
    const uint32_t stride = b.run_stride;
    for (uint64_t q = at; q < n; q += threads) {
        const uint32_t id_q = use_pending ? b.pending[q] : (uint32_t)q;
        const uint64_t r = b.s_run[q];
        const uint32_t start = b.run_start[r];
        const RunCell* row = b.run_cell + r * stride;
        if (b.run_start[r + 1] - start == 1) {
            // a single slice: its rail stands in the row of the longer run it was bound with, or in its own
            const bool joined = r > 0 && start - b.run_start[r - 1] > 1;
            const RunCell* own = joined ? row - stride : row;
            const uint32_t d = own->tail & 63u;
            uint64_t off = (uint64_t)own[d].T;
            if (joined) {
                const uint32_t before = b.run_start[r - 1];
                off += (uint64_t)own[d].K * b.s_len[use_pending ? b.pending[before] : before];
            }
            b.s_rail[id_q] = d;
            b.s_stage_off[id_q] = off;
            b.s_state[id_q] = TENT_SLICE_BOUND;
            continue;
        }
        const uint32_t l = b.s_len[id_q];
        const double inv_l = 1.0 / (double)l;
        // slot t -> (d, k)
        const uint32_t t = (uint32_t)(q - start);
        uint32_t d = R, k = 0, before = 0;
        for (uint32_t o0 = 0; o0 < R; o0 += kCells) {
            uint32_t K[kCells];
#pragma unroll
            for (uint32_t e = 0; e < kCells; ++e) K[e] = row[o0 + e].K;
#pragma unroll
            for (uint32_t e = 0; e < kCells; ++e) {
                const uint32_t ko = ((er.admitted >> (o0 + e)) & 1) ? K[e] : 0;
                const bool here = t - before < ko;                   // (t - before wraps behind the slot: never below ko then)
                d = here ? o0 + e : d;
                k = here ? t - before : k;
                before += ko;
            }
        }
        if (d >= R) continue;
        const uint64_t T_d = (uint64_t)row[d].T;
        const uint64_t f = slot_cost(Rail{er.c0[d], er.c1[d], er.inv[d]}, er.A[d] + T_d, l, k);
        uint64_t rank = k;
        for (uint32_t o0 = 0; o0 < R; o0 += kCells) {
            RunCell cell[kCells];
#pragma unroll
            for (uint32_t e = 0; e < kCells; ++e) cell[e] = row[o0 + e];
#pragma unroll
            for (uint32_t e = 0; e < kCells; ++e) {
                const uint32_t o = o0 + e;
                if (o == d || cell[e].K == 0 || !((er.admitted >> o) & 1)) continue;
                // slots of a lower rail win ties, slots of a higher rail lose them
                rank += slots_upto_fast(Rail{er.c0[o], er.c1[o], er.inv[o]}, er.A[o] + (uint64_t)cell[e].T, l, inv_l,
                                        o < d ? (int64_t)f : (int64_t)f - 1, cell[e].K);
            }
        }
        const uint64_t pos = (uint64_t)start + rank;
        const uint32_t id = use_pending ? b.pending[pos] : (uint32_t)pos;
        b.s_rail[id] = d;
        b.s_stage_off[id] = T_d + (uint64_t)k * l;
        b.s_state[id] = TENT_SLICE_BOUND;
    }
}

__global__ void __launch_bounds__(256) bind_emit_kernel(BatchDev b, RailParams rp, int use_pending, Report told)
{
    __shared__ EmitRails er;
    const uint32_t blocks = told.to ? gridDim.x - 1 : gridDim.x;
    if (blockIdx.x == blocks) {                                      // one more for the report
        if (threadIdx.x < 64) tell_totals(*b.plan, told);
        return;
    }
    bind_emit(b, rp, use_pending, er, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, (uint64_t)blocks * blockDim.x);
}

// ---- a small batch's first plan in one workgroup ----------------------------------------------------
// Prefixes, slice table, run table, chain, tile tables and emit one after the other with barriers in between, the tile
// tables beside the chain as in the large form.  What bounds a small plan is launches, not work: 64 transfers, 626 extents,
// 182 slices took five launches and 44 us of device time in a graph and take one of 32 us.
constexpr uint32_t kSmallThreads = 1024;
constexpr uint32_t kSmallExtents = 2048;         // per side; two per thread
constexpr uint32_t kSmallDescs = 2048;           // two per thread
constexpr uint32_t kSmallSlices = 2048;
constexpr uint32_t kFrontExtents = 4096;         // per side; four per thread
constexpr uint32_t kFrontSlices = 3072;          // three per thread; two beside four extents
constexpr uint64_t kSmallTiles = 16384;          // 20 per thread that the chain, its feeder and its drainer leave over

// What the front part of a plan keeps in LDS: extent prefixes of both sides, first slice and runs before every transfer.
template <int kItems>
struct FrontTables {
    uint64_t src_pre[kSmallThreads * kItems + 1], dst_pre[kSmallThreads * kItems + 1];
    uint32_t first[kSmallDescs + 1], runs_before[kSmallDescs + 1];
    uint64_t wave_out[kSmallThreads / 64];
};

template <int kWide>
struct SmallPlan {
    FrontTables<2> front;
    union {
        Ring<kWide> ring;
        EmitRails er;
    };
    LevelModel lm;
};

// Exclusive prefix of a thread's value over the workgroup.
__device__ __forceinline__ uint64_t thread_prefix(uint64_t v, uint64_t* wave_out)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t inc = wave_inclusive_scan(v);
    __syncthreads();
    if (lane == 63) wave_out[wave] = inc;
    __syncthreads();
    uint64_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before += wave_out[w];
    return before + inc - v;
}

// Prefixes, slice table and run table by one workgroup of kSmallThreads, with barriers; kItems extents a side and two transfers per
// thread.  A barrier follows before anyone else reads what it leaves.
template <int kItems>
__device__ __forceinline__ void plan_front(const BatchDev& b, FrontTables<kItems>& sh)
{
    const uint32_t t = threadIdx.x, base = kItems * t;
    const uint32_t ns = (uint32_t)b.n_src_ext, nd = (uint32_t)b.n_dst_ext, D = b.n_desc, N = (uint32_t)b.n_slices;
    const SliceDiv div(b.slice_bytes);
    {   // extent prefixes of both sides, and in address order where a table goes by it
        uint64_t s[kItems], d[kItems], o[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint32_t e = base + k;
            s[k] = e < ns ? b.src_ext[e].len : 0;
            d[k] = e < nd ? b.dst_ext[e].len : 0;
            o[k] = b.ord_pre && e < nd ? b.dst_order[e] : 0;
        }
        if (b.ord_pre) {
#pragma unroll
            for (int k = 0; k < kItems; ++k) o[k] = base + k < nd ? b.dst_ext[o[k]].len : 0;
        }
        auto put = [&](uint64_t* out, uint64_t* in_lds, uint32_t n, const uint64_t (&v)[kItems]) {
            uint64_t sum = 0;
#pragma unroll
            for (int k = 0; k < kItems; ++k) sum += v[k];
            uint64_t at = thread_prefix(sum, sh.wave_out);
#pragma unroll
            for (int k = 0; k <= kItems; ++k) {
                const uint32_t e = base + k;
                if (k == kItems && e != n) break;                    // (entry n otherwise comes from the thread behind)
                if (e <= n) {
                    out[e] = at;
                    if (in_lds) in_lds[e] = at;
                }
                if (k < kItems) at += v[k];
            }
        };
        put(b.src_pre, sh.src_pre, ns, s);
        put(b.dst_pre, sh.dst_pre, nd, d);
        if (b.ord_pre) put(b.ord_pre, nullptr, nd, o);
    }
    __syncthreads();
    {   // first slice and runs before every transfer
        const uint32_t e0 = 2 * t, e1 = 2 * t + 1;
        const TransferCounts counts{b.src_ptr, sh.src_pre, div};
        const uint64_t c0 = e0 < D ? counts(e0) : 0, c1 = e1 < D ? counts(e1) : 0;
        const uint64_t at = thread_prefix(c0 + c1, sh.wave_out);
        auto one = [&](uint32_t j, uint64_t v) {
            if (j > D) return;
            b.first[j] = v & 0xFFFFFFFFu;
            b.runs_before[j] = (uint32_t)(v >> 32);
            sh.first[j] = (uint32_t)v;
            sh.runs_before[j] = (uint32_t)(v >> 32);
        };
        one(e0, at);
        one(e1, at + c0);
        if (e1 + 1 == D) one(D, at + c0 + c1);
    }
    __syncthreads();
    for (uint32_t i = t; i < N; i += kSmallThreads) {
        uint32_t lo = 0, hi = D;                                      // last transfer that starts at or before slice i
        while (hi - lo > 1) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if (sh.first[mid] <= i) lo = mid; else hi = mid;
        }
        write_slice(b, div, i, lo, sh.first[lo], sh.runs_before[lo], sh.src_pre, sh.dst_pre);
    }
    if (t == 0) {
        const uint32_t n_runs = sh.runs_before[D];
        b.run_start[n_runs] = N;
        b.plan->n_runs = n_runs;
        b.plan->n_pending = N;
    }
}

// The front part alone, for batches whose tile tables or slices are too many for one workgroup: in place of three to five launches in
// a row (extent prefixes, counts, slices).  MI355X: a recorded cycle of 2,427 extents a side and 615 slices 134 -> 129.5 us, a life of
// 2,768 and 768 155 -> 149, cycles in turn of 3,347 and 261 65 -> 56; with eight extents a thread, cycles of 4,224 and 2,112 take
// 144 us against 137.  A slice costs one thread what it costs a thread of a whole launch, so beyond a few per thread the launches win again:
// recorded cycles of 3,000 extents and 3,480 slices 89.8 us against 87.4, of 3,860 and 2,868 88.8 against 87.6; cycles on their own of
// 2,048 and 2,608 191 against 199, of 1,792 and 3,584 175 against 180 and in turn 163.2 against 162.3.
template <int kItems>
__global__ void __launch_bounds__(kSmallThreads) plan_front_kernel(BatchDev b)
{
    __shared__ FrontTables<kItems> sh;
    plan_front(b, sh);
}

template <int kWide>
__global__ void __launch_bounds__(kSmallThreads) plan_small_kernel(BatchDev b, RailParams rp, Report told)
{
    __shared__ SmallPlan<kWide> sh;
    const uint32_t t = threadIdx.x;
    plan_front(b, sh.front);
    if (t == 0) start_ring(sh.ring);
    __syncthreads();
    build_level_model<kWide>(sh.lm, b, rp, kBindBuildTables);
    if (t < kChainThreads) chain_waves<kWide>(b, rp, kBindBuildTables, sh.ring, sh.lm);
    else build_tile_tables(b, t - kChainThreads, kSmallThreads - kChainThreads);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    bind_emit(b, rp, 0, sh.er, t, kSmallThreads);
    if (told.to && t >= kSmallThreads - 64) tell_totals(*b.plan, told);       // the wavefront with the fewest slices to emit
}

}  // namespace

bool plan_is_small(const BatchDev& b)
{
    return b.n_src_ext <= kSmallExtents && b.n_dst_ext <= kSmallExtents && b.n_slices <= kSmallSlices &&
           b.n_slices * (uint64_t)b.tiles_per_slice <= kSmallTiles;
}

bool plan_front_fits(const BatchDev& b)
{
    const uint64_t most = b.n_src_ext > b.n_dst_ext ? b.n_src_ext : b.n_dst_ext;
    return most <= kFrontExtents && b.n_desc <= kSmallDescs && b.n_slices <= (most <= kSmallExtents ? kFrontSlices : kSmallSlices);
}

hipError_t launch_plan_front(const BatchDev& b, hipStream_t s)
{
    const uint64_t most = b.n_src_ext > b.n_dst_ext ? b.n_src_ext : b.n_dst_ext;
    if (most <= 2 * kSmallThreads) hipLaunchKernelGGL(plan_front_kernel<2>, dim3(1), dim3(kSmallThreads), 0, s, b);
    else                           hipLaunchKernelGGL(plan_front_kernel<4>, dim3(1), dim3(kSmallThreads), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_plan_small(const BatchDev& b, const RailParams& rp, Report told, hipStream_t s)
{
    const dim3 grid(1), block(kSmallThreads);
    if (rp.n_rails <= 16)      hipLaunchKernelGGL(plan_small_kernel<16>, grid, block, 0, s, b, rp, told);
    else if (rp.n_rails <= 32) hipLaunchKernelGGL(plan_small_kernel<32>, grid, block, 0, s, b, rp, told);
    else                       hipLaunchKernelGGL(plan_small_kernel<64>, grid, block, 0, s, b, rp, told);
    return hipGetLastError();
}

hipError_t launch_bind_runs(const BatchDev& b, const RailParams& rp, int mode, Report told, hipStream_t s)
{
    const bool use_pending = (mode & kBindUsePending) != 0;
    const int up = use_pending ? 1 : 0;
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    auto launch_chain = [&](auto wide) {
        constexpr int kW = decltype(wide)::value;
        if (mode & kBindBuildTables)
            hipLaunchKernelGGL(bind_chain_tables_kernel<kW>, dim3(1 + tile_table_blocks(b)), dim3(256), 0, s, b, rp, mode);
        else
            hipLaunchKernelGGL(bind_chain_kernel<kW>, dim3(1), dim3(kChainThreads), 0, s, b, rp, mode);
    };
    if (rp.n_rails <= 16)      launch_chain(std::integral_constant<int, 16>{});
    else if (rp.n_rails <= 32) launch_chain(std::integral_constant<int, 32>{});
    else                       launch_chain(std::integral_constant<int, 64>{});
    hipLaunchKernelGGL(bind_emit_kernel, dim3((uint32_t)blocks + (told.to ? 1u : 0u)), dim3(256), 0, s, b, rp, up, told);
    return hipGetLastError();
}

}  // namespace tent
