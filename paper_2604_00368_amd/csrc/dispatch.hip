// Request-level dispatch (Algorithm 1 of the paper, Stages 1-3; Section 4.2 "Slice Dispatching" and
// "Quality of Service").  The algorithm runs once per request -- here per declared transfer, in
// declaration order:
//   Stage 1  admitted rails = non-excluded rails whose priority slot accepts the request
//            (the host passes one mask per priority level for the current window);
//   Stage 2  s_d = c0_d + (((A_d + L) * c1_d) >> 16) with the queue state at the start of the request;
//   Stage 3  mice (request shorter than theta): the whole request goes to one rail, picked round robin
//            among the admitted rails with s_d <= s_min + floor(gamma * s_min / 256);
//            elephants: weighted proportional spraying with weights 1 / s_d -- the request's pending
//            slices are dealt in order, each to the rail with the smallest (m_d + 1) * s_d (m_d = slices
//            of the request already on d, ties to the lowest rail).
//
// Requests depend on each other through A_d, so the per-request decisions form a chain: one
// wavefront, lane d = rail d.  Inside an elephant request nothing depends on A_d any more: dealing by
// smallest (m_d + 1) * s_d is the merge of the rails' arithmetic sequences s_d, 2 s_d, 3 s_d, ..., so the
// chain only needs the number of slots K_d each rail takes among the first n merged elements (a
// floating-point estimate of the cut level, repaired with exact integer comparisons), and a second,
// fully parallel kernel gives every slot its rank in the merge in closed form (R integer divisions).
#include <type_traits>

#include "scan.h"
#include "tile_tables.h"
#include "wave.h"

namespace tent {
namespace {

constexpr uint64_t kNoKey = ~0ull;

__device__ __forceinline__ uint32_t priority_of(const BatchDev& b, const DispatchParams& dp, const PriorityBits& bits, uint32_t j)
{
    return dp.all_high ? 2u : dp.by_bits ? (bits.word[j / 16] >> (2 * (j % 16))) & 3u : b.priority[j];
}

// ---- the chain over requests -------------------------------------------------------------------
// kWide = 16, 32 or 64: smallest of these that covers the rails; lanes beyond the rails only tag along
// (uniform decisions are read from lane 0's row).
// Runs in the first wavefront of a workgroup (lane = threadIdx.x < 64).
template <int kWide>
__device__ __forceinline__ void dispatch_chain(const BatchDev& b, const RailParams& rp, const DispatchParams& dp, const PriorityBits& bits)
{
    const int lane = threadIdx.x;
    const uint64_t S = b.slice_bytes;
    const uint32_t D = b.n_desc;
    const uint32_t stride = b.run_stride;
    const uint64_t c0 = rp.c0[lane];
    const uint64_t c1 = rp.c1[lane];
    uint64_t A = rp.A[lane], T = 0, cnt = 0;
    uint64_t rr = dp.rr_start, n_mice = 0, n_elephant = 0, n_deferred = 0, n_bound = 0, n_pending = 0;
    const uint64_t lanes_below = (1ull << lane) - 1;

    for (uint32_t blk = 0; blk < D; blk += 64) {
        // lane t fetches the description of request blk + t
        const uint32_t jl = blk + lane;
        uint32_t my_n = 0, my_short = 0, my_prio = 2;
        uint64_t my_len = 0;
        if (jl < D) {
            const uint64_t f0 = b.first[jl], f1 = b.first[jl + 1];
            my_n = (uint32_t)(dp.all_pending ? f1 - f0 : b.scan_tmp[f1] - b.scan_tmp[f0]);       // slices of the request not DONE
            my_len = b.src_pre[b.src_ptr[jl + 1]] - b.src_pre[b.src_ptr[jl]];
            const uint64_t last_len = my_len - (f1 - f0 - 1) * S;
            if (b.s_state[f1 - 1] != TENT_SLICE_DONE) my_short = (uint32_t)(S - last_len);
            my_prio = priority_of(b, dp, bits, jl);
        }
        const int m = (int)(D - blk < 64 ? D - blk : 64);
        uint32_t my_mode = 0;
        for (int t = 0; t < m; ++t) {
            const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)my_n, t);
            if (n == 0) continue;
            n_pending += n;
            const uint32_t prio = (uint32_t)__builtin_amdgcn_readlane((int)my_prio, t);
            const uint64_t adm = dp.adm[prio > 2 ? 2 : prio];
            if (adm == 0) {                                                  // Stage 1: nothing admitted
                if (lane == t) my_mode = 3;
                ++n_deferred;
                continue;
            }
            const uint64_t L_req = read_lane64(my_len, t);
            const uint32_t short_by = (uint32_t)__builtin_amdgcn_readlane((int)my_short, t);
            const bool live = (adm >> lane) & 1;
            const bool mice = L_req < dp.theta;
            const uint64_t L = mice ? L_req : (L_req < S ? L_req : S);
            uint64_t s = c0 + (((A + L) * c1) >> 16);                        // Stage 2
            uint64_t K = 0, bytes = 0;
            if (mice) {
                const uint64_t s_min = wave_reduce64(live ? s : kNoKey, kWide, OpMin{});
                const uint64_t limit = s_min + ((s_min * dp.gamma_q8) >> 8);
                const uint64_t cand = __ballot(live && s <= limit);
                const uint32_t idx = (uint32_t)(rr % (uint64_t)__popcll(cand));
                ++rr;
                const bool me = ((cand >> lane) & 1) && (uint32_t)__popcll(cand & lanes_below) == idx;
                if (me) { K = n; bytes = (uint64_t)n * S - short_by; }
                if (lane == t) my_mode = 1;
                ++n_mice;
            } else {
                if (s == 0) s = 1;
                // cut level of the merge: x with sum_d floor(x / s_d) ~ n
                const double inv = live ? 1.0 / (double)s : 0.0;
                const double sum_inv = wave_sum_f64(inv, kWide);
                const double n_live = (double)__popcll(adm);
                const double x = ((double)n + 0.5 * n_live) / sum_inv;
                if (live) {
                    const double kf = x * inv;
                    K = kf >= (double)n ? n : (uint64_t)kf;
                }
                uint64_t total = uniform64(wave_reduce64(K, kWide, OpAdd{}));
                // exact repair: grow by the cheapest free slot / shrink by the dearest held slot
#pragma clang loop unroll(disable)
                while (total < n) {
                    const int win = argmin_cost((K + 1) * s, live, lane, kWide);
                    if (lane == win) ++K;
                    ++total;
                }
#pragma clang loop unroll(disable)
                while (total > n) {
                    const int win = argmax_cost(K * s, live && K, lane, kWide);
                    if (lane == win) --K;
                    --total;
                }
                // the held slots must be exactly the first n of the merge: the dearest held slot
                // (ties: highest rail last) precedes the cheapest free slot (ties: lowest rail first)
                int last = 0;
#pragma clang loop unroll(disable)
                for (int guard = 0; guard < 4096; ++guard) {
                    last = argmax_cost(K * s, live && K, lane, kWide);
                    const int next = argmin_cost((K + 1) * s, live, lane, kWide);
                    const uint64_t held = read_lane64(K * s, last);
                    const uint64_t free_ = read_lane64((K + 1) * s, next);
                    if (held < free_ || (held == free_ && last < next)) break;
                    if (lane == last) --K;
                    if (lane == next) ++K;
                }
                // the request's last pending slice is the last element of the merge
                bytes = K * S - (lane == last ? short_by : 0);
                if (lane == t) my_mode = 2;
                ++n_elephant;
            }
            if (lane < (int)stride) {
                const uint64_t row = (uint64_t)(blk + t) * stride + lane;
                b.run_cell[row] = RunCell{(double)T, (uint32_t)K, 0u};
            }
            A += bytes;
            T += bytes;
            cnt += K;
            n_bound += n;
        }
        if (jl < D) b.req_mode[jl] = (uint8_t)my_mode;
    }

    const uint64_t rounded = (T + 255) & ~255ull;
    uint64_t inc = rounded;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t up = (uint64_t)__shfl_up((unsigned long long)inc, d, 64);
        if (lane >= d) inc += up;
    }
    PlanState* ps = b.plan;
    ps->T[lane] = T;
    ps->cnt[lane] = cnt;
    ps->A_after[lane] = A;
    ps->base[lane] = inc - rounded;
    if (lane == 0) {
        ps->n_bound = n_bound;
        ps->n_pending = n_pending;
        ps->n_mice = n_mice;
        ps->n_elephant = n_elephant;
        ps->n_deferred = n_deferred;
        ps->rr_next = rr;
    }
}

// ---- the chain of up to 16 rails ---------------------------------------------------------------
// The same decisions where every cost fits what is computed with here (dispatch_is_near).  What bounds it is one wavefront's
// instruction latency, about 5 clocks an instruction whatever its kind and 40 for a branch on a fresh comparison, so:
//   - costs are doubles that hold whole numbers; a slot's key is its cost times 16 plus its rail, below 2^53, so one
//     comparison settles cost and tie;
//   - the cut level comes from 32-bit reciprocals: any level will do, because the slots a rail takes are those that cost no
//     more than it, which is checked with the exact products.  What costs no more than a level is the beginning of the merge,
//     and stays so with every slot that is added cheapest first or dropped dearest first: no exchange of slots is needed;
//   - the guess is meant to be half a slot low.  Where nothing or one slot is missing (three requests in four), the reduction that
//     names the dearest slot taken or the cheapest free one is the only one, and only the check of all that is a branch;
//   - a second wavefront looks up the requests a block of 64 ahead, and sums up the rails' bytes and writes the rows a block
//     behind; they meet at a barrier per block.
// All four rows of the wavefront hold the same state (lane % 16 = rail).
// MI355X, chain and emit, against the chain above: 1,110 requests on three rails 815 -> 343 us, 512 on nine with priorities 431 -> 201, all
// HIGH 431 -> 300 (eight of the nine move in step, so that more slots are missing or too many at a time), 64 on three 59 -> 41.
typedef uint32_t Quad __attribute__((ext_vector_type(4)));
struct Request {
    Quad a;                                // slices not DONE (0: nothing to do) with kMice, bytes that the last of them is shorter than a
                                           // slice, and what Stage 2 counts: the request for mice, at most a slice for elephants
    Quad b;                                // rails whose slot takes the request; elephants: the slots the cut level is for, as a float;
                                           // mice: the round-robin counter modulo kTurns
};
constexpr uint32_t kMice = 1u << 31;
constexpr uint32_t kRequests = 64;         // of a block
constexpr uint32_t kTurns = 720720;        // a multiple of every number up to 16
constexpr uint32_t kLast = 1u << 28;       // found: slots of the rail, and whether it takes the request's last one
constexpr double kNoRail = 1125899906842624.0;   // 2^50: more than any cost, for rails that do not take the request

struct RequestRing {
    Request req[2][kRequests];
    uint32_t found[2][kRequests][16];
    uint64_t n_pending, n_deferred, n_mice, n_elephant, n_bound;
};

// Requests [64 blk, 64 blk + 64), one per lane.
__device__ __forceinline__ void feed_requests(const BatchDev& b, const DispatchParams& dp, const PriorityBits& bits, RequestRing& ring, uint32_t blk, uint32_t lane)
{
    const uint32_t j = blk * kRequests + lane;
    uint32_t mode = 0, pending = 0, admitted = 0, short_by = 0;
    uint64_t len = 0;
    bool mice = false;
    if (j < b.n_desc) {
        const uint64_t f0 = b.first[j], f1 = b.first[j + 1];
        len = b.src_pre[b.src_ptr[j + 1]] - b.src_pre[b.src_ptr[j]];
        const uint32_t prio = priority_of(b, dp, bits, j);
        pending = (uint32_t)(dp.all_pending ? f1 - f0 : b.scan_tmp[f1] - b.scan_tmp[f0]);
        admitted = (uint32_t)dp.adm[prio > 2 ? 2 : prio] & 0xFFFFu;
        mice = len < dp.theta;
        if (b.s_state[f1 - 1] != TENT_SLICE_DONE) short_by = (uint32_t)(b.slice_bytes - (len - (f1 - f0 - 1) * b.slice_bytes));
        if (!mice && len > b.slice_bytes) len = b.slice_bytes;
        mode = pending == 0 ? 0u : admitted == 0 ? 3u : mice ? 1u : 2u;
        b.req_mode[j] = (uint8_t)mode;
    }
    const uint64_t mice_mask = __ballot(mode == 1);
    const uint32_t n = mode == 1 || mode == 2 ? pending : 0;
    const uint64_t turn = (dp.rr_start + ring.n_mice + (uint64_t)__popcll(mice_mask & ((1ull << lane) - 1))) % kTurns;
    // half a slot per rail, because the counts are rounded down, less the half that the guess is meant to be low by
    const float want = (float)n + 0.5f * ((float)__popc(admitted) - 1.0f);
    ring.req[blk & 1][lane].a = Quad{n | (mode == 1 ? kMice : 0u), short_by, (uint32_t)len, (uint32_t)(len >> 32)};
    ring.req[blk & 1][lane].b = Quad{admitted, mode == 1 ? (uint32_t)turn : __float_as_uint(want), 0u, 0u};
    const uint64_t all = wave_reduce64(pending, 64, OpAdd{}), bound = wave_reduce64(n, 64, OpAdd{});
    const uint64_t elephant = __popcll(__ballot(mode == 2)), deferred = __popcll(__ballot(mode == 3));
    if (lane != 0) return;
    ring.n_pending += all;
    ring.n_bound += bound;
    ring.n_mice += __popcll(mice_mask);
    ring.n_elephant += elephant;
    ring.n_deferred += deferred;
}

__device__ __forceinline__ double row_max_f64(double x)
{
    auto step = [](double v, uint64_t other) {
        double r;
        asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(v), "v"(__longlong_as_double((long long)other)));
        return r;
    };
    x = step(x, dpp64<0xB1>((uint64_t)__double_as_longlong(x)));
    x = step(x, dpp64<0x4E>((uint64_t)__double_as_longlong(x)));
    x = step(x, dpp64<0x141>((uint64_t)__double_as_longlong(x)));
    return step(x, dpp64<0x140>((uint64_t)__double_as_longlong(x)));
}
__device__ __forceinline__ float row_sum_f32(float x)
{
    x += __uint_as_float(dpp32<0xB1>(__float_as_uint(x)));
    x += __uint_as_float(dpp32<0x4E>(__float_as_uint(x)));
    x += __uint_as_float(dpp32<0x141>(__float_as_uint(x)));
    return x + __uint_as_float(dpp32<0x140>(__float_as_uint(x)));
}
// a whole number below 2^52 as a double, and back
__device__ __forceinline__ double whole_f64(uint64_t v)
{
    return __longlong_as_double((long long)(v | 0x4330000000000000ull)) - 4503599627370496.0;
}
__device__ __forceinline__ uint64_t f64_whole(double x)
{
    return (uint64_t)__double_as_longlong(x + 4503599627370496.0) & 0xFFFFFFFFFFFFFull;
}

// One request's slots by adding and dropping one at a time, from a guess.  Out of the loop's way: one request in four.
struct Slots {
    uint32_t K;
    bool last;
};
__device__ __attribute__((noinline)) Slots settle_slots(uint32_t K, uint32_t n, double cost, double level, double rail)
{
    K += (double)(K + 1) * cost <= level ? 1u : 0u;              // (off by one at most, see walk_requests)
    K -= (double)K * cost > level ? 1u : 0u;
    int miss = __builtin_amdgcn_readfirstlane((int)(n - wave_reduce32(K, 16, Add32{})));
    if (miss > 0) {
        double key = fma((double)(K + 1) * cost, -16.0, -rail);
        bool won;
        do {                                                     // the cheapest free slot
            won = key == row_max_f64(key);
            K += won ? 1u : 0u;
            key -= won ? cost * 16.0 : 0.0;
        } while (--miss > 0);
        return Slots{K, won};
    }
    double key = fma((double)K * cost, 16.0, rail);              // (a rail without slots: its number)
    for (;; ++miss) {                                            // the dearest slot taken: the request's last one, or one too many
        const bool won = key == row_max_f64(key);
        if (miss == 0) return Slots{K, won};
        K -= won ? 1u : 0u;
        key -= won ? cost * 16.0 : 0.0;
    }
}

// The block's requests; Q: cost of the rail's next byte in units of 2^-16 ps, (c0 << 16) + A c1, below 2^63.
__device__ __forceinline__ void walk_requests(const BatchDev& b, const DispatchParams& dp, uint32_t c1, RequestRing& ring, uint32_t blk,
                                              uint64_t& Q)
{
    const uint32_t who = threadIdx.x & 15u;
    const uint64_t Sc1 = b.slice_bytes * c1;
    const double rail = (double)who;
    const Request* req = ring.req[blk & 1];
    uint32_t* found = &ring.found[blk & 1][0][who];
    const uint32_t m = b.n_desc - blk * kRequests < kRequests ? b.n_desc - blk * kRequests : kRequests;
    Quad ra = req[0].a, rb = req[0].b;
    for (uint32_t t = 0; t < m; ++t, found += 16) {
        const Quad a = ra, w = rb;
        const uint32_t head = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.x);
        const uint32_t next_at = t + 1 < m ? t + 1 : t;
        ra = req[next_at].a;
        rb = req[next_at].b;
        if (head == 0) continue;
        const bool live = (w.x >> who) & 1;
        const uint64_t len = ((uint64_t)a.w << 32) | a.z;
        const uint64_t s = (Q + len * c1) >> 16;                             // Stage 2
        const uint64_t short_c1 = (uint64_t)a.y * c1;
        uint32_t K;
        bool last;
        double cost = whole_f64(s & 0xFFFFFFFFFFFFFull);                     // (rails that take nothing may cost anything)
        if (head & kMice) {
            const uint32_t n = head & ~kMice;
            const uint64_t least = uniform64(f64_whole(-row_max_f64(live ? -cost : -kNoRail)));
            const uint32_t cand = (uint32_t)__ballot(live && s <= least + ((least * dp.gamma_q8) >> 8)) & 0xFFFFu;
            const uint32_t n_cand = (uint32_t)__popc(cand);
            // turn % n_cand, whole numbers below 2^24 in floats
            uint32_t idx = w.y - (uint32_t)((float)w.y * __builtin_amdgcn_rcpf((float)n_cand)) * n_cand;
            idx += (int)idx < 0 ? n_cand : 0u;
            idx -= idx >= n_cand ? n_cand : 0u;
            last = ((cand >> who) & 1) && (uint32_t)__popc(cand & ((1u << who) - 1)) == idx;
            K = last ? n : 0;
        } else {
            asm("v_max_f64 %0, %0, 1.0" : "+v"(cost));
            cost = live ? cost : kNoRail;
            const float inv = __builtin_amdgcn_rcpf((float)cost);
            const float level_f = __uint_as_float(w.y) * __builtin_amdgcn_rcpf(row_sum_f32(inv));
            const double level = (double)level_f;
            K = (uint32_t)(level_f * inv);                                   // off by one at most below 2^20 slots
            const double held = (double)K * cost, next = held + cost;
            const uint32_t miss = head - wave_reduce32(K, 16, Add32{});
            // the cheapest free slot, the dearest taken one otherwise
            const bool add = miss == 1;
            const double held_key = fma(held, 16.0, rail), next_key = fma(next, -16.0, -rail);
            const double key = add ? next_key : held_key;
            const bool guess_off = next <= level || held > level || miss > 1;
            last = key == row_max_f64(key);
            const uint32_t K_guess = K;
            K += add && last ? 1u : 0u;
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(guess_off) != 0, 0)) {
                const Slots r = settle_slots(K_guess, head, cost, level, rail);
                K = r.K;
                last = r.last;
            }
        }
        // the request's last pending slice is the last element of the merge
        Q += (uint64_t)K * Sc1 - (last ? short_c1 : 0);
        *found = K | (last ? kLast : 0u);
    }
}

// T, whole and below 2^53, is exact as a double.
struct RailTotals {
    double T;
    uint64_t cnt;
};
__device__ __forceinline__ void drain_requests(const BatchDev& b, const RequestRing& ring, uint32_t blk, RailTotals& sum, uint32_t lane)
{
    const uint32_t who = lane & 15u;
    const double S = (double)b.slice_bytes;
    const uint32_t m = b.n_desc - blk * kRequests < kRequests ? b.n_desc - blk * kRequests : kRequests;
    RunCell* cell = b.run_cell + (uint64_t)blk * kRequests * b.run_stride + who;
#pragma unroll 4
    for (uint32_t t = 0; t < m; ++t, cell += b.run_stride) {
        const Quad r = ring.req[blk & 1][t].a;
        const uint32_t word = ring.found[blk & 1][t][who];
        if (r.x == 0) continue;
        const uint32_t K = word & (kLast - 1);
        if (lane < 16) *cell = RunCell{sum.T, K, 0u};
        sum.T = fma((double)K, S, sum.T) - (double)(word & kLast ? r.y : 0u);
        sum.cnt += K;
    }
}

// By a whole workgroup of at least kChainThreads16, with barriers: the first wavefront walks, the second feeds and drains.
constexpr uint32_t kChainThreads16 = 128;
__device__ __forceinline__ void dispatch_chain16(const BatchDev& b, const RailParams& rp, const DispatchParams& dp, const PriorityBits& bits,
                                                 RequestRing& ring)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, who = lane & 15u;
    const uint32_t blocks = (b.n_desc + kRequests - 1) / kRequests;
    if (threadIdx.x == 0) ring.n_pending = ring.n_deferred = ring.n_mice = ring.n_elephant = ring.n_bound = 0;
    __syncthreads();
    const uint32_t c1 = (uint32_t)rp.c1[who];
    uint64_t Q = (rp.c0[who] << 16) + rp.A[who] * c1;
    RailTotals sum{0.0, 0};
    if (wave == 0) __builtin_amdgcn_s_setprio(3);
    if (wave == 1) feed_requests(b, dp, bits, ring, 0, lane);
    for (uint32_t k = 0; k < blocks; ++k) {                                  // block k walked, k + 1 fed, k - 1 drained
        __syncthreads();
        if (wave == 0) walk_requests(b, dp, c1, ring, k, Q);
        // (block k - 1 is drained first: its records' place is the next block's)
        if (wave == 1 && k > 0) drain_requests(b, ring, k - 1, sum, lane);
        if (wave == 1 && k + 1 < blocks) feed_requests(b, dp, bits, ring, k + 1, lane);
    }
    __syncthreads();
    if (wave != 1) return;
    drain_requests(b, ring, blocks - 1, sum, lane);
    const uint64_t T = (uint64_t)sum.T, rounded = (T + 255) & ~255ull;
    uint64_t inc = rounded;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const uint64_t up = (uint64_t)__shfl_up((unsigned long long)inc, d, 16);
        if ((int)who >= d) inc += up;
    }
    PlanState* ps = b.plan;
    // (rails from 16 on: none, and behind all others)
    const uint64_t all = (uint64_t)__shfl((unsigned long long)inc, 15, 64);
    ps->T[lane] = lane < 16 ? T : 0;
    ps->cnt[lane] = lane < 16 ? sum.cnt : 0;
    ps->A_after[lane] = rp.A[lane] + (lane < 16 ? T : 0);
    ps->base[lane] = lane < 16 ? inc - rounded : all;
    if (lane != 0) return;
    ps->n_bound = ring.n_bound;
    ps->n_pending = ring.n_pending;
    ps->n_mice = ring.n_mice;
    ps->n_elephant = ring.n_elephant;
    ps->n_deferred = ring.n_deferred;
    ps->rr_next = dp.rr_start + ring.n_mice;
}

// kWide = 0: dispatch_chain16
template <int kWide>
__device__ __forceinline__ void dispatch_workgroup(const BatchDev& b, const RailParams& rp, const DispatchParams& dp, const PriorityBits& bits)
{
    if constexpr (kWide == 0) {
        __shared__ RequestRing ring;
        dispatch_chain16(b, rp, dp, bits, ring);
    } else {
        if (threadIdx.x < 64) dispatch_chain<kWide>(b, rp, dp, bits);
    }
}

template <int kWide>
__global__ void __launch_bounds__(256) dispatch_chain_kernel(BatchDev b, RailParams rp, DispatchParams dp, PriorityBits bits)
{
    dispatch_workgroup<kWide>(b, rp, dp, bits);
}

// First plan of a batch: the tile tables of the copy kernels are built by the other workgroups of the
// chain's launch (they depend on the slice table only).
template <int kWide>
__global__ void __launch_bounds__(256) dispatch_chain_tables_kernel(BatchDev b, RailParams rp, DispatchParams dp, PriorityBits bits)
{
    if (blockIdx.x == 0) {
        dispatch_workgroup<kWide>(b, rp, dp, bits);
        return;
    }
    build_tile_tables_in(b, blockIdx.x - 1, gridDim.x - 1);
}

// ---- emit: one lane per pending position ---------------------------------------------------------
// Position q of the pending list belongs to request j; inside the request the lane takes slot
// number t = q - (first pending position of j) in rail-major order, i.e. slot k of rail d, computes
// the slot's rank in the merge and hands it to the request's rank-th pending slice.
__global__ void __launch_bounds__(256) dispatch_emit_kernel(BatchDev b, RailParams rp, DispatchParams dp, Report told)
{
    const uint32_t blocks = told.to ? gridDim.x - 1 : gridDim.x;
    if (blockIdx.x == blocks) {                                      // one more for the report
        if (threadIdx.x < 64) tell_totals(*b.plan, told);
        return;
    }
    const uint32_t R = rp.n_rails;
    const uint32_t stride = b.run_stride;
    const uint64_t S = b.slice_bytes;
    const uint64_t n = dp.all_pending ? b.n_slices : b.scan_tmp[b.n_slices];         // slices not DONE
    const uint64_t gstride = (uint64_t)blocks * blockDim.x;
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gstride) {
        const uint32_t i_q = dp.all_pending ? (uint32_t)q : b.pending[q];
        const uint32_t j = b.s_desc[i_q];
        const uint32_t mode = b.req_mode[j];
        if (mode != 1 && mode != 2) continue;                        // deferred
        const uint64_t q0 = dp.all_pending ? b.first[j] : b.scan_tmp[b.first[j]];    // first pending position of the request
        const uint64_t row = (uint64_t)j * stride;
        uint32_t t = (uint32_t)(q - q0), d = 0;
        for (; d < R; ++d) {
            const uint32_t kd = b.run_cell[row + d].K;
            if (t < kd) break;
            t -= kd;
        }
        if (d >= R) continue;
        const uint32_t k = t;
        uint64_t rank = k;
        if (mode == 2) {
            const uint64_t req_len = b.src_pre[b.src_ptr[j + 1]] - b.src_pre[b.src_ptr[j]];
            const uint64_t L = req_len < S ? req_len : S;
            uint64_t s_d = rp.c0[d] + (((rp.A[d] + (uint64_t)b.run_cell[row + d].T + L) * rp.c1[d]) >> 16);
            if (s_d == 0) s_d = 1;
            const uint64_t key = (uint64_t)(k + 1) * s_d;
            for (uint32_t o = 0; o < R; ++o) {
                const uint32_t ko = b.run_cell[row + o].K;
                if (o == d || ko == 0) continue;
                uint64_t s_o = rp.c0[o] + (((rp.A[o] + (uint64_t)b.run_cell[row + o].T + L) * rp.c1[o]) >> 16);
                if (s_o == 0) s_o = 1;
                // slots of a lower rail win ties, slots of a higher rail lose them
                const uint64_t before = (o < d ? key : key - 1) / s_o;
                rank += before < ko ? before : ko;
            }
        }
        const uint32_t id = dp.all_pending ? (uint32_t)(q0 + rank) : b.pending[q0 + rank];
        b.s_rail[id] = d;
        b.s_stage_off[id] = (uint64_t)b.run_cell[row + d].T + (uint64_t)k * S;
        b.s_state[id] = TENT_SLICE_BOUND;
    }
}

struct NotDone {
    const uint8_t* state;
    __device__ uint64_t operator()(uint64_t i) const { return state[i] != TENT_SLICE_DONE; }
};

__global__ void __launch_bounds__(256) pending_list_kernel(BatchDev b)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b.n_slices; i += stride)
        if (b.s_state[i] != TENT_SLICE_DONE) {
            b.pending[b.scan_tmp[i]] = (uint32_t)i;
            b.s_state[i] = TENT_SLICE_PENDING;                       // a slice bound earlier and never moved is dealt again
        }
}

}  // namespace

hipError_t launch_dispatch(const BatchDev& b, const RailParams& rp, const DispatchParams& dp, const PriorityBits& bits, bool first_plan,
                           Report told, hipStream_t s)
{
    uint64_t blocks = (b.n_slices + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (!first_plan) {
        hipError_t e = exclusive_scan(NotDone{b.s_state}, b.n_slices, b.scan_tmp, b.scan_partials, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(pending_list_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, b);
    }
    auto launch_chain = [&](auto wide) {
        constexpr int kW = decltype(wide)::value;
        if (first_plan)
            hipLaunchKernelGGL(dispatch_chain_tables_kernel<kW>, dim3(1 + tile_table_blocks(b)), dim3(256), 0, s, b, rp, dp, bits);
        else
            hipLaunchKernelGGL(dispatch_chain_kernel<kW>, dim3(1), dim3(kW == 0 ? kChainThreads16 : 64), 0, s, b, rp, dp, bits);
    };
    if (dp.near)               launch_chain(std::integral_constant<int, 0>{});
    else if (rp.n_rails <= 16) launch_chain(std::integral_constant<int, 16>{});
    else if (rp.n_rails <= 32) launch_chain(std::integral_constant<int, 32>{});
    else                       launch_chain(std::integral_constant<int, 64>{});
    hipLaunchKernelGGL(dispatch_emit_kernel, dim3((uint32_t)blocks + (told.to ? 1u : 0u)), dim3(256), 0, s, b, rp, dp, told);
    return hipGetLastError();
}

}  // namespace tent
