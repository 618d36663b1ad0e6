// Host runtime behind the C ABI: argument validation, device tables, rail-state conversion and
// kernel sequencing.  Every step of the hot path itself runs in the HIP kernels of this library.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstring>
#include <mutex>
#include <thread>
#include <new>
#include <utility>
#include <vector>

#include "tent_internal.h"

using namespace tent;

// Static workspace of tent_declare_static: callers that must not allocate get their batch's tables
// here.  One copy per GPU, held until the process ends.  In host code the array's name is only a
// stand-in: its address on a GPU is looked up once, with that GPU current, and host code uses the
// looked-up pointer and nothing else.
//
// The array is 5/16 larger than the limit that a batch is held to (static_measure): the tables of a batch at the
// limit take at most 1.28 times what it is counted with (64 rails: 2,078 against 1,626 bytes per transfer).
constexpr uint64_t kStaticArea = (uint64_t)TENT_STATIC_WORKSPACE_BYTES + TENT_STATIC_WORKSPACE_BYTES / 16 * 5;
static __device__ __align__(256) unsigned char scratch[kStaticArea];

namespace {

struct Segment { uint8_t* base; uint64_t len; };

// A stream on which work of a batch was enqueued, with an event recorded after the latest such work.
struct StreamMark {
    hipStream_t stream = nullptr;
    hipEvent_t event = nullptr;
    bool used = false;
};
constexpr int kMarks = 5;               // four streams of the caller's and the context's own

struct Batch {
    bool alive = false;
    bool planned = false;        // a plan has been enqueued since declare / reset
    bool has_done = false;       // execute ran since declare / reset: DONE slices may exist
    bool has_retry = false;      // a rail failed since declare / reset: slices with a retry count may exist
    bool broken = false;         // an execute failed after its slices were marked DONE: only reset or release help
    uint64_t bound_hint = 0;     // upper bound on the number of BOUND slices, as far as the host knows
    uint64_t tile_hint = ~0ull;  // upper bound on the copy tiles of the BOUND slices, as far as the host knows
    uint32_t generation = 0;
    uint64_t payload = 0;
    uint64_t max_req_slices = 0; // most slices any one transfer has
    uint64_t records = 0;        // transfers that start with a slice of another length than the one before ends with
    uint64_t chain_steps = 0;    // what the last plan's chain went through one by one: such transfers, or all of them (a dispatch)
    RailParams last_rails{};     // telemetry of the last plan (for the rail simulator)
    uint32_t last_lat_ns[TENT_MAX_RAILS] = {};
    // The last execute's bookkeeping (staging addresses, tile lists, DONE marks) ends on exec_stream; its
    // copies, which follow, read none of what a re-plan writes, and end at done_at.
    hipStream_t exec_stream = nullptr;
    hipEvent_t replan_at = nullptr;          // what a re-plan on another stream waits for: prep_event, done_at, or nothing
    bool done_recorded = false;
    hipEvent_t done_at = nullptr;            // the event that ends the last execute: its stream's mark, or done_event
    // A call that has reported something may have returned before its last kernel had quite ended: the mark that ends it, and its
    // stream (which the caller may have destroyed since: it is only compared with).
    hipEvent_t report_at = nullptr;
    hipStream_t report_stream = nullptr;
    // What the batch's tables were last worked on by: nothing yet (or only its declaration), a call on a stream of the caller's, an
    // execute, or a call that ran beside earlier copies (see work_stream).
    enum class Last { kNothing, kCaller, kExecute, kBeside } last = Last::kNothing;
    uint64_t execute_no = 0;                 // which of its stream's executes the last one was
    uint64_t execute_bytes = 0;              // what it moved at most, as far as the host knows
    hipStream_t beside = nullptr;            // the context's stream for such calls
    bool may_replan = false;                 // slices may be left over by the next execute: the simulator or a dispatch ran since the plan
    // The declaration's device work (descriptor upload, address sort, overlap check) runs on the
    // context's own stream and ends at decl_event; `verdict` (pinned host memory) then holds the
    // overlap check's result.
    bool decl_pending = false;
    // Device memory of the tables: an allocation of the batch's own, or the library's static workspace.
    void* block = nullptr;
    uint64_t block_bytes = 0;
    bool in_static = false;
    uint64_t static_generation = 0;
    bool marks_lost = false;     // work was enqueued that no mark covers: waiting for the batch means waiting for the device
    BatchDev dev{};

    // Created once per slot and kept across the batches that use it.
    hipEvent_t prep_event = nullptr, done_event = nullptr, decl_event = nullptr;
    uint32_t* verdict = nullptr;
    StreamMark marks[kMarks];
};

// Event pairs recorded around the launches of one stage since the last tent_get_timings.
struct Timing {
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;   // every pair ever created for the stage
    size_t used = 0;                                        // pairs recorded since the last read-out
};

struct Block { void* ptr; uint64_t bytes; };

// What a stream's work is given: its priority, and the compute units that it may run on, a bit each.
struct StreamTerms {
    static constexpr uint32_t kWords = 16;
    int priority = 0;
    uint32_t cu_mask[kWords] = {};
    bool operator==(const StreamTerms& o) const { return priority == o.priority && std::memcmp(cu_mask, o.cu_mask, sizeof(cu_mask)) == 0; }
};

}  // namespace

struct tent_ctx {
    int device = 0;
    tent_config cfg{};
    uint32_t max_rails = TENT_MAX_RAILS;
    std::vector<Segment> segments;
    uint64_t* seg_base_dev = nullptr;       // device table of segment base addresses
    uint32_t seg_capacity = 0;
    std::vector<Batch> batches;
    Batch static_batch;                     // the one batch whose tables live in the static workspace
    PlanState* host_plan = nullptr;         // pinned result block, written by the kernels of calls that report something
    uint64_t reports = 0;                   // such calls so far: the number a kernel writes behind its figures
    hipStream_t aux_stream = nullptr;       // second stream of the pipelined bounded execute (default priority)
    std::vector<hipEvent_t> sync_events;    // ordering events of the pipelined bounded execute, reused
    // tent_declare: its device work runs on a stream of the library's own, so that it neither waits for
    // nor holds up the caller's streams; host arrays travel through two pinned buffers used in turn.
    hipStream_t decl_stream = nullptr;
    uint8_t* stage[2] = {nullptr, nullptr};
    uint64_t stage_bytes[2] = {0, 0};
    hipEvent_t stage_event[2] = {nullptr, nullptr};
    bool stage_busy[2] = {false, false};
    uint32_t stage_turn = 0;
    hipStream_t beside = nullptr;           // calls that only work on a batch's tables, beside earlier copies (work_stream)
    StreamTerms beside_terms;               // of that stream
    uint32_t cu_words = 0;                  // words that hold a bit per compute unit of the device
    hipEvent_t copies_end = nullptr;        // the event that ends the last execute, and its stream
    hipStream_t copies_stream = nullptr;
    void* order_ws = nullptr;               // workspace of the address sort, grown when a declaration needs more
    uint64_t order_ws_bytes = 0;
    std::vector<Block> spare;               // table allocations of released batches, handed to later declarations
    Timing timing[TENT_T_COUNT];
};

namespace {

constexpr uint32_t kMaxSegments = 4096;
constexpr size_t kMaxTimedIntervals = 1u << 16;   // per stage, between two tent_get_timings calls
constexpr size_t kSpareBlocks = 4;                // released table allocations kept for reuse
constexpr uint64_t kStageInitial = 1ull << 20;    // pinned bytes per staging buffer at tent_create
constexpr uint32_t kStaticSlot = 0xFFFFFFFFu;     // slot field of a handle whose tables live in the static workspace

struct StaticArea {
    void* ptr = nullptr;         // device address of `scratch` on this GPU
    uint64_t generation = 0;     // goes up with every tent_declare_static on this GPU: older static batches are dead
};
constexpr int kMaxDevices = 64;
StaticArea g_static[kMaxDevices];
std::mutex g_static_mutex;

#define HIP_TRY(expr) do { if ((expr) != hipSuccess) return TENT_ERR_HIP; } while (0)

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
        if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
        target = dev;
    }
    ~DeviceGuard() { if (prev >= 0 && prev != target) (void)hipSetDevice(prev); }
    int target = -1;
};

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) { (void)hipGetLastError(); return false; }
    return cap != hipStreamCaptureStatusNone;
}

// Where the kernels of the next call that reports something put it; nowhere without `wanted`.
Report next_report(tent_ctx* ctx, bool wanted)
{
    return wanted ? Report{ctx->host_plan, ++ctx->reports} : Report{nullptr, 0};
}

// Remember that work of the batch was just enqueued on `s` (nothing is recorded into a stream that is
// being captured into a graph: such work is only known to be over when the device is idle).
StreamMark* note_stream(Batch& b, hipStream_t s)
{
    if (capturing(s)) { b.marks_lost = true; return nullptr; }
    StreamMark* slot = nullptr;
    for (StreamMark& m : b.marks) {
        if (m.used && m.stream == s) { slot = &m; break; }
        if (!m.used && !slot) slot = &m;
    }
    if (!slot || !slot->event || hipEventRecord(slot->event, s) != hipSuccess) {
        (void)hipGetLastError();
        b.marks_lost = true;
        return nullptr;
    }
    slot->stream = s;
    slot->used = true;
    return slot;
}

// Records the batch's stream use when an entry point returns, whichever way it returns.
struct StreamNote {
    Batch& b;
    hipStream_t s;
    bool noted = false;          // an event recorded by the call itself covers its work
    StreamNote(Batch& batch, hipStream_t stream) : b(batch), s(stream) {}
    ~StreamNote()
    {
        if (!b.alive || noted) return;
        const StreamMark* mark = note_stream(b, s);
        if (s != b.beside) return;
        // who goes on with the batch on the caller's stream waits for it, as for what a report left
        if (!mark) { (void)hipStreamSynchronize(s); return; }
        b.report_at = mark->event;
        b.report_stream = s;
    }
};

// Waits until the figures of `told` are there: everything enqueued on `s` before the kernel that tells them has ended then, and
// that kernel is past its last look at what it counts (a plan's goes on to write the slices' rails).  After kReportSpin, under
// capture (where it is refused) and behind an error this is a wait for the stream: a call of more than a millisecond does not
// notice the 4 us.
constexpr std::chrono::microseconds kReportSpin{1000};
hipError_t await_figures(const Report& told, hipStream_t s, bool* looked = nullptr)
{
    if (looked) *looked = false;                         // the figures were there before the stream had been waited for
    if (capturing(s)) return hipStreamSynchronize(s);
    const auto until = std::chrono::steady_clock::now() + kReportSpin;
    do {
        for (int k = 0; k < 64; ++k) {
            if (__atomic_load_n(&told.to->call, __ATOMIC_ACQUIRE) == told.call) {
                if (looked) *looked = true;
                return hipSuccess;
            }
            __builtin_ia32_pause();
        }
    } while (std::chrono::steady_clock::now() < until);
    return hipStreamSynchronize(s);
}

// The same for a call that writes the batch's tables: what is left of it then ends at the stream's mark, which the call records itself,
// while its kernels run.  Without a mark it waits for the stream.  (A call that only counts leaves nothing: its figures go out
// behind its last access to the batch.)
hipError_t await_report(Batch& b, const Report& told, hipStream_t s, StreamNote& note)
{
    const StreamMark* mark = note_stream(b, s);
    note.noted = true;
    if (!mark) return hipStreamSynchronize(s);
    b.report_at = mark->event;
    b.report_stream = s;
    return await_figures(told, s);
}

// Host calls on an event outside a graph that would invalidate a capture in progress, although what is captured does not depend on them.
struct CaptureAside {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    bool set = false;
    CaptureAside() { set = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess; }
    ~CaptureAside() { if (set) (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Callers may go on with the batch on another stream without an event of their own behind a call that waits.  What is left of its last
// kernel is waited for there, on the device; so is a call that ran on the context's own stream.  A stream that is being
// captured permits no wait for work outside the graph: when the graph runs is its caller's to order, but behind the context's own stream
// the caller cannot order anything, so that is waited for by the host.
hipError_t order_after_report(Batch& b, hipStream_t s)
{
    if (!b.report_at || s == b.report_stream) return hipSuccess;
    const bool captured = capturing(s);
    if (captured && b.report_stream != b.beside) return hipSuccess;
    const hipEvent_t end = b.report_at;
    b.report_at = nullptr;
    if (!captured) return hipStreamWaitEvent(s, end, 0);
    const CaptureAside aside;
    return hipEventSynchronize(end);
}

// Host-side wait for everything that was enqueued for the batch.
void wait_batch_idle(Batch& b)
{
    if (b.decl_pending) (void)hipEventSynchronize(b.decl_event);
    for (StreamMark& m : b.marks)
        if (m.used) (void)hipEventSynchronize(m.event);
    if (b.marks_lost) (void)hipDeviceSynchronize();
    (void)hipGetLastError();
}

bool init_slot(Batch& b)
{
    // Every one keeps its release to the whole system: the host waits for the marks before it frees or reuses what
    // the work wrote, and an event without that release (1.2 us cheaper) promises such a wait nothing.
    bool ok = hipEventCreateWithFlags(&b.prep_event, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&b.done_event, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&b.decl_event, hipEventDisableTiming) == hipSuccess &&
              hipHostMalloc((void**)&b.verdict, 64, hipHostMallocDefault) == hipSuccess;
    for (StreamMark& m : b.marks)
        ok = ok && hipEventCreateWithFlags(&m.event, hipEventDisableTiming) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    return ok;
}

void destroy_slot(Batch& b)
{
    if (b.prep_event) (void)hipEventDestroy(b.prep_event);
    if (b.done_event) (void)hipEventDestroy(b.done_event);
    if (b.decl_event) (void)hipEventDestroy(b.decl_event);
    if (b.verdict) (void)hipHostFree(b.verdict);
    for (StreamMark& m : b.marks)
        if (m.event) (void)hipEventDestroy(m.event);
    b.prep_event = b.done_event = b.decl_event = nullptr;
    b.verdict = nullptr;
    for (StreamMark& m : b.marks) m = StreamMark{};
}

// Start a new batch in a slot: everything but the slot's events, its pinned word and its generation starts afresh.
void renew_slot(Batch& b)
{
    Batch fresh;
    fresh.generation = b.generation + 1;
    fresh.prep_event = b.prep_event;
    fresh.done_event = b.done_event;
    fresh.decl_event = b.decl_event;
    fresh.verdict = b.verdict;
    for (int k = 0; k < kMarks; ++k) fresh.marks[k].event = b.marks[k].event;
    b = fresh;
}

// The batch's tables go back to the context (an allocation is kept for a later declaration of
// similar size; what the context cannot keep is freed).  The caller has waited for the batch.
void free_batch(tent_ctx* ctx, Batch& b)
{
    if (b.block && !b.in_static) {
        bool kept = false;
        if (ctx->spare.size() < kSpareBlocks) {
            try { ctx->spare.push_back({b.block, b.block_bytes}); kept = true; } catch (const std::bad_alloc&) {}
        } else {
            // keep the larger allocations: replace the smallest spare one if this one is larger
            size_t least = 0;
            for (size_t k = 1; k < ctx->spare.size(); ++k)
                if (ctx->spare[k].bytes < ctx->spare[least].bytes) least = k;
            if (ctx->spare[least].bytes < b.block_bytes) {
                (void)hipFree(ctx->spare[least].ptr);
                ctx->spare[least] = {b.block, b.block_bytes};
                kept = true;
            }
        }
        if (!kept) (void)hipFree(b.block);
    }
    b.block = nullptr;
    b.block_bytes = 0;
    b.alive = false;
    b.decl_pending = false;
    if (ctx->copies_end == b.done_at) ctx->copies_end = nullptr;       // (it has ended, and the slot's next batch records the event anew)
    b.replan_at = nullptr;
    b.report_at = nullptr;
    b.done_recorded = false;
    b.marks_lost = false;
    for (StreamMark& m : b.marks) { m.used = false; m.stream = nullptr; }
    b.dev = BatchDev{};
}

Batch* find_batch(tent_ctx* ctx, tent_batch_t h)
{
    const uint64_t idx = (h & 0xFFFFFFFFull);
    const uint32_t gen = (uint32_t)(h >> 32);
    if (idx == kStaticSlot) {
        Batch* b = &ctx->static_batch;
        if (!b->alive || b->generation != gen) return nullptr;
        // a later tent_declare_static on this GPU (from any context) has taken the workspace over
        uint64_t now = 0;
        {
            std::lock_guard<std::mutex> lk(g_static_mutex);
            now = ctx->device < kMaxDevices ? g_static[ctx->device].generation : 0;
        }
        if (now != b->static_generation) { b->alive = false; return nullptr; }
        return b;
    }
    if (idx == 0 || idx > ctx->batches.size()) return nullptr;
    Batch* b = &ctx->batches[idx - 1];
    return (b->alive && b->generation == gen) ? b : nullptr;
}

// Every per-batch table is carved from ONE range of device memory: a declaration asks for about fifty
// arrays, and fifty allocator calls cost more than everything else a declaration does.  The requests
// are collected first and then laid out at 256-byte aligned offsets.
struct Carver {
    struct Want { void** slot; uint64_t bytes; };
    static constexpr int kMost = 80;
    Want wants[kMost];
    int n = 0;
    bool overflow = false;
    template <class T>
    void want(T** out, uint64_t count)
    {
        if (n == kMost) { overflow = true; return; }
        wants[n++] = {reinterpret_cast<void**>(out), std::max<uint64_t>(count, 1) * sizeof(T)};
    }
    uint64_t total() const
    {
        uint64_t t = 0;
        for (int k = 0; k < n; ++k) t += (wants[k].bytes + 255) & ~255ull;
        return t;
    }
    void place(void* base) const
    {
        uint64_t at = 0;
        for (int k = 0; k < n; ++k) {
            *wants[k].slot = static_cast<char*>(base) + at;
            at += (wants[k].bytes + 255) & ~255ull;
        }
    }
};

// What a batch counts against the limit of tent_declare_static.  The entries and their sizes are the limit's definition, so
// that the batches which are accepted and refused stay the same whatever the tables look like: several of them are no size of
// a table or structure of today's (a run counts 12 bytes per rail and a record, its cells take 16 bytes per rail; retried
// slices count in chunks of 1024).  That the tables of an accepted batch fit the array is checked by the caller.
uint64_t static_measure(const BatchDev& d, bool bounded, uint64_t order_bytes)
{
    constexpr uint64_t kView = 528, kResult = 4712, kRunRecord = 32, kRotation = 1024;
    uint64_t t = order_bytes;
    const auto add = [&t](uint64_t count, uint64_t size) { t += (std::max<uint64_t>(count, 1) * size + 255) & ~255ull; };
    const uint64_t D = d.n_desc, ns = d.n_src_ext, nd = d.n_dst_ext, N = d.n_slices, q = d.n_sc_tiles;
    const uint64_t scan_n = std::max(std::max(ns, nd), std::max(N, D)), runs = 2 * D;
    const uint64_t rot = (N + kRotation - 1) / kRotation * TENT_MAX_RAILS;
    add(D + 1, 4); add(D + 1, 4); add(ns, 16); add(nd, 16);              // descriptors
    add(ns + 1, 8); add(nd + 1, 8); add(D + 1, 8);                       // prefixes
    for (int k = 0; k < 5; ++k) add(N, 4);                               // slices: transfer, length, extents, rail;
    for (int k = 0; k < 3; ++k) add(N, 8);                               //   offset, staging offset, latency;
    add(N, 1); add(N, 1); add(N, 16);                                    //   state, retries, copy record
    add(D, 1); add(D, 1); add(1, kView); add(1, 4);                      // priority, mode, the batch itself, verdict
    if (q == 0) { add(N * d.tiles_per_slice, 8); add(N * d.tiles_per_slice, 8); }
    add(runs + 1, 4); add(runs * d.run_stride, 8); add(runs * d.run_stride, 4); add(runs + 1, kRunRecord);
    add(N + 1, 8); add(nd, 4); add(nd, 4);
    if (q) {
        add(nd + 1, 8);
        for (int k = 0; k < 4; ++k) { add(q, 8); add(q, 4); }            // tiles, by either order
        if (bounded) add(q, 8);
        add(N + 1, 8); add(scan_partials_capacity(N), 8);
        for (int k = 0; k < 3; ++k) add(q / 2 + 1, 8);                   // tiles of a partial execute
    }
    if (bounded)
        for (int k = 0; k < 3; ++k) add((uint64_t)kMaxChunks * TENT_MAX_RAILS, 8);
    add(N, 4); add(N, 4); add(rot, 8); add(rot, 4);                      // pending and retried slices
    add(scan_n + 1, 8); add(scan_partials_capacity(scan_n), 8); add(scan_partials_capacity(scan_n), 8);
    add(1, kResult);                                                     // the result block
    return t;
}

// Device memory for a batch's tables: a spare allocation of a released batch when one is large enough
// (and not absurdly larger), else a new one.
int acquire_block(tent_ctx* ctx, uint64_t need, void** out, uint64_t* out_bytes)
{
    size_t best = ctx->spare.size();
    for (size_t k = 0; k < ctx->spare.size(); ++k) {
        const uint64_t have = ctx->spare[k].bytes;
        if (have >= need && have <= 4 * need + (1ull << 20) &&
            (best == ctx->spare.size() || have < ctx->spare[best].bytes))
            best = k;
    }
    if (best != ctx->spare.size()) {
        *out = ctx->spare[best].ptr;
        *out_bytes = ctx->spare[best].bytes;
        ctx->spare.erase(ctx->spare.begin() + (long)best);
        return TENT_OK;
    }
    void* p = nullptr;
    if (hipMalloc(&p, need) != hipSuccess) {
        (void)hipGetLastError();
        return TENT_ERR_NOMEM;
    }
    *out = p;
    *out_bytes = need;
    return TENT_OK;
}

// Pinned buffer for the host arrays of one declaration: the two buffers are used in turn, so a
// declaration seldom has to wait for the upload of the one before.  With `may_grow` unset a buffer
// that is too small is reported (nullptr) instead of being replaced.
uint8_t* acquire_stage(tent_ctx* ctx, uint64_t need, bool may_grow, int* which)
{
    const int k = (int)(ctx->stage_turn & 1);
    if (ctx->stage_busy[k]) {
        (void)hipEventSynchronize(ctx->stage_event[k]);
        ctx->stage_busy[k] = false;
    }
    if (ctx->stage_bytes[k] < need) {
        if (!may_grow) return nullptr;
        uint8_t* p = nullptr;
        const uint64_t want = need + need / 4;
        if (hipHostMalloc((void**)&p, want, hipHostMallocDefault) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        if (ctx->stage[k]) (void)hipHostFree(ctx->stage[k]);
        ctx->stage[k] = p;
        ctx->stage_bytes[k] = want;
    }
    ++ctx->stage_turn;
    *which = k;
    return ctx->stage[k];
}

// Host array -> device through the pinned buffer whose turn it is, one buffer-full at a time, waiting
// for each piece (used when the buffer cannot hold a declaration's arrays and must not be replaced).
bool upload_in_pieces(tent_ctx* ctx, void* dev, const void* host, uint64_t bytes)
{
    const int k = (int)(ctx->stage_turn & 1);
    if (ctx->stage_busy[k]) {
        if (hipEventSynchronize(ctx->stage_event[k]) != hipSuccess) return false;
        ctx->stage_busy[k] = false;
    }
    const uint64_t cap = ctx->stage_bytes[k];
    if (cap == 0) return false;
    for (uint64_t at = 0; at < bytes; at += cap) {
        const uint64_t n = std::min(cap, bytes - at);
        std::memcpy(ctx->stage[k], static_cast<const uint8_t*>(host) + at, n);
        if (hipMemcpyAsync(static_cast<uint8_t*>(dev) + at, ctx->stage[k], n, hipMemcpyHostToDevice, ctx->decl_stream) != hipSuccess ||
            hipStreamSynchronize(ctx->decl_stream) != hipSuccess)
            return false;
    }
    return true;
}

// CSR pointer arrays: start at 0, strictly increasing (no empty transfer).
bool pointers_ok(uint32_t n_desc, const uint32_t* p)
{
    if (p[0] != 0) return false;
    for (uint32_t j = 0; j < n_desc; ++j)
        if (p[j + 1] <= p[j]) return false;
    return true;
}

// Walks both extent lists of the transfers [j0, j1): structure, bounds, equal lengths; every extent is
// copied to `se_out` / `de_out` (if not null) on the way.
struct WalkResult {
    int rc = TENT_OK;
    uint64_t total = 0, slices = 0, bits = 0, most = 0, records = 0;
    uint64_t dst_apart = 0;                     // address bits in which a destination extent differs from the first one
};

// One side's extents.  What a check needs of a segment is kept from extent to extent, because a list seldom changes its
// segment: looking it up for every extent made tent_declare of 2 x 646,336 extents take 498 us instead of 390, and of 2 x 883,668
// 690 instead of 550 (host time of the call).
struct SideWalk {
    const Segment* seg;
    size_t n_seg;
    uint64_t origin;                            // address that all others are compared with
    uint32_t id = 0xFFFFFFFFu;                  // segment in hand; none yet, and no extent fits its length of 0
    uint64_t base = 0, seg_len = 0;
    uint64_t apart = 0, bits = 0;
    SideWalk(const tent_ctx* ctx, uint64_t org) : seg(ctx->segments.data()), n_seg(ctx->segments.size()), origin(org) {}
    // extents [e, end); adds up their length, false for one that is empty or outside its segment
    bool operator()(const tent_extent* ext, tent_extent* copy, uint32_t e, uint32_t end, uint64_t* total)
    {
        uint64_t sum = 0;
        for (; e < end; ++e) {
            const tent_extent x = ext[e];
            if (x.seg != id) {
                if (x.seg >= n_seg) return false;
                id = x.seg;
                base = (uint64_t)seg[id].base;
                seg_len = seg[id].len;
            }
            if (x.len == 0 || x.off > seg_len || x.len > seg_len - x.off) return false;
            if (copy) copy[e] = x;
            apart |= (base + x.off) ^ origin;
            bits |= x.len;
            sum += x.len;
        }
        *total = sum;
        return true;
    }
};

void validate_range(const tent_ctx* ctx, uint32_t j0, uint32_t j1, const uint32_t* sp, const tent_extent* se,
                    const uint32_t* dp, const tent_extent* de, tent_extent* se_out, tent_extent* de_out, WalkResult* out)
{
    const uint64_t S = ctx->cfg.slice_bytes;
    const uint64_t origin = de[0].seg < ctx->segments.size() ? (uint64_t)ctx->segments[de[0].seg].base + de[0].off : 0;
    WalkResult r;
    SideWalk src(ctx, origin), dst(ctx, origin);
    uint64_t last = 0;                          // length of the slice before
    for (uint32_t j = j0; j < j1; ++j) {
        uint64_t ls = 0, ld = 0;
        if (!src(se, se_out, sp[j], sp[j + 1], &ls) || !dst(de, de_out, dp[j], dp[j + 1], &ld) || ls != ld) {
            r.rc = TENT_ERR_INVALID;
            break;
        }
        r.total += ls;
        const uint64_t cnt = (ls + S - 1) / S;
        r.slices += cnt;
        r.most = std::max(r.most, cnt);
        r.records += last != std::min(ls, S);
        last = ls - (cnt - 1) * S;
    }
    r.bits = src.bits | dst.bits;
    r.dst_apart = dst.apart;
    *out = r;
}

// The whole batch, with the payload and the number of slices the device splitter will produce.
// Large batches are walked by a few threads, each over a range of transfers with about the same number of
// extents: the walk streams some tens of megabytes and is the longest part of a declaration.
int validate(const tent_ctx* ctx, uint32_t n_desc, const uint32_t* sp, const tent_extent* se,
             const uint32_t* dp, const tent_extent* de, tent_extent* se_out, tent_extent* de_out,
             WalkResult* all, bool may_spawn)
{
    constexpr uint32_t kMaxWalkers = 4;
    constexpr uint64_t kExtentsPerWalker = 1ull << 16;
    const uint64_t n_ext = (uint64_t)sp[n_desc] + dp[n_desc];
    uint32_t walkers = (uint32_t)std::min<uint64_t>(kMaxWalkers, n_ext / kExtentsPerWalker);
    walkers = std::min(walkers, std::max(1u, std::thread::hardware_concurrency()));
    if (!may_spawn) walkers = 1;                       // a thread's stack is an allocation: not for callers that forbid them
    WalkResult part[kMaxWalkers];
    uint32_t used = 1;
    if (walkers >= 2) {
        // cut points: transfers at which the running count of extents passes k / walkers of the total
        uint32_t cut[kMaxWalkers + 1];
        cut[0] = 0;
        for (uint32_t k = 1; k < walkers; ++k) {
            const uint64_t want = n_ext * k / walkers;
            uint32_t lo = cut[k - 1], hi = n_desc;
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if ((uint64_t)sp[mid] + dp[mid] < want) lo = mid + 1; else hi = mid;
            }
            cut[k] = lo;
        }
        cut[walkers] = n_desc;
        std::thread th[kMaxWalkers];
        uint32_t started = 0;
        try {
            for (uint32_t k = 1; k < walkers; ++k) {
                th[k] = std::thread(validate_range, ctx, cut[k], cut[k + 1], sp, se, dp, de, se_out, de_out, &part[k]);
                ++started;
            }
        } catch (...) {
            // no more threads to be had: the ranges not handed out are walked here
        }
        validate_range(ctx, cut[0], cut[1], sp, se, dp, de, se_out, de_out, &part[0]);
        for (uint32_t k = 1; k <= started; ++k) th[k].join();
        for (uint32_t k = started + 1; k < walkers; ++k)
            validate_range(ctx, cut[k], cut[k + 1], sp, se, dp, de, se_out, de_out, &part[k]);
        used = walkers;
    } else {
        validate_range(ctx, 0, n_desc, sp, se, dp, de, se_out, de_out, &part[0]);
    }
    for (uint32_t k = 0; k < used; ++k) {
        if (part[k].rc != TENT_OK) return part[k].rc;
        all->total += part[k].total;
        all->slices += part[k].slices;
        all->bits |= part[k].bits;
        all->most = std::max(all->most, part[k].most);
        all->records += part[k].records;
        all->dst_apart |= part[k].dst_apart;
    }
    return TENT_OK;
}

// Brackets the launches of one stage with a pair of HIP events on the caller's stream.
struct StageTimer {
    hipEvent_t stop = nullptr;
    hipStream_t s;
    StageTimer(tent_ctx* c, int stage, hipStream_t stream) : s(stream)
    {
        if (!(c->cfg.flags & TENT_FLAG_PROFILE)) return;
        Timing& t = c->timing[stage];
        if (t.used >= kMaxTimedIntervals) return;          // nobody reads the timings: stop collecting
        if (t.used == t.pool.size()) {
            hipEvent_t a = nullptr, b = nullptr;
            if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) {
                if (a) (void)hipEventDestroy(a);
                return;
            }
            try { t.pool.emplace_back(a, b); } catch (const std::bad_alloc&) {
                (void)hipEventDestroy(a); (void)hipEventDestroy(b);
                return;
            }
        }
        (void)hipEventRecord(t.pool[t.used].first, s);
        stop = t.pool[t.used].second;
        ++t.used;
    }
    ~StageTimer() { if (stop) (void)hipEventRecord(stop, s); }
};

// A re-plan enqueued on another stream than the last execute's may overlap that execute's copies: it
// only has to come after the execute's bookkeeping.  An execute that could leave nothing over records no
// event for that (each is a bubble of 6 us on the stream): a plan on another stream waits for its end, as it does for a
// bounded execute's.  What is being captured into a graph runs when its caller replays it: no wait is recorded there.
// A first plan (`whole`) rewrites what the copies read and waits for their end.
hipError_t order_after_execute_bookkeeping(const Batch& b, hipStream_t s, bool whole = false)
{
    const hipEvent_t end = whole && b.done_recorded ? b.done_at : b.replan_at;
    if (!end || s == b.exec_stream || capturing(s)) return hipSuccess;
    return hipStreamWaitEvent(s, end, 0);
}

// Marks the end of an execute's bookkeeping on its stream.  Nothing is recorded into a stream that is
// being captured into a graph; a graph holds its launches in stream order anyway.
hipError_t record_execute_bookkeeping(Batch& b, hipStream_t s)
{
    b.replan_at = nullptr;
    b.done_recorded = false;
    if (!b.may_replan || capturing(s)) return hipSuccess;
    hipError_t e = hipEventRecord(b.prep_event, s);
    if (e != hipSuccess) return e;
    b.exec_stream = s;
    b.replan_at = b.prep_event;
    return hipSuccess;
}

// Marks the end of an execute's copies on its stream: what batch-level completion waits for.
// It is the stream's mark as well (a later call on the same stream moves it on, which only makes it later).
hipError_t record_execute_done(Batch& b, hipStream_t s, StreamNote& note)
{
    b.done_recorded = false;
    if (capturing(s)) return hipSuccess;
    if (const StreamMark* mark = note_stream(b, s)) {
        note.noted = true;
        b.done_at = mark->event;
    } else {
        hipError_t e = hipEventRecord(b.done_event, s);
        if (e != hipSuccess) return e;
        b.done_at = b.done_event;
    }
    b.exec_stream = s;
    b.done_recorded = true;
    b.report_at = nullptr;               // what follows the execute follows the report
    return hipSuccess;
}

// Executes so far on a stream, of all contexts: tells a batch whether other copies have been enqueued there behind its own.
// Streams share the counters by their handles; those of two that meet only make a call change streams for nothing (see work_stream).
constexpr uint32_t kExecuteCounterBits = 10;
std::atomic<uint64_t> g_executes[1u << kExecuteCounterBits];

std::atomic<uint64_t>& executes_on(const tent_ctx* ctx, hipStream_t s)
{
    // (a default stream has the same handle on every device)
    const uint64_t key = (reinterpret_cast<uint64_t>(s) ^ ((uint64_t)ctx->device << 56)) * 0x9E3779B97F4A7C15ull;
    return g_executes[key >> (64 - kExecuteCounterBits)];
}

// An execute that was enqueued: what may run beside its copies (with `apart`, nothing).
void note_execute(tent_ctx* ctx, Batch& b, hipStream_t s, bool apart = false)
{
    b.last = b.done_recorded && !apart ? Batch::Last::kExecute : Batch::Last::kCaller;
    b.execute_no = ++executes_on(ctx, s);
    if (apart) ctx->copies_end = nullptr;
    if (!b.done_recorded || apart) return;
    ctx->copies_end = b.done_at;
    ctx->copies_stream = s;
}

// Whether the work behind which `end` was recorded has not ended.
bool running(hipEvent_t end)
{
    if (!end) return false;
    const CaptureAside aside;
    const bool yes = hipEventQuery(end) == hipErrorNotReady;
    if (yes) (void)hipGetLastError();
    return yes;
}

bool stream_terms(hipStream_t s, uint32_t cu_words, StreamTerms* out)
{
    if (hipStreamGetPriority(s, &out->priority) == hipSuccess && hipExtStreamGetCUMask(s, cu_words, out->cu_mask) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Where a call that only works on the batch's tables runs: a plan, a reset, the rail simulator and the probe read and write no byte
// of a segment or the arena, so they need not wait for copies that were enqueued on the caller's stream before -- those of other batches,
// and of the batch's own last execute as far as its bookkeeping.  Beside such copies they run on the context's own stream,
// ordered among themselves and behind that bookkeeping (`whole`, a reset or a first plan, which rewrite what the copies read:
// behind the batch's own copies); the next call of the batch on the caller's stream waits for them there.
// Only while copies are known to run on `s` that the call does not have to wait for, because the change of streams costs two waits:
// where executes on any stream counted as such, two contexts on a stream each, with 10 MB cycles, took 80 us for both instead of 60.
// MI355X, cycles of three batches in turn: 4,096 transfers 2060 -> 1540 us, 24,576 11534 -> 9095, 256 ragged ones 262 -> 198, 74
// slices (4 MB) 43 -> 37.  Beside the batch's own copies a re-plan has only those to hide behind, hence kBesideBytes: sixteen windows of
// 100 MB each 5808 -> 4807 us, and of a batch of 1 GiB three of 96 MiB 2263 -> 2210 and three of 64 2314 -> 2319 (2352 -> 2324 where the
// simulator's figures are read), but three of 32 2341 -> 2394, six of 2 2371 -> 2485, and of one of 70 MiB six of 2 440 -> 548.  Where
// other batches' copies lie behind them as well it is worth it in any case: two such batches in turn 877 -> 731.
// Not a call that reports figures: everything that was enqueued on `s` before it has ended when it returns.
// A batch that a graph holds a call of stays on its caller's streams, because replays are not seen here; so do batches in the
// static workspace, whose next owner's declaration waits for the caller's streams, and contexts that time their stages.  So do calls on a
// stream that its caller gave a priority or a share of the compute units (asking for both takes 0.4 us): they hold for what is enqueued there.
constexpr uint64_t kBesideBytes = 64ull << 20;
// Launches in a row lose up to 0.4 us each while another stream's kernels run or wait beside them, so a plan goes beside a bounded
// execute where its chain is worth that: kBesideChunks chunks, and one more for every kChunkSteps steps of the chain.  MI355X, cycles
// of three batches in turn, us a batch: 4,096 transfers of which three in four end in a short slice, in 16 chunks of 16 MiB 720 -> 403,
// in 126 2175 -> 1923, in 247 of 4 MiB 1765 -> 1591; 1,024 in 79 of 16 MiB 1215 -> 1165 and in 127 1846 -> 1817 (behind the line); 256 in
// 25 405 -> 373, in 65 935 -> 931, in 81 1144 -> 1154; 64 in 16 217 -> 202, in 47 674 -> 677, in 124 1698 -> 1742.  4,096 of whole slices,
// a single step, in 16 247 -> 225, in 32 485 -> 483, in 64 909 -> 923, in 128 1768 -> 1814.
constexpr uint64_t kBesideChunks = 16, kChunkSteps = 8;
bool worth_beside(const tent_ctx* ctx, const Batch& b, hipStream_t s, bool whole)
{
    if (b.last == Batch::Last::kBeside) return true;
    if (b.last == Batch::Last::kExecute) {
        if (b.exec_stream != s || !b.replan_at) return false;
        // where nothing has been enqueued behind its copies, what has to wait for them runs beside nothing
        const bool alone = b.execute_no == executes_on(ctx, s).load();
        if (whole || b.replan_at == b.done_at) {
            if (alone) return false;
        } else if (b.payload < kBesideBytes || (alone && b.execute_bytes < kBesideBytes)) {
            return false;
        }
        return running(b.done_at);
    }
    if (ctx->copies_stream != s || !running(ctx->copies_end)) return false;
    for (const StreamMark& m : b.marks)                  // (calls on the caller's streams that have not ended)
        if (m.used && running(m.event)) return false;
    return true;
}

hipStream_t work_stream(const tent_ctx* ctx, const Batch& b, hipStream_t s, bool whole, bool reports)
{
    if (reports || b.marks_lost || b.in_static || (ctx->cfg.flags & TENT_FLAG_PROFILE) || capturing(s) || !worth_beside(ctx, b, s, whole)) return s;
    StreamTerms terms;
    return stream_terms(s, ctx->cu_words, &terms) && terms == ctx->beside_terms ? b.beside : s;
}

// Prefixes, slice and run table of a first plan, and with `tables` the tile tables (where no chain's launch builds them).  A caller that
// asks for the time of every stage gets the launches of a large batch.
int split(tent_ctx* ctx, const BatchDev& d, bool tables, hipStream_t s)
{
    if (!(ctx->cfg.flags & TENT_FLAG_PROFILE) && plan_front_fits(d)) {
        HIP_TRY(launch_plan_front(d, s));
        if (tables) HIP_TRY(launch_tile_tables(d, s));
        return TENT_OK;
    }
    {
        StageTimer t(ctx, TENT_T_EXTENT_SCAN, s);
        HIP_TRY(launch_extent_scans(d, s));
    }
    {
        StageTimer t(ctx, TENT_T_SLICE_SCAN, s);
        HIP_TRY(launch_slice_scan(d, s));
    }
    StageTimer t(ctx, TENT_T_EXPAND, s);
    HIP_TRY(launch_expand(d, s));
    if (tables) HIP_TRY(launch_tile_tables(d, s));
    return TENT_OK;
}

// The first call that needs the batch's tables waits (on the host) for the declaration's device work
// and learns the verdict of the overlap check.  A batch that fails it is released.
int finish_declare(tent_ctx* ctx, Batch& b)
{
    if (!b.decl_pending) return TENT_OK;
    HIP_TRY(hipEventSynchronize(b.decl_event));
    b.decl_pending = false;
    if (*b.verdict != 0) {
        wait_batch_idle(b);
        free_batch(ctx, b);
        return TENT_ERR_INVALID;
    }
    return TENT_OK;
}

// The same for a plan that enqueues first and asks afterwards: the declaration's device work, the host's launches and the plan
// then follow each other without a host wait in between (20-40 us for a small batch).  A batch whose destinations overlap
// is planned like any other -- its tables are sound, only no byte may move -- and released here.
int finish_declare_behind(tent_ctx* ctx, Batch& b, hipStream_t s)
{
    if (!b.decl_pending) return TENT_OK;
    HIP_TRY(hipEventSynchronize(b.decl_event));
    if (*b.verdict != 0) HIP_TRY(hipStreamSynchronize(s));
    return finish_declare(ctx, b);
}

// Telemetry -> integer coefficients (Eq. 1 with the topology penalty folded in).
int convert_rails(const tent_rail_state* rails, uint32_t n_rails, uint64_t pending_bytes, RailParams* rp)
{
    std::memset(rp, 0, sizeof(*rp));
    rp->n_rails = n_rails;
    uint64_t max_c1 = 0, max_A = 0;
    for (uint32_t d = 0; d < n_rails; ++d) {
        const tent_rail_state& r = rails[d];
        if (r.health > 2) return TENT_ERR_INVALID;
        if (r.bw_MBps == 0) return TENT_ERR_RANGE;
        const uint64_t bp = (uint64_t)r.beta1_q8 * r.penalty_q8;
        // a degraded rail keeps half its weight: its predicted cost counts twice (Section 4.3)
        const uint64_t weight = r.health == 1 ? 2 : 1;
        const uint64_t c1 = weight * ((1000000ull * bp) / r.bw_MBps);
        if (c1 >= (1ull << 32)) return TENT_ERR_RANGE;
        rp->c1[d] = c1;
        rp->c0[d] = weight * (((uint64_t)r.lat_ns * 1000ull * r.penalty_q8) >> 8);
        rp->A[d] = r.queued_bytes;
        if (r.health != 2) {
            rp->admitted |= 1ull << d;
            max_c1 = std::max(max_c1, c1);
            max_A = std::max(max_A, r.queued_bytes);
        }
    }
    // (max A + pending bytes) * max c1 must stay below 2^63 so that no cost wraps
    const unsigned __int128 worst = ((unsigned __int128)max_A + pending_bytes) * max_c1;
    if (worst >= ((unsigned __int128)1 << 63)) return TENT_ERR_RANGE;
    // the binding chains count the bytes they bind to a rail in doubles (RunCell::T): whole numbers below 2^53 are exact.  No
    // device has room for the tables of such a batch
    if (pending_bytes >= (1ull << 53)) return TENT_ERR_RANGE;
    return TENT_OK;
}

// Whether the staging arena shares no byte with a registered segment: only then may a destination byte be written
// before every source byte has been read into staging.
bool arena_apart(const tent_ctx* ctx)
{
    const uint64_t a = (uint64_t)ctx->cfg.staging_arena, n = ctx->cfg.staging_bytes;
    for (const Segment& s : ctx->segments) {
        const uint64_t b = (uint64_t)s.base;
        if (b < a ? a - b < s.len : b - a < n) return false;
    }
    return true;
}

// tent_declare and tent_declare_static.  With `use_static` the tables and the sort's workspace are
// carved from the static workspace of the context's GPU and nothing is allocated, on the device or
// on the host.
int declare_impl(tent_ctx* ctx, uint32_t n_desc, const uint32_t* src_ptr, const tent_extent* src_ext,
                 const uint32_t* dst_ptr, const tent_extent* dst_ext, tent_batch_t* out, bool use_static)
{
    if (!ctx || !src_ptr || !src_ext || !dst_ptr || !dst_ext || !out || n_desc == 0) return TENT_ERR_INVALID;
    *out = 0;
    if (n_desc >= 0x7FFFFFFFu) return TENT_ERR_RANGE;
    if (!pointers_ok(n_desc, src_ptr) || !pointers_ok(n_desc, dst_ptr)) return TENT_ERR_INVALID;
    const uint64_t ns = src_ptr[n_desc], nd = dst_ptr[n_desc];
    if (ns + nd >= 0xFFFFFFFFull) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;

    // Host arrays -> pinned buffer (laid out as they will lie in the upload): both pointer arrays,
    // both extent lists, then the device view of the batch.
    const uint64_t ptr_bytes = ((uint64_t)n_desc + 1) * sizeof(uint32_t);
    const uint64_t o_sp = 0, o_dp = (o_sp + ptr_bytes + 15) & ~15ull, o_se = (o_dp + ptr_bytes + 15) & ~15ull;
    const uint64_t o_de = o_se + ns * sizeof(tent_extent), o_self = o_de + nd * sizeof(tent_extent);
    const uint64_t stage_need = o_self + sizeof(BatchDev);
    int which = -1;
    uint8_t* st = acquire_stage(ctx, stage_need, !use_static, &which);
    if (!st && !use_static) return TENT_ERR_NOMEM;

    WalkResult walk;
    int rc = validate(ctx, n_desc, src_ptr, src_ext, dst_ptr, dst_ext, st ? (tent_extent*)(st + o_se) : nullptr,
                      st ? (tent_extent*)(st + o_de) : nullptr, &walk, !use_static);
    if (rc != TENT_OK) return rc;
    const uint64_t payload = walk.total, n_slices = walk.slices, len_bits = walk.bits, max_req_slices = walk.most;
    if (n_slices >= 0xFFFFFFFEull) return TENT_ERR_RANGE;

    Batch* slot_b = nullptr;
    size_t slot = 0;
    if (use_static) {
        slot_b = &ctx->static_batch;
        if (slot_b->alive) {                              // the context's earlier static batch gives way
            wait_batch_idle(*slot_b);
            free_batch(ctx, *slot_b);
        }
    } else {
        // reuse a dead slot or append
        slot = ctx->batches.size();
        for (size_t k = 0; k < ctx->batches.size(); ++k) if (!ctx->batches[k].alive) { slot = k; break; }
        if (slot == ctx->batches.size()) {
            if (slot + 1 >= kStaticSlot) return TENT_ERR_RANGE;
            try { ctx->batches.emplace_back(); } catch (const std::bad_alloc&) { return TENT_ERR_NOMEM; }
            if (!init_slot(ctx->batches[slot])) {
                destroy_slot(ctx->batches[slot]);
                ctx->batches.pop_back();
                return TENT_ERR_NOMEM;
            }
        }
        slot_b = &ctx->batches[slot];
    }
    Batch& b = *slot_b;
    renew_slot(b);
    b.beside = ctx->beside;
    b.payload = payload;
    b.max_req_slices = max_req_slices;
    b.records = walk.records;
    BatchDev& d = b.dev;
    d.n_desc = n_desc;
    d.n_src_ext = ns;
    d.n_dst_ext = nd;
    d.n_slices = n_slices;
    d.slice_bytes = ctx->cfg.slice_bytes;
    d.seg_base = ctx->seg_base_dev;
    // Tile size: the largest power of two in [1 KiB, 4 KiB] that divides the slice size and every
    // extent length, so that no tile crosses an extent boundary; geometry that allows no such size
    // gets 1 KiB tiles, and the tiles that do cross a boundary take the generic copy path.
    {
        const uint64_t bits = len_bits | d.slice_bytes | kCopyBlockBytes;
        uint32_t tile = (uint32_t)(bits & (~bits + 1));
        d.tile_bytes = tile < 1024 ? 1024 : tile;
        d.tiles_per_slice = (uint32_t)((d.slice_bytes + d.tile_bytes - 1) / d.tile_bytes);
    }
    const uint64_t n_tiles = n_slices * d.tiles_per_slice;
    // Destination-ordered scatter needs every boundary on a tile boundary (addresses may have any
    // alignment); other geometry keeps the slice-ordered scatter.
    {
        const uint64_t bits = len_bits | d.slice_bytes;
        d.n_sc_tiles = (bits & (d.tile_bytes - 1)) == 0 ? payload / d.tile_bytes : 0;
    }

    uint8_t* upload = nullptr;                            // pointers, extents and the device view, laid out as in the pinned buffer
    const uint64_t scan_n = std::max<uint64_t>(std::max(ns, nd), std::max<uint64_t>(n_slices, n_desc));
    uint32_t* order_dev = nullptr;
    uint32_t* rank_dev = nullptr;
    Carver cv;
    cv.want(&upload, stage_need);
    cv.want(&d.src_pre, ns + 1);
    cv.want(&d.dst_pre, nd + 1);
    cv.want(&d.first, (uint64_t)n_desc + 1);
    cv.want(&d.s_desc, n_slices);
    cv.want(&d.s_off, n_slices);
    cv.want(&d.s_pos, n_slices);
    cv.want(&d.s_len, n_slices);
    cv.want(&d.s_src_e0, n_slices);
    cv.want(&d.s_dst_e0, n_slices);
    cv.want(&d.s_rail, n_slices);
    cv.want(&d.s_stage_off, n_slices);
    cv.want(&d.s_state, n_slices);
    cv.want(&d.s_tau, n_slices);
    cv.want(&d.s_rec, n_slices);
    cv.want(&d.s_retry, n_slices);
    cv.want(&d.priority, (uint64_t)n_desc);
    cv.want(&d.req_mode, (uint64_t)n_desc);
    if (d.n_sc_tiles == 0) {                              // per-slice tile tables only for untiled geometry
        cv.want(&d.src_tile, n_tiles);
        cv.want(&d.dst_tile, n_tiles);
    }
    d.run_capacity = 2u * n_desc;
    d.run_stride = ctx->max_rails <= 16 ? 16u : ctx->max_rails <= 32 ? 32u : 64u;   // a row per run, one entry per lane of the chain
    cv.want(&d.runs_before, (uint64_t)n_desc + 1);
    cv.want(&d.s_run, n_slices);
    cv.want(&d.run_start, (uint64_t)d.run_capacity + 1);
    cv.want(&d.run_cell, (uint64_t)d.run_capacity * d.run_stride);
    cv.want(&d.len_pre, n_slices + 1);
    cv.want(&order_dev, nd);
    cv.want(&rank_dev, nd);
    const bool bounded = (ctx->cfg.flags & TENT_FLAG_BOUNDED_STAGING) != 0;
    const bool check = !(ctx->cfg.flags & TENT_FLAG_SKIP_OVERLAP_CHECK);
    d.one_pass = check && arena_apart(ctx) && d.n_sc_tiles < 0xFFFFFFFFull ? 1u : 0u;
    if (d.n_sc_tiles) {
        // one-pass copies go by destination address (a context with bounded staging: by payload position, as its chunks
        // do), two passes by either order
        if (!d.one_pass || !bounded) cv.want(&d.ord_pre, nd + 1);
        if (!d.one_pass || bounded) {
            cv.want(&d.ga_slice, d.n_sc_tiles);
            cv.want(&d.ga_x, d.n_sc_tiles);
        }
        if (d.one_pass) {
            cv.want(&d.op_src, d.n_sc_tiles);
            cv.want(&d.op_dst, d.n_sc_tiles);
            cv.want(&d.op_lin, d.n_sc_tiles);
            if (!bounded) cv.want(&d.tile_pos, d.n_sc_tiles);
        } else {
            cv.want(&d.ga_src, d.n_sc_tiles);
            cv.want(&d.ga_lin, d.n_sc_tiles);
            if (bounded) cv.want(&d.ga_dst, d.n_sc_tiles);
            cv.want(&d.sc_dst, d.n_sc_tiles);
            cv.want(&d.sc_lin, d.n_sc_tiles);
            cv.want(&d.sc_slice, d.n_sc_tiles);
            cv.want(&d.sc_x, d.n_sc_tiles);
        }
        // an execute goes over a list of tiles only when at most half of the batch's tiles can move
        d.act_capacity = d.n_sc_tiles / 2 + 1;
        if (!d.one_pass) {
            cv.want(&d.tile_scan, n_slices + 1);
            cv.want(&d.tile_partials, scan_partials_capacity(n_slices));
        }
        cv.want(&d.act_src, d.act_capacity);
        cv.want(&d.act_lin, d.act_capacity);
        cv.want(&d.act_dst, d.act_capacity);
    }
    if (bounded) {
        cv.want(&d.ch_lo, (uint64_t)kMaxChunks * TENT_MAX_RAILS);
        cv.want(&d.ch_hi, (uint64_t)kMaxChunks * TENT_MAX_RAILS);
        cv.want(&d.ch_base, (uint64_t)kMaxChunks * TENT_MAX_RAILS);
        if (d.n_sc_tiles == 0) cv.want(&d.range_slice, payload / 1024 + 1);
    }
    cv.want(&d.pending, n_slices);
    cv.want(&d.retry_ids, n_slices);
    const uint64_t rot_chunks = (n_slices + kRotChunk - 1) / kRotChunk;
    cv.want(&d.rot_bytes, rot_chunks * TENT_MAX_RAILS);
    cv.want(&d.rot_cnt, rot_chunks * TENT_MAX_RAILS);
    cv.want(&d.scan_tmp, scan_n + 1);
    cv.want(&d.scan_partials, scan_partials_capacity(scan_n));
    cv.want(&d.scan_partials2, scan_partials_capacity(scan_n));
    cv.want(&d.scan_partials3, scan_partials_capacity(scan_n));
    cv.want(&d.plan, 1);
    if (cv.overflow) return TENT_ERR_NOMEM;

    // destination extents in address order (for the scatter) and the overlap check run on the device
    const bool order = check || d.n_sc_tiles != 0;
    OrderPlan order_plan{};
    KeyBits key_bits{0, 1};
    if (walk.dst_apart) key_bits = KeyBits{(uint32_t)__builtin_ctzll(walk.dst_apart), 64u - (uint32_t)__builtin_clzll(walk.dst_apart)};
    uint64_t order_bytes = ~0ull;                         // what the order may take
    if (order && use_static && order_measure(nd, ns, check, &order_bytes) != hipSuccess) { (void)hipGetLastError(); return TENT_ERR_HIP; }
    if (order && plan_order(nd, ns, check, key_bits, (uint64_t)ctx->segments[dst_ext[0].seg].base + dst_ext[0].off, order_bytes,
                            &order_plan) != hipSuccess) { (void)hipGetLastError(); return TENT_ERR_HIP; }
    const uint64_t ws_need = order_plan.bytes;
    const uint64_t table_bytes = cv.total();
    void* workspace = nullptr;
    if (use_static) {
        if (static_measure(d, bounded, order ? order_bytes : 0) > TENT_STATIC_WORKSPACE_BYTES) return TENT_ERR_RANGE;
        if (table_bytes + ws_need > kStaticArea) return TENT_ERR_RANGE;   // (not reached by a batch within the limit)
        uint8_t* area = nullptr;
        {
            std::lock_guard<std::mutex> lk(g_static_mutex);
            if (ctx->device >= kMaxDevices || !g_static[ctx->device].ptr) return TENT_ERR_STATE;
            area = static_cast<uint8_t*>(g_static[ctx->device].ptr);
            b.static_generation = ++g_static[ctx->device].generation;
        }
        b.block = area;
        b.block_bytes = table_bytes;
        b.in_static = true;
        workspace = area + table_bytes;
    } else {
        rc = acquire_block(ctx, table_bytes, &b.block, &b.block_bytes);
        if (rc != TENT_OK) return rc;
        if (ws_need > ctx->order_ws_bytes) {
            // the stream that used the old workspace is the context's own: wait for it, then replace
            (void)hipStreamSynchronize(ctx->decl_stream);
            if (ctx->order_ws) (void)hipFree(ctx->order_ws);
            ctx->order_ws = nullptr;
            ctx->order_ws_bytes = 0;
            const uint64_t want = ws_need + ws_need / 4;
            if (hipMalloc(&ctx->order_ws, want) != hipSuccess) {
                (void)hipGetLastError();
                ctx->order_ws = nullptr;
                free_batch(ctx, b);
                return TENT_ERR_NOMEM;
            }
            ctx->order_ws_bytes = want;
        }
        workspace = ctx->order_ws;
    }
    cv.place(b.block);
    d.src_ptr = reinterpret_cast<uint32_t*>(upload + o_sp);
    d.dst_ptr = reinterpret_cast<uint32_t*>(upload + o_dp);
    d.src_ext = reinterpret_cast<tent_extent*>(upload + o_se);
    d.dst_ext = reinterpret_cast<tent_extent*>(upload + o_de);
    d.dst_order = order_dev;
    d.dst_rank = rank_dev;
    d.self = reinterpret_cast<BatchDev*>(upload + o_self);

    // Everything from here on is enqueued on the context's own stream; nothing waits for the device
    // unless the host arrays could not go through the pinned buffer.
    hipStream_t ds = ctx->decl_stream;
    bool ok = true;
    if (st) {
        std::memcpy(st + o_sp, src_ptr, ptr_bytes);
        std::memcpy(st + o_dp, dst_ptr, ptr_bytes);
        std::memcpy(st + o_self, &d, sizeof(BatchDev));
        ok = hipMemcpyAsync(upload, st, stage_need, hipMemcpyHostToDevice, ds) == hipSuccess &&
             hipEventRecord(ctx->stage_event[which], ds) == hipSuccess;
        if (ok) ctx->stage_busy[which] = true;
    } else {
        // the pinned buffer is too small and may not grow: the arrays go through it piece by piece
        ok = upload_in_pieces(ctx, upload + o_sp, src_ptr, ptr_bytes) && upload_in_pieces(ctx, upload + o_dp, dst_ptr, ptr_bytes) &&
             upload_in_pieces(ctx, upload + o_se, src_ext, ns * sizeof(tent_extent)) &&
             upload_in_pieces(ctx, upload + o_de, dst_ext, nd * sizeof(tent_extent)) &&
             upload_in_pieces(ctx, upload + o_self, &d, sizeof(BatchDev));
    }
    *b.verdict = 0;
    ok = ok && launch_declare(d, order, check, order_plan, order_dev, rank_dev, b.verdict, workspace, ds) == hipSuccess &&
         hipEventRecord(b.decl_event, ds) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(ds);
        free_batch(ctx, b);
        return TENT_ERR_HIP;
    }
    b.decl_pending = true;
    b.alive = true;
    *out = ((uint64_t)b.generation << 32) | (use_static ? (uint64_t)kStaticSlot : (uint64_t)(slot + 1));
    return TENT_OK;
}

}  // namespace

extern "C" {

const char* tent_strerror(int status)
{
    switch (status) {
        case TENT_OK:          return "ok";
        case TENT_DEFER:       return "deferred: no admitted rail";
        case TENT_ERR_INVALID: return "invalid argument";
        case TENT_ERR_RANGE:   return "value out of range";
        case TENT_ERR_STATE:   return "call out of order";
        case TENT_ERR_NOMEM:   return "out of memory";
        case TENT_ERR_HIP:     return "HIP runtime error";
        default:               return "unknown status";
    }
}

int tent_create(tent_ctx** out, const tent_config* cfg)
{
    if (!out || !cfg) return TENT_ERR_INVALID;
    *out = nullptr;
    if (cfg->slice_bytes == 0 || cfg->slice_bytes > 0x80000000ull) return TENT_ERR_INVALID;
    if (!cfg->staging_arena || cfg->staging_bytes == 0) return TENT_ERR_INVALID;
    if (cfg->max_rails > TENT_MAX_RAILS) return TENT_ERR_RANGE;
    tent_ctx* ctx = new (std::nothrow) tent_ctx;
    if (!ctx) return TENT_ERR_NOMEM;
    ctx->cfg = *cfg;
    ctx->max_rails = cfg->max_rails ? cfg->max_rails : TENT_MAX_RAILS;
    if (hipGetDevice(&ctx->device) != hipSuccess) { delete ctx; return TENT_ERR_HIP; }
    ctx->seg_capacity = kMaxSegments;
    bool ok = true;
    try { ctx->spare.reserve(kSpareBlocks); ctx->batches.reserve(16); } catch (const std::bad_alloc&) { ok = false; }
    ok = ok && hipMalloc((void**)&ctx->seg_base_dev, sizeof(uint64_t) * ctx->seg_capacity) == hipSuccess &&
         hipHostMalloc((void**)&ctx->host_plan, sizeof(PlanState), hipHostMallocCoherent) == hipSuccess &&
         hipStreamCreateWithFlags(&ctx->decl_stream, hipStreamNonBlocking) == hipSuccess &&
         hipStreamCreateWithFlags(&ctx->beside, hipStreamNonBlocking) == hipSuccess &&
         init_slot(ctx->static_batch);
    if (ok) {
        int n_cu = 0;
        ok = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, ctx->device) == hipSuccess;
        ctx->cu_words = std::min<uint32_t>((n_cu + 31) / 32, StreamTerms::kWords);
        (void)stream_terms(ctx->beside, ctx->cu_words, &ctx->beside_terms);
        ctx->host_plan->call = 0;
    }
    for (int k = 0; k < 2 && ok; ++k) {
        ok = hipHostMalloc((void**)&ctx->stage[k], kStageInitial, hipHostMallocDefault) == hipSuccess &&
             hipEventCreateWithFlags(&ctx->stage_event[k], hipEventDisableTiming) == hipSuccess;
        if (ok) ctx->stage_bytes[k] = kStageInitial;
    }
    // the static workspace's address on this GPU, looked up once per device with the device current
    int rc = ok ? TENT_OK : TENT_ERR_NOMEM;
    if (ok && ctx->device < kMaxDevices) {
        std::lock_guard<std::mutex> lk(g_static_mutex);
        if (!g_static[ctx->device].ptr) {
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) rc = TENT_ERR_HIP;
            else g_static[ctx->device].ptr = p;
        }
    }
    if (rc != TENT_OK) {
        (void)hipGetLastError();
        (void)tent_destroy(ctx);
        return rc;
    }
    *out = ctx;
    return TENT_OK;
}

int tent_destroy(tent_ctx* ctx)
{
    if (!ctx) return TENT_ERR_INVALID;
    DeviceGuard g(ctx->device);
    (void)hipDeviceSynchronize();
    for (Batch& b : ctx->batches) {
        if (b.alive) free_batch(ctx, b);
        destroy_slot(b);
    }
    if (ctx->static_batch.alive) free_batch(ctx, ctx->static_batch);
    destroy_slot(ctx->static_batch);
    for (Block& blk : ctx->spare) (void)hipFree(blk.ptr);
    for (Timing& t : ctx->timing)
        for (auto& pr : t.pool) { (void)hipEventDestroy(pr.first); (void)hipEventDestroy(pr.second); }
    for (hipEvent_t e : ctx->sync_events) (void)hipEventDestroy(e);
    for (int k = 0; k < 2; ++k) {
        if (ctx->stage[k]) (void)hipHostFree(ctx->stage[k]);
        if (ctx->stage_event[k]) (void)hipEventDestroy(ctx->stage_event[k]);
    }
    if (ctx->order_ws) (void)hipFree(ctx->order_ws);
    if (ctx->decl_stream) (void)hipStreamDestroy(ctx->decl_stream);
    if (ctx->beside) (void)hipStreamDestroy(ctx->beside);
    if (ctx->aux_stream) (void)hipStreamDestroy(ctx->aux_stream);
    if (ctx->seg_base_dev) (void)hipFree(ctx->seg_base_dev);
    if (ctx->host_plan) (void)hipHostFree(ctx->host_plan);
    delete ctx;
    return TENT_OK;
}

int tent_register_segment(tent_ctx* ctx, void* dev_base, uint64_t len, uint32_t* seg_out)
{
    if (!ctx || !dev_base || len == 0 || !seg_out) return TENT_ERR_INVALID;
    if (ctx->segments.size() >= ctx->seg_capacity) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    const uint32_t id = (uint32_t)ctx->segments.size();
    const uint64_t addr = (uint64_t)dev_base;
    try { ctx->segments.reserve(ctx->segments.size() + 1); } catch (const std::bad_alloc&) { return TENT_ERR_NOMEM; }
    HIP_TRY(hipMemcpy(ctx->seg_base_dev + id, &addr, sizeof(addr), hipMemcpyHostToDevice));
    ctx->segments.push_back({static_cast<uint8_t*>(dev_base), len});
    *seg_out = id;
    return TENT_OK;
}

int tent_declare(tent_ctx* ctx, uint32_t n_desc, const uint32_t* src_ptr, const tent_extent* src_ext,
                 const uint32_t* dst_ptr, const tent_extent* dst_ext, tent_batch_t* out)
{
    return declare_impl(ctx, n_desc, src_ptr, src_ext, dst_ptr, dst_ext, out, false);
}

int tent_declare_static(tent_ctx* ctx, uint32_t n_desc, const uint32_t* src_ptr, const tent_extent* src_ext,
                        const uint32_t* dst_ptr, const tent_extent* dst_ext, tent_batch_t* out)
{
    return declare_impl(ctx, n_desc, src_ptr, src_ext, dst_ptr, dst_ext, out, true);
}

int tent_plan(tent_ctx* ctx, tent_batch_t batch, const tent_rail_state* rails, uint32_t n_rails,
              tent_plan_info* info, void* stream)
{
    if (!ctx || !rails) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (b->broken) return TENT_ERR_STATE;
    if (n_rails == 0 || n_rails > ctx->max_rails) return TENT_ERR_RANGE;
    RailParams rp;
    int rc = convert_rails(rails, n_rails, b->payload, &rp);
    if (rc != TENT_OK) return rc;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool too_small = !(ctx->cfg.flags & TENT_FLAG_BOUNDED_STAGING) && b->payload + 256ull * n_rails > ctx->cfg.staging_bytes;
    if (rp.admitted == 0 || too_small || capturing(s)) {
        rc = finish_declare(ctx, *b);
        if (rc != TENT_OK) return rc;
        if (rp.admitted == 0) return TENT_DEFER;
        if (too_small) return TENT_ERR_RANGE;
    }
    const BatchDev& d = b->dev;
    s = work_stream(ctx, *b, s, !b->has_done && !b->has_retry, info != nullptr);
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    if (b->decl_pending) HIP_TRY(hipStreamWaitEvent(s, b->decl_event, 0));
    HIP_TRY(order_after_execute_bookkeeping(*b, s, !b->has_done && !b->has_retry));
    b->last = s == b->beside ? Batch::Last::kBeside : Batch::Last::kCaller;

    // Retry rotation (Section 4.3, "Link-Level Resilience"): candidates are the HEALTHY rails, else the
    // DEGRADED rails without topology penalty, else every DEGRADED rail, in ascending index.
    RotateParams rot;
    std::memset(&rot, 0, sizeof(rot));
    if (b->has_retry) {
        for (int pass = 0; pass < 3 && rot.n_cand == 0; ++pass)
            for (uint32_t r = 0; r < n_rails; ++r) {
                const bool take = pass == 0 ? rails[r].health == 0
                                : pass == 1 ? rails[r].health == 1 && rails[r].penalty_q8 <= 256
                                            : rails[r].health == 1;
                if (take) rot.cand[rot.n_cand++] = (uint8_t)r;
            }
    }

    const bool replan = b->has_done || b->has_retry;
    // the run-parallel chain divides by c1, so a rail whose cost does not grow with bytes
    // (c1 = 0) sends the plan down the slice-by-slice kernel
    bool serial = (ctx->cfg.flags & TENT_FLAG_SERIAL_BINDING) != 0;
    for (uint32_t r = 0; r < n_rails; ++r)
        if (((rp.admitted >> r) & 1) && rp.c1[r] == 0) serial = true;
    const bool small = !replan && !serial && plan_is_small(d);
    const Report told = next_report(ctx, info && !serial);
    if (small) {
        // one launch does it all and counts as binding (so does a caller that asks for the time of every stage see it)
        StageTimer t(ctx, TENT_T_BIND, s);
        HIP_TRY(launch_plan_small(d, rp, told, s));
    } else if (!replan) {
        // the tile tables of the copy kernels are built beside the binding chain, in its launch
        // (the slice-by-slice binder has no such launch: there they are built here)
        rc = split(ctx, d, serial, s);
        if (rc != TENT_OK) return rc;
    } else {
        StageTimer t(ctx, TENT_T_COMPACT, s);
        HIP_TRY(launch_compact(d, s));
    }
    int mode = replan ? kBindUsePending : 0;
    if (b->has_retry) {
        StageTimer t(ctx, TENT_T_BIND, s);
        HIP_TRY(launch_rotate(d, rot, s));
        mode |= kBindAfterRotation;
    }
    if (!small) {
        StageTimer t(ctx, TENT_T_BIND, s);
        if (serial) HIP_TRY(launch_bind_serial(d, rp, mode, s));
        else        HIP_TRY(launch_bind_runs(d, rp, mode | (replan ? 0 : kBindBuildTables), told, s));
    }
    // Only a batch whose verdict has been read counts as planned: an execute relies on there being no overlap.
    rc = finish_declare_behind(ctx, *b, s);
    if (rc != TENT_OK) return rc;
    b->planned = true;
    b->may_replan = false;                                    // every pending slice is BOUND now
    b->chain_steps = b->records;
    b->bound_hint = b->dev.n_slices;
    b->tile_hint = ~0ull;
    b->last_rails = rp;
    for (uint32_t r = 0; r < n_rails; ++r) b->last_lat_ns[r] = rails[r].lat_ns;

    if (info) {
        if (serial) {
            HIP_TRY(hipMemcpyAsync(ctx->host_plan, d.plan, sizeof(PlanState), hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
        } else {
            HIP_TRY(await_report(*b, told, s, note));
        }
        const PlanState& ps = *ctx->host_plan;
        std::memset(info, 0, sizeof(*info));
        b->bound_hint = ps.n_bound;
        info->n_slices = ps.n_bound;
        info->n_pending_before = ps.n_pending;
        for (uint32_t r = 0; r < TENT_MAX_RAILS; ++r) {
            info->rail_bytes[r] = ps.T[r];
            info->rail_slices[r] = ps.cnt[r];
            info->queued_after[r] = r < n_rails ? ps.A_after[r] : 0;
            info->stage_base[r] = r < n_rails ? ps.base[r] : 0;
        }
    }
    return TENT_OK;
}

int tent_plan_dispatch(tent_ctx* ctx, tent_batch_t batch, const tent_rail_state* rails, uint32_t n_rails,
                       const tent_dispatch_params* params, const uint8_t* priority, tent_dispatch_info* info,
                       void* stream)
{
    if (!ctx || !rails || !params) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (b->broken) return TENT_ERR_STATE;
    if (n_rails == 0 || n_rails > ctx->max_rails) return TENT_ERR_RANGE;
    if (params->gamma_q8 > 65535u) return TENT_ERR_RANGE;
    RailParams rp;
    int rc = convert_rails(rails, n_rails, b->payload, &rp);
    if (rc != TENT_OK) return rc;
    {
        DeviceGuard g0(ctx->device);
        if (!g0.ok) return TENT_ERR_HIP;
        rc = finish_declare(ctx, *b);
        if (rc != TENT_OK) return rc;
    }
    if (rp.admitted == 0) return TENT_DEFER;
    if (!(ctx->cfg.flags & TENT_FLAG_BOUNDED_STAGING) && b->payload + 256ull * n_rails > ctx->cfg.staging_bytes)
        return TENT_ERR_RANGE;
    const uint32_t n_desc = b->dev.n_desc;
    const bool by_bits = priority && n_desc <= kPriorityBits;
    PriorityBits bits;
    std::memset(&bits, 0, sizeof(bits));
    if (priority)
        for (uint32_t j = 0; j < n_desc; ++j) {
            if (priority[j] > 2) return TENT_ERR_INVALID;
            if (by_bits) bits.word[j / 16] |= (uint32_t)priority[j] << (2 * (j % 16));
        }
    // The slot keys (m + 1) * s_d are packed with a 6-bit rail index and the tolerance multiplies a
    // cost by gamma: bound the largest cost any rail can show during this plan.
    DispatchParams dp;
    std::memset(&dp, 0, sizeof(dp));
    {
        unsigned __int128 worst = 0;
        for (uint32_t d = 0; d < n_rails; ++d) {
            if (!((rp.admitted >> d) & 1)) continue;
            const unsigned __int128 c = (unsigned __int128)rp.c0[d] +
                                        ((((unsigned __int128)rp.A[d] + b->payload) * rp.c1[d]) >> 16);
            worst = std::max(worst, c);
        }
        if (worst * (b->max_req_slices + 1) >= ((unsigned __int128)1 << 57)) return TENT_ERR_RANGE;
        if (worst * (params->gamma_q8 + 1u) >= ((unsigned __int128)1 << 63)) return TENT_ERR_RANGE;
        dp.near = n_rails <= 16 && dispatch_is_near(worst, b->max_req_slices) ? 1u : 0u;
    }
    dp.theta = params->theta_bytes;
    dp.rr_start = params->rr_start;
    dp.gamma_q8 = params->gamma_q8;
    // Priority slots (Section 4.2, "Quality of Service"): in window w rail d sits in slot (w + d) mod 3;
    // slot 0 takes HIGH only, slot 1 HIGH and MID, slot 2 everything.
    for (uint32_t d = 0; d < n_rails; ++d) {
        if (!((rp.admitted >> d) & 1)) continue;
        const uint32_t slot = (uint32_t)(((uint64_t)params->window + d) % 3);
        const uint32_t lowest = slot == 0 ? 2 : slot == 1 ? 1 : 0;
        for (uint32_t p = lowest; p <= 2; ++p) dp.adm[p] |= 1ull << d;
    }

    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    const bool first_plan = !b->planned;
    const hipStream_t s = work_stream(ctx, *b, static_cast<hipStream_t>(stream), first_plan, info != nullptr);
    const BatchDev& d = b->dev;
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    HIP_TRY(order_after_execute_bookkeeping(*b, s, first_plan));
    b->last = s == b->beside ? Batch::Last::kBeside : Batch::Last::kCaller;
    dp.all_high = priority ? 0u : 1u;
    dp.all_pending = first_plan ? 1u : 0u;
    dp.by_bits = by_bits ? 1u : 0u;
    if (priority && !by_bits) HIP_TRY(hipMemcpyAsync(d.priority, priority, d.n_desc, hipMemcpyHostToDevice, s));
    const Report told = next_report(ctx, info != nullptr);
    if (first_plan) {
        rc = split(ctx, d, false, s);
        if (rc != TENT_OK) return rc;
    }
    {
        StageTimer t(ctx, TENT_T_BIND, s);
        HIP_TRY(launch_dispatch(d, rp, dp, bits, first_plan, told, s));
    }
    b->planned = true;
    b->may_replan = true;                                     // deferred transfers stay pending
    b->chain_steps = n_desc;
    b->bound_hint = b->dev.n_slices;
    b->tile_hint = ~0ull;
    b->last_rails = rp;
    for (uint32_t r = 0; r < n_rails; ++r) b->last_lat_ns[r] = rails[r].lat_ns;

    if (info) {
        HIP_TRY(await_report(*b, told, s, note));
        const PlanState& ps = *ctx->host_plan;
        std::memset(info, 0, sizeof(*info));
        b->bound_hint = ps.n_bound;
        info->plan.n_slices = ps.n_bound;
        info->plan.n_pending_before = ps.n_pending;
        for (uint32_t r = 0; r < n_rails; ++r) {
            info->plan.rail_bytes[r] = ps.T[r];
            info->plan.rail_slices[r] = ps.cnt[r];
            info->plan.queued_after[r] = ps.A_after[r];
            info->plan.stage_base[r] = ps.base[r];
        }
        info->n_mice = ps.n_mice;
        info->n_elephant = ps.n_elephant;
        info->n_deferred = ps.n_deferred;
        info->rr_next = ps.rr_next;
    }
    return TENT_OK;
}

int tent_get_modes(tent_ctx* ctx, tent_batch_t batch, uint8_t* host_out, uint64_t cap)
{
    if (!ctx || !host_out) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (cap < b->dev.n_desc) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(host_out, b->dev.req_mode, b->dev.n_desc, hipMemcpyDeviceToHost));
    return TENT_OK;
}

int tent_sim_advance(tent_ctx* ctx, tent_batch_t batch, const uint64_t* budget_bytes, uint64_t* n_done,
                     void* stream)
{
    if (!ctx || !budget_bytes) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned) return TENT_ERR_STATE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    const hipStream_t s = work_stream(ctx, *b, static_cast<hipStream_t>(stream), false, n_done != nullptr);
    BudgetParams bp;
    std::memset(&bp, 0, sizeof(bp));
    for (uint32_t d = 0; d < b->last_rails.n_rails; ++d) {
        bp.queued[d] = b->last_rails.A[d];
        bp.budget[d] = budget_bytes[d];
    }
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    if (s == b->beside) HIP_TRY(order_after_execute_bookkeeping(*b, s));
    b->last = s == b->beside ? Batch::Last::kBeside : Batch::Last::kCaller;
    b->may_replan = true;
    const Report told = next_report(ctx, n_done != nullptr);
    HIP_TRY(launch_retire(b->dev, bp, told, s));
    // What stays BOUND on rail d fits in budget_d - queued_d bytes, which bounds the tiles the next execute
    // copies without asking the device (slices of a tiled batch are whole tiles).
    uint64_t tiles = 0;
    for (uint32_t d = 0; d < b->last_rails.n_rails; ++d)
        if (bp.budget[d] > bp.queued[d]) tiles += (bp.budget[d] - bp.queued[d]) / (b->dev.tile_bytes ? b->dev.tile_bytes : 1u);
    b->tile_hint = tiles;
    if (!n_done) return TENT_OK;
    HIP_TRY(await_report(*b, told, s, note));
    b->bound_hint = ctx->host_plan->n_done;
    *n_done = ctx->host_plan->n_done;
    return TENT_OK;
}

int tent_sim_fail(tent_ctx* ctx, tent_batch_t batch, const uint8_t* rail_failed, uint64_t* failed_per_rail,
                  void* stream)
{
    if (!ctx || !rail_failed) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned) return TENT_ERR_STATE;
    const uint32_t n_rails = b->last_rails.n_rails;
    FailParams fp;
    std::memset(&fp, 0, sizeof(fp));
    bool any = false;
    for (uint32_t d = 0; d < n_rails; ++d) {
        fp.failed[d] = rail_failed[d] ? 1 : 0;
        any = any || rail_failed[d];
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    const hipStream_t s = work_stream(ctx, *b, static_cast<hipStream_t>(stream), false, any && failed_per_rail);
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    const Report told = next_report(ctx, any && failed_per_rail);
    if (any) {
        if (s == b->beside) HIP_TRY(order_after_execute_bookkeeping(*b, s));
        b->last = s == b->beside ? Batch::Last::kBeside : Batch::Last::kCaller;
        b->may_replan = true;
        HIP_TRY(launch_fail(b->dev, fp, told, s));
        b->has_retry = true;
    }
    if (failed_per_rail) {
        for (uint32_t d = 0; d < n_rails; ++d) failed_per_rail[d] = 0;
        if (any) {
            HIP_TRY(await_report(*b, told, s, note));
            for (uint32_t d = 0; d < n_rails; ++d) failed_per_rail[d] = ctx->host_plan->fail_cnt[d];
        }
    }
    return TENT_OK;
}

int tent_get_retries(tent_ctx* ctx, tent_batch_t batch, uint8_t* host_out, uint64_t cap)
{
    if (!ctx || !host_out) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (cap < b->dev.n_slices) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(host_out, b->dev.s_retry, b->dev.n_slices, hipMemcpyDeviceToHost));
    return TENT_OK;
}

int tent_sim_latency(tent_ctx* ctx, tent_batch_t batch, const uint32_t* true_bw_MBps, void* stream)
{
    if (!ctx || !true_bw_MBps) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned) return TENT_ERR_STATE;
    LatencyParams lp;
    std::memset(&lp, 0, sizeof(lp));
    uint64_t max_q = 0;
    for (uint32_t d = 0; d < TENT_MAX_RAILS; ++d) lp.bw_MBps[d] = 1;
    for (uint32_t d = 0; d < b->last_rails.n_rails; ++d) {
        if (true_bw_MBps[d] == 0) return TENT_ERR_RANGE;
        lp.queued[d] = b->last_rails.A[d];
        lp.lat_ns[d] = b->last_lat_ns[d];
        lp.bw_MBps[d] = true_bw_MBps[d];
        max_q = std::max(max_q, lp.queued[d]);
    }
    if (max_q >= (1ull << 53) || b->payload >= (1ull << 53) || max_q + b->payload >= (1ull << 53)) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    const hipStream_t s = work_stream(ctx, *b, static_cast<hipStream_t>(stream), false, false);
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    if (s == b->beside) HIP_TRY(order_after_execute_bookkeeping(*b, s));
    b->last = s == b->beside ? Batch::Last::kBeside : Batch::Last::kCaller;
    HIP_TRY(launch_sim_latency(b->dev, lp, s));
    return TENT_OK;
}

int tent_update_bandwidth(tent_ctx* ctx, tent_batch_t batch, const tent_probe_params* params, tent_rail_state* rails,
                          uint32_t n_rails, uint32_t* probe_MBps_out, void* stream)
{
    if (!ctx || !params || !rails) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned) return TENT_ERR_STATE;
    if (n_rails != b->last_rails.n_rails) return TENT_ERR_RANGE;
    ProbeParams pp;
    std::memset(&pp, 0, sizeof(pp));
    pp.n_rails = n_rails;
    for (uint32_t d = 0; d < n_rails; ++d) {
        if (params[d].alpha_q8 > 65535u || params[d].ewma_q8 > 256u) return TENT_ERR_RANGE;
        pp.cal[d] = params[d];
        pp.bw_MBps[d] = rails[d].bw_MBps;
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(order_after_report(*b, s));
    const Report told = next_report(ctx, true);
    {
        StageTimer t(ctx, TENT_T_FEEDBACK, s);
        HIP_TRY(launch_probe(b->dev, pp, told, s));
    }
    HIP_TRY(await_figures(told, s));
    for (uint32_t d = 0; d < n_rails; ++d) {
        rails[d].bw_MBps = ctx->host_plan->bw_next[d];
        if (probe_MBps_out) probe_MBps_out[d] = ctx->host_plan->probe[d];
    }
    return TENT_OK;
}

int tent_get_latencies(tent_ctx* ctx, tent_batch_t batch, uint64_t* host_out, uint64_t cap)
{
    if (!ctx || !host_out) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned) return TENT_ERR_STATE;
    if (cap < b->dev.n_slices) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(host_out, b->dev.s_tau, b->dev.n_slices * sizeof(uint64_t), hipMemcpyDeviceToHost));
    return TENT_OK;
}

int tent_execute(tent_ctx* ctx, tent_batch_t batch, void* stream)
{
    if (!ctx) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned || b->broken) return TENT_ERR_STATE;
    if (b->payload + 256ull * b->last_rails.n_rails > ctx->cfg.staging_bytes) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    b->last = Batch::Last::kCaller;
    // When the host knows that only a small part of the batch is BOUND (after the rail simulator), the
    // copies run over a list of the tiles of the BOUND slices and their launches are sized by that part.
    uint64_t max_tiles = b->bound_hint * b->dev.tiles_per_slice;
    if (b->tile_hint < max_tiles) max_tiles = b->tile_hint;
    const bool compact = b->dev.n_sc_tiles != 0 && max_tiles * 2 <= b->dev.n_sc_tiles;
    // The copies below are driven by the tables that the bookkeeping writes and read no slice state, so the slices
    // are marked DONE ahead of them: in stream order nothing changes, and the next re-plan, if it
    // is enqueued on another stream, can run beside the copies.  tent_poll, on whatever stream, waits
    // for the end of the copies (done_at), so a slice is never reported complete while its bytes move.
    uint8_t* arena = static_cast<uint8_t*>(ctx->cfg.staging_arena);
    if (b->dev.one_pass) {
        HIP_TRY(launch_stage_and_mark(b->dev, arena, compact, max_tiles, s));
    } else {
        HIP_TRY(launch_finalize(b->dev, arena, compact, max_tiles, s));
        HIP_TRY(launch_mark_done(b->dev, compact, s));
    }
    // From here on a failure would leave slices marked DONE whose bytes were never moved: the batch
    // is then flagged, and every call but tent_reset and tent_release refuses it.
    auto record_end = [&]() -> hipError_t {
        hipError_t e = record_execute_done(*b, s, note);
        if (e == hipSuccess && b->done_recorded && !b->replan_at) b->replan_at = b->done_at;
        return e;
    };
    auto copies = [&]() -> hipError_t {
        hipError_t e = record_execute_bookkeeping(*b, s);
        if (e != hipSuccess) return e;
        if (b->dev.one_pass) {
            StageTimer t(ctx, TENT_T_GATHER, s);
            e = launch_copy_one_pass(b->dev, compact, max_tiles, s);
            if (e != hipSuccess) return e;
            return record_end();
        }
        {
            StageTimer t(ctx, TENT_T_GATHER, s);
            e = compact ? launch_copy_compact(b->dev, true, max_tiles, s)
                : b->dev.n_sc_tiles ? launch_copy_ordered(b->dev, true, s) : launch_copy(b->dev, true, s);
        }
        if (e != hipSuccess) return e;
        {
            StageTimer t(ctx, TENT_T_SCATTER, s);
            e = compact ? launch_copy_compact(b->dev, false, max_tiles, s)
                : b->dev.n_sc_tiles ? launch_copy_ordered(b->dev, false, s) : launch_copy(b->dev, false, s);
        }
        if (e != hipSuccess) return e;
        return record_end();
    };
    b->has_done = true;
    b->bound_hint = 0;
    b->execute_bytes = max_tiles < b->payload / b->dev.tile_bytes ? max_tiles * b->dev.tile_bytes : b->payload;
    const bool moved = copies() == hipSuccess;
    note_execute(ctx, *b, s);
    if (!moved) {
        (void)hipGetLastError();
        b->broken = true;
        return TENT_ERR_HIP;
    }
    return TENT_OK;
}

int tent_execute_bounded(tent_ctx* ctx, tent_batch_t batch, uint64_t chunk_bytes, uint32_t slots, void* stream)
{
    if (!ctx) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned || b->broken || !(ctx->cfg.flags & TENT_FLAG_BOUNDED_STAGING)) return TENT_ERR_STATE;
    const BatchDev& d = b->dev;
    // chunks are cut on 1 MiB boundaries, so that the 256 consecutive tiles of a workgroup of the tables' kernels lie in one chunk and
    // a chunk begins with a whole tile or range (a workgroup of bounded_ranges_kernel may reach into several chunks)
    if (chunk_bytes == 0 || (chunk_bytes & ((1ull << 20) - 1)) != 0 || slots < 1 || slots > 2) return TENT_ERR_INVALID;
    const uint64_t slot_bytes = chunk_bytes + 256ull * b->last_rails.n_rails;
    if (slot_bytes > ctx->cfg.staging_bytes / slots) return TENT_ERR_RANGE;
    const uint64_t n_chunks = (b->payload + chunk_bytes - 1) / chunk_bytes;
    if (n_chunks > kMaxChunks) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(order_after_report(*b, s));
    StreamNote note(*b, s);
    b->last = Batch::Last::kCaller;
    uint8_t* arena = static_cast<uint8_t*>(ctx->cfg.staging_arena);
    const uint64_t payload = b->payload;
    HIP_TRY(launch_bounded_prepare(d, chunk_bytes, (uint32_t)n_chunks, slot_bytes, slots, arena, s));
    if (d.one_pass) {
        // both directions of a chunk in one launch; a chunk's launch ends before the next one may reuse its slot
        for (uint32_t c = 0; c < n_chunks; ++c) {
            StageTimer t(ctx, TENT_T_GATHER, s);
            HIP_TRY(launch_bounded_copy(d, true, c, payload, chunk_bytes, slot_bytes, slots, arena, s));
        }
    } else if (slots == 1) {
        for (uint32_t c = 0; c < n_chunks; ++c) {
            {
                StageTimer t(ctx, TENT_T_GATHER, s);
                HIP_TRY(launch_bounded_copy(d, true, c, payload, chunk_bytes, slot_bytes, slots, arena, s));
            }
            {
                StageTimer t(ctx, TENT_T_SCATTER, s);
                HIP_TRY(launch_bounded_copy(d, false, c, payload, chunk_bytes, slot_bytes, slots, arena, s));
            }
        }
    } else {
        // Two slots: gathers stay on the caller's stream, scatters go to a second stream.  Scatter c
        // waits for gather c; gather c + 2 waits for scatter c, which frees its slot; gather c + 1
        // overlaps scatter c (Section 4.1: consecutive stages of the staging pipeline overlap).
        if (!ctx->aux_stream && hipStreamCreateWithFlags(&ctx->aux_stream, hipStreamNonBlocking) != hipSuccess) {
            (void)hipGetLastError();
            ctx->aux_stream = nullptr;
            return TENT_ERR_HIP;
        }
        try {
            while (ctx->sync_events.size() < 2 * n_chunks + 1) {
                hipEvent_t e = nullptr;
                if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                    (void)hipGetLastError();
                    return TENT_ERR_HIP;
                }
                ctx->sync_events.push_back(e);
            }
        } catch (const std::bad_alloc&) { return TENT_ERR_NOMEM; }
        hipStream_t x = ctx->aux_stream;
        hipEvent_t prepared = ctx->sync_events[2 * n_chunks];
        HIP_TRY(hipEventRecord(prepared, s));
        HIP_TRY(hipStreamWaitEvent(x, prepared, 0));
        for (uint32_t c = 0; c < n_chunks; ++c) {
            hipEvent_t gathered = ctx->sync_events[2 * c], scattered = ctx->sync_events[2 * c + 1];
            if (c >= 2) HIP_TRY(hipStreamWaitEvent(s, ctx->sync_events[2 * (c - 2) + 1], 0));
            {
                StageTimer t(ctx, TENT_T_GATHER, s);
                HIP_TRY(launch_bounded_copy(d, true, c, payload, chunk_bytes, slot_bytes, slots, arena, s));
            }
            HIP_TRY(hipEventRecord(gathered, s));
            HIP_TRY(hipStreamWaitEvent(x, gathered, 0));
            {
                StageTimer t(ctx, TENT_T_SCATTER, x);
                HIP_TRY(launch_bounded_copy(d, false, c, payload, chunk_bytes, slot_bytes, slots, arena, x));
            }
            HIP_TRY(hipEventRecord(scattered, x));
        }
        // the caller's stream continues once every scatter has finished
        HIP_TRY(hipStreamWaitEvent(s, ctx->sync_events[2 * (n_chunks - 1) + 1], 0));
        if (n_chunks >= 2) HIP_TRY(hipStreamWaitEvent(s, ctx->sync_events[2 * (n_chunks - 2) + 1], 0));
    }
    HIP_TRY(launch_mark_done_bounded(d, s));
    b->replan_at = nullptr;
    b->has_done = true;
    b->bound_hint = 0;
    HIP_TRY(record_execute_done(*b, s, note));
    // the range copies read what a re-plan rewrites, and the DONE marks come last: a re-plan on another stream waits for it all
    if (b->done_recorded) b->replan_at = b->done_at;
    note_execute(ctx, *b, s, n_chunks > kBesideChunks + b->chain_steps / kChunkSteps);
    return TENT_OK;
}

int tent_poll(tent_ctx* ctx, tent_batch_t batch, uint64_t* remaining, void* stream)
{
    if (!ctx || !remaining) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (b->broken) return TENT_ERR_STATE;
    if (!b->planned) { *remaining = b->dev.n_slices; return TENT_OK; }
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(order_after_report(*b, s));
    // slices are marked DONE ahead of their copies: completion is only reported once the last
    // execute's copies have ended, whichever stream the caller polls on
    if (b->done_recorded && s != b->exec_stream) HIP_TRY(hipStreamWaitEvent(s, b->done_at, 0));
    const Report told = next_report(ctx, true);
    HIP_TRY(launch_count_remaining(b->dev, told, s));
    bool looked = false;
    HIP_TRY(await_figures(told, s, &looked));
    const uint64_t left = ctx->host_plan->n_remaining;
    // The figure says that the copies have ended, not that what they wrote has left the caches: that is what the event behind them, or
    // the stream's end, waits for.
    if (left == 0 && looked) HIP_TRY(b->done_recorded && !b->marks_lost ? hipEventSynchronize(b->done_at) : hipStreamSynchronize(s));
    *remaining = left;
    return TENT_OK;
}

int tent_reset(tent_ctx* ctx, tent_batch_t batch, void* stream)
{
    if (!ctx) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    // The next plan writes the slice table afresh, states included, and nothing looks at it before.  What else a reset clears are the
    // retry counts, so without any there is nothing to launch -- in a graph, whose replays other calls come between, there always is.
    // (MI355X: 74 slices, cycles of three batches in turn 32 -> 30 us and alone 52 -> 47.5, 80 slices of 1 MiB 58 -> 52 and 98 -> 84.)
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (b->planned && !b->has_retry && !b->broken && !b->marks_lost && !b->report_at && !capturing(s)) {
        if (b->done_recorded && s != b->exec_stream) HIP_TRY(hipStreamWaitEvent(s, b->done_at, 0));
    } else {
        s = work_stream(ctx, *b, s, true, false);
        if (b->planned || s != b->beside) HIP_TRY(order_after_report(*b, s));
        if (b->planned) {
            StreamNote note(*b, s);
            b->last = s == b->beside ? Batch::Last::kBeside : Batch::Last::kCaller;
            // the reset must not overtake the copies of an execute that runs on another stream
            if (b->done_recorded && s != b->exec_stream && !capturing(s)) HIP_TRY(hipStreamWaitEvent(s, b->done_at, 0));
            HIP_TRY(launch_reset(b->dev, s));
        }
    }
    b->planned = false;
    b->has_done = false;
    b->has_retry = false;
    b->broken = false;
    return TENT_OK;
}

int tent_slice_count(tent_ctx* ctx, tent_batch_t batch, uint64_t* n_slices)
{
    if (!ctx || !n_slices) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    *n_slices = b->dev.n_slices;
    return TENT_OK;
}

int tent_get_plan(tent_ctx* ctx, tent_batch_t batch, tent_slice* host_out, uint64_t cap)
{
    if (!ctx || !host_out) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    if (!b->planned) return TENT_ERR_STATE;
    const BatchDev& d = b->dev;
    const uint64_t n = d.n_slices;
    if (cap < n) return TENT_ERR_RANGE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    HIP_TRY(hipDeviceSynchronize());
    std::vector<uint32_t> desc, len, rail;
    std::vector<uint64_t> off, stage;
    std::vector<uint8_t> state;
    try {
        desc.resize(n); len.resize(n); rail.resize(n); off.resize(n); stage.resize(n); state.resize(n);
    } catch (const std::bad_alloc&) { return TENT_ERR_NOMEM; }
    HIP_TRY(hipMemcpy(desc.data(), d.s_desc, n * 4, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(len.data(), d.s_len, n * 4, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(rail.data(), d.s_rail, n * 4, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(off.data(), d.s_off, n * 8, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(stage.data(), d.s_stage_off, n * 8, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(state.data(), d.s_state, n, hipMemcpyDeviceToHost));
    for (uint64_t i = 0; i < n; ++i)
        host_out[i] = tent_slice{desc[i], len[i], off[i], stage[i], rail[i], state[i]};
    return TENT_OK;
}

int tent_get_timings(tent_ctx* ctx, float* ms_out, uint32_t* launches_out)
{
    if (!ctx || !ms_out || !launches_out) return TENT_ERR_INVALID;
    if (!(ctx->cfg.flags & TENT_FLAG_PROFILE)) return TENT_ERR_STATE;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    int rc = TENT_OK;
    for (int st = 0; st < TENT_T_COUNT; ++st) {
        Timing& t = ctx->timing[st];
        double total = 0.0;
        for (size_t k = 0; k < t.used; ++k) {
            float ms = 0.0f;
            if (hipEventSynchronize(t.pool[k].second) != hipSuccess ||
                hipEventElapsedTime(&ms, t.pool[k].first, t.pool[k].second) != hipSuccess) {
                (void)hipGetLastError();
                rc = TENT_ERR_HIP;
            }
            total += ms;
        }
        ms_out[st] = (float)total;
        launches_out[st] = (uint32_t)t.used;
        t.used = 0;
    }
    return rc;
}

int tent_release(tent_ctx* ctx, tent_batch_t batch)
{
    if (!ctx) return TENT_ERR_INVALID;
    Batch* b = find_batch(ctx, batch);
    if (!b) return TENT_ERR_INVALID;
    DeviceGuard g(ctx->device);
    if (!g.ok) return TENT_ERR_HIP;
    wait_batch_idle(*b);
    free_batch(ctx, *b);
    return TENT_OK;
}

}  // extern "C"
