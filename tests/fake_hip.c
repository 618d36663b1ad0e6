/* A HIP runtime without a device, for tests of the library's host side: memory is host memory, launches do nothing, and
 * every launch, event and wait is written to a log with its stream.  Loaded in place of libamdhip64 by a child process. */
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

enum { LAUNCH = 1, RECORD = 2, WAIT = 3, HOST_WAIT = 4, COPY = 5 };
enum { MOST = 1 << 16, KERNELS = 512 };

static struct { int kind; void *stream, *what; } log_[MOST];
static int n_log, n_kernels, fail_host_waits;
static struct { const void *fn; const char *name; } kernel[KERNELS];
static void *capturing_stream, *termed_stream;
static int termed_priority;
static uint32_t termed_mask;
static int answer, n_host, busy;
static struct { char *at; size_t n; } host[64];

static void note(int kind, void *stream, void *what)
{
    if (n_log < MOST) { log_[n_log].kind = kind; log_[n_log].stream = stream; log_[n_log].what = what; ++n_log; }
}

/* ---- for the tests ---- */
int fake_log_size(void) { return n_log; }
void fake_log_clear(void) { n_log = 0; }
int fake_log_at(int i, void **stream, void **what)
{
    *stream = log_[i].stream;
    *what = log_[i].what;
    return log_[i].kind;
}
const char *fake_kernel_name(const void *fn)
{
    for (int k = 0; k < n_kernels; ++k) if (kernel[k].fn == fn) return kernel[k].name;
    return "";
}
void fake_fail_host_waits(int n) { fail_host_waits = n; }
void fake_capture(void *stream) { capturing_stream = stream; }
/* the one stream that has a priority or whose first word of compute units is not full */
void fake_terms(void *stream, int priority, unsigned mask) { termed_stream = stream; termed_priority = priority; termed_mask = mask; }
/* whether what has been enqueued has not ended yet */
void fake_busy(int on) { busy = on; }
/* a launch that reports answers its report, a block of host memory and a number: the number goes to the block's last word (1), with
 * figures that are not zero in front of it (2) */
void fake_answer_reports(int on) { answer = on; }
static const struct { const char *name; int arg; } reporter[] = {
    {"plan_small_kernel", 2}, {"dispatch_emit_kernel", 3}, {"retire_kernel", 2}, {"fail_kernel", 2}, {"probe_kernel", 2}, {"count_remaining_kernel", 1},
};

/* ---- the runtime ---- */
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
int hipGetStreamDeviceId(hipStream_t s) { (void)s; return 0; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int d)
{
    (void)d;
    memset(p, 0, sizeof(*p));
    strcpy(p->gcnArchName, "gfx950");
    p->warpSize = 64;
    p->multiProcessorCount = 256;
    p->maxThreadsPerBlock = 1024;
    return hipSuccess;
}

/* the library writes from the host to the first part of an allocation only, so a large one need not be there as a whole */
static void *map(size_t n)
{
    const size_t most = (size_t)1 << 32;
    void *p = mmap(NULL, n < most ? n : most, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return p == MAP_FAILED ? NULL : p;
}
hipError_t hipMalloc(void **p, size_t n) { *p = map(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { (void)p; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags)
{
    (void)flags;
    *p = calloc(n, 1);
    if (n_host < 64) { host[n_host].at = *p; host[n_host].n = n; ++n_host; }
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *symbol)
{
    static void *area;
    (void)symbol;
    if (!area) area = map((size_t)1 << 27);
    *p = area;
    return area ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    note(COPY, st, d);
    return hipMemcpy(d, s, n, k);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) { (void)d; (void)v; (void)n; (void)st; return hipSuccess; }

static hipError_t new_event(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return new_event(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags) { (void)flags; return new_event(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { (void)a; (void)b; *ms = 0; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { note(RECORD, s, e); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned flags) { (void)flags; note(WAIT, s, e); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { (void)e; return busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *mode) { (void)mode; return hipSuccess; }
static hipError_t host_wait(void *stream, void *what)
{
    if (fail_host_waits > 0) { --fail_host_waits; return hipErrorUnknown; }
    note(HOST_WAIT, stream, what);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return host_wait(NULL, e); }
hipError_t hipStreamSynchronize(hipStream_t s) { return host_wait(s, NULL); }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned flags) { (void)flags; *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamGetPriority(hipStream_t s, int *priority)
{
    *priority = s && s == termed_stream ? termed_priority : 0;
    return hipSuccess;
}
hipError_t hipExtStreamGetCUMask(hipStream_t s, uint32_t words, uint32_t *mask)
{
    if (words * 32 < 256) return hipErrorInvalidValue;
    for (uint32_t k = 0; k < words; ++k) mask[k] = 0xFFFFFFFFu;
    if (s && s == termed_stream) mask[0] = termed_mask;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *to, hipDeviceAttribute_t what, int d)
{
    (void)d;
    if (what != hipDeviceAttributeMultiprocessorCount) return hipErrorInvalidValue;
    *to = 256;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    *st = s && s == capturing_stream ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}

static dim3 grid_, block_;
static size_t shared_;
static hipStream_t stream_;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s)
{
    grid_ = g; block_ = b; shared_ = sh; stream_ = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s)
{
    *g = grid_; *b = block_; *sh = shared_; *s = stream_;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **args, size_t sh, hipStream_t s)
{
    (void)g; (void)b; (void)sh;
    note(LAUNCH, s, (void *)fn);
    for (size_t r = 0; answer && r < sizeof(reporter) / sizeof(reporter[0]); ++r) {
        if (!strstr(fake_kernel_name(fn), reporter[r].name)) continue;
        const struct { char *to; unsigned long long call; } *report = args[reporter[r].arg];
        for (int k = 0; k < n_host; ++k)
            if (host[k].at == report->to) {
                memset(host[k].at, answer - 1, host[k].n - 8);
                memcpy(host[k].at + host[k].n - 8, &report->call, 8);
            }
    }
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *data) { static void *handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *fn, char *device_fn, const char *name, unsigned limit, void *tid, void *bid,
                           void *bdim, void *gdim, int *wsize)
{
    (void)h; (void)device_fn; (void)limit; (void)tid; (void)bid; (void)bdim; (void)gdim; (void)wsize;
    if (n_kernels < KERNELS) { kernel[n_kernels].fn = fn; kernel[n_kernels].name = name; ++n_kernels; }
}
void __hipRegisterVar(void **h, void *var, char *host, char *name, int ext, size_t size, int constant, int global)
{
    (void)h; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
