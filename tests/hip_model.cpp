// A model of the HIP runtime for host tests of the library: it lets libca_hip.so run its host code without a GPU and
// records what is queued where.  Nothing queued is done until the host waits for it (the worst case a caller can meet);
// per operation the model knows which other operations must be done before it starts.  Streams are independent of each
// other (non-blocking), every device has a default stream of its own, hipStreamPerThread is one per thread and device.
// Built with the runtime's soname and loaded first, it takes the runtime's place in the process.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "../paper_2403_19708_amd/csrc/ca_internal.h"

namespace {

struct Stream {
    int device;
    std::set<int> behind;      // operations a new one on this stream is behind
    bool alive = true, capturing = false, spoilt = false;      // spoilt: a call that a capture does not survive
};
struct Event {
    int device;
    std::set<int> ops;
    bool captured = false;
    Stream *stream = nullptr;  // it was recorded on
};
struct Op {
    std::string what;
    Stream *stream;
    std::set<int> behind;
    unsigned workgroups;       // kernels: of the grid's first dimension
    std::vector<char> args;    // attention kernels: their AttnArgs; moves: their MoveArgs or MoveArgs2
};
struct Range {
    size_t size;
    hipMemoryType type;
    int device;
    ptrdiff_t device_shift;    // device address - host address
    bool extent_known;
};

std::recursive_mutex lock;
#define MODEL std::lock_guard<std::recursive_mutex> hold(lock)
int n_devices = 2, launches_until_failure = -1, n_cus = 256;
thread_local int current = 0;
std::map<int, Stream *> default_stream;
thread_local std::map<int, Stream *> thread_stream;
std::vector<Op> ops;
std::set<int> done;
std::set<Stream *> streams;
std::map<uintptr_t, Range> ranges;
std::map<const void *, std::string> kernels;

Stream *stream_of(hipStream_t s) {
    if (s == nullptr || s == hipStreamLegacy || s == hipStreamPerThread) {
        Stream *&own = s != hipStreamPerThread ? default_stream[current] : thread_stream[current];
        if (!own) own = new Stream{current};
        return own;
    }
    Stream *x = (Stream *)s;
    return streams.count(x) && x->alive ? x : nullptr;
}
void finish(const std::set<int> &what) {
    for (int op : what)
        if (done.insert(op).second) finish(ops[op].behind);
}
// A call that is not allowed while a stream is under capture (in global mode): unless its thread is in relaxed mode it ends
// the capture.
thread_local hipStreamCaptureMode capture_mode = hipStreamCaptureModeGlobal;
bool spoils() {
    bool any = false;
    if (capture_mode != hipStreamCaptureModeRelaxed)
        for (Stream *s : streams) if (s->capturing) any = s->spoilt = true;
    return any;
}
// its stream has come under capture since the event was recorded: no capture survives being asked about it
bool out_of_reach(const Event *e) { return e->stream && e->stream->capturing && !e->captured; }
bool spoils(const Event *e) {
    if (out_of_reach(e)) e->stream->spoilt = true;
    return spoils() || out_of_reach(e);
}
bool finished(const std::set<int> &what) {
    for (int op : what) if (!done.count(op)) return false;
    return true;
}
int queue(const std::string &what, Stream *s) {
    ops.push_back({what, s, s->behind, 0, {}});
    s->behind.insert((int)ops.size() - 1);
    return (int)ops.size() - 1;
}
const Range *range_of(const void *p, uintptr_t *base = nullptr) {
    auto it = ranges.upper_bound((uintptr_t)p);
    if (it == ranges.begin()) return nullptr;
    --it;
    if ((uintptr_t)p >= it->first + it->second.size) return nullptr;
    if (base) *base = it->first;
    return &it->second;
}
void *allocate(size_t size, hipMemoryType type, ptrdiff_t shift = 0, bool extent_known = true) {
    MODEL;
    void *p = mmap(nullptr, size + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) return nullptr;
    ranges[(uintptr_t)p] = Range{size, type, current, shift, extent_known};
    return p;
}
bool holds(const void *p, size_t bytes) {
    uintptr_t base;
    const Range *r = range_of(p, &base);
    return r && (uintptr_t)p + bytes <= base + r->size;
}

}  // namespace

extern "C" {

// ---- the runtime's functions the library uses ----
hipError_t hipGetDeviceCount(int *n) { *n = n_devices; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { if (d < 0 || d >= n_devices) return hipErrorInvalidDevice; current = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error of the model"; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { std::memset(p, 0, sizeof *p); p->multiProcessorCount = n_cus; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { if (spoils()) return hipErrorStreamCaptureUnsupported; *p = allocate(n, hipMemoryTypeDevice); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = allocate(n, hipMemoryTypeHost); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { MODEL; if (spoils()) return hipErrorStreamCaptureUnsupported; finish([] { std::set<int> all; for (int i = 0; i < (int)ops.size(); ++i) all.insert(i); return all; }()); ranges.erase((uintptr_t)p); return hipSuccess; }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static void *held[64]; if (!held[current]) held[current] = allocate(32 << 20, hipMemoryTypeDevice); *p = held[current]; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t stream) {
    MODEL;
    Stream *x = stream_of(stream);
    if (!x || !holds(d, n) || !holds(s, n)) return hipErrorInvalidValue;
    queue("copy", x);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    MODEL;
    const Range *r = range_of(p);
    if (!r) return hipErrorInvalidValue;
    std::memset(a, 0, sizeof *a);
    a->type = r->type;
    a->device = r->device;
    a->devicePointer = (char *)p + r->device_shift;
    a->hostPointer = r->type == hipMemoryTypeHost ? (void *)p : nullptr;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p) {
    MODEL;
    uintptr_t b;
    const Range *r = range_of(p, &b);
    if (!r || !r->extent_known) return hipErrorNotFound;
    *base = (char *)b + r->device_shift;
    *size = r->size;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { MODEL; Stream *x = new Stream{current}; streams.insert(x); *s = (hipStream_t)x; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { MODEL; Stream *x = stream_of(s); if (!x) return hipErrorInvalidHandle; x->alive = false; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { std::swap(*m, capture_mode); return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) { MODEL; Stream *x = stream_of(s); if (s && spoils()) return hipErrorStreamCaptureUnsupported; if (x && x->capturing) { x->spoilt = true; return hipErrorStreamCaptureUnsupported; } return !x ? hipErrorInvalidHandle : finished(x->behind) ? hipSuccess : hipErrorNotReady; }
hipError_t hipStreamSynchronize(hipStream_t s) { MODEL; Stream *x = stream_of(s); if (s && spoils()) return hipErrorStreamCaptureUnsupported; if (!x) return hipErrorInvalidHandle; finish(x->behind); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) { MODEL; Stream *x = stream_of(s); if (!x) return hipErrorInvalidHandle; *st = x->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipDeviceSynchronize() { MODEL; for (int i = 0; i < (int)ops.size(); ++i) if (ops[i].stream->device == current) finish({i}); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t) new Event{current}; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    MODEL;
    Stream *x = stream_of(s);
    if (!x || x->device != ((Event *)e)->device) return hipErrorInvalidHandle;
    ((Event *)e)->ops = x->behind;
    ((Event *)e)->captured = x->capturing;
    ((Event *)e)->stream = x;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    MODEL;
    Stream *x = stream_of(s);
    if (!x) return hipErrorInvalidHandle;
    if (out_of_reach((Event *)e)) return hipErrorStreamCaptureIsolation;
    if (x->capturing != ((Event *)e)->captured) { x->spoilt |= x->capturing; return hipErrorStreamCaptureIsolation; }
    x->behind.insert(((Event *)e)->ops.begin(), ((Event *)e)->ops.end());
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { MODEL; if (spoils((Event *)e)) return hipErrorStreamCaptureUnsupported; return ((Event *)e)->captured ? hipErrorCapturedEvent : finished(((Event *)e)->ops) ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t e) { MODEL; if (spoils((Event *)e)) return hipErrorStreamCaptureUnsupported; if (((Event *)e)->captured) return hipErrorCapturedEvent; finish(((Event *)e)->ops); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.001f; return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
namespace { thread_local struct { dim3 grid, block; size_t shared; hipStream_t stream; } call; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) { call = {g, b, m, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) { *g = call.grid; *b = call.block; *m = call.shared; *s = call.stream; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t s) {
    MODEL;
    Stream *x = stream_of(s);
    if (!x) return hipErrorInvalidHandle;
    if (launches_until_failure >= 0 && launches_until_failure-- == 0) return hipErrorLaunchFailure;
    const int op = queue(kernels[f], x);
    const std::string &name = ops[op].what;
    ops[op].workgroups = grid.x;
    const size_t bytes = name.find("8AttnArgs") != std::string::npos ? sizeof(ca::AttnArgs)
                         : name.find("9MoveArgs2") != std::string::npos ? sizeof(ca::MoveArgs2)
                         : name.find("8MoveArgs") != std::string::npos ? sizeof(ca::MoveArgs) : 0;
    ops[op].args.assign((char *)args[0], (char *)args[0] + bytes);
    if (name.find("10RebaseArgs") != std::string::npos) {      // its copy of the plan is done, so that a test can read the plan
        const ca::RebaseArgs *a = (const ca::RebaseArgs *)args[0];
        std::memcpy(a->meta, a->image, (size_t)a->image_vecs * 16);
    }
    return hipSuccess;
}

// ---- what the tests ask ----
// kind: 0 device memory, 1 pinned host memory, 2 pinned at another device address, of unknown extent (registered memory)
void *model_alloc(size_t size, int kind) { return allocate(size, kind ? hipMemoryTypeHost : hipMemoryTypeDevice, kind == 2 ? (ptrdiff_t)1 << 40 : 0, kind != 2); }
int model_capture(hipStream_t s, int on) { stream_of(s)->capturing = on; return !stream_of(s)->spoilt; }      // 1: the capture is whole
void model_cus(int n) { n_cus = n; }
void model_fail_launch(int after) { launches_until_failure = after; }
int model_ops() { MODEL; return (int)ops.size(); }
const char *model_what(int op) { MODEL; return ops[op].what.c_str(); }
void *model_stream(int op) { MODEL; return ops[op].stream; }
int model_workgroups(int op) { MODEL; return (int)ops[op].workgroups; }
int model_device(int op) { MODEL; return ops[op].stream->device; }
int model_done(int op) { MODEL; return done.count(op); }
int model_behind(int op, int other) { MODEL; return ops[op].behind.count(other); }
int model_stream_behind(hipStream_t s, int op) { MODEL; return stream_of(s)->behind.count(op); }
int model_streams_alive() { MODEL; int n = 0; for (Stream *s : streams) n += s->alive; return n; }
size_t model_device_bytes() { MODEL; size_t n = 0; for (auto &r : ranges) n += r.second.type == hipMemoryTypeDevice ? r.second.size : 0; return n; }
void *model_attn_pointer(int op, int which) {
    MODEL;
    const ca::AttnArgs *a = (const ca::AttnArgs *)ops[op].args.data();
    return which == 0 ? (void *)a->partial : (void *)a->arrived;
}

// the tier pointers of conversation i of a move (keys, values)
void *model_move_pointer(int op, int i, int values) {
    MODEL;
    if (ops[op].args.size() == sizeof(ca::MoveArgs2)) {
        const ca::MoveArgs2 *a = (const ca::MoveArgs2 *)ops[op].args.data();
        return values ? a->dst_v[i] : a->dst_k[i];
    }
    const ca::MoveArgs *a = (const ca::MoveArgs *)ops[op].args.data();
    return values ? a->contig_v[i] : a->contig_k[i];
}

}  // extern "C"
