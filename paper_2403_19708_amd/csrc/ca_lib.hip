// Host side of the C ABI declared in include/ca.h: argument validation, the context (streams,
// events, staging ring, rotary table, plan metadata) and the stream choreography of the
// layer-wise load / save pipeline (Section 3.2).  Every step of the path itself runs in the
// kernels of ca_move.hip and ca_attn_*.hip; nothing here computes on the CPU except prefix
// sums over the batch (a few dozen integers) and the one-time rotary table.
#include "../../include/ca.h"
#include "ca_internal.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <list>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace ca;

// Partial-result buffer of ca_cached_prefill_attn_static: lives in the code object (one copy per GPU the library
// runs on, held until the process ends), so that entry point needs no allocation anywhere.  The name below is a
// host-side stand-in, not a device address: host code uses the per-device pointer that hipGetSymbolAddress
// returned (static_scratch_ptr), never the array itself.
// Plans cut for their last round only have at most one share to a workgroup place, 256 of 256 rows x 130 floats (32.5 MiB), and
// always fit; others are held to 32 MiB.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20, kStaticArrayBytes = (size_t)34 << 20;
static __device__ __align__(256) uint8_t scratch[kStaticArrayBytes];
constexpr int kMaxDevices = 64;
static void *static_scratch_ptr[kMaxDevices] = {nullptr};   // [device ordinal], filled by ca_create with that device current

// The internal streams (copy-in, unpack, save) of a GPU, shared by the contexts of the process that work behind the same
// stream of the caller: the stream a plan is made on for loads, the one a save follows for saves.  A process has four
// hardware queues here, and streams that share one wait for each other's unfinished work: with three streams per context the
// append of one context's turn sat behind another context's loads as soon as a second context existed (three contexts in
// turn, 236 MB of pinned history each: 6.4 ms a turn, 4.6 ms with one context's three streams).  Contexts behind different
// streams of the caller have streams of their own: an internal stream waits for its caller's, and what another context queued
// behind that wait would wait too (with 16 hardware queues and one of two contexts behind a stream that is busy for 14 ms, the
// other one's turn: 22.8 ms with one set, 5.6 with its own; with four queues the streams wait for each other either way).
// Contexts on different threads may use a stream at once: enqueueing is thread-safe, and
// every wait is on an event recorded right behind the work it stands for.
// There are at most as many of a kind as there were contexts at once.  A stream goes with the context that used it last; one
// that a context left for another serves the next context that needs one, or goes with the GPU's last context.
enum StreamKind { kCopyStream = 0, kUnpackStream = 1, kSaveStream = 2, kStreamKinds = 3 };
struct SharedStream {
    hipStream_t stream = nullptr, caller = nullptr;
    uint64_t owner = 0;                // see stream_owner
    int users = 0;
};
static std::mutex shared_streams_mutex;
static std::list<SharedStream> shared_streams[kMaxDevices][kStreamKinds];   // [device ordinal]
static int contexts_on[kMaxDevices];

struct ca_ctx {
    ca_config cfg{};
    SharedStream *held[kStreamKinds] = {nullptr, nullptr, nullptr};
    hipStream_t s_copy = nullptr, s_unpack = nullptr, s_save = nullptr;   // their handles (s_copy: with staged loads only)
    bool counted = false;              // in contexts_on
    // What the streams still owe this context.  An event costs the stream it is recorded on about 3 us and a wait across
    // streams about 11 us of host time and 20 us from one stream's kernel to the other's, so none is made that nothing needs.
    bool copy_waits_plan = false, unpack_waits_plan = false, save_waits_plan = false;   // the stream has not yet been told to wait for ev_plan
    hipEvent_t load_done = nullptr;    // event behind the newest load on the unpack stream (one of ev_ready), null: none outstanding
    bool save_pending = false;         // ev_saved stands behind work on the save stream that may be unfinished
    int32_t link_layer = -1;           // layer of the newest load across the host link under this plan (-1: none)
    bool saves_under_plan = false;     // some of it was queued under the current plan
    bool joined_null = false;          // the default stream (of the context's GPU) already waits for all of it
    // short moves run on a stream of the caller's instead (see runs_inline): the newest one, and the event behind it (null on
    // the default stream, which outlives the context and can be asked or recorded on when it matters)
    bool inline_pending = false;
    hipStream_t inline_stream = nullptr;
    uint64_t inline_owner = 0;         // see stream_owner
    hipEvent_t inline_done = nullptr, ev_inline = nullptr;
    hipStream_t plan_stream = nullptr; // the stream ca_rope_rebase was given
    std::vector<uint8_t> ready_inline; // per layer: loaded on the plan's stream
    hipEvent_t ev_saved = nullptr;
    // staging rings, each for its staged mode only: `depth` slots for loads, `depth` for saves; slot = [K tokens | V tokens]
    uint8_t *load_slots = nullptr, *save_slots = nullptr;
    size_t slot_bytes = 0, half_slot_bytes = 0;
    std::vector<hipEvent_t> ev_slot_copied, ev_slot_copied2, ev_slot_free;  // per load slot
    std::vector<uint8_t> slot_used;
    int64_t load_count = 0, save_count = 0;
    float2 *rope = nullptr;
    // plan metadata: one pinned host image, one device image
    uint8_t *h_meta = nullptr, *h_meta_dev = nullptr, *d_meta = nullptr;   // (h_meta_dev: h_meta as the GPU addresses it)
    size_t meta_bytes = 0;
    hipEvent_t ev_plan = nullptr, ev_after = nullptr;
    bool meta_in_flight = false;
    // offsets (bytes) inside the metadata image; those of the uploaded part change from plan to plan (its arrays lie back
    // to back, so that only what the plan uses crosses the host link)
    size_t off_table = 0, off_n_keep = 0, off_cu_q = 0, off_cu_k = 0, off_items = 0, off_combine = 0, off_q_pos = 0,
           off_q_seq = 0, off_slot_map = 0, upload_capacity = 0;
    size_t items_capacity = 0;         // work items the image has room for
    float *partial = nullptr;          // shares of row tiles whose keys were split over workgroups
    uint16_t *k_rot = nullptr;         // keys of the batch context rotated once per layer (dense pages)
    uint16_t *v_t = nullptr;           // values of the batch context transposed once per layer (same pages)
    bool pipelined = false;             // the plan runs the software-pipelined kernel on the two scratch copies
    size_t off_rot_nvalid = 0;
    size_t k_rot_pages = 0;
    size_t off_dense0 = 0, off_rot_src = 0, off_rot_pos = 0;
    int32_t n_dense_pages = 0;
    bool prerotate = false;
    int32_t n_cus = 256;               // compute units of the device (balancing target)
    // current plan (host copies)
    bool has_plan = false;
    int32_t n_seqs = 0, max_pages = 0, num_pages = 0, n_items = 0, n_combine = 0, tile_rows = 128;
    int32_t max_unit_rows = 0;   // most stacked query rows of any (conversation, kv head) of the plan
    // plan of the few-rows kernel (launch_attn_rows): its workgroups' item ranges, and one counter per merge for each of the
    // two attention entry points, which may run at once (zero between calls, and set to zero with every plan)
    int32_t n_wgs = 0, wg_wavefronts = 4;
    bool rows_runs = false;
    bool last_round_cut = false;   // tile kernels: only items of the last round of workgroups are cut
    int32_t wgs_per_cu = 0;        // tile kernels: workgroups that run on a compute unit at a time
    size_t off_wg_first = 0, off_rows_items = 0;
    uint32_t *arrived = nullptr, *static_arrived = nullptr;
    int32_t n_split_parts = 0;   // shares of split row tiles of the plan (slots of the partial-result buffer in use)
    float *static_partial = nullptr;   // this device's copy of the static scratch array (ca_cached_prefill_attn_static)
    int64_t total_q = 0, total_k = 0, total_n = 0;
    std::vector<int32_t> hist_len, new_len, n_keep, cu_q, cu_k;
    // kept saved tokens of conversation i: ranges keep_rng[keep_rng_at[i] .. keep_rng_at[i+1]) of (begin, end)
    std::vector<int32_t> keep_rng_at;
    std::vector<std::pair<int32_t, int32_t>> keep_rng;
    std::vector<int64_t> cu_n;
    std::vector<hipEvent_t> ev_ready;  // per layer
    std::vector<uint8_t> loaded;
    // optional timing of the library's own GPU work (ca_profile_*)
    struct Interval { int32_t kind; hipEvent_t start, stop; };
    bool profiling = false;
    uint32_t profile_mask = ~0u;       // bit k: intervals of kind k are recorded
    std::vector<Interval> intervals;
    std::vector<hipEvent_t> spare_events;
    std::string err;
};

namespace {

void set_err(char *dst, int32_t len, const char *fmt, ...) {
    if (!dst || len <= 0) return;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(dst, (size_t)len, fmt, ap);
    va_end(ap);
}

ca_status fail(ca_ctx *ctx, ca_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (ctx) ctx->err = buf;
    return st;
}

#define CA_HIP(ctx, expr)                                                                        \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess) {                                                                  \
            (void)hipGetLastError();                                                             \
            return fail((ctx), CA_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));      \
        }                                                                                        \
    } while (0)

// Cuts of a few-rows plan (and its workgroups, where it has runs) are at most this many: two workgroups of four wavefronts per compute
// unit.  A unit that is cut has at most twice as many shares as cuts, hence kAttnMaxParts / 2.
constexpr int kRowsMaxWorkgroups = kAttnMaxParts / 2;
constexpr int kRowsCutPages = 20;
constexpr size_t kMetaAlign = 64;            // alignment of the arrays of the metadata image
// Workgroups of a kernel that moves between the pool and pinned host memory (32 KB in flight each), measured on MI355X with
// 16 conversations of a grouped-query layer (169 MB to load, 18 MB to save): the rate alone, the rate beside the attention of
// another layer (563 us), and how that attention is slowed down (its own times differ by 7 % from run to run)
//   loads   4: 46, 30 GB/s, not   8: 57, 51, not   10: 57, 54, not   16: 56, 56, 1.36 x   32: 57, 55, 2.0 x
//   saves   2: 31, 31 GB/s, not   4: 45, 44, not    8: 52, 51, 1.4 x   16: 54, 54, 1.9 x
// Past what the link holds the requests queue up in the memory system in front of everyone else's.  Whole turns (two layers
// of 64 such conversations, us): 27648 with 6 load workgroups, 27006 with 8, 26780 with 10, 26706 with 12.
// That is with the attention that rotates keys itself.  Beside the one over keys rotated beforehand and two save workgroups, a step of
// 16 layers of 64 such conversations: 8 load workgroups 195.1 ms and 2150 to 2190 us of attention a layer, 10: 194.4 and 2200,
// 12: 196.9 and 2375.  (Fewer and larger workgroups, which would leave more compute units alone, cannot have as many requests
// under way: 3 of 1024 threads load 34 GB/s.)
constexpr int kLinkLoadWorkgroups = 10;
constexpr int kLinkSaveWorkgroups = 4;
constexpr int kLinkSaveBesideLoads = 2;

enum ProfileKind { kProfCopyIn = 0, kProfUnpack = 1, kProfAppend = 2, kProfAttn = 3, kProfPack = 4, kProfCopyOut = 5, kProfKinds = 6 };

hipError_t prof_event(ca_ctx *ctx, hipEvent_t *ev) {
    if (!ctx->spare_events.empty()) {
        *ev = ctx->spare_events.back();
        ctx->spare_events.pop_back();
        return hipSuccess;
    }
    return hipEventCreate(ev);
}

// Opens a timed interval on `stream`; returns its index or -1 when profiling is off.
hipError_t prof_begin(ca_ctx *ctx, int kind, hipStream_t stream, int *idx) {
    *idx = -1;
    if (!ctx->profiling || !(ctx->profile_mask & (1u << kind))) return hipSuccess;
    ca_ctx::Interval iv{kind, nullptr, nullptr};
    hipError_t e = prof_event(ctx, &iv.start);
    if (e != hipSuccess) return e;
    e = prof_event(ctx, &iv.stop);
    if (e != hipSuccess) return e;
    e = hipEventRecord(iv.start, stream);
    if (e != hipSuccess) return e;
    ctx->intervals.push_back(iv);
    *idx = (int)ctx->intervals.size() - 1;
    return hipSuccess;
}

hipError_t prof_end(ca_ctx *ctx, int idx, hipStream_t stream) {
    if (idx < 0) return hipSuccess;
    return hipEventRecord(ctx->intervals[idx].stop, stream);
}

// Makes a GPU current for the length of a scope.
class OnDevice {
public:
    hipError_t enter(int device) {
        const hipError_t e = hipGetDevice(&before_);
        if (e != hipSuccess || before_ == device) { before_ = -1; return e; }
        return hipSetDevice(device);
    }
    bool other() const { return before_ >= 0; }      // another GPU was current
    void leave() { if (before_ >= 0) (void)hipSetDevice(before_); before_ = -1; }
    ~OnDevice() { leave(); }

private:
    int before_ = -1;
};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int64_t row_bytes(const ca_config &c) { return (int64_t)c.n_kv_heads * c.head_dim * 2; }

enum class MemKind { kDevice, kPinnedHost, kUnknown };

// *shift = where the GPU addresses p, as a distance from p: zero but for host memory that was allocated without the runtime and
// registered with it later, for which the two addresses may differ
MemKind mem_kind(const void *p, ptrdiff_t *shift) {
    hipPointerAttribute_t attr;
    *shift = 0;
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return MemKind::kUnknown;
    }
    if (attr.type == hipMemoryTypeDevice) return MemKind::kDevice;
    if (attr.type == hipMemoryTypeHost) {
        if (attr.devicePointer) *shift = (const uint8_t *)attr.devicePointer - (const uint8_t *)p;
        return MemKind::kPinnedHost;
    }
    if (attr.type == hipMemoryTypeManaged) return MemKind::kDevice;
    return MemKind::kUnknown;
}

// Kind and extent of the allocations a call's pointers lie in.  One API call asks about up to two pointers per
// conversation and they mostly come out of one or two allocations: the last answer is kept for the length of the call
// (never longer, an allocation may be gone by the next one).
class MemMap {
public:
    // kind of p; *room = bytes from p to the end of its allocation (SIZE_MAX where the runtime cannot tell); *gpu = p as the GPU
    // addresses it
    MemKind look(const void *p, size_t *room, uint8_t **gpu) {
        const uint8_t *q = (const uint8_t *)p;
        if (base_ && q >= base_ && q < base_ + size_) {
            *room = (size_t)(base_ + size_ - q);
            *gpu = const_cast<uint8_t *>(q) + shift_;
            return kind_;
        }
        ptrdiff_t shift;
        const MemKind k = mem_kind(p, &shift);
        *room = SIZE_MAX;
        *gpu = const_cast<uint8_t *>(q) + shift;
        if (k == MemKind::kUnknown) return k;
        hipDeviceptr_t base = nullptr;
        size_t size = 0;
        if (hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
            (void)hipGetLastError();
            return k;
        }
        const uint8_t *b = (const uint8_t *)base;
        if (q < b || q >= b + size) {       // host memory the GPU has at another address: the range does not say where p ends
            if (k == MemKind::kDevice) *room = 0;
            return k;
        }
        base_ = b; size_ = size; kind_ = k; shift_ = shift;
        *room = (size_t)(b + size - q);
        return k;
    }
    // true if [p, p+bytes) lies inside one device allocation
    bool device_range_ok(const void *p, size_t bytes) {
        size_t room = 0;
        uint8_t *gpu;
        return p && look(p, &room, &gpu) == MemKind::kDevice && bytes <= room;
    }

private:
    const uint8_t *base_ = nullptr;
    size_t size_ = 0;
    MemKind kind_ = MemKind::kUnknown;
    ptrdiff_t shift_ = 0;
};

// ---- which stream a move runs on, and what waits for it ---------------------------------------------------------
// A move between the tier and the pool has an internal stream so that it overlaps with the caller's kernels.  Getting
// there and back costs about 20 us on the GPU and as much on the host (measured: a kernel, event, wait, kernel, event, wait
// loop over two streams 27 us, the two kernels on one stream 7.5 us), so a move that is shorter than that runs on the
// caller's stream: one to or from device memory of at most 16 MB (about 8 us), one across the host link of at most 128 KB
// for a save (4 us; stores) and 512 KB for a load (12 us; reads).
constexpr int64_t kInlineDeviceBytes = (int64_t)16 << 20;
constexpr int64_t kInlineHostSaveBytes = (int64_t)128 << 10;
constexpr int64_t kInlineHostLoadBytes = (int64_t)512 << 10;

// Work queued on a stream that is being captured becomes part of a graph: the caller orders it where the graph is launched, and
// nothing outside can wait for it.
bool is_captured(hipStream_t stream) {
    if (stream == nullptr) return false;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) != hipSuccess) (void)hipGetLastError();
    return st != hipStreamCaptureStatusNone;
}

// What a capture does not survive (measured): hipEventQuery and hipStreamQuery while some other stream is under capture (by any
// thread, if in global mode), unless the calling thread is in relaxed mode; and in every mode a query of, or a host's wait
// for, an event whose stream has come under capture since it was recorded.  Another stream's wait for such an event is refused
// with hipErrorStreamCaptureIsolation, the capture stays whole; the host then waits instead.
class RelaxedCapture {
public:
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }

private:
    hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};
// The host waits for the GPU, as hipFree does, which a capture survives in relaxed mode (hipDeviceSynchronize it does not).
hipError_t finish_device() {
    RelaxedCapture relaxed;
    void *p = nullptr;
    const hipError_t e = hipMalloc(&p, 256);
    return e == hipSuccess ? hipFree(p) : e;
}
// `stream` waits for an event that was recorded on a stream of the caller's, which may have come under capture since
hipError_t wait_for(hipStream_t stream, hipEvent_t event) {
    const hipError_t e = hipStreamWaitEvent(stream, event, 0);
    if (e != hipErrorStreamCaptureIsolation || is_captured(stream)) return e;
    (void)hipGetLastError();
    return finish_device();
}
hipError_t query(hipEvent_t event) { RelaxedCapture relaxed; return hipEventQuery(event); }
hipError_t query(hipStream_t stream) { RelaxedCapture relaxed; return hipStreamQuery(stream); }

// May a move be queued on the stream the plan was made on?  The caller may have destroyed it, or be capturing it (a capture
// would take the move in, and would not survive being asked whether the stream is done).
bool stream_usable(hipStream_t stream) {
    if (stream == nullptr) return true;
    if (is_captured(stream)) return false;
    const hipError_t e = query(stream);
    if (e == hipSuccess) return true;
    (void)hipGetLastError();
    return e == hipErrorNotReady;
}

// hipStreamPerThread is one handle for a stream in each thread: a number of the calling thread's own, 0 for other streams
uint64_t stream_owner(hipStream_t stream) {
    static std::atomic<uint64_t> threads{0};
    static thread_local uint64_t own = 0;
    if (stream != hipStreamPerThread) return 0;
    if (own == 0) own = ++threads;
    return own;
}

// ctx->held[kind] becomes the internal stream that works behind the caller's stream `caller`
hipError_t stream_for(ca_ctx *ctx, StreamKind kind, hipStream_t caller) {
    SharedStream *&held = ctx->held[kind];
    const uint64_t owner = stream_owner(caller);
    if (held && held->caller == caller && held->owner == owner) return hipSuccess;     // (changed by its only user alone)
    std::lock_guard<std::mutex> hold(shared_streams_mutex);
    auto &all = shared_streams[ctx->cfg.device][kind];
    SharedStream *take = nullptr, *spare = held && held->users == 1 ? held : nullptr;
    for (SharedStream &s : all) {
        if (s.users > 0 && s.caller == caller && s.owner == owner) take = &s;
        if (s.users == 0 && !spare) spare = &s;
    }
    if (!take && !spare) {
        hipStream_t created;
        const hipError_t e = hipStreamCreateWithFlags(&created, hipStreamNonBlocking);
        if (e != hipSuccess) return e;
        all.emplace_back();
        spare = &all.back();
        spare->stream = created;
    }
    if (!take) {
        take = spare;
        take->caller = caller;
        take->owner = owner;
    }
    if (held != take) {
        if (held) --held->users;
        ++take->users;
        held = take;
    }
    return hipSuccess;
}

// the streams for loads under a plan made on `caller`
hipError_t load_streams_for(ca_ctx *ctx, hipStream_t caller) {
    hipError_t e = stream_for(ctx, kUnpackStream, caller);
    if (e == hipSuccess && ctx->cfg.load_mode == 1) e = stream_for(ctx, kCopyStream, caller);
    if (e != hipSuccess) return e;
    ctx->s_unpack = ctx->held[kUnpackStream]->stream;
    ctx->s_copy = ctx->held[kCopyStream] ? ctx->held[kCopyStream]->stream : nullptr;
    return hipSuccess;
}

// the stream for saves behind `caller`; one that takes over continues behind the plan and the saves so far
hipError_t save_stream_for(ca_ctx *ctx, hipStream_t caller) {
    hipError_t e = stream_for(ctx, kSaveStream, caller);
    if (e != hipSuccess || ctx->s_save == ctx->held[kSaveStream]->stream) return e;
    ctx->s_save = ctx->held[kSaveStream]->stream;
    if (ctx->save_pending) e = hipStreamWaitEvent(ctx->s_save, ctx->ev_saved, 0);
    ctx->save_waits_plan = ctx->has_plan;
    return e;
}

void leave_streams(ca_ctx *ctx) {
    if (!ctx->counted) return;
    std::lock_guard<std::mutex> hold(shared_streams_mutex);
    const bool last = --contexts_on[ctx->cfg.device] == 0;
    for (int kind = 0; kind < kStreamKinds; ++kind) {
        SharedStream *held = ctx->held[kind];
        if (held) --held->users;
        auto &all = shared_streams[ctx->cfg.device][kind];
        for (auto s = all.begin(); s != all.end();) {
            if (s->users > 0 || (&*s != held && !last)) { ++s; continue; }
            (void)hipStreamDestroy(s->stream);
            s = all.erase(s);
        }
    }
}

// Is the stream of the newest short move under capture?  (That of another thread's hipStreamPerThread cannot be asked.)
bool inline_captured(const ca_ctx *ctx) {
    return ctx->inline_owner == stream_owner(ctx->inline_stream) && is_captured(ctx->inline_stream);
}

// May the next short move run on `stream`?  Only one stream's inline moves are kept track of at a time.
bool inline_free(ca_ctx *ctx, hipStream_t stream) {
    if (!ctx->inline_pending || (ctx->inline_stream == stream && ctx->inline_owner == stream_owner(stream))) return true;
    if (inline_captured(ctx)) return false;
    if ((ctx->inline_stream != nullptr ? query(ctx->inline_done) : query((hipStream_t) nullptr)) == hipSuccess) {
        ctx->inline_pending = false;
        return true;
    }
    (void)hipGetLastError();
    return false;
}

// a short move has been queued on `stream`; `done`: the event recorded behind it (may be null on the default stream only)
void note_inline(ca_ctx *ctx, hipStream_t stream, hipEvent_t done) {
    ctx->inline_pending = true;
    ctx->inline_stream = stream;
    ctx->inline_owner = stream_owner(stream);
    ctx->inline_done = done;
}

hipError_t note_inline(ca_ctx *ctx, hipStream_t stream) {
    if (stream != nullptr) {
        const hipError_t e = hipEventRecord(ctx->ev_inline, stream);
        if (e != hipSuccess) return e;
    }
    note_inline(ctx, stream, stream != nullptr ? ctx->ev_inline : nullptr);
    return hipSuccess;
}

// first use of an internal stream under a plan: it waits for the plan's metadata
hipError_t after_plan(ca_ctx *ctx, hipStream_t stream, bool *waits) {
    if (!*waits) return hipSuccess;
    const hipError_t e = wait_for(stream, ctx->ev_plan);
    if (e == hipSuccess) *waits = false;
    return e;
}

// a stream of the caller's waits for the plan's metadata (nothing to do for HIP on the stream the plan was made on)
hipError_t caller_after_plan(ca_ctx *ctx, hipStream_t stream) {
    return stream == nullptr && ctx->plan_stream == nullptr ? hipSuccess : wait_for(stream, ctx->ev_plan);
}

// `stream` waits for the load of `layer`
hipError_t after_load(ca_ctx *ctx, int32_t layer, hipStream_t stream) {
    if (ctx->ready_inline[layer] && ctx->plan_stream == nullptr) {
        if (stream == nullptr) return hipSuccess;      // same stream
        const hipError_t e = hipEventRecord(ctx->ev_ready[layer], nullptr);
        if (e != hipSuccess) return e;
    }
    return wait_for(stream, ctx->ev_ready[layer]);   // (nothing to do for HIP on the stream it was recorded on)
}

}  // namespace

extern "C" {

const char *ca_status_string(ca_status s) {
    switch (s) {
        case CA_OK: return "CA_OK";
        case CA_ERR_INVALID_ARG: return "CA_ERR_INVALID_ARG";
        case CA_ERR_OUT_OF_RANGE: return "CA_ERR_OUT_OF_RANGE";
        case CA_ERR_UNSUPPORTED: return "CA_ERR_UNSUPPORTED";
        case CA_ERR_NOMEM: return "CA_ERR_NOMEM";
        case CA_ERR_NOT_READY: return "CA_ERR_NOT_READY";
        case CA_ERR_HIP: return "CA_ERR_HIP";
    }
    return "CA_ERR_?";
}

void ca_config_default(ca_config *c) {
    if (!c) return;
    std::memset(c, 0, sizeof *c);
    c->n_layers = 1;
    c->n_q_heads = c->n_kv_heads = 1;
    c->head_dim = 128;
    c->page_size = kPageSize;
    c->max_positions = 4096;
    c->rope_base = 10000.0f;
    c->rope_style = 0;
    c->pipeline_depth = 2;
    c->max_seqs = 64;
    c->max_batch_kv_tokens = 1 << 16;
    c->max_batch_q_tokens = 1 << 14;
    c->load_mode = 0;
    c->save_mode = 0;
    c->attn_variant = 0;
    c->attn_tile_rows = 0;
    c->attn_split = 0;
    c->attn_prerotate = 0;
    c->attn_schedule = 0;
    c->require_load = 1;
    c->device = 0;
}

ca_status ca_config_validate(const ca_config *c, char *err, int32_t err_len) {
    if (!c) { set_err(err, err_len, "config is NULL"); return CA_ERR_INVALID_ARG; }
    if (c->n_layers < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1) {
        set_err(err, err_len, "n_layers, n_q_heads, n_kv_heads must be >= 1");
        return CA_ERR_INVALID_ARG;
    }
    if (c->n_q_heads % c->n_kv_heads != 0) {
        set_err(err, err_len, "n_q_heads (%d) is not a multiple of n_kv_heads (%d)", c->n_q_heads, c->n_kv_heads);
        return CA_ERR_INVALID_ARG;
    }
    if (c->head_dim != 64 && c->head_dim != 128) {
        set_err(err, err_len, "head_dim %d unsupported (64 or 128)", c->head_dim);
        return CA_ERR_UNSUPPORTED;
    }
    if (c->page_size != kPageSize) {
        set_err(err, err_len, "page_size %d unsupported (%d)", c->page_size, kPageSize);
        return CA_ERR_UNSUPPORTED;
    }
    if (c->rope_style != 0 && c->rope_style != 1) {
        set_err(err, err_len, "rope_style %d unsupported (0 or 1)", c->rope_style);
        return CA_ERR_UNSUPPORTED;
    }
    if (!(c->rope_base > 1.0f) || !std::isfinite(c->rope_base)) {
        set_err(err, err_len, "rope_base must be finite and > 1");
        return CA_ERR_INVALID_ARG;
    }
    if (c->max_positions < 1 || c->max_positions > (1 << 20)) {
        set_err(err, err_len, "max_positions %d out of range [1, 2^20]", c->max_positions);
        return CA_ERR_OUT_OF_RANGE;
    }
    if (c->pipeline_depth < 1 || c->pipeline_depth > 64) {
        set_err(err, err_len, "pipeline_depth %d out of range [1, 64]", c->pipeline_depth);
        return CA_ERR_OUT_OF_RANGE;
    }
    if (c->max_seqs < 1 || c->max_seqs > 4096) {
        set_err(err, err_len, "max_seqs %d out of range [1, 4096]", c->max_seqs);
        return CA_ERR_OUT_OF_RANGE;
    }
    if (c->max_batch_kv_tokens < 1 || c->max_batch_kv_tokens > ((int64_t)1 << 26) ||
        c->max_batch_q_tokens < 1 || c->max_batch_q_tokens > c->max_batch_kv_tokens) {
        set_err(err, err_len, "max_batch_kv_tokens / max_batch_q_tokens out of range");
        return CA_ERR_OUT_OF_RANGE;
    }
    if (c->save_mode < 0 || c->save_mode > 2) {
        set_err(err, err_len, "save_mode (0..2) out of range");
        return CA_ERR_INVALID_ARG;
    }
    if (c->load_mode < 0 || c->load_mode > 2 || c->attn_variant < 0 || c->attn_variant > 4) {
        set_err(err, err_len, "load_mode (0..2) or attn_variant (0..4) out of range");
        return CA_ERR_INVALID_ARG;
    }
    if (c->attn_variant == 3) {
        set_err(err, err_len, "attn_variant 3 (the register-staged kernel) was removed: the LDS-direct kernel serves every window");
        return CA_ERR_UNSUPPORTED;
    }
    if (c->attn_tile_rows != 0 && c->attn_tile_rows != 128 && c->attn_tile_rows != 256) {
        set_err(err, err_len, "attn_tile_rows %d unsupported (0, 128 or 256)", c->attn_tile_rows);
        return CA_ERR_UNSUPPORTED;
    }
    if (c->attn_prerotate < 0 || c->attn_prerotate > 2) { set_err(err, err_len, "attn_prerotate must be 0, 1 or 2"); return CA_ERR_INVALID_ARG; }
    if (c->attn_schedule < 0 || c->attn_schedule > 1) { set_err(err, err_len, "attn_schedule must be 0 or 1"); return CA_ERR_INVALID_ARG; }
    if (c->attn_split < 0 || c->attn_split > 1) { set_err(err, err_len, "attn_split must be 0 or 1"); return CA_ERR_INVALID_ARG; }
    if (c->device < 0) { set_err(err, err_len, "device < 0"); return CA_ERR_INVALID_ARG; }
    return CA_OK;
}

ca_status ca_batch_validate(const ca_config *c, const ca_batch *b, char *err, int32_t err_len) {
    ca_status st = ca_config_validate(c, err, err_len);
    if (st != CA_OK) return st;
    if (!b || !b->hist_len || !b->new_len || !b->block_table) {
        set_err(err, err_len, "batch or one of its arrays is NULL");
        return CA_ERR_INVALID_ARG;
    }
    if ((b->keep_ranges == nullptr) != (b->keep_range_count == nullptr)) {
        set_err(err, err_len, "keep_ranges and keep_range_count must both be given or both NULL");
        return CA_ERR_INVALID_ARG;
    }
    if (!b->keep_ranges && !b->keep_start) {
        set_err(err, err_len, "neither keep_start nor keep_ranges is given");
        return CA_ERR_INVALID_ARG;
    }
    if (b->n_seqs < 1 || b->n_seqs > c->max_seqs) {
        set_err(err, err_len, "n_seqs %d out of range [1, max_seqs=%d]", b->n_seqs, c->max_seqs);
        return CA_ERR_OUT_OF_RANGE;
    }
    if (b->max_pages < 1 || b->num_pages < 1) {
        set_err(err, err_len, "max_pages and num_pages must be >= 1");
        return CA_ERR_INVALID_ARG;
    }
    if ((int64_t)b->num_pages * c->page_size > ((int64_t)1 << 31) - 1) {
        set_err(err, err_len, "num_pages %d: slot index would overflow int32", b->num_pages);
        return CA_ERR_OUT_OF_RANGE;
    }
    int64_t tot_k = 0, tot_q = 0, range_at = 0;
    std::vector<uint8_t> seen((size_t)b->num_pages, 0);
    for (int32_t i = 0; i < b->n_seqs; ++i) {
        const int64_t h = b->hist_len[i], n = b->new_len[i];
        if (h < 0 || n < 1) {
            set_err(err, err_len, "conversation %d: hist_len %lld < 0 or new_len %lld < 1", i, (long long)h, (long long)n);
            return CA_ERR_INVALID_ARG;
        }
        int64_t kept = 0;
        if (b->keep_ranges) {
            const int64_t cnt = b->keep_range_count[i];
            if (cnt < 0 || cnt > h) {
                set_err(err, err_len, "conversation %d: keep_range_count %lld outside [0, hist_len=%lld]", i, (long long)cnt, (long long)h);
                return CA_ERR_OUT_OF_RANGE;
            }
            int64_t prev_end = 0;
            for (int64_t r = 0; r < cnt; ++r) {
                const int64_t rb = b->keep_ranges[2 * (range_at + r)], re = b->keep_ranges[2 * (range_at + r) + 1];
                if (rb < prev_end || re <= rb || re > h) {
                    set_err(err, err_len, "conversation %d: kept range %lld = [%lld, %lld) is empty, out of order or outside [0, hist_len=%lld]",
                            i, (long long)r, (long long)rb, (long long)re, (long long)h);
                    return CA_ERR_OUT_OF_RANGE;
                }
                kept += re - rb;
                prev_end = re;
            }
            range_at += cnt;
        } else {
            const int64_t s = b->keep_start[i];
            if (s < 0 || s > h) {
                set_err(err, err_len, "conversation %d: keep_start %lld outside [0, hist_len=%lld]", i, (long long)s, (long long)h);
                return CA_ERR_OUT_OF_RANGE;
            }
            kept = h - s;
        }
        const int64_t ctx_len = kept + n;
        if (ctx_len > c->max_positions) {
            set_err(err, err_len, "conversation %d: context %lld exceeds max_positions %d (truncate first)", i,
                    (long long)ctx_len, c->max_positions);
            return CA_ERR_OUT_OF_RANGE;
        }
        const int64_t pages = (ctx_len + c->page_size - 1) / c->page_size;
        if (pages > b->max_pages) {
            set_err(err, err_len, "conversation %d: needs %lld pages, block table has %d columns", i, (long long)pages, b->max_pages);
            return CA_ERR_OUT_OF_RANGE;
        }
        for (int64_t p = 0; p < pages; ++p) {
            const int32_t page = b->block_table[(int64_t)i * b->max_pages + p];
            if (page < 0 || page >= b->num_pages) {
                set_err(err, err_len, "conversation %d: block_table[%lld] = %d outside [0, num_pages=%d)", i, (long long)p, page, b->num_pages);
                return CA_ERR_OUT_OF_RANGE;
            }
            if (seen[(size_t)page]) {
                set_err(err, err_len, "conversation %d: page %d is used twice in the batch", i, page);
                return CA_ERR_INVALID_ARG;
            }
            seen[(size_t)page] = 1;
        }
        tot_k += ctx_len;
        tot_q += n;
    }
    if (tot_k > c->max_batch_kv_tokens || tot_q > c->max_batch_q_tokens) {
        set_err(err, err_len, "batch has %lld context / %lld new tokens, limits are %lld / %lld", (long long)tot_k,
                (long long)tot_q, (long long)c->max_batch_kv_tokens, (long long)c->max_batch_q_tokens);
        return CA_ERR_OUT_OF_RANGE;
    }
    return CA_OK;
}

ca_status ca_truncate_plan_sinks(const int32_t *hist_len, const int32_t *new_len, int32_t window, double ratio,
                                 int32_t n_sink, int32_t n, int32_t *ranges_out, int32_t *count_out) {
    if (!hist_len || !new_len || !ranges_out || !count_out || n < 0 || n_sink < 0) return CA_ERR_INVALID_ARG;
    if (window < 1 || !(ratio > 0.0) || !(ratio < 1.0)) return CA_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i)
        if (hist_len[i] < 0 || new_len[i] < 0) return CA_ERR_INVALID_ARG;
    const int64_t keep_target = (int64_t)std::floor((double)window * (1.0 - ratio));
    for (int32_t i = 0; i < n; ++i) {
        const int64_t h = hist_len[i], fresh = new_len[i];
        int32_t *r = ranges_out + 4 * (int64_t)i;
        r[0] = r[1] = r[2] = r[3] = 0;
        int32_t cnt = 0;
        if (h + fresh <= window) {
            if (h > 0) { r[0] = 0; r[1] = (int32_t)h; cnt = 1; }
        } else {
            const int64_t budget = std::min<int64_t>(h, std::max<int64_t>(0, keep_target - fresh));
            const int64_t sinks = std::min<int64_t>(n_sink, budget);
            const int64_t recent = budget - sinks;                 // tokens [h - recent, h)
            if (sinks > 0 && recent > 0 && h - recent <= sinks) {  // the two pieces touch or overlap
                r[0] = 0; r[1] = (int32_t)h; cnt = 1;              // (only when everything is kept)
            } else {
                if (sinks > 0) { r[2 * cnt] = 0; r[2 * cnt + 1] = (int32_t)sinks; ++cnt; }
                if (recent > 0) { r[2 * cnt] = (int32_t)(h - recent); r[2 * cnt + 1] = (int32_t)h; ++cnt; }
            }
        }
        count_out[i] = cnt;
    }
    return CA_OK;
}

ca_status ca_tier_compact(int32_t n, const int32_t *hist_len, const int32_t *keep_start, const int32_t *keep_ranges,
                          const int32_t *keep_range_count, int64_t row_bytes, void *const *tier_k, void *const *tier_v,
                          int32_t *hist_len_out) {
    if (n < 0 || !hist_len || !tier_k || !tier_v || !hist_len_out || row_bytes <= 0) return CA_ERR_INVALID_ARG;
    if ((keep_ranges == nullptr) != (keep_range_count == nullptr)) return CA_ERR_INVALID_ARG;
    if (!keep_ranges && !keep_start) return CA_ERR_INVALID_ARG;
    // everything is checked before the first byte moves
    int64_t at = 0;
    for (int32_t c = 0; c < n; ++c) {
        if (hist_len[c] < 0) return CA_ERR_INVALID_ARG;
        if (keep_ranges) {
            if (keep_range_count[c] < 0) return CA_ERR_INVALID_ARG;
            int32_t prev_end = 0;
            for (int32_t r = 0; r < keep_range_count[c]; ++r, ++at) {
                const int32_t b = keep_ranges[2 * at], e = keep_ranges[2 * at + 1];
                if (b < prev_end || e <= b || e > hist_len[c]) return CA_ERR_OUT_OF_RANGE;
                prev_end = e;
            }
            if (keep_range_count[c] > 0 && (!tier_k[c] || !tier_v[c])) return CA_ERR_INVALID_ARG;
        } else {
            if (keep_start[c] < 0 || keep_start[c] > hist_len[c]) return CA_ERR_OUT_OF_RANGE;
            if (keep_start[c] < hist_len[c] && (!tier_k[c] || !tier_v[c])) return CA_ERR_INVALID_ARG;
        }
    }
    at = 0;
    for (int32_t c = 0; c < n; ++c) {
        int64_t dst = 0;   // rows written so far; a range never starts below it, so the moves go towards lower addresses
        auto move = [&](int32_t b, int32_t e) {
            const size_t bytes = (size_t)(e - b) * (size_t)row_bytes;
            if (b != dst) {
                std::memmove((uint8_t *)tier_k[c] + (size_t)dst * row_bytes, (const uint8_t *)tier_k[c] + (size_t)b * row_bytes, bytes);
                std::memmove((uint8_t *)tier_v[c] + (size_t)dst * row_bytes, (const uint8_t *)tier_v[c] + (size_t)b * row_bytes, bytes);
            }
            dst += e - b;
        };
        if (keep_ranges) {
            for (int32_t r = 0; r < keep_range_count[c]; ++r, ++at) move(keep_ranges[2 * at], keep_ranges[2 * at + 1]);
        } else if (keep_start[c] < hist_len[c]) {
            move(keep_start[c], hist_len[c]);
        }
        hist_len_out[c] = (int32_t)dst;
    }
    return CA_OK;
}

ca_status ca_truncate_plan(const int32_t *hist_len, const int32_t *new_len, int32_t window, double ratio,
                           int32_t policy, int32_t n, int32_t *keep_start_out) {
    if (!hist_len || !new_len || !keep_start_out || n < 0) return CA_ERR_INVALID_ARG;
    if (window < 1 || !(ratio > 0.0) || !(ratio < 1.0)) return CA_ERR_INVALID_ARG;
    if (policy < 0 || policy > 2) return CA_ERR_UNSUPPORTED;
    for (int32_t i = 0; i < n; ++i)
        if (hist_len[i] < 0 || new_len[i] < 0) return CA_ERR_INVALID_ARG;
    const int64_t keep_target = (int64_t)std::floor((double)window * (1.0 - ratio));
    const int64_t drop_fixed = std::max<int64_t>(1, (int64_t)std::floor((double)window * ratio));
    for (int32_t i = 0; i < n; ++i) {
        const int64_t h = hist_len[i], fresh = new_len[i];
        int64_t first = 0;  // first surviving history token
        if (h + fresh > window) {
            switch (policy) {
                case 0:
                    first = h - std::min(h, std::max<int64_t>(0, keep_target - fresh));
                    break;
                case 1:
                    while (first < h && h - first + fresh > window) first = std::min(h, first + drop_fixed);
                    break;
                default:
                    while (first < h && h - first + fresh > window) {
                        const int64_t d = (int64_t)std::floor(ratio * (double)(h - first + fresh));
                        first = std::min(h, first + std::max<int64_t>(1, d));
                    }
            }
        }
        keep_start_out[i] = (int32_t)first;
    }
    return CA_OK;
}

const char *ca_last_error(const ca_ctx *ctx) { return ctx ? ctx->err.c_str() : "context is NULL"; }

void ca_destroy(ca_ctx *ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->cfg.device);
    (void)ca_sync(ctx);
    for (auto e : ctx->ev_slot_copied) if (e) (void)hipEventDestroy(e);
    for (auto e : ctx->ev_slot_copied2) if (e) (void)hipEventDestroy(e);
    for (auto e : ctx->ev_slot_free) if (e) (void)hipEventDestroy(e);
    for (auto e : ctx->ev_ready) if (e) (void)hipEventDestroy(e);
    if (ctx->ev_saved) (void)hipEventDestroy(ctx->ev_saved);
    if (ctx->ev_inline) (void)hipEventDestroy(ctx->ev_inline);
    if (ctx->ev_plan) (void)hipEventDestroy(ctx->ev_plan);
    if (ctx->ev_after) (void)hipEventDestroy(ctx->ev_after);
    for (auto &iv : ctx->intervals) { (void)hipEventDestroy(iv.start); (void)hipEventDestroy(iv.stop); }
    for (auto e : ctx->spare_events) (void)hipEventDestroy(e);
    if (ctx->load_slots) (void)hipFree(ctx->load_slots);
    if (ctx->save_slots) (void)hipFree(ctx->save_slots);
    if (ctx->rope) (void)hipFree(ctx->rope);
    if (ctx->partial) (void)hipFree(ctx->partial);
    if (ctx->arrived) (void)hipFree(ctx->arrived);
    if (ctx->k_rot) (void)hipFree(ctx->k_rot);
    if (ctx->v_t) (void)hipFree(ctx->v_t);
    if (ctx->d_meta) (void)hipFree(ctx->d_meta);
    if (ctx->h_meta) (void)hipHostFree(ctx->h_meta);
    leave_streams(ctx);
    delete ctx;
}

// every variant but the scalar check kernel stages K/V through LDS without registers (any window: the kernels keep a
// moving window of page ids in LDS)
static bool direct_variant(const ca_config &c) { return c.attn_variant != 1; }

static ca_status create_impl(ca_ctx *ctx) {
    const ca_config &c = ctx->cfg;
    int n_dev = 0;
    CA_HIP(ctx, hipGetDeviceCount(&n_dev));
    if (c.device >= n_dev) return fail(ctx, CA_ERR_OUT_OF_RANGE, "device %d of %d", c.device, n_dev);
    CA_HIP(ctx, hipSetDevice(c.device));
    if (c.device >= kMaxDevices) return fail(ctx, CA_ERR_OUT_OF_RANGE, "device %d: at most %d are served", c.device, kMaxDevices);
    {
        std::lock_guard<std::mutex> hold(shared_streams_mutex);
        ++contexts_on[c.device];
        ctx->counted = true;
    }
    CA_HIP(ctx, load_streams_for(ctx, nullptr));       // (most programs plan on one stream; a plan on another changes them)
    CA_HIP(ctx, save_stream_for(ctx, nullptr));
    const int depth = c.pipeline_depth;
    ctx->half_slot_bytes = align_up((size_t)c.max_batch_kv_tokens * (size_t)row_bytes(c), 256);
    ctx->slot_bytes = 2 * ctx->half_slot_bytes;
    if (c.save_mode == 1) CA_HIP(ctx, hipMalloc((void **)&ctx->save_slots, ctx->slot_bytes * depth));
    if (c.load_mode == 1) {
        CA_HIP(ctx, hipMalloc((void **)&ctx->load_slots, ctx->slot_bytes * depth));
        ctx->ev_slot_copied.assign(depth, nullptr);
        ctx->ev_slot_copied2.assign(depth, nullptr);
        ctx->ev_slot_free.assign(depth, nullptr);
        ctx->slot_used.assign(depth, 0);
        for (int i = 0; i < depth; ++i) {
            CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_slot_copied[i], hipEventDisableTiming));
            CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_slot_copied2[i], hipEventDisableTiming));
            CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_slot_free[i], hipEventDisableTiming));
        }
    }
    ctx->ev_ready.assign(c.n_layers, nullptr);
    ctx->loaded.assign(c.n_layers, 0);
    ctx->ready_inline.assign(c.n_layers, 0);
    for (int i = 0; i < c.n_layers; ++i)
        CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_ready[i], hipEventDisableTiming));
    CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_saved, hipEventDisableTiming));
    CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_inline, hipEventDisableTiming));
    CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_plan, hipEventDisableTiming));
    CA_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_after, hipEventDisableTiming));

    // Rotary table (Section 3.4): cos/sin of pos * base^(-2i/D), evaluated in fp64, stored fp32.
    {
        const int half = c.head_dim / 2;
        const int rows = std::max(c.max_positions, kRopeMinRows);
        std::vector<float2> tab((size_t)rows * half);
        std::vector<double> inv_freq(half);
        for (int i = 0; i < half; ++i)
            inv_freq[i] = std::exp(-std::log((double)c.rope_base) * (2.0 * i) / (double)c.head_dim);
        for (int p = 0; p < rows; ++p)
            for (int i = 0; i < half; ++i) {
                const double ang = (double)p * inv_freq[i];
                tab[(size_t)p * half + i] = make_float2((float)std::cos(ang), (float)std::sin(ang));
            }
        CA_HIP(ctx, hipMalloc((void **)&ctx->rope, tab.size() * sizeof(float2)));
        CA_HIP(ctx, hipMemcpy(ctx->rope, tab.data(), tab.size() * sizeof(float2), hipMemcpyHostToDevice));
    }

    // Capacity of the metadata image: the uploaded part (its layout is a plan's own, see ca_rope_rebase; block table rows
    // have at most ceil(max_positions/page)+1 columns), then the device-computed arrays.
    {
        const size_t max_cols = (size_t)(c.max_positions + c.page_size - 1) / c.page_size + 1;
        const size_t units = (size_t)c.max_seqs * c.n_kv_heads;
        const size_t g = (size_t)c.n_q_heads / c.n_kv_heads;
        // tiles: sum over units of ceil(rows/tile) <= total_q*g*n_kv_heads/tile + units, padded per die
        // (+ the extra items that splitting keys can add)
        const size_t max_items = (size_t)c.max_batch_q_tokens * g * c.n_kv_heads / kAttnTileRowsMin + units + kAttnMaxParts;
        const size_t max_items_padded = (max_items + 1) * kXcds;  // worst case: every tile on one die
        ctx->items_capacity = max_items_padded;
        ctx->k_rot_pages = (size_t)c.max_batch_kv_tokens / c.page_size + (size_t)c.max_seqs;
        size_t off = 0;
        const auto add = [&off](size_t bytes) { const size_t at = off; off = align_up(off + bytes, kMetaAlign); return at; };
        add((size_t)c.max_seqs * max_cols * 4);                       // block table
        for (int i = 0; i < 4; ++i) add(((size_t)c.max_seqs + 1) * 4); // n_keep, cu_q, cu_k, dense0
        for (int i = 0; i < 3; ++i) add(ctx->k_rot_pages * 4);        // rot_src, rot_pos, rot_nvalid
        add((size_t)kAttnMaxParts * sizeof(CombineItem));
        add(max_items_padded * sizeof(WorkItem));
        add((kRowsMaxWorkgroups + units + 1) * (4 + sizeof(WorkItem) + sizeof(RowsItem)));   // few-rows plan: one item per unit and cut
        ctx->upload_capacity = off = align_up(off, 256);
        ctx->off_q_pos = off;   off = align_up(off + (size_t)c.max_batch_q_tokens * 4, 256);
        ctx->off_q_seq = off;   off = align_up(off + (size_t)c.max_batch_q_tokens * 4, 256);
        ctx->off_slot_map = off; off = align_up(off + (size_t)c.max_batch_kv_tokens * 4, 256);
        ctx->meta_bytes = off;
        CA_HIP(ctx, hipMalloc((void **)&ctx->d_meta, ctx->meta_bytes));
        CA_HIP(ctx, hipHostMalloc((void **)&ctx->h_meta, ctx->upload_capacity, hipHostMallocMapped));
        CA_HIP(ctx, hipHostGetDevicePointer((void **)&ctx->h_meta_dev, ctx->h_meta, 0));
    }
    // Partial results of row tiles whose keys are split over workgroups (only the LDS-direct kernel splits).
    const bool may_split = c.attn_split == 0 && direct_variant(c);
    if (may_split) {
        const size_t bytes = (size_t)kAttnMaxParts * 256 * (size_t)(c.head_dim + 2) * sizeof(float);
        CA_HIP(ctx, hipMalloc((void **)&ctx->partial, bytes));
        CA_HIP(ctx, hipMalloc((void **)&ctx->arrived, (size_t)2 * kAttnMaxParts * sizeof(uint32_t)));
        ctx->static_arrived = ctx->arrived + kAttnMaxParts;
    }
    const bool may_direct = direct_variant(c);
    if (may_direct && c.attn_prerotate != 1) {
        CA_HIP(ctx, hipMalloc((void **)&ctx->k_rot, ctx->k_rot_pages * (size_t)c.page_size * (size_t)row_bytes(c)));
        if (c.head_dim == 128 && c.attn_schedule == 1)
            CA_HIP(ctx, hipMalloc((void **)&ctx->v_t, ctx->k_rot_pages * (size_t)c.page_size * (size_t)row_bytes(c)));
    }
    {
        hipDeviceProp_t prop;
        CA_HIP(ctx, hipGetDeviceProperties(&prop, c.device));
        ctx->n_cus = std::max(8, prop.multiProcessorCount);
    }
    // address of this device's copy of the static scratch array (the device is current here)
    if (c.device < kMaxDevices) {
        if (!static_scratch_ptr[c.device]) {
            void *p = nullptr;
            CA_HIP(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            static_scratch_ptr[c.device] = p;
        }
        ctx->static_partial = (float *)static_scratch_ptr[c.device];
    }
    return CA_OK;
}

ca_status ca_create(const ca_config *cfg, ca_ctx **out) {
    if (!out) return CA_ERR_INVALID_ARG;
    *out = nullptr;
    char msg[256] = {0};
    ca_status st = ca_config_validate(cfg, msg, sizeof msg);
    if (st != CA_OK) return st;
    ca_ctx *ctx = new (std::nothrow) ca_ctx();
    if (!ctx) return CA_ERR_NOMEM;
    ctx->cfg = *cfg;
    st = create_impl(ctx);
    if (st != CA_OK) {
        if (st == CA_ERR_HIP && ctx->err.find("out of memory") != std::string::npos) st = CA_ERR_NOMEM;
        std::fprintf(stderr, "ca_create: %s\n", ctx->err.c_str());
        ca_destroy(ctx);
        return st;
    }
    *out = ctx;
    return CA_OK;
}

ca_status ca_sync(ca_ctx *ctx) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    OnDevice on;
    CA_HIP(ctx, on.enter(ctx->cfg.device));
    if (ctx->load_done) CA_HIP(ctx, hipEventSynchronize(ctx->load_done));
    ctx->load_done = nullptr;
    if (ctx->save_pending) CA_HIP(ctx, hipEventSynchronize(ctx->ev_saved));
    ctx->save_pending = false;
    if (ctx->inline_pending) {
        if (inline_captured(ctx)) CA_HIP(ctx, finish_device());
        else if (ctx->inline_done) CA_HIP(ctx, hipEventSynchronize(ctx->inline_done));
        else CA_HIP(ctx, hipStreamSynchronize(nullptr));
    }
    ctx->inline_pending = false;
    return CA_OK;
}

ca_status ca_join(ca_ctx *ctx, void *stream) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    // The default stream is the context's GPU's, as in every other call, and where another GPU is current that one's as well.
    OnDevice on;
    CA_HIP(ctx, on.enter(ctx->cfg.device));
    const bool other_too = on.other() && (s == nullptr || s == hipStreamLegacy || s == hipStreamPerThread);
    hipEvent_t short_moves = nullptr;
    if (ctx->inline_pending && (s != nullptr || ctx->inline_stream != nullptr || other_too)) {
        if (!ctx->inline_done) CA_HIP(ctx, hipEventRecord(ctx->ev_inline, nullptr));
        short_moves = ctx->inline_done ? ctx->inline_done : ctx->ev_inline;
    }
    // (the copies of a staged load are in front of its unpack kernel, which waits for both halves)
    if ((ctx->load_done || ctx->save_pending) && !(s == nullptr && ctx->joined_null)) {
        if (ctx->load_done) CA_HIP(ctx, hipStreamWaitEvent(s, ctx->load_done, 0));
        if (ctx->save_pending) CA_HIP(ctx, hipStreamWaitEvent(s, ctx->ev_saved, 0));
        if (s == nullptr) ctx->joined_null = true;
    }
    if (short_moves && !(s == nullptr && ctx->inline_stream == nullptr)) CA_HIP(ctx, wait_for(s, short_moves));
    if (other_too) {
        on.leave();
        if (ctx->load_done) CA_HIP(ctx, hipStreamWaitEvent(s, ctx->load_done, 0));
        if (ctx->save_pending) CA_HIP(ctx, hipStreamWaitEvent(s, ctx->ev_saved, 0));
        if (short_moves) CA_HIP(ctx, wait_for(s, short_moves));
    }
    return CA_OK;
}

// ----------------------------------------------------------------------------------------------
// Section 3.4: rebase
// ----------------------------------------------------------------------------------------------
// Does the few-rows kernel serve the current plan?  It reads a unit's keys once for up to 32 stacked rows; one or two rows
// go to the streaming kernel of decode steps, which needs no matrix cores, more rows to the tile kernels.
static bool rows_plan(const ca_ctx *ctx) {
    const ca_config &c = ctx->cfg;
    return c.attn_variant == 0 && c.attn_tile_rows == 0 && c.attn_prerotate != 2 && ctx->max_unit_rows > kAttnDecodeMaxRows &&
           ctx->max_unit_rows <= kAttnRowsMax;
}

// Work list of the few-rows kernel.  Cuts inside a (conversation, kv head) unit lie on multiples of 64 keys.
// Much to stream (eight pages per wavefront and more): the pages of all units, laid end to end, are cut into one run per
// workgroup; a cut leaves at least kAttnMinPartKeys on either side (a share costs a merge), so runs are equal up to 256 keys.
// Less: a workgroup has one share, and the time is a chain: a wavefront takes 0.9 us a page (heads of 128), and the workgroup that
// merges reads all shares of its unit, about 45 KB/us, some 2 us at least.  Units of kRowsCutPages pages and more are cut into
// shares of about the square root of their pages, which balances the two for 8 rows of 128 (neither heads of 64 nor other
// numbers of rows are asked about), or what an equal spread over the compute units gives where that is more.  us of one attention
// call of one conversation with the rule's share (in brackets) and with shares of 8, 12, 16, 24 and 32 pages:
//                  8 kv heads, 8 rows of 128                    2 kv heads, 4 rows of 128                    4 kv heads, 8 rows of 64
//    100 pages     11.4 (12)  10.8 11.4 11.5 13.3 15.1          10.6 (12)   9.7 10.5 10.9 12.7 14.3           8.6 (12)   7.7  8.5  9.0 10.2 11.3
//    174           12.0 (12)  12.7 11.9 12.7 13.5 15.2          10.5 (12)  10.5 10.5 11.6 12.8 14.4           8.7 (12)   8.9  8.7  9.7 10.2 11.3
//    250           13.0 (16)  14.3 13.6 13.0 14.5 15.3          11.6 (16)  11.1 11.6 11.4 13.3 14.6           9.6 (16)   9.8  9.7  9.5 10.8 11.4
//    500           16.4 (24)  16.3 16.3 16.3 16.2 16.6          13.9 (24)  14.3 13.6 13.1 14.2 15.2          11.7 (24)  13.9 12.5 11.7 11.8 12.1
//   1876           27.5 (60)  27.3 27.4 27.4 27.3 27.4          20.5 (44)  21.9 21.9 21.9 19.6 19.6          17.3 (44)  17.8 17.8 17.8 17.8 17.8
// Where the line of kRowsCutPages lies is not the best for few units (us whole and cut, 8 kv heads): one conversation of 12, 16, 20
// and 24 pages 9.1, 7.5; 10.7, 7.6; 11.4, 7.6; 12.3, 7.7; 16 conversations 9.2, 9.8; 11.0, 9.8; 11.8, 10.9; 12.9, 10.9; one turn
// of 32 rows of 128 11.2, 12.4; 12.9, 12.4; 13.8, 12.5; 15.2, 12.6.
static ca_status plan_rows(ca_ctx *ctx, size_t &up) {
    const ca_config &c = ctx->cfg;
    const int B = ctx->n_seqs, Hkv = c.n_kv_heads, G = c.n_q_heads / Hkv;
    const auto put = [&up](size_t bytes) { const size_t at = up; up = align_up(up + bytes, kMetaAlign); return at; };
    ctx->prerotate = ctx->pipelined = false;
    ctx->n_dense_pages = 0;
    ctx->tile_rows = ctx->max_unit_rows <= 16 ? 16 : 32;
    constexpr int kCut = 64 / kPageSize, kMin = kAttnMinPartKeys / kPageSize;    // pages
    int64_t total = 0;
    for (int i = 0; i < B; ++i) total += (int64_t)((ctx->n_keep[i] + ctx->new_len[i] + kPageSize - 1) / kPageSize) * Hkv;
    const int n_units = B * Hkv;
    const bool split = ctx->partial != nullptr;
    const bool runs = total >= (int64_t)2 * ctx->n_cus * 32;
    const int wgs = !runs ? 0 : split ? std::min(kRowsMaxWorkgroups, 2 * ctx->n_cus) : n_units;
    const int spread = std::min(kRowsMaxWorkgroups, ctx->n_cus);
    const int even = (int)std::max<int64_t>(kCut, (total / spread + kCut - 1) / kCut * kCut);        // pages, where there are no runs
    // A unit of p pages is cut into shares of at least `even` pages, at most p / even times.
    const int cuts = !split ? 0 : runs ? wgs : (int)(total / even);      // at most
    ctx->rows_runs = runs;
    ctx->off_wg_first = put((size_t)(wgs + 1) * 4);
    ctx->off_items = put((size_t)(n_units + cuts) * sizeof(WorkItem));
    ctx->off_rows_items = put((size_t)(n_units + cuts) * sizeof(RowsItem));
    if (cuts > kRowsMaxWorkgroups || up > ctx->upload_capacity)
        return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rope_rebase: internal: %d cuts, image of %zu bytes (room for %zu)", cuts, up, ctx->upload_capacity);
    int32_t *wg_first = (int32_t *)(ctx->h_meta + ctx->off_wg_first);
    WorkItem *items = (WorkItem *)(ctx->h_meta + ctx->off_items);
    RowsItem *rows_items = (RowsItem *)(ctx->h_meta + ctx->off_rows_items);
    int n_items = 0, n_merges = 0, n_parts = 0, w = 0;
    int64_t done = 0;                       // pages of the units before this one
    wg_first[0] = 0;
    for (int i = 0; i < B; ++i) {
        const int keys = ctx->n_keep[i] + ctx->new_len[i], rows = ctx->new_len[i] * G;
        const int pages = (keys + kPageSize - 1) / kPageSize;
        const int32_t *table = (const int32_t *)(ctx->h_meta + ctx->off_table) + (size_t)i * ctx->max_pages;
        const int share = std::max(even, (int)(std::sqrt((double)pages) / kCut + 0.5) * kCut);
        for (int g = 0; g < Hkv; ++g, done += pages) {
            const int first_item = n_items;
            for (int at = 0; at < pages;) {
                int cut = pages;
                bool next_wg = false;
                if (!split) {
                    next_wg = true;
                } else if (runs) {
                    const int64_t end = (w + 1) * total / wgs - done;        // of workgroup w's run, as a page of this unit
                    if (end < pages) {
                        cut = end <= 0 ? 0 : (int)((end + kCut / 2) / kCut * kCut);
                        if (cut - at < kMin) cut = at;
                        else if (keys / kPageSize - cut < kMin) cut = pages;
                    }
                    next_wg = end <= pages;
                } else if (pages >= kRowsCutPages) {
                    cut = std::min(pages, at + share);
                }
                if (cut > at) {
                    items[n_items] = WorkItem{i, g, 0, rows, at * kPageSize, cut == pages ? keys : cut * kPageSize, -1, 0};
                    RowsItem &r = rows_items[n_items++];
                    r = RowsItem{i, g, rows, at * kPageSize, cut == pages ? keys : cut * kPageSize, -1, ctx->n_keep[i], ctx->cu_q[i], 0, 0, 0, {}, {}};
                    for (int p = 0; p < 16; ++p) r.page[p] = table[std::min(at + p, pages - 1)];
                }
                at = cut;
                if (next_wg && w + 1 < wgs) wg_first[++w] = n_items;
            }
            if (n_items - first_item > 1) {
                const int first_part = n_parts;
                for (int k = first_item; k < n_items; ++k) {
                    items[k].part = rows_items[k].part = n_parts++;
                    rows_items[k].merge = n_merges;
                    rows_items[k].first_part = first_part;
                    rows_items[k].n_parts = n_items - first_item;
                }
                ++n_merges;
            }
        }
    }
    while (w < wgs) wg_first[++w] = n_items;
    ctx->n_wgs = runs ? wgs : n_items;
    // Whole units that leave compute units over: eight wavefronts take half the steps (a turn of 256 + 32 tokens, 4 heads of 64:
    // 29.0 us, 30.5 with four).  Where a workgroup's loads are the longer part they are no gain (shares of 16 pages: 1558 us, 1330).
    ctx->wg_wavefronts = !runs && n_merges == 0 && n_items < ctx->n_cus ? 8 : 4;
    ctx->n_items = n_items;
    ctx->n_combine = n_merges;
    ctx->n_split_parts = n_parts;
    if (n_parts > kAttnMaxParts) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rope_rebase: internal: %d shares", n_parts);
    return CA_OK;
}

// Whether a plan that has units of more than 128 rows is better served by 128-row tiles, keys rotated in the kernel.  Two
// such workgroups share a compute unit: one walks while the other loads its queries and first keys or writes its output,
// and no wavefront is without rows; but units of more than 128 rows read and rotate their keys once more.  Costs in 64-key tiles
// of a full 256-row workgroup: per tile of a 128-row workgroup and of a 256-row one that has at most 128 rows, and the fixed part
// of either, which the neighbour hides most of for 128 rows.  Where the tiles do not fill both places of every compute unit they
// would be cut into twice the shares, and with few rounds of them the last one is felt, hence the margin.  Fitted to 133
// random batches (2 to 64 conversations, no history to 4000 tokens, 4 to 2048 new) timed with either tile: 128 rows are taken for
// 46 of them, for 0.70 to 1.02 of the time with 256, 0.88 on average, and 8 more would gain over 5 %.  us of one attention call, 256
// and 128 rows, with ratio of costs and rounds:
//   17 first turns of 303-311 tokens, 32 heads  103, 80 (0.76, 3.2)   32 turns, 8-512 new, most below 128, 40 heads  585, 548 (0.95, 3.6)
//   40 first turns of 80-137, 40 heads          100, 70 (0.62, 3.6)   52 first turns of 18-114, 32/4 heads of 64     27, 23 (0.94, 2.0)
// and the other way round:
//   16 turns of 1536 + 19-178, 32 heads         116, 137 (0.96, 1.3)  32 of 3080-3206 + 41-168, 32 heads             399, 460 (1.00, 2.6)
//   10 of 347-383 + 168-369, 32 heads           75, 79 (0.91, 1.6)    64 of 343-417 + 279-344, 4 heads of 64         47, 56 (1.05, 1.5)
static bool half_tiles_pay(const ca_ctx *ctx) {
    struct Costs { double tile128, item128, half_full256, item256, margin; };
    const Costs cost = ctx->cfg.head_dim == 64 ? Costs{0.61, 1.0, 0.48, 2.3, 0.04} : Costs{0.555, 1.3, 0.56, 3.2, 0.15};
    const int G = ctx->cfg.n_q_heads / ctx->cfg.n_kv_heads;
    int64_t tiles128 = 0;
    double cost128 = 0, cost256 = 0;
    for (int i = 0; i < ctx->n_seqs; ++i) {
        const int rows = ctx->new_len[i] * G;
        const auto key_tiles = [&](int end_row) { return (ctx->n_keep[i] + (end_row - 1) / G + 64) / 64; };    // of 64, that rows below end_row see
        for (int at = 0; at < rows; at += 128) cost128 += cost.tile128 * key_tiles(std::min(rows, at + 128)) + cost.item128;
        for (int at = 0; at < rows; at += 256)
            cost256 += (rows - at <= 128 ? cost.half_full256 : 1.0) * key_tiles(std::min(rows, at + 256)) + cost.item256;
        tiles128 += (rows + 127) / 128;
    }
    tiles128 *= ctx->cfg.n_kv_heads;
    const double rounds = (double)tiles128 / (2 * ctx->n_cus);
    return rounds >= 1 && cost128 < (1 - cost.margin / rounds) * cost256;
}

// Cutting the last round only is taken where it is estimated to take at most this share of the better one of the other two plans.
// Of 3000 drawn batches of 1 to 64 conversations it changes the plans of 36, whose attention takes 0.77 to 0.99 of the time, 0.87 on
// average (one layer of 4 conversations of 1667-1800 tokens with 177-497 new ones, 40 heads: 133 -> 106 us).  With 0.97 it would be
// half as many again, none of 26 measured ones slower, among them 8 conversations of 2048 with 64-512 new ones, 32 heads (4 layers of
// it 892 -> 868 us); the line lies below that batch because its plan is held to be whole, from a time when there was only whole and cut.
constexpr double kLastRoundGain = 0.89;

// A row tile or a share of one, as the planner of the tile kernels handles it
struct Item { WorkItem w; double cost; int32_t parent; };

// Estimated us of a plan of the tile kernels (`bins` workgroups run on a die at a time), to decide whether its row tiles are left
// whole, cut into shares, or cut only where the last round of workgroups would leave compute units idle.  Shares fill those
// units, but each is launched, fetches its queries and fills its load pipeline, is written and read back (its valid rows),
// and the merge is a launch.  The items are laid out on the dies in time: us per 64-key tile on a compute unit that other
// workgroups share and on one of a workgroup's own, and per item, by kernel and shape; 3 us and 1.75 TB/s of shares for the
// merge, 7 us a launch in either case; `shares` is a factor on the time with shares, where the decisions came out best.  Fitted to
// 1236 random plans (1 to 64 conversations, no history to 31000 tokens, 2 to 2048 new, seven shapes of heads) timed whole and
// cut: whole is taken 391 times, for 0.51 to 1.08 of the time with shares, 0.83 on average, and the plan taken is the slower one by
// more than 3 % in 19.  (One layer of 13 conversations of 2134-2392 tokens with 9-45 new ones, 16/8 heads of 64: 38 us in
// 832 shares, 72 whole.)
static double plan_time(const ca_ctx *ctx, const std::vector<std::vector<Item>> &plan, const std::vector<int32_t> &parts_of, int bins) {
    struct Times { double tile, tile_alone, item, shares; };
    const bool d64 = ctx->cfg.head_dim == 64, small = ctx->tile_rows == 128;
    const Times t = ctx->prerotate ? (!d64 ? Times{1.65, 1.45, 9.2, 1.05} : small ? (ctx->wgs_per_cu == 4 ? Times{1.55, 1.10, 6.8, 1.10} : Times{1.25, 1.10, 5.5, 1.10}) : Times{1.05, 0.95, 4.1, 0.95})
                    : d64          ? (small ? Times{1.85, 1.65, 0.5, 1.05} : Times{1.45, 1.30, 2.5, 1.00})
                                   : (small ? Times{2.60, 1.95, 3.0, 1.00} : Times{2.10, 1.85, 5.6, 1.00});
    const size_t die_cus = std::max(1, ctx->n_cus / kXcds);
    std::vector<double> heap;
    double longest = 0, share_bytes = 0;
    for (const auto &items : plan) {
        const double tile = items.size() <= die_cus ? t.tile_alone : t.tile;
        heap.assign(bins, 0.0);
        for (const Item &it : items) {
            const double part = !small && it.w.n_rows <= 128 ? 0.78 : 1.0;      // (four of eight wavefronts have rows)
            std::pop_heap(heap.begin(), heap.end(), std::greater<double>());
            heap.back() += t.item + part * tile * ((it.w.key_end + 63) / 64 - it.w.key_begin / 64);
            longest = std::max(longest, heap.back());
            std::push_heap(heap.begin(), heap.end(), std::greater<double>());
            if (parts_of[it.parent] > 1) share_bytes += (double)it.w.n_rows * (ctx->cfg.head_dim + 2) * sizeof(float);
        }
    }
    return share_bytes > 0 ? t.shares * (longest + 7.0 + 3.0 + share_bytes / 1.75e6) : longest + 7.0;
}

ca_status ca_rope_rebase(ca_ctx *ctx, const ca_batch *b, void *stream_) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    char msg[384] = {0};
    ca_status st = ca_batch_validate(&ctx->cfg, b, msg, sizeof msg);
    if (st != CA_OK) return fail(ctx, st, "ca_rope_rebase: %s", msg);
    const ca_config &c = ctx->cfg;
    hipStream_t stream = (hipStream_t)stream_;
    CA_HIP(ctx, hipSetDevice(c.device));

    const int B = b->n_seqs;

    // the pinned image may still be the source of the previous plan's upload
    if (ctx->meta_in_flight) {
        CA_HIP(ctx, hipEventSynchronize(ctx->ev_plan));
        ctx->meta_in_flight = false;
    }

    // from here on the host copy of the plan is rewritten: until the new metadata has been queued for upload
    // the context has no usable plan (a failure below must not leave new host counts beside old device tables)
    ctx->has_plan = false;
    ctx->hist_len.assign(b->hist_len, b->hist_len + B);
    ctx->keep_rng_at.assign(B + 1, 0);
    ctx->keep_rng.clear();
    for (int i = 0, at = 0; i < B; ++i) {
        if (b->keep_ranges) {
            for (int r = 0; r < b->keep_range_count[i]; ++r, ++at)
                ctx->keep_rng.push_back({b->keep_ranges[2 * at], b->keep_ranges[2 * at + 1]});
        } else if (b->keep_start[i] < b->hist_len[i]) {
            ctx->keep_rng.push_back({b->keep_start[i], b->hist_len[i]});
        }
        ctx->keep_rng_at[i + 1] = (int32_t)ctx->keep_rng.size();
    }
    ctx->new_len.assign(b->new_len, b->new_len + B);
    ctx->n_keep.resize(B);
    ctx->cu_q.assign(B + 1, 0);
    ctx->cu_k.assign(B + 1, 0);
    ctx->cu_n.assign(B + 1, 0);
    for (int i = 0; i < B; ++i) {
        int32_t kept = 0;
        for (int r = ctx->keep_rng_at[i]; r < ctx->keep_rng_at[i + 1]; ++r) kept += ctx->keep_rng[r].second - ctx->keep_rng[r].first;
        ctx->n_keep[i] = kept;
        ctx->cu_q[i + 1] = ctx->cu_q[i] + b->new_len[i];
        ctx->cu_k[i + 1] = ctx->cu_k[i] + ctx->n_keep[i] + b->new_len[i];
        ctx->cu_n[i + 1] = ctx->cu_n[i] + ctx->n_keep[i];
    }
    int cols = 1;   // block table columns in use
    for (int i = 0; i < B; ++i) cols = std::max(cols, (ctx->n_keep[i] + b->new_len[i] + c.page_size - 1) / c.page_size);
    ctx->n_seqs = B;
    ctx->max_pages = cols;
    ctx->num_pages = b->num_pages;
    ctx->total_q = ctx->cu_q[B];
    ctx->total_k = ctx->cu_k[B];
    ctx->total_n = ctx->cu_n[B];

    // ---- host image -------------------------------------------------------------------------
    // The arrays of the plan lie back to back.  Each is no longer than what ca_create made room for.
    size_t up = 0;
    const auto put = [&up](size_t bytes) { const size_t at = up; up = align_up(up + bytes, kMetaAlign); return at; };
    ctx->off_n_keep = put((size_t)B * 4);
    ctx->off_cu_q = put((size_t)(B + 1) * 4);
    ctx->off_cu_k = put((size_t)(B + 1) * 4);
    ctx->off_table = put((size_t)B * cols * 4);
    int32_t *h_table = (int32_t *)(ctx->h_meta + ctx->off_table);
    for (int i = 0; i < B; ++i) {
        const int pages = (ctx->n_keep[i] + b->new_len[i] + c.page_size - 1) / c.page_size;
        const int32_t *from = b->block_table + (int64_t)i * b->max_pages;
        std::memcpy(h_table + (size_t)i * cols, from, (size_t)pages * 4);
        std::fill(h_table + (size_t)i * cols + pages, h_table + (size_t)(i + 1) * cols, from[0]);  // always a valid page
    }
    std::memcpy(ctx->h_meta + ctx->off_n_keep, ctx->n_keep.data(), (size_t)B * 4);
    std::memcpy(ctx->h_meta + ctx->off_cu_q, ctx->cu_q.data(), (size_t)(B + 1) * 4);
    std::memcpy(ctx->h_meta + ctx->off_cu_k, ctx->cu_k.data(), (size_t)(B + 1) * 4);

    // ---- attention work list ------------------------------------------------------------------
    ctx->n_wgs = 0;
    ctx->last_round_cut = false;
    ctx->max_unit_rows = 0;
    for (int i = 0; i < B; ++i) ctx->max_unit_rows = std::max(ctx->max_unit_rows, b->new_len[i] * (c.n_q_heads / c.n_kv_heads));
    if (rows_plan(ctx)) {
        st = plan_rows(ctx, up);
        if (st != CA_OK) return st;
    } else
    // Tiles of stacked query rows, placed die by die.
    // All tiles of one (conversation, kv head) read the same keys/values, so they are given to the
    // same die (workgroup i runs on die i % 8), in plans of many rounds one after the other, and share its L2.
    // Units go longest-first to the least loaded die; dies are padded to equal length.
    {
        const int G = c.n_q_heads / c.n_kv_heads;
        // 256-row tiles (8 wavefronts) halve the K/V re-reads and the rotary work per row when a
        // (conversation, kv head) has more than 128 stacked rows; small turns keep 128-row tiles, and so do mixed batches in which
        // these cost less (half_tiles_pay).  Keys of 64 dimensions
        // that were rotated beforehand are cheap to read again, and three or four workgroups of four wavefronts to a compute unit,
        // none in step with another, beat one of eight: 16 first turns of 128-2048 tokens (32/4 heads) 158 -> 138 us a
        // layer, 8 turns of 1000-3000 + 64-300 tokens 74 -> 62 (with heads of 128: 1750 -> 1975, the other way round).  Where
        // the tiles are fewer than half the compute units, their keys are split many times over, and tiles of half the rows
        // would need twice the shares.
        int tile = c.attn_tile_rows;
        const int most = ctx->max_unit_rows;
        if (tile == 0) tile = most > 128 ? 256 : 128;
        const bool direct_for_rot = direct_variant(c);
        {   // rotate the keys once per layer when on average three or more row tiles would each rotate them (48 batches, 4 to 64
            // conversations of 500 to 3000 tokens, four shapes of heads, rotated beforehand against in the kernel: with one tile
            // 1.11 to 1.31 of the time, with two 0.94 to 1.15, three 0.90 to 1.07, four 0.85 to 1.10)
            int64_t tiles256 = 0;
            for (int i = 0; i < B; ++i) tiles256 += ((int64_t)b->new_len[i] * G + 255) / 256;
            ctx->prerotate = ctx->k_rot && direct_for_rot &&
                             (c.attn_prerotate == 2 || (c.attn_prerotate == 0 && tiles256 >= (int64_t)3 * B));
            if (ctx->prerotate && c.attn_tile_rows == 0) tile = c.head_dim == 64 && tiles256 * c.n_kv_heads * 2 >= ctx->n_cus ? 128 : 256;
            if (c.attn_tile_rows == 0 && tile == 256 && direct_for_rot && !ctx->prerotate && half_tiles_pay(ctx)) tile = 128;
            ctx->pipelined = ctx->prerotate && ctx->v_t && tile == 256 && c.attn_variant != 3 && c.attn_variant != 1;
            size_t dense_pages = 0;
            if (ctx->prerotate)
                for (int i = 0; i < B; ++i) dense_pages += (size_t)((ctx->n_keep[i] + b->new_len[i] + c.page_size - 1) / c.page_size);
            if (dense_pages > ctx->k_rot_pages) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rope_rebase: internal: %zu dense pages exceed %zu", dense_pages, ctx->k_rot_pages);
            ctx->off_dense0 = put((size_t)B * 4);
            ctx->off_rot_src = put(dense_pages * 4);
            ctx->off_rot_pos = put(dense_pages * 4);
            ctx->off_rot_nvalid = put(dense_pages * 4);
            int32_t *dense0 = (int32_t *)(ctx->h_meta + ctx->off_dense0);
            int32_t *rot_src = (int32_t *)(ctx->h_meta + ctx->off_rot_src), *rot_pos = (int32_t *)(ctx->h_meta + ctx->off_rot_pos);
            int32_t *rot_nvalid = (int32_t *)(ctx->h_meta + ctx->off_rot_nvalid);
            int32_t at = 0;
            for (int i = 0; i < B; ++i) {
                dense0[i] = at;
                if (!ctx->prerotate) continue;
                const int pages = (ctx->n_keep[i] + b->new_len[i] + c.page_size - 1) / c.page_size;
                for (int p = 0; p < pages; ++p, ++at) {
                    rot_src[at] = b->block_table[(int64_t)i * b->max_pages + p];
                    rot_pos[at] = p * c.page_size;
                    rot_nvalid[at] = std::min(c.page_size, ctx->n_keep[i] + b->new_len[i] - p * c.page_size);
                }
            }
            ctx->n_dense_pages = at;
        }
        ctx->tile_rows = tile;
        const bool direct_kernel = direct_variant(c);
        struct Unit { int32_t seq, head; int64_t work; };
        std::vector<Unit> units;
        units.reserve((size_t)B * c.n_kv_heads);
        for (int i = 0; i < B; ++i) {
            const int64_t ln = b->new_len[i], n = ctx->n_keep[i];
            const int64_t work = (int64_t)G * (ln * n + ln * (ln + 1) / 2);
            for (int g = 0; g < c.n_kv_heads; ++g) units.push_back({i, g, work});
        }
        std::stable_sort(units.begin(), units.end(), [](const Unit &x, const Unit &y) { return x.work > y.work; });
        int64_t total_tiles = 0;
        for (const Unit &u : units) total_tiles += (b->new_len[u.seq] * G + tile - 1) / tile;
        // a unit with more tiles than a die's fair share is cut into chunks so that a small batch
        // still spreads over all dies
        const int chunk_cap = (int)std::max<int64_t>(1, (total_tiles + kXcds - 1) / kXcds);
        // Cost of an item in the time a full workgroup needs for one 64-key tile (measured on single items:
        // a 256-row workgroup whose rows fill at most four wavefronts, one per SIMD, takes 0.72 of that per
        // tile; rotating Q, filling the load pipeline and the epilogue cost about three tiles).
        // A plan of decode steps goes to the streaming kernel, which reaches its bandwidth with one workgroup
        // per compute unit: shares (and the merge they need) only pay when there are fewer items than that.
        const bool decode_plan = direct_kernel && c.attn_variant != 2 && !ctx->prerotate && most >= 1 && most <= kAttnDecodeMaxRows;
        auto item_cost = [&](int n_rows, int keys) {
            const double per_tile = (tile == 256 && n_rows <= 128) ? 0.72 : 1.0;
            return per_tile * ((keys + 63) / 64) + 3.0;
        };
        std::vector<std::vector<Item>> per_die(kXcds);
        double load[kXcds] = {0};
        int32_t n_parents = 0;
        for (const Unit &u : units) {
            const int rows = b->new_len[u.seq] * G;
            const int n_tiles = (rows + tile - 1) / tile;
            const int n = ctx->n_keep[u.seq];
            for (int hi = n_tiles; hi > 0; hi -= chunk_cap) {  // later rows see more keys: longest first
                const int lo = std::max(0, hi - chunk_cap);
                int die = 0;
                for (int d = 1; d < kXcds; ++d) if (load[d] < load[die]) die = d;
                for (int t = hi - 1; t >= lo; --t) {
                    const int n_rows = std::min(tile, rows - t * tile);
                    const int keys = n + (t * tile + n_rows - 1) / G + 1;       // what the tile's rows see
                    const double cost = item_cost(n_rows, keys);
                    load[die] += cost;
                    per_die[die].push_back({WorkItem{u.seq, u.head, t * tile, n_rows, 0, keys, -1, 0}, cost, n_parents++});
                }
            }
        }

        // Few, long items leave compute units idle at the end (or, for a small batch, from the start): split
        // the keys of the longest items over several workgroups until a longest-first schedule of the die's
        // items over its compute units is within 12 % of the ideal.  Shares are merged by combine_tiles_kernel.
        // Up to four rounds per die; a round halves every item longer than 0.7 of the ideal load of a
        // compute unit (so 16 shares per row tile at most).
        size_t n_live = 0;
        for (auto &v : per_die) n_live += v.size();
        // Workgroups that run on a compute unit at a time: one of eight wavefronts, two of four, and with heads of 64 whose keys are
        // rotated beforehand, three of four, or four with 128 registers, where the fullest die has more row tiles than that many places:
        // three spread a single round better (24 random plans left whole, us of the attention with three and four: 18688 tiles 408, 378;
        // 4604 102, 96; 2236 41, 39; 1312 39, 38; 820 22.3, 22.0; 816 24.4, 25.5; 340 20.8, 21.6).  Decided before anything is cut, so
        // that the plan is cut for what is launched: 63 random plans of 700 to 1300 tiles that were laid out for three and launched with four
        // where shares made the items more take 0.90 to 1.035 of that time so, 0.97 on average (1144 tiles whole 273, last
        // round cut for four 246; 792 cut for three, launched with four 193, with three 187; 944 cut for three 187, 194).
        size_t fullest = 0;
        for (auto &v : per_die) fullest = std::max(fullest, v.size());
        const size_t die_cus = std::max(1, ctx->n_cus / kXcds);
        ctx->wgs_per_cu = tile != 128 ? 1 : c.head_dim == 128 || !ctx->prerotate ? 2 : fullest > 4 * die_cus ? 4 : 3;
        std::vector<int32_t> parts_of(n_parents, 1);
        int32_t n_split_parts = 0;          // shares that need a slot in the partial-result buffer
        const auto by_cost = [](const Item &x, const Item &y) { return x.cost > y.cost; };
        if (ctx->partial && direct_kernel && n_live < (size_t)(decode_plan ? 1 : 6) * ctx->n_cus) {
            const int bins = (int)die_cus * ctx->wgs_per_cu;
            // tiles of 128 rows where there would be 256-row ones: no more shares than the static scratch array holds, so that
            // ca_cached_prefill_attn_static takes the plans it would take with 256-row tiles
            const bool smaller = tile == 128 && most > 128 && c.attn_tile_rows == 0;
            const int max_parts = smaller ? (int)std::min<size_t>(kAttnMaxParts, kStaticScratchBytes / (128 * (size_t)(c.head_dim + 2) * sizeof(float)))
                                          : kAttnMaxParts;
            std::vector<double> heap;
            // sorts the items and returns the makespan of their longest-first list schedule over `bins` compute units
            // (min-heap of their loads)
            const auto schedule = [&](std::vector<Item> &v, double &total) {
                std::stable_sort(v.begin(), v.end(), by_cost);
                heap.assign(bins, 0.0);
                total = 0;
                for (const Item &it : v) {
                    std::pop_heap(heap.begin(), heap.end(), std::greater<double>());
                    heap.back() += it.cost;
                    std::push_heap(heap.begin(), heap.end(), std::greater<double>());
                    total += it.cost;
                }
                return *std::max_element(heap.begin(), heap.end());
            };
            std::vector<Item> shares, best;
            std::vector<std::vector<Item>> whole_of(kXcds);
            for (int d = 0; d < kXcds; ++d) {
                auto &v = per_die[d];
                std::vector<Item> &whole = whole_of[d];
                const int32_t parts_before = n_split_parts;
                double uncut = 0;
                for (int round = 0; round < 4 && !v.empty(); ++round) {
                    double total;
                    const double makespan = schedule(v, total);
                    const double ideal = total / bins;
                    if (makespan <= 1.12 * ideal + 1.0) break;   // (cutting further was measured to cost more than it gains)
                    if (round == 0) {
                        whole = v;
                        uncut = ideal;
                    }
                    const size_t n_before = v.size();
                    bool cut_any = false;
                    for (size_t k = 0; k < n_before && v[k].cost > 0.7 * ideal; ++k) {
                        Item &it = v[k];
                        const int len = it.w.key_end - it.w.key_begin;
                        const int extra = parts_of[it.parent] == 1 ? 2 : 1;   // slots a cut of this item adds
                        if (len < 2 * kAttnMinPartKeys || parts_of[it.parent] >= kAttnMaxPartsPerTile ||
                            n_split_parts + extra > max_parts) continue;
                        Item hi_half = it;
                        const int tiles64 = (len + 63) / 64;
                        const int mid = it.w.key_begin + (tiles64 / 2) * 64;
                        it.w.key_end = mid;
                        hi_half.w.key_begin = mid;
                        it.cost = item_cost(it.w.n_rows, mid - it.w.key_begin);
                        hi_half.cost = item_cost(hi_half.w.n_rows, hi_half.w.key_end - mid);
                        n_split_parts += extra;
                        parts_of[it.parent] += 1;
                        v.push_back(hi_half);          // (invalidates `it`)
                        cut_any = true;
                    }
                    if (!cut_any) break;
                }
                if (uncut <= 0) continue;           // nothing was cut, and the schedule has left the items sorted
                double total;
                double makespan = schedule(v, total);
                // Halving leaves shares of like length, whose number need not divide well among the compute units: one
                // conversation of 31003 + 301 tokens on 8 kv heads gets 76 shares a die for 32 compute units, three rounds
                // where 2.4 would do.  So equal shares of at most a few fractions of a compute unit's ideal load are tried
                // as well, and taken where their schedule is at least 5 % shorter and they need no more scratch than
                // halving.  Below sixteen tiles between halving and ideal the search costs the host what it could gain.
                // (That conversation, 8 layers: 3327 -> 2905 us a pass.  Of 52 batches, 13 length mixes of one to four
                // conversations of 4100 to 60000 tokens on 64/8, 32/32 and 8/2 heads of 128 and 32/4 of 64, the rule changes
                // the plan of 11: their attention takes 0.83 to 0.99 of what it took, 0.90 in the middle.  The search costs
                // the host up to 27 us a plan.)
                const double halved = makespan;
                if (halved < 1.05 * uncut + 16.0) continue;
                bool found = false;
                for (const double fraction : {1.18, 1.02, 0.87, 0.70, 0.56}) {
                    const double cap = std::max(fraction * uncut - item_cost(1, 0), 1.0);
                    int32_t parts = parts_before;
                    shares.clear();
                    for (const Item &it : whole) {
                        const int len = it.w.key_end - it.w.key_begin, tiles64 = len / 64;
                        const int n = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)kAttnMaxPartsPerTile, len / kAttnMinPartKeys,
                                                                                 (int64_t)std::ceil((it.cost - item_cost(1, 0)) / cap)}));
                        if (n > 1) parts += n;
                        for (int k = 0; k < n; ++k) {
                            Item share = it;
                            share.w.key_begin = it.w.key_begin + (int)((int64_t)tiles64 * k / n) * 64;
                            if (k + 1 < n) share.w.key_end = it.w.key_begin + (int)((int64_t)tiles64 * (k + 1) / n) * 64;
                            share.cost = item_cost(it.w.n_rows, share.w.key_end - share.w.key_begin);
                            shares.push_back(share);
                        }
                    }
                    if (parts > n_split_parts) continue;
                    const double with_shares = schedule(shares, total);
                    if (with_shares >= makespan || with_shares > 0.95 * halved) continue;
                    makespan = with_shares;
                    best.swap(shares);
                    found = true;
                }
                if (!found) continue;
                for (const Item &it : whole) parts_of[it.parent] = 0;
                for (const Item &it : best) ++parts_of[it.parent];
                n_split_parts = parts_before;
                for (const Item &it : whole)
                    if (parts_of[it.parent] > 1) n_split_parts += parts_of[it.parent];
                v.swap(best);
            }
            if (n_split_parts > 0 && !decode_plan) {
                for (int d = 0; d < kXcds; ++d)
                    if (whole_of[d].empty()) whole_of[d] = per_die[d];          // not cut, or cut in vain
                // Whole rounds of workgroups stay whole and the items left over for the last round, the shortest ones of the die,
                // are cut so that they fill it.
                std::vector<std::vector<Item>> last_of(kXcds);
                std::vector<int32_t> last_parts(n_parents, 1), one(n_parents, 1);
                int32_t n_last_parts = 0;
                // (never more than the static array holds: ca_cached_prefill_attn_static takes the plan whole, and so it takes it cut)
                const int32_t room = (int32_t)std::min<size_t>(kAttnMaxParts, kStaticArrayBytes / ((size_t)tile * (c.head_dim + 2) * sizeof(float)));
                for (int d = 0; d < kXcds; ++d) {
                    const auto &whole = whole_of[d];
                    auto &v = last_of[d];
                    const int n = (int)whole.size(), rest = n > bins ? n % bins : 0;
                    v.assign(whole.begin(), whole.end() - rest);
                    for (int k = n - rest; k < n; ++k) {
                        const Item &it = whole[k];
                        const int len = it.w.key_end - it.w.key_begin, tiles64 = len / 64;
                        int shares = std::min({bins / rest, kAttnMaxPartsPerTile, len / kAttnMinPartKeys});
                        if (shares < 2 || n_last_parts + shares > room) shares = 1;
                        for (int i = 0; i < shares; ++i) {
                            Item share = it;
                            share.w.key_begin = it.w.key_begin + tiles64 * i / shares * 64;
                            if (i + 1 < shares) share.w.key_end = it.w.key_begin + tiles64 * (i + 1) / shares * 64;
                            share.cost = item_cost(it.w.n_rows, share.w.key_end - share.w.key_begin);
                            v.push_back(share);
                        }
                        last_parts[it.parent] = shares;
                        if (shares > 1) n_last_parts += shares;
                    }
                    std::stable_sort(v.begin(), v.end(), by_cost);
                }
                const double us_whole = plan_time(ctx, whole_of, one, bins), us_cut = plan_time(ctx, per_die, parts_of, bins);
                const double us_last = n_last_parts > 0 ? plan_time(ctx, last_of, last_parts, bins) : INFINITY;
                if (us_last < kLastRoundGain * std::min(us_whole, us_cut)) {
                    for (int d = 0; d < kXcds; ++d) per_die[d].swap(last_of[d]);
                    parts_of = last_parts;
                    n_split_parts = n_last_parts;
                    ctx->last_round_cut = true;
                } else if (us_whole < us_cut) {
                    for (int d = 0; d < kXcds; ++d) per_die[d].swap(whole_of[d]);
                    parts_of.assign(n_parents, 1);
                    n_split_parts = 0;
                }
            }
        }
        // The last items of a die are launched longest first: within a unit the tiles of early rows see few keys, and few rows on a long
        // context take as long as many.  In front of them the tiles of a unit follow each other and share their keys in the die's
        // L2 (64 turns of 1024-4096 + 64-512 tokens, 64/8 heads, 4776 tiles: the attention reads 1.51 GB, sorted throughout 2.67).  Four a
        // compute unit are sorted of tiles of 256 rows, sixteen of 128 rows, whose units have few tiles (of 64-wide heads as
        // many rounds).  us of one attention call by units, with two, four, six and eight rounds sorted, and all:
        //   11 of 1402 + 850-1275 tokens, 40 heads      608, 591, 607, 625, 638, 639
        //   12 of 1000-1050 + 867-2048, 40 heads        811, 807, 827, 837, 858, 872
        //   47 of 1268 + 200, 64/8 heads                504, 501, 497, 511, 514, 534
        //   60 first turns of 607-2048, 32 heads        1563, 1554, 1550, 1558, 1555, 1670
        //   33 first turns of 632-948, 32 heads         445, 440, 439, 444, 436, 427
        //   45 of 167-250, 40 heads, 128 rows           122, 119, 116, 112, 110, 109
        //   63 of 3809-3999 + 453-679, 32/4 of 64       1367, 1356, 1386, 1401, 1415, 1436
        //   11 first turns of 681-2048, 32/8 of 64      129, 124, 123, 123, 123, 123
        // 40 random plans of this size take 0.92 to 1.03 of the time with all sorted, 0.97 on average.
        // (Where shares were considered, in plans of few rounds, all items are sorted already.)
        for (auto &v : per_die)
            std::stable_sort(v.end() - std::min(v.size(), die_cus * (tile == 128 ? 16 : 4)), v.end(), by_cost);
        // number the shares of split row tiles consecutively and list the tiles for the merge
        ctx->off_combine = put((size_t)n_split_parts * sizeof(CombineItem));    // (a tile has at least two shares)
        CombineItem *combine = (CombineItem *)(ctx->h_meta + ctx->off_combine);
        int32_t n_combine = 0;
        {
            std::vector<int32_t> first_part(n_parents, -1), next_part(n_parents, 0);
            int32_t at = 0;
            for (auto &v : per_die)
                for (Item &it : v) {
                    if (parts_of[it.parent] == 1) continue;
                    if (first_part[it.parent] < 0) {
                        first_part[it.parent] = at;
                        at += parts_of[it.parent];
                        combine[n_combine++] = CombineItem{it.w.seq, it.w.kv_head, it.w.row0, it.w.n_rows,
                                                           first_part[it.parent], parts_of[it.parent], {0, 0}};
                    }
                    it.w.part = first_part[it.parent] + next_part[it.parent]++;
                }
            if (at != n_split_parts || at > kAttnMaxParts) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rope_rebase: internal: %d shares numbered, %d planned", at, n_split_parts);
        }
        ctx->n_combine = n_combine;
        ctx->n_split_parts = n_split_parts;

        size_t longest = 0;
        for (auto &v : per_die) longest = std::max(longest, v.size());
        const size_t n_items = longest * kXcds;
        if (n_items > ctx->items_capacity) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rope_rebase: %zu work items exceed capacity %zu", n_items, ctx->items_capacity);
        ctx->off_items = put(n_items * sizeof(WorkItem));
        WorkItem *items = (WorkItem *)(ctx->h_meta + ctx->off_items);
        for (size_t s = 0; s < longest; ++s)
            for (int d = 0; d < kXcds; ++d)
                items[s * kXcds + d] = s < per_die[d].size() ? per_die[d][s].w : WorkItem{-1, 0, 0, 0, 0, 0, -1, 0};
        ctx->n_items = (int32_t)n_items;
    }

    // ---- order against everything still using the previous plan, then upload + per-token arrays in one kernel --
    if (up > ctx->upload_capacity) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rope_rebase: internal: image of %zu bytes exceeds %zu", up, ctx->upload_capacity);
    st = ca_join(ctx, stream_);
    if (st != CA_OK) return st;
    CA_HIP(ctx, load_streams_for(ctx, stream));
    RebaseArgs ra{};
    ra.n_seqs = B;
    ra.max_pages = cols;
    ra.image = ctx->h_meta_dev;
    ra.meta = ctx->d_meta;
    ra.image_vecs = (int64_t)(up / 16);
    ra.off_table = (int64_t)ctx->off_table;
    ra.off_n_keep = (int64_t)ctx->off_n_keep;
    ra.off_cu_q = (int64_t)ctx->off_cu_q;
    ra.off_cu_k = (int64_t)ctx->off_cu_k;
    ra.q_pos = (int32_t *)(ctx->d_meta + ctx->off_q_pos);
    ra.q_seq = (int32_t *)(ctx->d_meta + ctx->off_q_seq);
    ra.slot_map = (int32_t *)(ctx->d_meta + ctx->off_slot_map);
    ra.arrived[0] = ctx->arrived;
    ra.arrived[1] = ctx->static_arrived;
    ra.n_merges = ctx->n_wgs > 0 ? ctx->n_combine : 0;
    CA_HIP(ctx, launch_rebase(ra, stream));

    // internal streams start work of this plan only after the metadata exists (each waits when it is first used)
    CA_HIP(ctx, hipEventRecord(ctx->ev_plan, stream));
    ctx->meta_in_flight = true;
    ctx->copy_waits_plan = ctx->unpack_waits_plan = ctx->save_waits_plan = true;
    ctx->saves_under_plan = false;
    ctx->link_layer = -1;
    ctx->plan_stream = stream;
    std::fill(ctx->loaded.begin(), ctx->loaded.end(), 0);
    std::fill(ctx->ready_inline.begin(), ctx->ready_inline.end(), 0);
    ctx->has_plan = true;
    return CA_OK;
}

ca_status ca_rebase_read(ca_ctx *ctx, int32_t which, int32_t *out, int64_t capacity, int64_t *count) {
    if (!ctx || !out || !count || capacity < 0) return CA_ERR_INVALID_ARG;
    if (!ctx->has_plan) return fail(ctx, CA_ERR_NOT_READY, "ca_rebase_read: no plan (call ca_rope_rebase first)");
    size_t off;
    int64_t n;
    switch (which) {
        case 0: off = ctx->off_n_keep; n = ctx->n_seqs; break;
        case 1: off = ctx->off_cu_q; n = ctx->n_seqs + 1; break;
        case 2: off = ctx->off_cu_k; n = ctx->n_seqs + 1; break;
        case 3: off = ctx->off_q_pos; n = ctx->total_q; break;
        case 4: off = ctx->off_q_seq; n = ctx->total_q; break;
        case 5: off = ctx->off_slot_map; n = ctx->total_k; break;
        case 6: off = ctx->off_items; n = (int64_t)ctx->n_items * 8; break;
        default: return fail(ctx, CA_ERR_INVALID_ARG, "ca_rebase_read: which = %d", which);
    }
    if (n > capacity) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_rebase_read: need %lld elements, capacity %lld", (long long)n, (long long)capacity);
    CA_HIP(ctx, hipSetDevice(ctx->cfg.device));
    CA_HIP(ctx, hipDeviceSynchronize());
    CA_HIP(ctx, hipMemcpy(out, ctx->d_meta + off, (size_t)n * 4, hipMemcpyDeviceToHost));
    *count = n;
    return CA_OK;
}

// ----------------------------------------------------------------------------------------------
// Section 3.2: movement between the contiguous tier and the paged pool
// ----------------------------------------------------------------------------------------------
namespace {

struct Segment {  // one conversation's share of a move
    uint8_t *k, *v;
    int64_t contig_tok0;
    int32_t ctx_tok0, count, seq;
};

MoveShape move_shape(const ca_ctx *ctx, int max_tokens) {
    const ca_config &c = ctx->cfg;
    MoveShape shape{};
    shape.block_table = (const int32_t *)(ctx->d_meta + ctx->off_table);
    shape.n_keep = (const int32_t *)(ctx->d_meta + ctx->off_n_keep);
    shape.cu_q = (const int32_t *)(ctx->d_meta + ctx->off_cu_q);
    shape.max_pages = ctx->max_pages;
    shape.n_kv_heads = c.n_kv_heads;
    shape.vec_shift = c.head_dim == 128 ? 4 : 3;      // 16-byte vectors per head and token: 16 or 8
    // one 256-lane pass of kMoveUnroll x 16 bytes per lane covers the tokens of a page (of a decode step: one) of this many heads
    const int tokens = std::max(1, std::min(kPageSize, max_tokens));
    shape.heads_per_wg = std::max(1, std::min(c.n_kv_heads, (kMoveUnroll * 256 / tokens) >> shape.vec_shift));
    return shape;
}

// where a context token of a conversation lies in the pool (the host copy of the plan's block table)
int32_t token_slot(const ca_ctx *ctx, int seq, int token) {
    const int32_t *table = (const int32_t *)(ctx->h_meta + ctx->off_table);
    return table[(size_t)seq * ctx->max_pages + token / kPageSize] * kPageSize + token % kPageSize;
}

// link_workgroups > 0: the contiguous side is pinned host memory; a kernel of that many workgroups moves it
ca_status run_move(ca_ctx *ctx, bool to_pool, const std::vector<Segment> &segs, void *k_pool, void *v_pool,
                   hipStream_t stream, int link_workgroups = 0) {
    for (size_t at = 0; at < segs.size(); at += kMaxSeqsPerLaunch) {
        MoveArgs args;
        const int n = (int)std::min<size_t>(kMaxSeqsPerLaunch, segs.size() - at);
        int max_touched = 0, max_tokens = 0;
        for (int i = 0; i < n; ++i) {
            const Segment &s = segs[at + i];
            args.contig_k[i] = s.k;
            args.contig_v[i] = s.v;
            args.contig_tok0[i] = s.contig_tok0;
            args.ctx_tok0[i] = s.ctx_tok0;
            args.count[i] = s.count;
            args.seq[i] = s.seq;
            max_tokens = std::max(max_tokens, s.count);
            if (s.count > 0)
                max_touched = std::max(max_touched, (s.ctx_tok0 + s.count - 1) / kPageSize - s.ctx_tok0 / kPageSize + 1);
        }
        MoveShape shape = move_shape(ctx, max_tokens);
        shape.n_in_launch = n;
        shape.max_pages_touched = max_touched;
        if (link_workgroups > 0) {
            CA_HIP(ctx, launch_link(to_pool, args, shape, link_workgroups, (uint8_t *)k_pool, (uint8_t *)v_pool, stream));
            continue;
        }
        // A decode step's write-back: the host has looked up the slots.  (Not into a graph: its replays may follow another
        // plan's table.)
        if (!to_pool && max_tokens == 1 && !is_captured(stream)) {
            TokenSlots slots;
            TokenRows rows;
            const int64_t rb = row_bytes(ctx->cfg);
            for (int i = 0; i < n; ++i) {
                const Segment &s = segs[at + i];
                slots.slot[i] = token_slot(ctx, s.seq, s.ctx_tok0);
                rows.k[i] = s.k + s.contig_tok0 * rb;
                rows.v[i] = s.v + s.contig_tok0 * rb;
            }
            CA_HIP(ctx, launch_save_tokens(slots, rows, n, shape, (const uint8_t *)k_pool, (const uint8_t *)v_pool, stream));
            continue;
        }
        CA_HIP(ctx, launch_move(to_pool, args, shape, (uint8_t *)k_pool, (uint8_t *)v_pool, stream));
    }
    return CA_OK;
}

// shape of a launch that moves the new turn of conversations [first, first + n)
MoveShape new_turn_shape(const ca_ctx *ctx, int first, int n) {
    int max_touched = 0, max_tokens = 0;
    for (int q = first; q < first + n; ++q) {
        max_tokens = std::max(max_tokens, ctx->new_len[q]);
        max_touched = std::max(max_touched, (ctx->n_keep[q] + ctx->new_len[q] - 1) / kPageSize - ctx->n_keep[q] / kPageSize + 1);
    }
    MoveShape shape = move_shape(ctx, max_tokens);
    shape.n_in_launch = n;
    shape.max_pages_touched = max_touched;
    return shape;
}

// the new turn's K/V -> pool, on `stream`
ca_status run_append(ca_ctx *ctx, const void *new_k, const void *new_v, void *k_pool, void *v_pool, hipStream_t stream) {
    int iv;
    CA_HIP(ctx, prof_begin(ctx, kProfAppend, stream, &iv));
    // One new token per conversation, as many as the arguments hold: the host has looked up the slots.  (Not into a graph, whose
    // replays read the plan of their time.)
    if (ctx->total_q == ctx->n_seqs && ctx->n_seqs <= kMaxSeqsPerLaunch && !is_captured(stream)) {
        TokenSlots slots;
        for (int i = 0; i < ctx->n_seqs; ++i) slots.slot[i] = token_slot(ctx, i, ctx->n_keep[i]);
        CA_HIP(ctx, launch_append_tokens(slots, ctx->n_seqs, move_shape(ctx, 1), (const uint8_t *)new_k, (const uint8_t *)new_v, (uint8_t *)k_pool,
                                         (uint8_t *)v_pool, stream));
        CA_HIP(ctx, prof_end(ctx, iv, stream));
        return CA_OK;
    }
    CA_HIP(ctx, launch_append(new_turn_shape(ctx, 0, ctx->n_seqs), (const uint8_t *)new_k, (const uint8_t *)new_v, (uint8_t *)k_pool,
                              (uint8_t *)v_pool, stream));
    CA_HIP(ctx, prof_end(ctx, iv, stream));
    return CA_OK;
}

ca_status check_pools(ca_ctx *ctx, const char *who, const void *k_pool, const void *v_pool, MemMap &map) {
    if (!k_pool || !v_pool) return fail(ctx, CA_ERR_INVALID_ARG, "%s: pool pointer is NULL", who);
    const size_t bytes = (size_t)ctx->num_pages * ctx->cfg.page_size * (size_t)row_bytes(ctx->cfg);
    if (!map.device_range_ok(k_pool, bytes) || !map.device_range_ok(v_pool, bytes))
        return fail(ctx, CA_ERR_INVALID_ARG, "%s: a pool is not device memory holding num_pages=%d pages (%zu bytes)", who,
                    ctx->num_pages, bytes);
    return CA_OK;
}

// Workgroups of a write-back of `tokens` of `layer` to pinned memory.  Both directions of the link at once hold up the attention
// over keys rotated beforehand, which has a tile's time for its loads where the one that rotates them has two.  So beside
// it and the loads of later layers two workgroups write back, as long as the loads, at twice their rate, bring at least
// twice as much.  A step of 64 conversations of 1024-4096 + 64-512 tokens, 64/8 heads, 80 layers: attention 2705 us with four
// and 2137 with two (1660 alone), the link 55.1 and 56.5 GB/s, the step 986.5 and 961.2 ms; nine other batches of such plans
// 0.92 to 1.00 of their time.  Beside the other kernel four are the better: 16 conversations of 512-2048 + 32-256, 32 heads, 32
// layers, 199 ms a step, 207 with two.
int save_workgroups(const ca_ctx *ctx, int32_t layer, int64_t tokens) {
    const bool beside_loads = ctx->link_layer >= 0 && ctx->link_layer != layer;
    return ctx->prerotate && beside_loads && ctx->total_n >= 2 * tokens ? kLinkSaveBesideLoads : kLinkSaveWorkgroups;
}

// Is a save of `bytes` so short that it runs on the caller's stream?  (save_mode 1 keeps what it asks for, the staging slot.)
bool save_is_short(const ca_ctx *ctx, bool to_host, int64_t bytes) {
    return ctx->cfg.save_mode != 1 && bytes <= (to_host ? kInlineHostSaveBytes : kInlineDeviceBytes);
}

// Saves are done in the order they were asked for (two may write the same rows of the tier): none goes to the caller's stream
// while another under this plan is on the save stream, and the save stream waits for those on the caller's streams.  (Earlier
// plans' saves are in front of the plan.)
bool save_stream_idle(ca_ctx *ctx) {
    if (!ctx->saves_under_plan) return true;
    if (query(ctx->ev_saved) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    ctx->saves_under_plan = false;
    return true;
}

// the save stream continues behind the plan, the work queued so far on `after` and the short moves on other streams
ca_status save_follows(ca_ctx *ctx, hipStream_t after) {
    CA_HIP(ctx, save_stream_for(ctx, after));
    if (ctx->inline_pending && (ctx->inline_stream != after || ctx->inline_owner != stream_owner(after))) {
        if (!ctx->inline_done) CA_HIP(ctx, hipEventRecord(ctx->ev_inline, nullptr));
        CA_HIP(ctx, wait_for(ctx->s_save, ctx->inline_done ? ctx->inline_done : ctx->ev_inline));
    }
    if (after != nullptr || ctx->plan_stream != nullptr) CA_HIP(ctx, after_plan(ctx, ctx->s_save, &ctx->save_waits_plan));
    ctx->save_waits_plan = false;          // (behind the default stream: the plan is in front there)
    CA_HIP(ctx, hipEventRecord(ctx->ev_after, after));
    CA_HIP(ctx, hipStreamWaitEvent(ctx->s_save, ctx->ev_after, 0));
    return CA_OK;
}

hipError_t note_save(ca_ctx *ctx) {
    ctx->save_pending = ctx->saves_under_plan = true;
    ctx->joined_null = false;
    return hipEventRecord(ctx->ev_saved, ctx->s_save);
}

ca_status check_layer_plan(ca_ctx *ctx, const char *who, int32_t layer) {
    if (!ctx->has_plan) return fail(ctx, CA_ERR_NOT_READY, "%s: no plan (call ca_rope_rebase first)", who);
    if (layer < 0 || layer >= ctx->cfg.n_layers)
        return fail(ctx, CA_ERR_OUT_OF_RANGE, "%s: layer %d outside [0, %d)", who, layer, ctx->cfg.n_layers);
    return CA_OK;
}

}  // namespace

ca_status ca_kv_load_layer(ca_ctx *ctx, int32_t layer, const void *const *src_k, const void *const *src_v,
                           void *k_pool, void *v_pool) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    ca_status st = check_layer_plan(ctx, "ca_kv_load_layer", layer);
    if (st != CA_OK) return st;
    if (!src_k || !src_v) return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_load_layer: source pointer array is NULL");
    if (ctx->loaded[layer]) return fail(ctx, CA_ERR_NOT_READY, "ca_kv_load_layer: layer %d already loaded under this plan", layer);
    const ca_config &c = ctx->cfg;
    CA_HIP(ctx, hipSetDevice(c.device));
    MemMap map;
    st = check_pools(ctx, "ca_kv_load_layer", k_pool, v_pool, map);
    if (st != CA_OK) return st;

    const int B = ctx->n_seqs;
    const int64_t rb = row_bytes(c);
    bool any_host = false, any_unknown = false;
    std::vector<uint8_t *> gpu_k(B), gpu_v(B);      // the sources as a kernel reads them
    MemMap map_k;          // (keys and values may be in an allocation each)
    for (int i = 0; i < B; ++i) {
        if (ctx->n_keep[i] == 0) continue;
        if (!src_k[i] || !src_v[i]) return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_load_layer: source of conversation %d is NULL", i);
        // device memory holds the saved history; of pinned memory only what is read has to be there, up to the last kept range
        const size_t saved = (size_t)ctx->hist_len[i] * rb, read = (size_t)ctx->keep_rng[ctx->keep_rng_at[i + 1] - 1].second * rb;
        size_t k_room, v_room;
        const MemKind kk = map_k.look(src_k[i], &k_room, &gpu_k[i]), kv = map.look(src_v[i], &v_room, &gpu_v[i]);
        if (kk == MemKind::kUnknown || kv == MemKind::kUnknown) any_unknown = true;
        if (kk == MemKind::kPinnedHost || kv == MemKind::kPinnedHost) any_host = true;
        if (k_room < (kk == MemKind::kDevice ? saved : read))
            return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_load_layer: K source of conversation %d is smaller than hist_len tokens", i);
        if (v_room < (kv == MemKind::kDevice ? saved : read))
            return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_load_layer: V source of conversation %d is smaller than hist_len tokens", i);
    }
    if (any_unknown)
        return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_load_layer: a source is neither pinned host nor device memory");
    const int64_t move_bytes = 2 * ctx->total_n * rb;
    const bool small = move_bytes <= (any_host ? kInlineHostLoadBytes : kInlineDeviceBytes);
    const bool staged = c.load_mode == 1;
    const bool on_caller = small && !staged && stream_usable(ctx->plan_stream) && inline_free(ctx, ctx->plan_stream);
    hipStream_t mover = on_caller ? ctx->plan_stream : ctx->s_unpack;
    if (on_caller) CA_HIP(ctx, caller_after_plan(ctx, mover));
    else CA_HIP(ctx, after_plan(ctx, ctx->s_unpack, &ctx->unpack_waits_plan));

    std::vector<Segment> segs;
    segs.reserve(B);
    if (staged) {
        const int slot = (int)(ctx->load_count % c.pipeline_depth);
        uint8_t *sk = ctx->load_slots + (size_t)slot * ctx->slot_bytes;
        uint8_t *sv = sk + ctx->half_slot_bytes;
        // The K half is copied on the copy stream and the V half on the unpack stream, ahead of the kernel that needs
        // both: two copy queues keep the host link busier than one (each fills the gaps between the other's
        // per-conversation copies), and a stream of its own for the second queue would be one more than the hardware
        // queues a process has, which makes unrelated streams wait for each other.
        CA_HIP(ctx, after_plan(ctx, ctx->s_copy, &ctx->copy_waits_plan));
        // the slot is free again once the unpack that last read it has finished (the unpack stream is behind it anyway)
        if (ctx->slot_used[slot]) CA_HIP(ctx, hipStreamWaitEvent(ctx->s_copy, ctx->ev_slot_free[slot], 0));
        int iv_copy;
        CA_HIP(ctx, prof_begin(ctx, kProfCopyIn, ctx->s_copy, &iv_copy));
        for (int i = 0; i < B; ++i) {
            const int64_t n = ctx->n_keep[i];
            if (n == 0) continue;
            // the kept ranges land back to back in the slot: truncation and discarding are source offsets
            size_t dst_off = (size_t)ctx->cu_n[i] * rb;
            for (int r = ctx->keep_rng_at[i]; r < ctx->keep_rng_at[i + 1]; ++r) {
                const size_t src_off = (size_t)ctx->keep_rng[r].first * rb;
                const size_t bytes = (size_t)(ctx->keep_rng[r].second - ctx->keep_rng[r].first) * rb;
                CA_HIP(ctx, hipMemcpyAsync(sk + dst_off, (const uint8_t *)src_k[i] + src_off, bytes, hipMemcpyDefault, ctx->s_copy));
                CA_HIP(ctx, hipMemcpyAsync(sv + dst_off, (const uint8_t *)src_v[i] + src_off, bytes, hipMemcpyDefault, ctx->s_unpack));
                dst_off += bytes;
            }
            segs.push_back({sk, sv, ctx->cu_n[i], 0, (int32_t)n, i});
        }
        if (iv_copy >= 0) {
            // a timed copy-in ends when both halves have landed (only then do the two queues meet once per layer)
            CA_HIP(ctx, hipEventRecord(ctx->ev_slot_copied2[slot], ctx->s_unpack));
            CA_HIP(ctx, hipStreamWaitEvent(ctx->s_copy, ctx->ev_slot_copied2[slot], 0));
        }
        CA_HIP(ctx, prof_end(ctx, iv_copy, ctx->s_copy));
        CA_HIP(ctx, hipEventRecord(ctx->ev_slot_copied[slot], ctx->s_copy));
        CA_HIP(ctx, hipStreamWaitEvent(ctx->s_unpack, ctx->ev_slot_copied[slot], 0));
        int iv_unpack;
        CA_HIP(ctx, prof_begin(ctx, kProfUnpack, ctx->s_unpack, &iv_unpack));
        st = run_move(ctx, true, segs, k_pool, v_pool, ctx->s_unpack);
        if (st != CA_OK) return st;
        CA_HIP(ctx, prof_end(ctx, iv_unpack, ctx->s_unpack));
        CA_HIP(ctx, hipEventRecord(ctx->ev_slot_free[slot], ctx->s_unpack));
        ctx->slot_used[slot] = 1;
        ctx->load_count++;
    } else {
        for (int i = 0; i < B; ++i) {
            const int64_t n = ctx->n_keep[i];
            if (n == 0) continue;
            int32_t at = 0;      // context token the range starts at
            for (int r = ctx->keep_rng_at[i]; r < ctx->keep_rng_at[i + 1]; ++r) {
                const int32_t len = ctx->keep_rng[r].second - ctx->keep_rng[r].first;
                segs.push_back({gpu_k[i], gpu_v[i], ctx->keep_rng[r].first, at, len, i});
                at += len;
            }
        }
        // Across the host link one kernel reads the tier in place and scatters it into the pages.  It counts as the layer's
        // copy-in; the unpacking, which is part of it, as an empty interval behind it.
        const bool link = any_host && !on_caller;
        int iv_in = -1, iv_unpack;
        if (link) CA_HIP(ctx, prof_begin(ctx, kProfCopyIn, mover, &iv_in));
        else CA_HIP(ctx, prof_begin(ctx, kProfUnpack, mover, &iv_unpack));
        st = run_move(ctx, true, segs, k_pool, v_pool, mover, link ? kLinkLoadWorkgroups : 0);
        if (st != CA_OK) return st;
        CA_HIP(ctx, prof_end(ctx, iv_in, mover));
        if (link) ctx->link_layer = layer;
        if (link) CA_HIP(ctx, prof_begin(ctx, kProfUnpack, mover, &iv_unpack));
        CA_HIP(ctx, prof_end(ctx, iv_unpack, mover));
    }
    if (!on_caller || mover != nullptr) CA_HIP(ctx, hipEventRecord(ctx->ev_ready[layer], mover));
    if (on_caller) {
        note_inline(ctx, mover, mover != nullptr ? ctx->ev_ready[layer] : nullptr);
    } else {
        ctx->load_done = ctx->ev_ready[layer];
        ctx->joined_null = false;
    }
    ctx->ready_inline[layer] = on_caller ? 1 : 0;
    ctx->loaded[layer] = 1;
    return CA_OK;
}

ca_status ca_kv_append_layer(ca_ctx *ctx, int32_t layer, const void *new_k, const void *new_v, void *k_pool,
                             void *v_pool, void *stream) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    ca_status st = check_layer_plan(ctx, "ca_kv_append_layer", layer);
    if (st != CA_OK) return st;
    const ca_config &c = ctx->cfg;
    CA_HIP(ctx, hipSetDevice(c.device));
    MemMap map;
    st = check_pools(ctx, "ca_kv_append_layer", k_pool, v_pool, map);
    if (st != CA_OK) return st;
    const size_t bytes = (size_t)ctx->total_q * (size_t)row_bytes(c);
    if (!map.device_range_ok(new_k, bytes) || !map.device_range_ok(new_v, bytes))
        return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_append_layer: new_k/new_v must be device memory of %zu bytes", bytes);
    return run_append(ctx, new_k, new_v, k_pool, v_pool, (hipStream_t)stream);
}

ca_status ca_kv_save_layer(ca_ctx *ctx, int32_t layer, const int32_t *tok_begin, const int32_t *tok_end,
                           const void *k_pool, const void *v_pool, void *const *dst_k, void *const *dst_v,
                           const int64_t *dst_tok_offset, void *after_stream) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    ca_status st = check_layer_plan(ctx, "ca_kv_save_layer", layer);
    if (st != CA_OK) return st;
    if (!dst_k || !dst_v) return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_save_layer: destination pointer array is NULL");
    if ((tok_begin == nullptr) != (tok_end == nullptr))
        return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_save_layer: tok_begin and tok_end must both be given or both NULL");
    const ca_config &c = ctx->cfg;
    CA_HIP(ctx, hipSetDevice(c.device));
    MemMap map, map_k;
    st = check_pools(ctx, "ca_kv_save_layer", k_pool, v_pool, map);
    if (st != CA_OK) return st;

    const int B = ctx->n_seqs;
    const int64_t rb = row_bytes(c);
    struct Range { int32_t b, e; int64_t off; };
    std::vector<Range> r(B);
    std::vector<uint8_t *> gpu_k(B), gpu_v(B);      // the destinations as a kernel writes them
    bool any_host = false;
    int64_t total = 0;
    for (int i = 0; i < B; ++i) {
        const int32_t ctx_len = ctx->n_keep[i] + ctx->new_len[i];
        r[i].b = tok_begin ? tok_begin[i] : ctx->n_keep[i];
        r[i].e = tok_end ? tok_end[i] : ctx_len;
        r[i].off = dst_tok_offset ? dst_tok_offset[i] : ctx->hist_len[i];
        if (r[i].b < 0 || r[i].e < r[i].b || r[i].e > ctx_len)
            return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_kv_save_layer: conversation %d: token range [%d, %d) outside the context [0, %d)", i,
                        r[i].b, r[i].e, ctx_len);
        if (r[i].off < 0) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_kv_save_layer: conversation %d: negative destination offset", i);
        if (r[i].e == r[i].b) continue;
        if (!dst_k[i] || !dst_v[i]) return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_save_layer: destination of conversation %d is NULL", i);
        const size_t need = (size_t)(r[i].off + (r[i].e - r[i].b)) * rb;
        size_t k_room, v_room;
        const MemKind kk = map_k.look(dst_k[i], &k_room, &gpu_k[i]), kv = map.look(dst_v[i], &v_room, &gpu_v[i]);
        if (kk == MemKind::kUnknown || kv == MemKind::kUnknown)
            return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_save_layer: destination of conversation %d is neither pinned host nor device memory", i);
        if (kk == MemKind::kPinnedHost || kv == MemKind::kPinnedHost) any_host = true;
        if (k_room < need || v_room < need)
            return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_save_layer: destination of conversation %d is smaller than offset + count tokens", i);
        total += r[i].e - r[i].b;
    }
    if (total > c.max_batch_kv_tokens) return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_kv_save_layer: %lld tokens exceed a staging slot", (long long)total);
    hipStream_t after = (hipStream_t)after_stream;
    const bool on_caller = save_is_short(ctx, any_host, 2 * total * rb) && save_stream_idle(ctx) && inline_free(ctx, after);
    const bool staged = c.save_mode == 1;

    // saving starts after the producer of this layer's K/V: the work queued on `after_stream`, and the load of
    // this layer if one was issued (its unpack runs on an internal stream and may still be writing the pages a
    // range of kept-history tokens reads)
    if (on_caller) {
        CA_HIP(ctx, caller_after_plan(ctx, after));
    } else {
        st = save_follows(ctx, after);
        if (st != CA_OK) return st;
    }
    hipStream_t saver = on_caller ? after : ctx->s_save;
    if (ctx->loaded[layer]) CA_HIP(ctx, after_load(ctx, layer, saver));

    std::vector<Segment> segs;
    segs.reserve(B);
    if (staged) {
        // pack and copy-out run on the one save stream, so a slot is never overwritten while it is
        // still being copied; several slots only let the caller queue saves without bound
        const int slot = (int)(ctx->save_count % c.pipeline_depth);
        uint8_t *sk = ctx->save_slots + (size_t)slot * ctx->slot_bytes;
        uint8_t *sv = sk + ctx->half_slot_bytes;
        int64_t at = 0;
        std::vector<int64_t> slot_tok0(B, 0);
        for (int i = 0; i < B; ++i) {
            const int32_t cnt = r[i].e - r[i].b;
            if (cnt == 0) continue;
            slot_tok0[i] = at;
            segs.push_back({sk, sv, at, r[i].b, cnt, i});
            at += cnt;
        }
        int iv_pack, iv_out;
        CA_HIP(ctx, prof_begin(ctx, kProfPack, ctx->s_save, &iv_pack));
        st = run_move(ctx, false, segs, (void *)k_pool, (void *)v_pool, ctx->s_save);
        if (st != CA_OK) return st;
        CA_HIP(ctx, prof_end(ctx, iv_pack, ctx->s_save));
        CA_HIP(ctx, prof_begin(ctx, kProfCopyOut, ctx->s_save, &iv_out));
        for (int i = 0; i < B; ++i) {
            const int32_t cnt = r[i].e - r[i].b;
            if (cnt == 0) continue;
            const size_t bytes = (size_t)cnt * rb, src_off = (size_t)slot_tok0[i] * rb, dst_off = (size_t)r[i].off * rb;
            CA_HIP(ctx, hipMemcpyAsync((uint8_t *)dst_k[i] + dst_off, sk + src_off, bytes, hipMemcpyDefault, ctx->s_save));
            CA_HIP(ctx, hipMemcpyAsync((uint8_t *)dst_v[i] + dst_off, sv + src_off, bytes, hipMemcpyDefault, ctx->s_save));
        }
        CA_HIP(ctx, prof_end(ctx, iv_out, ctx->s_save));
        ctx->save_count++;
    } else {
        for (int i = 0; i < B; ++i) {
            const int32_t cnt = r[i].e - r[i].b;
            if (cnt == 0) continue;
            segs.push_back({gpu_k[i], gpu_v[i], r[i].off, r[i].b, cnt, i});
        }
        int iv_pack;
        CA_HIP(ctx, prof_begin(ctx, kProfPack, saver, &iv_pack));
        st = run_move(ctx, false, segs, (void *)k_pool, (void *)v_pool, saver, any_host && !on_caller ? save_workgroups(ctx, layer, total) : 0);
        if (st != CA_OK) return st;
        CA_HIP(ctx, prof_end(ctx, iv_pack, saver));
    }
    if (on_caller) CA_HIP(ctx, note_inline(ctx, saver));
    else CA_HIP(ctx, note_save(ctx));
    return CA_OK;
}

// Appending and saving the new turn in one call: the saved bytes ARE the appended bytes (keys without positions,
// Section 3.4), so the pool need not be read back.  Device destinations (and pinned ones under save_mode 2, or when the
// turn is short): one kernel reads new_k/new_v once and stores every vector twice (pool and tier).  Pinned destinations by
// default, and all while another stream's short move is under way: append kernel, then the pack kernel writes the tier in place
// from the save stream.  Pinned destinations with staged saving: the
// copy-out on the save stream reads new_k/new_v directly; no pack kernel, no staging slot.
ca_status ca_kv_append_save_layer(ca_ctx *ctx, int32_t layer, const void *new_k, const void *new_v, void *k_pool,
                                  void *v_pool, void *const *dst_k, void *const *dst_v, void *stream_) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    ca_status st = check_layer_plan(ctx, "ca_kv_append_save_layer", layer);
    if (st != CA_OK) return st;
    if (!dst_k || !dst_v) return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_append_save_layer: destination pointer array is NULL");
    const ca_config &c = ctx->cfg;
    CA_HIP(ctx, hipSetDevice(c.device));
    MemMap map, map_k;
    st = check_pools(ctx, "ca_kv_append_save_layer", k_pool, v_pool, map);
    if (st != CA_OK) return st;
    const int64_t rb = row_bytes(c);
    const size_t bytes = (size_t)ctx->total_q * (size_t)rb;
    if (!map.device_range_ok(new_k, bytes) || !map.device_range_ok(new_v, bytes))
        return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_append_save_layer: new_k/new_v must be device memory of %zu bytes", bytes);
    const int B = ctx->n_seqs;
    std::vector<uint8_t *> gpu_k(B), gpu_v(B);      // the destinations as a kernel writes them
    bool any_host = false;
    for (int i = 0; i < B; ++i) {
        if (!dst_k[i] || !dst_v[i]) return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_append_save_layer: destination of conversation %d is NULL", i);
        const size_t need = (size_t)(ctx->hist_len[i] + ctx->new_len[i]) * rb;
        size_t k_room, v_room;
        const MemKind kk = map_k.look(dst_k[i], &k_room, &gpu_k[i]), kv = map.look(dst_v[i], &v_room, &gpu_v[i]);
        if (kk == MemKind::kUnknown || kv == MemKind::kUnknown)
            return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_append_save_layer: destination of conversation %d is neither pinned host nor device memory", i);
        if (kk == MemKind::kPinnedHost || kv == MemKind::kPinnedHost) any_host = true;
        if (k_room < need || v_room < need)
            return fail(ctx, CA_ERR_INVALID_ARG, "ca_kv_append_save_layer: destination of conversation %d is smaller than hist_len + new_len tokens", i);
    }
    hipStream_t stream = (hipStream_t)stream_;
    const bool captured = is_captured(stream);
    const bool one_kernel = (any_host ? c.save_mode == 2 || (save_is_short(ctx, any_host, 2 * (int64_t)bytes) && (captured || save_stream_idle(ctx)))
                                      : c.save_mode != 1) && (captured || inline_free(ctx, stream));
    if (!one_kernel) {
        // the append kernel on the caller's stream (which must not wait for stores that cross the host link); the write-back
        // follows it on the save stream
        st = run_append(ctx, new_k, new_v, k_pool, v_pool, stream);
        if (st == CA_OK) st = save_follows(ctx, stream);
        if (st != CA_OK) return st;
        int iv;
        if (c.save_mode != 1) {
            // the pack kernel writes the new tokens to the tier in place
            std::vector<Segment> segs;
            for (int i = 0; i < B; ++i)
                if (ctx->new_len[i] > 0)
                    segs.push_back({gpu_k[i], gpu_v[i], ctx->hist_len[i], ctx->n_keep[i], ctx->new_len[i], i});
            if (ctx->loaded[layer]) CA_HIP(ctx, after_load(ctx, layer, ctx->s_save));
            CA_HIP(ctx, prof_begin(ctx, kProfPack, ctx->s_save, &iv));
            st = run_move(ctx, false, segs, k_pool, v_pool, ctx->s_save, any_host ? save_workgroups(ctx, layer, ctx->total_q) : 0);
            if (st != CA_OK) return st;
        } else {
            // one copy per conversation, straight from new_k / new_v
            CA_HIP(ctx, prof_begin(ctx, kProfCopyOut, ctx->s_save, &iv));
            for (int i = 0; i < B; ++i) {
                const size_t n = (size_t)ctx->new_len[i] * rb, src_off = (size_t)ctx->cu_q[i] * rb, dst_off = (size_t)ctx->hist_len[i] * rb;
                CA_HIP(ctx, hipMemcpyAsync((uint8_t *)dst_k[i] + dst_off, (const uint8_t *)new_k + src_off, n, hipMemcpyDefault, ctx->s_save));
                CA_HIP(ctx, hipMemcpyAsync((uint8_t *)dst_v[i] + dst_off, (const uint8_t *)new_v + src_off, n, hipMemcpyDefault, ctx->s_save));
            }
        }
        CA_HIP(ctx, prof_end(ctx, iv, ctx->s_save));
        CA_HIP(ctx, note_save(ctx));
        return CA_OK;
    }
    // one pass: every vector of the new turn goes to its page and to its row of the tier
    int iv;
    CA_HIP(ctx, prof_begin(ctx, kProfAppend, stream, &iv));
    for (int at = 0; at < B; at += kMaxSeqsPerLaunch) {
        MoveArgs2 second;
        const int n = std::min(kMaxSeqsPerLaunch, B - at);
        for (int i = 0; i < n; ++i) {       // new token j is saved behind the history, at token hist_len + j
            second.dst_k[i] = gpu_k[at + i] + (size_t)ctx->hist_len[at + i] * rb;
            second.dst_v[i] = gpu_v[at + i] + (size_t)ctx->hist_len[at + i] * rb;
        }
        CA_HIP(ctx, launch_append_save(new_turn_shape(ctx, at, n), at, second, (const uint8_t *)new_k, (const uint8_t *)new_v,
                                       (uint8_t *)k_pool, (uint8_t *)v_pool, stream));
    }
    CA_HIP(ctx, prof_end(ctx, iv, stream));
    if (!captured) CA_HIP(ctx, note_inline(ctx, stream));    // ca_sync and ca_join cover it, as they would the save stream
    return CA_OK;
}

// ----------------------------------------------------------------------------------------------
// Sections 2.1 / 3.1 / 3.4: attention of the new tokens
// ----------------------------------------------------------------------------------------------
// partial, arrived: where the shares of split row tiles go and are counted (the context's buffer, or the static scratch array);
// timed: bracket the launch with profiling events when profiling is on (creating an event may allocate)
static ca_status attn_impl(ca_ctx *ctx, int32_t layer, const void *q, const void *k_pool, const void *v_pool, void *out,
                           float softmax_scale, void *stream_, float *partial, uint32_t *arrived, bool timed) {
    ca_status st = check_layer_plan(ctx, "ca_cached_prefill_attn", layer);
    if (st != CA_OK) return st;
    const ca_config &c = ctx->cfg;
    CA_HIP(ctx, hipSetDevice(c.device));
    MemMap map;
    st = check_pools(ctx, "ca_cached_prefill_attn", k_pool, v_pool, map);
    if (st != CA_OK) return st;
    if (!(softmax_scale > 0.f) || !std::isfinite(softmax_scale))
        return fail(ctx, CA_ERR_INVALID_ARG, "ca_cached_prefill_attn: softmax_scale must be finite and > 0");
    const size_t q_bytes = (size_t)ctx->total_q * c.n_q_heads * c.head_dim * 2;
    if (!map.device_range_ok(q, q_bytes) || !map.device_range_ok(out, q_bytes))
        return fail(ctx, CA_ERR_INVALID_ARG, "ca_cached_prefill_attn: q/out must be device memory of %zu bytes", q_bytes);
    hipStream_t stream = (hipStream_t)stream_;
    if (ctx->loaded[layer]) {
        CA_HIP(ctx, after_load(ctx, layer, stream));
    } else if (c.require_load && ctx->total_n > 0) {
        return fail(ctx, CA_ERR_NOT_READY, "ca_cached_prefill_attn: layer %d has kept history but was not loaded under this plan", layer);
    }
    AttnArgs a{};
    a.q = (const uint16_t *)q;
    a.out = (uint16_t *)out;
    a.k_pool = (const uint16_t *)k_pool;
    a.v_pool = (const uint16_t *)v_pool;
    a.block_table = (const int32_t *)(ctx->d_meta + ctx->off_table);
    a.n_keep = (const int32_t *)(ctx->d_meta + ctx->off_n_keep);
    a.cu_q = (const int32_t *)(ctx->d_meta + ctx->off_cu_q);
    a.q_pos = (const int32_t *)(ctx->d_meta + ctx->off_q_pos);
    a.q_seq = (const int32_t *)(ctx->d_meta + ctx->off_q_seq);
    a.items = (const WorkItem *)(ctx->d_meta + ctx->off_items);
    a.combine = (const CombineItem *)(ctx->d_meta + ctx->off_combine);
    a.partial = partial;
    a.k_rot = ctx->k_rot;
    a.dense_page0 = (const int32_t *)(ctx->d_meta + ctx->off_dense0);
    a.rot_src_page = (const int32_t *)(ctx->d_meta + ctx->off_rot_src);
    a.rot_pos0 = (const int32_t *)(ctx->d_meta + ctx->off_rot_pos);
    a.v_t = ctx->v_t;
    a.rot_nvalid = (const int32_t *)(ctx->d_meta + ctx->off_rot_nvalid);
    a.pipelined = ctx->pipelined ? 1 : 0;
    a.n_dense_pages = ctx->n_dense_pages;
    a.max_positions = c.max_positions;
    a.n_combine = ctx->n_combine;
    a.rope = ctx->rope;
    a.n_items = ctx->n_items;
    a.wg_first = (const int32_t *)(ctx->d_meta + ctx->off_wg_first);
    a.rows_items = (const RowsItem *)(ctx->d_meta + ctx->off_rows_items);
    a.arrived = arrived;
    a.n_wgs = ctx->n_wgs;
    a.total_q = (int32_t)ctx->total_q;
    a.max_pages = ctx->max_pages;
    a.n_q_heads = c.n_q_heads;
    a.n_kv_heads = c.n_kv_heads;
    a.head_dim = c.head_dim;
    a.rope_style = c.rope_style;
    a.tile_rows = ctx->tile_rows;
    a.wgs_per_cu = ctx->wgs_per_cu;
    a.softmax_scale = softmax_scale;
    int iv = -1;
    if (timed) CA_HIP(ctx, prof_begin(ctx, kProfAttn, stream, &iv));
    const bool direct = direct_variant(c);
    // a decode step (one or two stacked rows per (conversation, kv head)) is a matrix-vector product: streamed
    const bool decode = direct && c.attn_variant != 2 && !ctx->prerotate && ctx->max_unit_rows >= 1 &&
                        ctx->max_unit_rows <= kAttnDecodeMaxRows;
    if (c.attn_variant == 4 && !decode) {
        (void)prof_end(ctx, iv, stream);
        return fail(ctx, CA_ERR_UNSUPPORTED, "ca_cached_prefill_attn: attn_variant 4 needs at most %d stacked rows per (conversation, kv head), the plan has %d",
                    kAttnDecodeMaxRows, ctx->max_unit_rows);
    }
    if (c.attn_variant == 1) {
        CA_HIP(ctx, launch_attn_ref(a, stream));
    } else if (ctx->n_wgs > 0) {
        CA_HIP(ctx, launch_attn_rows(a, ctx->wg_wavefronts, ctx->rows_runs, stream));
    } else if (decode) {
        CA_HIP(ctx, launch_attn_decode(a, ctx->max_unit_rows, stream));
    } else if (direct && ctx->pipelined) {
        CA_HIP(ctx, launch_attn_pp(a, stream));
    } else if (direct && ctx->prerotate) {
        CA_HIP(ctx, launch_attn_prerot(a, stream));
    } else if (direct) {
        CA_HIP(ctx, launch_attn_dma(a, stream));
    } else {
        return fail(ctx, CA_ERR_UNSUPPORTED, "ca_cached_prefill_attn: attn_variant %d", c.attn_variant);
    }
    CA_HIP(ctx, prof_end(ctx, iv, stream));
    return CA_OK;
}

ca_status ca_cached_prefill_attn(ca_ctx *ctx, int32_t layer, const void *q, const void *k_pool, const void *v_pool,
                                 void *out, float softmax_scale, void *stream) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    return attn_impl(ctx, layer, q, k_pool, v_pool, out, softmax_scale, stream, ctx->partial, ctx->arrived, true);
}

ca_status ca_cached_prefill_attn_static(ca_ctx *ctx, int32_t layer, const void *q, const void *k_pool, const void *v_pool,
                                        void *out, float softmax_scale, void *stream) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    if (ctx->has_plan && ctx->n_split_parts > 0) {
        if (!ctx->static_partial)
            return fail(ctx, CA_ERR_UNSUPPORTED, "ca_cached_prefill_attn_static: no static scratch on device %d", ctx->cfg.device);
        const size_t need = (size_t)ctx->n_split_parts * (size_t)ctx->tile_rows * (size_t)(ctx->cfg.head_dim + 2) * sizeof(float);
        if (need > (ctx->last_round_cut ? kStaticArrayBytes : kStaticScratchBytes))
            return fail(ctx, CA_ERR_OUT_OF_RANGE, "ca_cached_prefill_attn_static: the plan's %d shares of split row tiles need %zu bytes of "
                        "partial results, the static scratch holds %zu", ctx->n_split_parts, need, kStaticScratchBytes);
    }
    return attn_impl(ctx, layer, q, k_pool, v_pool, out, softmax_scale, stream, ctx->static_partial, ctx->static_arrived, false);
}

// ----------------------------------------------------------------------------------------------
// timing of the library's own GPU work
// ----------------------------------------------------------------------------------------------
ca_status ca_profile_enable(ca_ctx *ctx, int32_t on) {
    if (!ctx) return CA_ERR_INVALID_ARG;
    ctx->profiling = on != 0;
    ctx->profile_mask = (on == 1 || on == 0) ? ~0u : ((uint32_t)on >> 1);
    return CA_OK;
}

ca_status ca_profile_read(ca_ctx *ctx, int32_t kind, double *total_ms, int64_t *count) {
    if (!ctx || !total_ms || !count) return CA_ERR_INVALID_ARG;
    if (kind < 0 || kind >= kProfKinds) return fail(ctx, CA_ERR_INVALID_ARG, "ca_profile_read: kind %d", kind);
    CA_HIP(ctx, hipSetDevice(ctx->cfg.device));
    CA_HIP(ctx, hipDeviceSynchronize());
    double sum = 0.0;
    int64_t n = 0;
    std::vector<ca_ctx::Interval> keep;
    for (auto &iv : ctx->intervals) {
        if (iv.kind != kind) { keep.push_back(iv); continue; }
        float ms = 0.f;
        CA_HIP(ctx, hipEventElapsedTime(&ms, iv.start, iv.stop));
        sum += ms;
        ++n;
        ctx->spare_events.push_back(iv.start);
        ctx->spare_events.push_back(iv.stop);
    }
    ctx->intervals.swap(keep);
    *total_ms = sum;
    *count = n;
    return CA_OK;
}

ca_status ca_profile_timeline(ca_ctx *ctx, int32_t *kinds, double *start_ms, double *stop_ms, int64_t capacity,
                              int64_t *count) {
    if (!ctx || !count || capacity < 0) return CA_ERR_INVALID_ARG;
    if (capacity > 0 && (!kinds || !start_ms || !stop_ms)) return fail(ctx, CA_ERR_INVALID_ARG, "ca_profile_timeline: null array");
    CA_HIP(ctx, hipSetDevice(ctx->cfg.device));
    CA_HIP(ctx, hipDeviceSynchronize());
    *count = (int64_t)ctx->intervals.size();
    const int64_t n = std::min<int64_t>(*count, capacity);
    for (int64_t i = 0; i < n; ++i) {
        const auto &iv = ctx->intervals[(size_t)i];
        float a = 0.f, b = 0.f;
        if (i > 0) CA_HIP(ctx, hipEventElapsedTime(&a, ctx->intervals[0].start, iv.start));
        CA_HIP(ctx, hipEventElapsedTime(&b, iv.start, iv.stop));
        kinds[i] = iv.kind;
        start_ms[i] = a;
        stop_ms[i] = (double)a + b;
    }
    return CA_OK;
}

}  // extern "C"
