// Order between the private streams of contexts set up on the null stream, and the streams themselves.
//
// The runtime orders such a stream with the caller's work on the null stream, but not with the private stream of another
// context, and most calls return before their work is done.  So every call states the ranges of caller memory it reads
// and writes, and first waits, on the device, for the earlier calls of other contexts that it conflicts with: a field one
// context writes and the next one reads, or memory that is in a call's use when the caller's allocator hands it out
// again.  Calls without a conflict are not ordered: contexts overlap (two contexts at 16^3 take 27 us a call,
// 38 us when each waits for the other).
#include <algorithm>
#include <mutex>

#include "common.h"

namespace ls {

namespace {

constexpr int kMaxStreamDevices = 64;
std::mutex g_order_mutex;            // guards everything below and Ctx::order of every context
std::vector<Ctx*> g_private;         // live contexts on private streams
std::vector<hipStream_t> g_idle_streams[kMaxStreamDevices];

bool conflict(const StreamOrder::Range* a, int na, const Span* s, int ns) {
    for (int i = 0; i < na; ++i)
        for (int k = 0; k < ns; ++k) {
            const uintptr_t lo = reinterpret_cast<uintptr_t>(s[k].p);
            if ((a[i].write || s[k].write) && a[i].lo < lo + s[k].bytes && lo < a[i].hi) return true;
        }
    return false;
}

// whether the work before the recorded event has ended (no error and no wait under a capture of the calling thread)
bool finished(const StreamOrder& o) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    const hipError_t e = hipEventQuery(o.ev);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

// whether a caller is recording the stream's work into a graph of its own: such work runs when the caller launches the
// graph, and its order is the caller's
bool captured(const Ctx* c) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// records the event behind the calls noted so far
int cover(Ctx* c) {
    StreamOrder& o = c->order;
    if (o.covered > 0 && finished(o)) {
        std::copy(o.range + o.covered, o.range + o.n, o.range);
        o.n -= o.covered;
    }
    if (o.n > StreamOrder::kMax / 2) {   // many calls in flight: their hull
        StreamOrder::Range h = o.range[0];
        for (int i = 1; i < o.n; ++i) h = {std::min(h.lo, o.range[i].lo), std::max(h.hi, o.range[i].hi), true};
        o.range[0] = h;
        o.n = 1;
    }
    LS_HIP(hipEventRecord(o.ev, c->stream));
    o.covered = o.n;
    return LS_OK;
}

// g_order_mutex held
int wait_for_others(Ctx* c, const Span* s, int ns) {
    for (Ctx* q : g_private) {
        StreamOrder& o = q->order;
        if (q == c || o.n == 0 || !conflict(o.range, o.n, s, ns)) continue;
        if (captured(c)) return LS_OK;
        // a stream inside a waiting call may be recording a graph: the ranges that are not covered are those of that
        // call, which its caller keeps until it returns
        if (o.covered < o.n && !o.waiting && !captured(q) && conflict(o.range + o.covered, o.n - o.covered, s, ns)) {
            const int rc = cover(q);
            if (rc) return rc;
        }
        if (o.covered == 0) continue;
        if (finished(o))
            std::copy(o.range + o.covered, o.range + o.n, o.range), o.n -= o.covered, o.covered = 0;
        else
            LS_HIP(hipStreamWaitEvent(c->stream, o.ev, 0));
    }
    return LS_OK;
}

}  // namespace

int order_begin(Ctx* c, const Span* s, int ns) {
    if (!c->own_stream) return LS_OK;
    std::lock_guard<std::mutex> lock(g_order_mutex);
    int rc = wait_for_others(c, s, ns);
    if (rc) return rc;
    StreamOrder& o = c->order;
    for (int k = 0; k < ns; ++k) {
        const uintptr_t lo = reinterpret_cast<uintptr_t>(s[k].p);
        const StreamOrder::Range r = {lo, lo + s[k].bytes, s[k].write};
        bool known = false;
        for (int i = o.covered; i < o.n && !known; ++i)
            known = o.range[i].lo <= r.lo && r.hi <= o.range[i].hi && (o.range[i].write || !r.write);
        if (known) continue;
        if (o.n == StreamOrder::kMax && (rc = cover(c))) return rc;
        o.range[o.n++] = r;
    }
    return LS_OK;
}

int order_begin_waiting(Ctx* c, const Span* s, int ns) {
    if (!c->own_stream) return LS_OK;
    std::lock_guard<std::mutex> lock(g_order_mutex);
    int rc = wait_for_others(c, s, ns);
    if (rc == LS_OK && c->order.covered < c->order.n) rc = cover(c);
    if (rc == LS_OK) c->order.waiting = true;
    return rc;
}

void order_end_waiting(Ctx* c) {
    if (!c->own_stream) return;
    (void)hipStreamSynchronize(c->stream);   // an early return leaves work behind
    std::lock_guard<std::mutex> lock(g_order_mutex);
    c->order.waiting = false;
    c->order.n = c->order.covered = 0;
}

int private_stream(Ctx* c) {
    std::lock_guard<std::mutex> lock(g_order_mutex);
    auto& idle = g_idle_streams[c->device % kMaxStreamDevices];
    hipStream_t s = nullptr;
    if (!idle.empty()) {
        s = idle.back();
        idle.pop_back();
    } else if (hipStreamCreate(&s) != hipSuccess) {
        (void)hipGetLastError();
        return fail(LS_ERR_HIP, "stream creation failed");
    }
    c->own_stream = c->stream = s;
    if (hipEventCreateWithFlags(&c->order.ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        c->order.ev = nullptr;
        return fail(LS_ERR_HIP, "event creation failed");
    }
    g_private.push_back(c);
    return LS_OK;
}

void private_stream_release(Ctx* c) {
    if (!c->own_stream) return;
    std::lock_guard<std::mutex> lock(g_order_mutex);
    g_private.erase(std::remove(g_private.begin(), g_private.end(), c), g_private.end());
    if (c->order.ev) (void)hipEventDestroy(c->order.ev);
    g_idle_streams[c->device % kMaxStreamDevices].push_back(c->own_stream);
    c->own_stream = c->stream = nullptr;
}

}  // namespace ls
