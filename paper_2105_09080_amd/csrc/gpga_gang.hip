// Order of the launches whose workgroups wait for each other (gpga_gang.hpp).
#include "gpga_gang.hpp"

#include <mutex>

namespace {

// The last launch's stream is looked up when the next one comes on another stream, and only then is there an event: one behind
// every launch cost 3 us each (9 x 1660, 8 iterations 39.8 -> 42.7).  The stream is the owner's, which says so before it lets go.
struct GangOrder {
    std::mutex lock;
    const gpga_ctx* owner = nullptr;  // of the last launch; NULL: there is none, or `behind` is behind it
    hipEvent_t behind = nullptr;      // lives as long as the process
    bool pending = false;             // `behind` was recorded and nothing has waited for it yet
};
constexpr int kMaxDevices = 64;
GangOrder& order_of(const gpga_ctx* c) {
    static GangOrder orders[kMaxDevices];
    return orders[c->device >= 0 && c->device < kMaxDevices ? c->device : 0];
}

bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// An event behind the owner's work.
bool mark(GangOrder* o) {
    if (capturing(o->owner->stream)) return false;
    if (!o->behind && hipEventCreateWithFlags(&o->behind, hipEventDisableTiming) != hipSuccess) {
        o->behind = nullptr;
        (void)hipGetLastError();
        return false;
    }
    if (hipEventRecord(o->behind, o->owner->stream) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    o->owner = nullptr;
    o->pending = true;
    return true;
}

}  // namespace

bool gang_begin(const gpga_ctx* c) {
    GangOrder& o = order_of(c);
    o.lock.lock();
    bool ok = !o.owner || o.owner->stream == c->stream || mark(&o);
    if (ok && o.pending) {
        ok = hipStreamWaitEvent(c->stream, o.behind, 0) == hipSuccess;
        if (!ok) (void)hipGetLastError();
    }
    if (!ok) o.lock.unlock();
    return ok;
}

void gang_end(const gpga_ctx* c, bool launched) {
    GangOrder& o = order_of(c);
    if (launched) {
        o.owner = c;
        o.pending = false;
    }
    o.lock.unlock();
}

void gang_forget(const gpga_ctx* c) {
    GangOrder& o = order_of(c);
    std::lock_guard<std::mutex> hold(o.lock);
    if (o.owner != c) return;
    if (!mark(&o)) {
        (void)hipStreamSynchronize(c->stream);
        (void)hipGetLastError();
        o.owner = nullptr;
    }
}
