// Order and memory of the launches whose workgroups wait for each other (gpga_gang.hpp).
#include "gpga_gang.hpp"

#include <mutex>

namespace {

struct GangDevice {
    std::mutex lock;
    GangTurn turn;
    uint32_t before = 0;        // the turn before the one that is being taken
    GangSpace space;
    uint32_t* ended = nullptr;  // pinned, as long as the process: number of the last launch that has ended
    int contexts = 0;
};
constexpr int kMaxDevices = 64;
// A device without contexts keeps so much until the process ends, for programs that make one context after the other
// (8 iterations on 8 x 1000, first call of such a context 148 us where the memory comes and goes, 73 where it stays).
constexpr size_t kKeptBytes = 8 << 20;
GangDevice* device_of(const gpga_ctx* c) {
    static GangDevice devices[kMaxDevices];
    return c->device >= 0 && c->device < kMaxDevices ? &devices[c->device] : nullptr;
}

// What GangSpace asks of a stream's device; no error is left behind.
struct StreamMemory {
    hipStream_t stream;
    static bool ok(hipError_t e) {
        if (e != hipSuccess) (void)hipGetLastError();
        return e == hipSuccess;
    }
    unsigned char* get(size_t bytes) {
        void* p = nullptr;
        return ok(hipMalloc(&p, bytes)) ? static_cast<unsigned char*>(p) : nullptr;
    }
    void put(unsigned char* p) { (void)ok(hipFree(p)); }
    bool wait() { return ok(hipStreamSynchronize(stream)); }
    bool clear(unsigned char* p, size_t bytes) { return ok(hipMemsetAsync(p, 0, bytes, stream)); }
};

}  // namespace

void gang_join(gpga_ctx* c) {
    GangDevice* const o = device_of(c);
    if (!o) return;
    std::lock_guard<std::mutex> hold(o->lock);
    if (!o->ended) {
        if (!StreamMemory::ok(hipHostMalloc(reinterpret_cast<void**>(&o->ended), sizeof(uint32_t), hipHostMallocCoherent))) {
            o->ended = nullptr;
            return;
        }
        *o->ended = 0;
    }
    ++o->contexts;
    c->in_gang = true;
}

void gang_leave(gpga_ctx* c) {
    GangDevice* const o = device_of(c);
    if (!o || !c->in_gang) return;
    std::lock_guard<std::mutex> hold(o->lock);
    c->in_gang = false;
    if (--o->contexts > 0 || o->space.cap <= kKeptBytes) return;
    StreamMemory memory{nullptr};
    if (*o->ended != o->turn.number) (void)StreamMemory::ok(hipDeviceSynchronize());  // of a context bound to another stream since
    memory.put(o->space.at);
    o->space = GangSpace();
}

bool gang_begin(const gpga_ctx* c, size_t bytes, GangArgs* g, unsigned char** base) {
    GangDevice* const o = device_of(c);
    if (!o || !c->in_gang) return false;
    o->lock.lock();
    o->before = o->turn.number;
    bool ok = o->turn.take(c->stream, c->stream == hipStreamPerThread, __atomic_load_n(o->ended, __ATOMIC_ACQUIRE));
    if (ok) {
        StreamMemory memory{c->stream};
        ok = o->space.room(bytes, o->turn.number < o->before, memory);
        if (!ok) o->turn.undo(o->before);
    }
    if (!ok) {
        o->lock.unlock();
        return false;
    }
    g->number = o->turn.number;
    g->ended = o->ended;
    *base = o->space.at;
    return true;
}

void gang_end(const gpga_ctx* c, bool launched) {
    GangDevice* const o = device_of(c);
    if (!launched) o->turn.undo(o->before);
    o->lock.unlock();
}
