// Order of the launches whose workgroups wait for each other (gpga_gang.hpp).
#include "gpga_gang.hpp"

#include <mutex>

namespace {

struct GangDevice {
    std::mutex lock;
    GangTurn turn;
    uint32_t* ended = nullptr;  // pinned, as long as the process: number of the last launch that has ended
};
constexpr int kMaxDevices = 64;
GangDevice* device_of(const gpga_ctx* c) {
    static GangDevice devices[kMaxDevices];
    return c->device >= 0 && c->device < kMaxDevices ? &devices[c->device] : nullptr;
}

}  // namespace

void gang_set_up(const gpga_ctx* c) {
    GangDevice* const o = device_of(c);
    if (!o) return;
    std::lock_guard<std::mutex> hold(o->lock);
    if (o->ended) return;
    if (hipHostMalloc(reinterpret_cast<void**>(&o->ended), sizeof(uint32_t), hipHostMallocCoherent) != hipSuccess) {
        o->ended = nullptr;
        (void)hipGetLastError();
        return;
    }
    *o->ended = 0;
}

bool gang_begin(const gpga_ctx* c, GangArgs* g) {
    GangDevice* const o = device_of(c);
    if (!o) return false;
    o->lock.lock();
    if (!o->ended || !o->turn.take(c->stream, c->stream == hipStreamPerThread, __atomic_load_n(o->ended, __ATOMIC_ACQUIRE))) {
        o->lock.unlock();
        return false;
    }
    g->turn = o->turn.number;
    g->ended = o->ended;
    return true;
}

void gang_end(const gpga_ctx* c, bool launched) {
    GangDevice* const o = device_of(c);
    if (!launched) o->turn.undo();
    o->lock.unlock();
}
