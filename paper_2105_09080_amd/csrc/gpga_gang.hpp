// Exchange between the workgroups of one launch, for kernels that run many iterations without going back to the host.
//
// Words: a value travels as one 64-bit word, 32 bits of payload under the launch's number.  A reader polls the word itself, so
// that one trip through memory (0.9 - 1.2 us between any two compute units of the chip, where a dependent launch costs 4 - 5)
// carries both the value and the news that it is there.  Every word is written once a launch and launches on a device have
// different numbers, so nothing is cleared in between, no reader can be overtaken, and one memory serves all contexts.
//
// Waits end: the launcher sees to it that such launches of one process do not overlap on a device (GangTurn), but others'
// kernels may hold compute units, so a wait that is not met within `limit` clock ticks gives up and marks the launch; all
// other workgroups see the mark in their own waits and leave as well.  The last workgroup to leave a marked launch does the
// launch's work alone.  A launch behind one that was given up waits a 64th of that: many may have been queued by then.
#pragma once

#include <thread>

#include "gpga_internal.hpp"

struct GangWords {
    uint32_t left;      // workgroups that have left
    uint32_t given_up;  // number of the last launch that was given up
};

struct GangArgs {
    GangWords* words;
    uint32_t* finished;  // [workgroups] number of the last launch in which the workgroup stored its results
    uint32_t number;     // of this launch among those of the device, never 0
    uint32_t limit;      // clock ticks a wait may take
    uint32_t* ended;     // host memory: the last workgroup to leave stores the number there
    uint32_t* count;     // host memory, the context's: launches that were given up
};

// Whose launch the last one on a device was.  Two at a time might each hold compute units that the other needs, so a launch is
// made only behind the last one in the same stream, or when that one is known to have ended; who is refused takes its iterations
// one at a time, which needs no order.  Nothing is asked of the other stream, which may be capturing or gone, and nothing waits
// for it: events behind the launches of one kind would order contexts that do not depend on each other (two contexts on two
// streams, 8 iterations on 8 x 1000: 141 us a round of calls in turn, 80 with one launch an iteration side by side).
struct GangTurn {
    const void* stream = nullptr;
    std::thread::id thread;  // of a stream that every thread has its own of
    uint32_t number = 0;     // of the last launch
    bool take(const void* to, bool per_thread, uint32_t ended) {
        const std::thread::id here = per_thread ? std::this_thread::get_id() : std::thread::id();
        if (number != ended && (to != stream || here != thread)) return false;
        stream = to;
        thread = here;
        if (++number == 0) number = 1;  // what older launches left is to be cleared
        return true;
    }
    void undo(uint32_t before) { number = before; }  // nothing was launched
};

// The memory that launches on a device exchange through, made when the first of them comes and grown rarely: a context of its own
// cost the first gpga_run of every context an allocation, and a clear of what the longest launch would take (8 iterations on
// 8 x 1000 113 us instead of 73).  Memory does what it says of its device: get, put, clear, and wait for the launches that use it.
struct GangSpace {
    unsigned char* at = nullptr;
    size_t cap = 0;
    bool clear = false;  // no word there carries the number of a launch to come
    template <typename Memory>
    bool room(size_t bytes, bool numbers_start_again, Memory& memory) {
        constexpr size_t kPiece = 2 << 20;
        if (cap < bytes) {
            size_t size = ((bytes > 2 * cap ? bytes : 2 * cap) + kPiece - 1) / kPiece * kPiece;
            unsigned char* more = memory.get(size);
            if (!more && size > bytes) more = memory.get(size = bytes);
            if (!more) return false;
            if (at) {
                if (!memory.wait()) {
                    memory.put(more);
                    return false;
                }
                memory.put(at);
            }
            at = more;
            cap = size;
            clear = false;
        }
        if (!clear || numbers_start_again) clear = memory.clear(at, cap);
        return clear;
    }
};

#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)
// Agent scope: past the caches that are not shared by the whole chip.
__device__ __forceinline__ void gang_put32(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t gang_get32(const uint32_t* p) {
    return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gang_put(uint64_t* p, uint32_t number, uint32_t payload) {
    __hip_atomic_store(p, ((uint64_t)number << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t gang_peek(const uint64_t* p) {
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t gang_peek_at(const uint64_t* base, uint32_t index) {  // base uniform
    return gang_peek(reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(base) + (size_t)(index * 8u)));
}
// By the workgroup that has done a launch alone.
__device__ __forceinline__ void gang_done_alone(const GangArgs& g) {
    const uint32_t before = __hip_atomic_load(g.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(g.count, before + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// By the last workgroup to leave: nobody waits in this launch any more, and the words' counter stands at 0 for the next one.
__device__ __forceinline__ void gang_ended(const GangArgs& g) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(g.ended, g.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Looks at N words at a time, look(v), until all of them carry the launch's number; *s_gone (LDS) is set if the wait was given up.
template <int N, typename Look>
__device__ __forceinline__ void gang_wait(const GangArgs& g, int* s_gone, Look look, uint32_t (&out)[N]) {
    uint64_t begin = 0;
#pragma unroll 1
    for (uint32_t polls = 0;; ++polls) {
        uint64_t v[N];
        look(v);
        uint32_t other = 0;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            out[k] = (uint32_t)v[k];
            other |= (uint32_t)(v[k] >> 32) ^ g.number;
        }
        if (other == 0) return;
        if (g.limit && polls % 32 != 31) {
            if (polls == 0) begin = __builtin_amdgcn_s_memrealtime();
            continue;
        }
        const uint32_t given_up = gang_get32(&g.words->given_up);
        const bool late = __builtin_amdgcn_s_memrealtime() - begin >= (given_up + 1 == g.number ? g.limit / 64 : g.limit);
        if (late) gang_put32(&g.words->given_up, g.number);
        if (late || given_up == g.number) {
            *s_gone = 1;
            return;
        }
    }
}
#endif

// A context comes to its device and goes; one that did not come makes no such launch.
void gang_join(gpga_ctx* c);
void gang_leave(gpga_ctx* c);
// Around a launch that exchanges through `bytes` of memory; false, and nothing is held, if it cannot be made now.
bool gang_begin(const gpga_ctx* c, size_t bytes, GangArgs* g, unsigned char** base);
void gang_end(const gpga_ctx* c, bool launched);
