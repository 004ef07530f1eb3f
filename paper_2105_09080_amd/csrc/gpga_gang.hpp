// Exchange between the workgroups of one launch, for kernels that run many iterations without going back to the host.
//
// Words: a value travels as one 64-bit word, 32 bits of payload under the launch's number.  A reader polls the word itself, so
// that one trip through memory (0.9 - 1.2 us between any two compute units of the chip, where a dependent launch costs 4 - 5)
// carries both the value and the news that it is there.  Every word is written once a launch and launches on a context have
// different numbers, so nothing is cleared in between and no reader can be overtaken.
//
// Waits end: the launcher sees to it that such launches of one process do not overlap on a device (GangOrder), but a foreign
// process may hold compute units, so a wait that is not met within `limit` clock ticks gives up and marks the launch; all
// other workgroups see the mark in their own waits and leave as well.  The last workgroup to leave a marked launch does the
// launch's work alone.
#pragma once

#include "gpga_internal.hpp"

struct GangWords {
    uint32_t left;      // workgroups that have left
    uint32_t given_up;  // number of the last launch that was given up
};

struct GangArgs {
    GangWords* words;
    uint32_t* finished;  // [workgroups] number of the last launch in which the workgroup stored its results
    uint32_t number;     // of this launch, never 0
    uint32_t limit;      // clock ticks a wait may take
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
        const bool late = __builtin_amdgcn_s_memrealtime() - begin >= g.limit;
        if (late) gang_put32(&g.words->given_up, g.number);
        if (late || gang_get32(&g.words->given_up) == g.number) {
            *s_gone = 1;
            return;
        }
    }
}
#endif

// Launches of this kind on one device, in the order of their calls: on another stream than the last one's, a launch waits for
// that one to end, since two of them at a time might each hold compute units that the other needs.  gang_begin is false, and
// nothing is held, where that cannot be arranged now (the other stream is being captured): the caller takes another way.
bool gang_begin(const gpga_ctx* c);
void gang_end(const gpga_ctx* c, bool launched);
// Before the context lets go of its stream.
void gang_forget(const gpga_ctx* c);
