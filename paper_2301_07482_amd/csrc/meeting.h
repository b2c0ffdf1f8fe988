// Words through which workgroups that are all there at once tell each other what they have counted. The waits are bounded: a workgroup that
// has polled often enough gives up, and then all of those that look at the word it waited for have to come to the same decision, since
// what they write (lists, slots, a header) only fits together.
//
// A workgroup's word is written once, by a compare-and-swap from zero: by itself with what it has to say, or by one that has
// waited too long, which says in its place that it is given up. Whatever is there then stays, and everybody reads the same.
//
// Mem: load, cas (returns what was there), add, pause, on memory that all of them see (device code: FgAgentMem).
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define FG_MEETING __device__ __forceinline__
#else
#define FG_MEETING inline
#endif

constexpr uint32_t FG_PUBLISHED = 0x80000000u, FG_GIVEN_UP = 0x40000000u;      // in a workgroup's word; the rest is its own
constexpr uint32_t FG_LOST = 0x10000u;                                          // in a counter of arrivals (at most 64 Ki - 1 of them)
constexpr int FG_POLLS = 1 << 20;                                               // before a wait gives up (never reached)

// What this workgroup has to say (the lower 30 bits of `value`, or FG_GIVEN_UP); it stays given up if somebody has waited too long for it.
template <typename Mem>
FG_MEETING void fg_publish(Mem mem, uint32_t* word, uint32_t value) {
    mem.cas(word, 0u, FG_PUBLISHED | value);
}

// The word as it stays: published by its workgroup, or given up.
template <typename Mem>
FG_MEETING uint32_t fg_settled(Mem mem, uint32_t* word, int polls) {
    for (int i = 0; i < polls; ++i) {
        const uint32_t w = mem.load(word);
        if (w & FG_PUBLISHED) return w;
        mem.pause();
    }
    const uint32_t w = mem.cas(word, 0u, FG_PUBLISHED | FG_GIVEN_UP);
    return w ? w : FG_PUBLISHED | FG_GIVEN_UP;
}

// Counts this workgroup in and waits until `n` have come. false: one of them has not within the polls, or has given up further up.
template <typename Mem>
FG_MEETING bool fg_meet(Mem mem, uint32_t* arrived, uint32_t n, int polls) {
    mem.add(arrived, 1u);
    uint32_t v = mem.load(arrived);
    for (int i = 0; (v & (FG_LOST - 1)) < n; v = mem.load(arrived)) {
        if (++i >= polls) return false;
        mem.pause();
    }
    return v < FG_LOST;
}

// A workgroup that has given up is counted in where it would still come, so that nobody waits for it there, and says so: the others then count
// without what it has not added.
template <typename Mem>
FG_MEETING void fg_lost_ahead(Mem mem, uint32_t* arrived) {
    mem.add(arrived, FG_LOST | 1u);
}

#ifdef __HIPCC__
struct FgAgentMem {
    static __device__ __forceinline__ uint32_t load(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    static __device__ __forceinline__ uint32_t cas(uint32_t* p, uint32_t was, uint32_t v) {
        __hip_atomic_compare_exchange_strong(p, &was, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return was;
    }
    static __device__ __forceinline__ void add(uint32_t* p, uint32_t v) { __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    static __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(1); }
};
#endif
