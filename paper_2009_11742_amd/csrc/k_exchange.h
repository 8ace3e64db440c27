// State exchange between the workgroups of one row-split group (all on one
// XCD, sharing its L2): published rows carry their own arrival.
//
// A group publishes its rows once per half-step ("phase") into a ring of
// kRing buffers, phase q in buffer q % kRing.  Every 32-bit word of an empty
// slot is kEmpty, a bit pattern that no published value has (publishers
// replace it by another NaN), so a reader polls the data itself: one store
// and one load on the critical path, against a completed store, an atomic
// add, a poll of the counter and then the load when a group meets at a
// counter barrier.
//
// Slot reuse.  A workgroup publishes phase q only after all its waves have
// read all of phase q - 1, so once a workgroup has read all of phase q - 1
// (its waves meet at a workgroup barrier), every member has finished reading
// phase q - 2.  Its publishing threads therefore, after the stores of phase
// q, empty their own slots of phase q - 2, and wait for those stores
// (publish_fence) before they publish phase q + 1.  Buffer (q - 2) % 4 is
// next read in phase q + 2, by workgroups that have read phase q + 1 from
// every member, hence after it was emptied.
//
// Loads are device-scope (the CU's vector L1 does not serve them); plain
// stores reach the shared L2.  Every poll is bounded: one that runs out
// records ROM_E_TIMEOUT and raises the abort word, and every later poll of
// the launch returns at once, so the kernel always ends.
//
// Repeatable runs.  A wait can run out although nothing is wrong: another
// stream's or process's kernel may hold CUs that a member of the group needs.
// A run that would not have waited on another kernel must not fail for that:
// its workgroups write V, S and the sums only at the end, and only if all of
// the group got there (agree); behind it the other kernel is launched with
// the groups' words and does the work of those that did not (committed).
#pragma once

#include <hip/hip_runtime.h>

#include "rom.h"
#include "rom_internal.h"

namespace rom {
namespace xch {

// A kernel's first argument, read where this is called: what only the end of a
// run needs would otherwise be held, and spilled, across its step loop.
template <class A>
__device__ __forceinline__ const __attribute__((address_space(4))) A &args_here() {
    typedef const __attribute__((address_space(4))) A Args;
    Args *p = (Args *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *p;
}

// Where the rows a wave reads do not fit in its registers at once, polling
// them one by one would put a branch and a wait into the pipelined loads;
// there each publishing wave counts its phases in a flag word, stored after
// its rows' stores have completed, a reader polls the flags of the blocks it
// needs and then streams the rows unchecked.  (Two buffers would do: whoever
// publishes phase q has read all of phase q - 1, so every member has read
// all of phase q - 2.)
//
constexpr unsigned kEmpty = 0xFFFFFFFFu;
constexpr int kRing = 4;
constexpr long kSpinMax = 1L << 20;   // polls of one bounded wait

// The abort state of a launch, per wave: `st` the status words ([1]
// ROM_E_TIMEOUT, [2] abort), `max` the poll budget, `forced` (host-forced
// time-outs): treat everything as missing.
struct Wait {
    int *st;
    long max;
    int forced;
    bool dead;
    // After a failed poll (wave-uniform call): whether to give up.
    __device__ __forceinline__ bool give_up(long &spins) {
        if (++spins > max) {
            __hip_atomic_store(&st[1], (int)ROM_E_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st[2], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            dead = true;
        } else if ((spins & 63) == 0 &&
                   __builtin_amdgcn_readfirstlane(__hip_atomic_load(&st[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0) {
            dead = true;
        }
        return dead;
    }
};

// Stores of this thread that are still in flight (the emptied slots of two
// phases ago) complete before anything that follows.
__device__ __forceinline__ void publish_fence() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Poll until the flag words of this lane (null: none) of all lanes of the
// wave have reached phase `want`.
__device__ __forceinline__ void wait_flags(Wait &wait, const unsigned *flag, unsigned want) {
    long spins = 0;
    for (;;) {
        bool late = false;
        if (flag != nullptr)
            late = (int)(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - want) < 0;
        if (wait.dead || (!wait.forced && __ballot(late) == 0)) break;
        if (wait.give_up(spins)) break;
    }
    asm volatile("" ::: "memory");
}

// This wave's rows of a phase are stored: count it (lane 0 of the wave).
__device__ __forceinline__ void raise_flag(unsigned *flag, unsigned phase) {
    publish_fence();
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(flag, phase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// The end of round t (0, 1, ..) of a group: whether all its R members have
// come this far without a wait that ran out.  `words`: the arrivals so far,
// and the rounds that all have agreed on, which the first member that gives
// up freezes, so that all of them and every later reader see one answer.
// Called by whole workgroups.  (Arrivals by compare-and-exchange on one word
// with the answer cost up to 150 us for 32 members, these about 2.)
constexpr unsigned kGivenUp = 0x80000000u;
__device__ __forceinline__ bool agree(unsigned *words, unsigned R, unsigned t, Wait &wait) {
    __shared__ int sh_all;
    const bool bad = __syncthreads_or(wait.dead) != 0;
    if (threadIdx.x == 0) {
        // the answer from t to `to`, unless it is there already
        auto settle = [&](unsigned to) {
            unsigned v = t;
            return __hip_atomic_compare_exchange_strong(&words[1], &v, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) ? to : v;
        };
        unsigned v = t;
        if (bad)
            v = settle(t | kGivenUp);
        else if (__hip_atomic_fetch_add(&words[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == (t + 1u) * R)
            v = settle(t + 1u);
        for (long spins = 0; v == t;) {
            v = __hip_atomic_load(&words[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v == t && wait.give_up(spins)) v = settle(t | kGivenUp);
        }
        sh_all = (v & ~kGivenUp) > t;
    }
    __syncthreads();
    return sh_all != 0;
}

// Whether the run that r repeats has done sample m.
__device__ __forceinline__ bool committed(const Repeat &r, int m) {
    const int g = m / r.nc;
    return (r.done[2 * (g % r.slots) + 1] & ~kGivenUp) > (unsigned)(g / r.slots);
}

__device__ __forceinline__ unsigned max3u(unsigned a, unsigned b, unsigned c) {
    const unsigned m = a > b ? a : b;
    return m > c ? m : c;
}

// 64-bit values: a slot is empty while its high word is kEmpty (8-byte
// loads and stores are single accesses).
typedef unsigned long long u64;
constexpr u64 kEmpty64 = ~0ull;
__device__ __forceinline__ void put64(u64 *p, double v) {
    u64 b = __builtin_bit_cast(u64, v);
    if ((unsigned)(b >> 32) == kEmpty) b = 0x7FF8000000000000ull;
    __hip_atomic_store(p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void clear64(u64 *p) {
    __hip_atomic_store(p, kEmpty64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ u64 get64(const u64 *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace xch
}  // namespace rom
