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
#pragma once

#include <hip/hip_runtime.h>

#include "rom.h"

namespace rom {
namespace xch {

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
