// A crew: blocks of one launch that run on one die and meet in its L2 (HIP, gfx950).
//
// A chain of small dependent steps launched one by one pays a kernel boundary and cold caches for each: 3.7 us between two
// empty launches.  A barrier over the whole chip costs more (9 us with a block on each of its 256 units), because the L2s of
// the eight dies meet in memory.  On one die a store goes through the L1 into the L2 that the other units read, so a
// hand-over is a store that has arrived, a flag and a poll: 0.73 us for 32 blocks that each write 2 KB, meet and read a
// neighbour's.  A chain whose steps are small enough for a die therefore runs as one launch.
//
// A launch of 8 N blocks puts every eighth on the same die; those with blockIdx % 8 == pick are the candidates, the others
// end at once.  Candidates that run on the die of the first of them sign the roll.  The first one there, the founder, begins
// when all N have, or after a while, with those that have; who signs later waits and is taken on with the next step.  So the
// members of a crew all run already, and a barrier between them ends whatever else the chip is doing and whichever blocks it
// still holds back; with fewer members each has more to do, until the units that others held come free.  The work's cut, and
// so every sum, does not depend on their number.
//
// What members write for each other: plain stores, which pass the L1.  What they read of each other: loads that miss the L1
// (fresh_*; ordinary ones may find an older line in it, and the scalar cache is not looked at either).
#pragma once
#include "eck_internal.h"

namespace eck {

constexpr unsigned CREW_DIES = 8;
constexpr unsigned CREW_MOST = 32; // members, one per compute unit of a die

struct CrewState { // device memory, zero before the launch: two lines
    uint32_t home;      // the members' die + 1, 0: none yet
    uint32_t pad;
    uint64_t muster;    // the founder's: who belongs to the crew and since which step (Crew::call)
    uint32_t roll[16];  // by die: candidates that signed
    uint32_t pad2[12];
    uint32_t met[CREW_MOST]; // by member: barriers it has reached
};
static_assert(sizeof(CrewState) == 256, "fits the place behind a workspace's last buffer");

// which of every eight blocks are candidates: crews of different workspaces on different dies
inline unsigned crew_pick(const void *state) { return (unsigned)(((uintptr_t)state >> 8) * 0x9E3779B1u >> 16) % CREW_DIES; }

__device__ __forceinline__ void crew_clear(CrewState *s) // by one wavefront of an earlier launch
{
    if (threadIdx.x < 64) reinterpret_cast<uint32_t *>(s)[threadIdx.x] = 0;
}

// Work in steps with two barriers each
struct Crew {
    CrewState *s;
    uint32_t rank, size, barriers;

    // `members` belong to the crew from `step` on, `before` of them already did; at_once: so many may be taken on together.  OVER:
    // nobody is any more.
    static constexpr uint64_t OVER = 1u << 24;
    static __device__ __forceinline__ uint64_t call(uint32_t step, uint32_t at_once, uint32_t before, uint32_t members)
    {
        return (uint64_t)step << 32 | at_once << 16 | before << 8 | members;
    }
    static __device__ __forceinline__ uint32_t part(uint64_t muster, int byte) { return (uint32_t)muster >> 8 * byte & 255; }
    static __device__ __forceinline__ uint32_t members(uint64_t muster) { return part(muster, 0); }

    static __device__ __forceinline__ uint32_t this_die() { return __builtin_amdgcn_s_getreg((31 << 11) | 20) & 15; } // HW_REG_XCC_ID

    // Called by every thread of a candidate block: the step that it begins with, or -1: not a member.  slot: four words of LDS.
    __device__ __forceinline__ int join(CrewState *state, uint32_t at_once, uint32_t *slot)
    {
        s = state;
        if (threadIdx.x == 0) {
            const uint32_t die = this_die();
            const uint32_t place = __hip_atomic_fetch_add(&s->roll[die], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t home = 0;
            uint64_t muster = 0;
            const bool first = __hip_atomic_compare_exchange_strong(&s->home, &home, die + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                    __HIP_MEMORY_SCOPE_AGENT);
            if (first || home == die + 1) {
                if (place == 0) {
                    constexpr int PATIENCE = 128; // polls, some 50 us
                    uint32_t there = 1;
                    for (int i = 0; i < PATIENCE && (there = relaxed(&s->roll[die])) < gridDim.x / CREW_DIES; ++i) {
                    }
                    muster = call(0, at_once, 0, min(there, at_once));
                    __hip_atomic_store(&s->muster, muster, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    do muster = relaxed(&s->muster); // (the founder runs)
                    while (members(muster) <= place && !(muster & OVER));
                }
            }
            slot[0] = place;
            slot[1] = members(muster);
            slot[2] = part(muster, 1);
            slot[3] = (uint32_t)(muster >> 32);
        }
        __syncthreads();
        rank = __builtin_amdgcn_readfirstlane(slot[0]);
        const uint32_t all = __builtin_amdgcn_readfirstlane(slot[1]), before = __builtin_amdgcn_readfirstlane(slot[2]);
        const uint32_t step = __builtin_amdgcn_readfirstlane(slot[3]);
        if (rank >= all) return -1;
        barriers = 2 * step;
        size = before;
        if (step > 0) meet(); // the others are through with the step before
        size = all;
        return (int)step;
    }

    // Between a step's first barrier and its second, by every thread: who has signed belongs to the crew from the next step on.
    // (The second barrier is the old members'; the next muster is written when all have met at the next first one.)
    __device__ __forceinline__ void summon(int next_step) const
    {
        if (full() || !founder()) return;
        const uint32_t there = relaxed(&s->roll[this_die()]), at_once = part(relaxed(&s->muster), 2);
        if (there > size)
            __hip_atomic_store(&s->muster, call(next_step, at_once, size, min(there, size + at_once)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ bool grown() // behind the second barrier
    {
        if (full()) return false;
        const uint32_t all = __builtin_amdgcn_readfirstlane(members(relaxed(&s->muster)));
        if (all == size) return false;
        size = all;
        return true;
    }
    __device__ __forceinline__ void dismiss() const // behind the last step's first barrier: who was called has come
    {
        if (founder()) __hip_atomic_store(&s->muster, relaxed(&s->muster) | OVER, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ bool full() const { return __builtin_expect(size == CREW_MOST, true); }
    __device__ __forceinline__ bool founder() const { return rank == 0 && threadIdx.x == 0; } // its first thread

    // The block's stores have arrived and its flag says so.  Every thread; first half of a barrier.
    __device__ __forceinline__ void arrive()
    {
        ++barriers;
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (threadIdx.x == 0) __hip_atomic_store(&s->met[rank], barriers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    // Every member has arrived.  Second half; loads requested between the two stay on their way.
    __device__ __forceinline__ void meet() const
    {
        if (threadIdx.x < 64) {
            const uint32_t *theirs = &s->met[threadIdx.x < size ? threadIdx.x : 0]; // (the founder; a block that joins has no flag yet)
            while (__ballot((int32_t)(relaxed(theirs) - barriers) < 0)) {
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }

    template <class T>
    static __device__ __forceinline__ T relaxed(const T *p)
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// The thread's index, worked out anew wherever it is asked for: what follows from it stays inside its phase, and the registers of
// one phase are the next one's (hoisted out of the loop over the steps, the addresses of all phases spilled a hundred registers).
__device__ __forceinline__ int crew_thread()
{
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// Loads of what other members wrote (FRESH: past the L1), or ordinary ones: `at` bytes behind a base that all lanes share, which
// `shared` is added to (a scalar, so that a row of loads needs one address)
constexpr int CREW_RSRC_FLAGS = 0x00020000; // buffer descriptor: raw 32-bit data
constexpr int CREW_SC1 = 16;                // cache policy: device scope
typedef int crew_i32x4 __attribute__((ext_vector_type(4)));
typedef crew_i32x4 crew_i32x4_any __attribute__((aligned(4))); // (a vector of an fp32 model of any widths starts on four bytes)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t crew_buffer(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, CREW_RSRC_FLAGS);
}

template <bool FRESH>
__device__ __forceinline__ crew_i32x4 fresh_16(const void *base, uint32_t at, uint32_t shared)
{
    if (!FRESH) return *reinterpret_cast<const crew_i32x4_any *>(static_cast<const char *>(base) + at + shared);
    return __builtin_amdgcn_raw_buffer_load_b128(crew_buffer(base), at, shared, CREW_SC1);
}

// (at and shared in bytes)
template <bool FRESH>
__device__ __forceinline__ float fresh_float(const float *base, uint32_t at, uint32_t shared)
{
    if (!FRESH) return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + shared + at);
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(crew_buffer(base), at, shared, CREW_SC1));
}

} // namespace eck
