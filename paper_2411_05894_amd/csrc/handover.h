// Hand-over of partial results between the workgroups of ONE launch that run on one die.
//
// A die (XCD) has one L2, every store of its compute units is written through to it, and a load that passes over the compute unit's
// own cache finds there what a neighbour stored: no data has to reach memory.  Workgroups i and i + 8 of a launch run on one die, so a
// launcher that gives the n workgroups of a group block indexes of one residue modulo 8 lets them exchange partial results inside the
// launch.  Between 256 workgroups of 256 threads in groups of four, each storing 16 KB and reading a quarter of every slice of its
// group: 1.0 us more than the stores alone, against 2.5 us for stores with device scope (through to memory) and 2.7 us for a second
// launch that reads them; with 64 KB 2.7, 8.0 and 5.8 us.
//
// Which of the eight dies takes the workgroups whose index is 0 modulo 8 depends on the hardware queue, and so on the stream (measured over
// nine streams: 0, 5, 6 and 7, always the same for one queue); that all of one residue run on one die does not.
//
// Nothing here relies on where a workgroup runs or on all of them running at once:
//  - every workgroup that arrives adds its die and the die's square to its group's word, so when all have arrived all of them know
//    whether they are on one die (n times the sum of squares is the square of the sum for equal numbers only);
//  - a workgroup that may not wait (no `polls`), or that has polled `polls` times for the others, gives the fast way up for its whole
//    group (HAND_GONE); that succeeds only while not everybody has arrived, so the group's workgroups agree on the way taken;
//  - where the fast way is given up, or leads over several dies, each makes its stores visible to the device (a release fence, about
//    20 us) and counts itself in a second time, and the last one to do so does the whole group's work.  So no wait is without a bound.
// Beside other work on the device: a launch's workgroups start in the order of their indexes, and a group's lie next to each other, so of each
// launch at most one group per die waits for workgroups that have not started, while the groups in front of it finish and make room.
// Two contexts stepping on two streams, a pair of steps of two 8B layers without / with hand-over, us: 9 rows 350 / 348, 36 rows 604 / 548,
// 160 rows 802 / 779, 512 rows 1774 / 1789; two processes, a step of each: 351 / 344, 466 / 441, 804 / 786, 1772 / 1772; a step beside two
// products of 4096 x 4096 x 4096 on another stream: 423 / 414, 503 / 476, 665 / 628, 1143 / 1120.
#pragma once
#include "common.h"

// One word per group, HAND_STRIDE apart (128 bytes: groups of different dies share no line); zero before and after every launch.
// Bits 0..7 arrivals, 8..15 departures, 16..23 arrivals on the slow way, 24 the fast way is given up, 32..47 and 48..63 the sum of the
// dies' numbers (up to 15) and of their squares.
constexpr int HAND_STRIDE = 16, HAND_GROUPS = 256;   // ... groups of a launch at most (of up to 255 workgroups)
constexpr uint64_t HAND_ARRIVE = 1u, HAND_LEAVE = 1u << 8, HAND_SLOW = 1u << 16, HAND_GONE = 1u << 24, HAND_DIE = (uint64_t)1 << 32, HAND_DIE2 = (uint64_t)1 << 48;
constexpr int HAND_POLLS = 400;   // 0.6 us each: past every difference between workgroups that start together
constexpr int HAND_LATE = HAND_GROUPS * HAND_STRIDE, HAND_WORD_COUNT = HAND_LATE + 1;   // behind the groups' words: how many groups went the slow way

constexpr size_t HAND_WORDS = (size_t)1 << 20, HAND_PARTS = (size_t)40 << 20;   // bytes for the words, and for the parts behind them

struct Hand {            // of a launch
    uint64_t *words;     // HAND_WORD_COUNT, or null: no hand-over
    float *parts;        // HAND_PARTS bytes for what GEMMs hand over: 256 workgroups of ten units of 2 KiB in each of eight waves
    int polls;           // HAND_POLLS, or 0: nobody waits, every group goes the slow way
};

enum HandWay {
    HAND_SHARE = 0,   // every workgroup of the group has stored its results: read them with die_load and do your share
    HAND_TURN_IN,     // the fast way is given up: store what the share would have kept back, then call hand_turn_in
    HAND_ALL,         // do the whole group's work
    HAND_NOTHING,     // another workgroup does it
};

__device__ __forceinline__ uint32_t own_die() { return __builtin_amdgcn_s_getreg(20 | 3 << 11); }   // XCC_ID, 4 bits

__device__ __forceinline__ uint64_t hand_add(uint64_t *word, uint64_t x)
{
    return __hip_atomic_fetch_add(word, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + x;
}

// The workgroup's stores so far are part of its group's results; n workgroups form the group.  All threads call both, in turn; what
// stands between them needs no other workgroup.  Stores count down vmcnt when the die's L2 has them.
__device__ __forceinline__ uint64_t hand_arrive(const Hand &h, int group)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x != 0) return 0;
    uint64_t *word = h.words + (size_t)group * HAND_STRIDE;
    const uint32_t die = own_die();
    if (h.polls > 0) return hand_add(word, HAND_ARRIVE + die * HAND_DIE + die * die * HAND_DIE2);
    // not counted in: the others cannot all arrive
    return __hip_atomic_fetch_or(word, HAND_GONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) | HAND_GONE;
}

__device__ __forceinline__ HandWay hand_wait(const Hand &h, int group, int n, uint64_t seen, int *way_s)
{
    if (threadIdx.x == 0) {
        uint64_t *word = h.words + (size_t)group * HAND_STRIDE;
        auto open = [&]() { return (int)(seen & 0xFFu) < n && !(seen & HAND_GONE); };
        for (int i = 0; i < h.polls && open(); ++i) {
            __builtin_amdgcn_s_sleep(1);
            seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        while (open())   // at most as often as others count themselves in
            if (__hip_atomic_compare_exchange_strong(word, &seen, seen | HAND_GONE, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                seen |= HAND_GONE;
        const uint32_t sum = (uint32_t)(seen >> 32) & 0xFFFFu, squares = (uint32_t)(seen >> 48);
        *way_s = seen & HAND_GONE || sum * sum != (uint32_t)n * squares ? HAND_TURN_IN : HAND_SHARE;
    }
    __syncthreads();
    return (HandWay)__builtin_amdgcn_readfirstlane(*way_s);
}

__device__ __forceinline__ HandWay hand_turn_in(const Hand &h, int group, int n, int *way_s)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t *word = h.words + (size_t)group * HAND_STRIDE;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const bool last = (int)(hand_add(word, HAND_SLOW) >> 16 & 0xFFu) == n;
        if (last) hand_add(h.words + HAND_LATE, 1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *way_s = last ? HAND_ALL : HAND_NOTHING;
    }
    __syncthreads();
    return (HandWay)__builtin_amdgcn_readfirstlane(*way_s);
}

// Every workgroup of the group leaves once it needs the word no more, and clears it at its end if it was the last to leave.
__device__ __forceinline__ uint64_t hand_leave(const Hand &h, int group)
{
    return threadIdx.x == 0 ? hand_add(h.words + (size_t)group * HAND_STRIDE, HAND_LEAVE) : 0;
}
__device__ __forceinline__ void hand_clear(const Hand &h, int group, int n, uint64_t left)
{
    if (threadIdx.x == 0 && (int)(left >> 8 & 0xFFu) == n)
        __hip_atomic_store(h.words + (size_t)group * HAND_STRIDE, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Loads that pass over the compute unit's own cache (sc1), which may hold what was there before: byte offset `at` behind `base`,
// `bytes` of which may be read (fewer than 2^31).
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
struct DieBuffer {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ DieBuffer(const void *base, size_t bytes) : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00027000)) {}
    __device__ __forceinline__ f32x4 load4(int at, int base = 0) const { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at, base, 16)); }
    __device__ __forceinline__ float2 load2(int at) const
    {
        const u32x2_t x = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, 16));
        return float2{bits_f32(x[0]), bits_f32(x[1])};
    }
};
