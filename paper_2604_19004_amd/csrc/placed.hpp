// One pass from A and B to C (kernels of placed.hip, and k_numeric_dspan): every row is written straight to its
// place in C, so there is no symbolic pass, no reserved slab that is compacted afterwards, and no binning.
//
// A row's place is the number of entries of the rows before it, which is known only when those are accumulated.  Units of
// rows (those of a workgroup) publish their number of entries as soon as it is known, a sorted row before its values are
// added up; workgroup 0 of the launch reads the numbers in row order and publishes the places; meanwhile the
// unit adds up its values, then waits for its place and writes.  Places are given by one workgroup and not by every unit looking
// back over the units before it, because thousands of units are between their two steps at any time: each would
// read that many words.
//
// Every wait ends: units wait only for units of lower numbers, which their XCD starts before them (units.hpp), and whatever the
// order in which workgroups start, the number of polls is limited.  A wait that runs out leaves bit 32 in flags and the call goes
// another way.  Workgroup 0 is dispatched first and holds its place until the last unit has published.
#pragma once

#include "ocean_internal.hpp"
#include "units.hpp"

namespace ocean {

namespace {

constexpr unsigned long long NO_PLACE = ~0ull;   // the placing wave gave up
constexpr int FLAG_GAVE_UP = 32;

template <typename T>
__device__ __forceinline__ T peek(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void post(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// A workgroup of 256 threads: places[u] = 1 + sum of (counts[v] - 1) over v < u, in the order in which the counts (0: not
// there yet) arrive.  A turn looks at 256 counts from the first that is missing on, a quarter per wave.  What bounds the rows is not
// how many places a turn gives but how long it takes, as it is in every row's way: turns of 1024 counts (2.7 us with the
// chip to themselves, 6 beside the sort) were 1.268 ms instead of 1.240 for the rectangular input, 2.00 instead of 1.95 for the
// clustered one, 278 us instead of 268 for the Laplacian of 1024^2 (whole calls).  Turns whose loads are on their way two, three
// or four at a time see older counts: 1.266, 1.378 and 1.430 ms.
struct Turn {
    int lead[2][4];              // counts of a wave's quarter that are there, by the parity of the turn
    unsigned int sum[2][4];      // entries among them that are new
};
__device__ __forceinline__ void place_units(const uint32_t *counts, unsigned long long *places, int64_t units,
                                            unsigned long long *total_out, int32_t *flags, int polls, Turn &turn)
{
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    __builtin_amdgcn_s_setprio(3);
    auto load = [&](int64_t from) {
        const int64_t i = from + wave * WAVE + lane;
        return i < units ? peek(counts + i) : 0u;
    };
    int64_t at = 0;                // units before this one have their places
    int64_t from = 0;              // the turn's first count, a multiple of the wave
    unsigned long long run = 0;
    int idle = 0;
    uint32_t c = load(0);
    for (int parity = 0; at < units; parity ^= 1) {
        const unsigned long long missing = __ballot(c == 0u);
        const int lead = missing == 0ull ? WAVE : __builtin_ctzll(missing);   // uniform
        const int old = (int)(at - from) - wave * WAVE;   // counts of the quarter that had been there before
        const uint32_t n = lane >= old && lane < lead ? c - 1u : 0u;
        const uint32_t upto = wave_inclusive_scan_u32(n);
        if (lane == WAVE - 1) {
            turn.lead[parity][wave] = lead;
            turn.sum[parity][wave] = upto;
        }
        __syncthreads();
        int total_lead = 0;
        unsigned long long before = run, after = run;
        bool mine = true, open = true;   // the quarters before this wave's, and so far, are complete
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int l = __builtin_amdgcn_readfirstlane(turn.lead[parity][w]);
            const unsigned int s = (unsigned int)__builtin_amdgcn_readfirstlane((int)turn.sum[parity][w]);
            total_lead += open ? l : 0;
            after += open ? s : 0u;
            if (w < wave) {
                before += s;
                mine = mine && l == WAVE;
            }
            open = open && l == WAVE;
        }
        const int64_t first = from + wave * WAVE;
        const int64_t next = from + total_lead;
        from = next & ~(int64_t)(WAVE - 1);
        c = load(from);
        if (next > at) {
            if (mine && lane >= old && lane < lead) post(places + first + lane, before + (unsigned long long)(upto - n) + 1ull);
            at = next;
            run = after;
            idle = 0;
        } else if (++idle > polls) {   // (all waves at the same turn)
            for (int64_t i = at + (int)threadIdx.x; i < units; i += 256) post(places + i, NO_PLACE);
            if (threadIdx.x == 0) atomicOr(flags, FLAG_GAVE_UP);
            return;
        }
    }
    if (threadIdx.x == 0) *total_out = run;
}

// The place of a unit, or -1.  The whole wave.
__device__ __forceinline__ int64_t wait_for_place(const unsigned long long *place, int32_t *flags, int polls)
{
    for (int i = 0; i < polls; ++i) {
        if (i > 0) __builtin_amdgcn_s_sleep(1);
        const unsigned long long v = peek(place);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
        const unsigned long long p = ((unsigned long long)hi << 32) | lo;
        if (p == NO_PLACE) return -1;
        if (p != 0ull) return (int64_t)p - 1;
    }
    if (lane_id() == 0) atomicOr(flags, FLAG_GAVE_UP);
    return -1;
}

}  // namespace

// What both kernels are given besides the matrices.  slots: entries that out_col and out_val hold; beyond them nothing is
// written, and the total tells.  counts, places: a word per unit, zero.
template <typename V>
struct Placing {
    int64_t m;
    int64_t *c_rp;
    int32_t *out_col;
    V *out_val;
    int64_t slots;
    uint32_t *counts;
    unsigned long long *places;
    unsigned long long *total;
    int32_t *flags;
    int placer_polls, unit_polls;   // before workgroup 0 and a unit give up
    bool by_xcd;                    // unit_of_workgroup's
};

}  // namespace ocean
