// Per-wave queue of entries to hook (internal to the device code of libhookcc).
#pragma once

#include "common.hpp"

namespace hookcc {

// A wave's pending entries, one per lane in lanes 0 .. count - 1.  The
// entries a filtered launch keeps are a few per wave and step, and hooking
// them where they are found costs the whole wave their chain of dependent
// tree accesses (2-4 us) for a few lanes' work, at every step.  Here they
// move to the next free lanes (one ds_permute per word; every call is a
// permutation of the 64 lanes, so no two lanes write one slot) and are
// hooked 64 at a time.  Held in registers: the LDS belongs to the table.
// All calls are made by whole waves.
struct PairQueue {
    int32_t a = 0, b = 0;
    uint32_t count = 0;  // uniform

    static __device__ __forceinline__ void hook_entry(int32_t x, int32_t y, int32_t* pi, bool halve) {
        if (halve) hook_pair<true>(pi, x, y, kHalveEveryFiltered);
        else hook_pair<false>(pi, x, y, kHalveEveryFiltered);
    }

    __device__ __forceinline__ void push(bool on, int32_t x, int32_t y, int32_t* pi, bool halve) {
        const uint64_t mask = __ballot(on);
        if (mask == 0) return;
        const uint32_t added = (uint32_t)__popcll(mask);
        const uint32_t rank = lane_prefix(mask);
        const uint32_t lane = threadIdx.x & 63;
        const uint32_t to = (on ? count + rank : count + added + (lane - rank)) & 63;
        const int32_t nx = __builtin_amdgcn_ds_permute((int)(to << 2), x);
        const int32_t ny = __builtin_amdgcn_ds_permute((int)(to << 2), y);
        if (lane >= count && lane < count + added) {
            a = nx;
            b = ny;
        }
        count += added;
        if (count < 64) return;
        hook_entry(a, b, pi, halve);
        count -= 64;
        a = nx;  // lanes below count hold the entries that wrapped around
        b = ny;
    }
    __device__ __forceinline__ void flush(int32_t* pi, bool halve) {
        if ((threadIdx.x & 63) < count) hook_entry(a, b, pi, halve);
        count = 0;
    }
};

}  // namespace hookcc
