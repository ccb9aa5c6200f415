// jatam_shapes.hpp - the shape table on the device: open addressing keyed by
// (hash, size) with 64-bit counts.
#pragma once

#include "jatam_internal.hpp"

namespace jatam {

__device__ __forceinline__ uint64_t shape_key(uint32_t hash, int32_t size)
{
    return ((uint64_t)(uint32_t)size << 32) | hash;   // size >= 1: never 0
}

__device__ __forceinline__ uint32_t slot_of(uint64_t key, int log2cap)
{
    return (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - log2cap));
}

// Adds `count` to the entry of `key` in the global table; false if the table
// has no free entry left.
__device__ __forceinline__ bool global_add(jatam_shape_count_t* table, int log2cap, uint64_t key,
                                           uint64_t count)
{
    const uint32_t mask = (1u << log2cap) - 1u;
    uint32_t s = slot_of(key, log2cap);
    for (uint32_t probe = 0; probe <= mask; ++probe, s = (s + 1) & mask) {
        unsigned long long* kp = reinterpret_cast<unsigned long long*>(&table[s]);
        const unsigned long long seen = atomicCAS(kp, 0ull, (unsigned long long)key);
        if (seen == 0ull || seen == key) {
            atomicAdd(reinterpret_cast<unsigned long long*>(&table[s].count),
                      (unsigned long long)count);
            return true;
        }
    }
    return false;
}

// A call's shape table (entries == nullptr: none).
struct ShapeTable {
    jatam_shape_count_t* entries = nullptr;
    int log2cap = 0;

    __device__ __forceinline__ void add(uint64_t key, uint64_t count) const
    {
        (void)global_add(entries, log2cap, key, count);
    }
};

}  // namespace jatam
