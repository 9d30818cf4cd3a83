// Lookup in the compressed row cache's table, shared by the kernels that gather through it.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "ibp_device.hpp"

namespace ibp {
namespace dev {

struct CacheSlot {
    uint64_t key;   // row id + 1; 0 = empty
    uint64_t val;   // cache entry
};

// Whether row `id` is cached; if so, `byte` is its first packed byte in the slab.
__device__ __forceinline__ bool cache_probe(const CacheView &c, uint64_t id, uint64_t &byte) {
    const CacheSlot *__restrict__ tab = reinterpret_cast<const CacheSlot *>(c.table);
    uint64_t h = (id * 0x9E3779B97F4A7C15ull) >> (64 - c.log2cap);
    // the table is at most half full, so an empty slot ends every probe sequence
    for (uint64_t k = 0; k <= c.mask; ++k) {
        const CacheSlot e = tab[h];
        if (e.key == id + 1) {
            byte = e.val & 0xFFFFFFFFFFull;
            return true;
        }
        if (e.key == 0) return false;
        h = (h + 1) & c.mask;
    }
    return false;
}

// Counts a wave's hits and misses (by one lane), spread over kCountLines 128-byte lines so
// that waves do not all contend for one address.
__device__ __forceinline__ void cache_count(const CacheView &c, uint32_t hits, uint32_t misses) {
    unsigned long long *cnt = c.counts + (blockIdx.x % kCountLines) * kCountStride;
    if (hits) atomicAdd(cnt, (unsigned long long)hits);
    if (misses) atomicAdd(cnt + 1, (unsigned long long)misses);
}

}  // namespace dev
}  // namespace ibp
