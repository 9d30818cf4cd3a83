// Lookup in the compressed row cache's table, shared by the kernels that gather through it.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "ibp_device.hpp"

namespace ibp {
namespace dev {

// A row's first table slot, in flight. A slot is one 16-byte load: as two, the second would
// wait for the first one's key to match, a round trip more for every row that hits.
struct CacheProbe {
    uint64_t h;   // index of the slot
    uint4 e;      // its key (row id + 1; 0 = empty) and entry
};

__device__ __forceinline__ CacheProbe cache_probe_begin(const CacheView &c, uint64_t id) {
    CacheProbe p;
    p.h = (id * 0x9E3779B97F4A7C15ull) >> (64 - c.log2cap);
    p.e = reinterpret_cast<const uint4 *>(c.table)[p.h];
    return p;
}

// Whether row `id` is cached; if so, `byte` is its first packed byte in the slab.
__device__ __forceinline__ bool cache_probe_end(const CacheView &c, uint64_t id, CacheProbe p, uint64_t &byte) {
    bool hit = false;
    // the table is at most half full, so an empty slot ends every probe sequence
    for (uint64_t k = 0;; ++k) {
        const uint64_t key = (uint64_t)p.e.y << 32 | p.e.x;
        if (key == id + 1) {
            hit = true;
            break;
        }
        if (key == 0 || k == c.mask) break;
        p.h = (p.h + 1) & c.mask;
        p.e = reinterpret_cast<const uint4 *>(c.table)[p.h];
    }
    if (hit) byte = ((uint64_t)p.e.w << 32 | p.e.z) & 0xFFFFFFFFFFull;
    return hit;
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
