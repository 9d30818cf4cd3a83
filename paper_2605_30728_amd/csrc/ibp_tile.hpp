// A tile of a row (64*K words of one cluster) as a wave decodes it: every word's variant
// positions as precomputed runs, and the word's rebuild from its packed bits.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "ibp_wave.hpp"

namespace ibp {
namespace dev {

// Per-wave decode state for one tile of a row (64*K words) of one cluster.
template <int K, int MAXR>
struct Tile {
    uint32_t bv[K];          // Bitval of the lane's words
    uint32_t nm[K];          // ~Mask: the variant positions
    uint32_t s[K];           // bit offset of the word inside the packed row
    uint32_t pk[K];          // packed width popcount(~Mask) (0 past the row's end)
    uint32_t rot[K][MAXR];   // rotate-right amount that lands run k at its position
    uint32_t rm[K][MAXR];    // run k's bits in place
    uint32_t bits;           // packed bits of this tile (wave-uniform)
    int nr;                  // runs applied per word (uniform); -1 = generic loop
};

// Words of the tile that starts at word w0: lane l owns w0 + l + 64j, or, ADJ, the K
// consecutive ones from w0 + K*l (then without bit offsets: s and bits are not set).
template <bool ADJ = false, int K, int MAXR>
__device__ __forceinline__ void tile_setup(Tile<K, MAXR> &t, const uint32_t *__restrict__ mg,
                                           uint32_t W, uint32_t w0, uint32_t carry) {
    const uint32_t l = lane_id();
    uint32_t c = carry;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const uint32_t w = w0 + (ADJ ? K * l + j : l + kWave * j);
        uint32_t m = 0xFFFFFFFFu, b = 0u;
        if (w < W) {
            m = mg[w];
            b = mg[W + w];
        }
        t.nm[j] = ~m;
        t.bv[j] = b;
        const uint32_t n = (uint32_t)__builtin_popcount(~m);
        t.pk[j] = n;
        if constexpr (!ADJ) {
            const uint32_t inc = wave_incl_scan(n);
            t.s[j] = c + inc - n;
            c += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
    }
    t.bits = c - carry;

    int cnt_max = 0;
    bool rest = false;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        uint32_t v = t.nm[j];
        uint32_t so = 0;
        int cnt = 0;
#pragma unroll
        for (int k = 0; k < MAXR; ++k) {
            const uint32_t low = v & (0u - v);
            const uint32_t tt = v + low;      // carries through the lowest run
            const uint32_t run = v & ~tt;
            v &= tt;
            const uint32_t lo = (uint32_t)__builtin_ctz(run | 0x80000000u);
            t.rot[j][k] = (so - lo) & 31u;
            t.rm[j][k] = run;
            so += (uint32_t)__builtin_popcount(run);
            cnt += run != 0u;
        }
        cnt_max = cnt > cnt_max ? cnt : cnt_max;
        rest = rest || v != 0u;
    }
    if (__any(rest)) {
        t.nr = -1;
    } else {
        int nr = 0;
#pragma unroll
        for (int k = 0; k < MAXR; ++k)
            if (__any(cnt_max > k)) nr = k + 1;
        t.nr = nr;
    }
}

// Rebuild one word from its 32-bit window x: Bitval | the NR runs of variant bits.
template <int NR, int K, int MAXR>
__device__ __forceinline__ uint32_t word_fast(const Tile<K, MAXR> &t, int j, uint32_t x) {
    uint32_t acc = t.bv[j];
#pragma unroll
    for (int k = 0; k < NR; ++k) acc |= __builtin_amdgcn_alignbit(x, x, t.rot[j][k]) & t.rm[j][k];
    return acc;
}

// Generic rebuild for any Mask: walk the runs of ~Mask from the lowest bit up.
__device__ __forceinline__ uint32_t word_generic(uint32_t bv, uint32_t nm, uint32_t x) {
    uint32_t acc = bv, v = nm;
    while (v) {
        const uint32_t low = v & (0u - v);
        const uint32_t tt = v + low;
        const uint32_t run = v & ~tt;
        v &= tt;
        acc |= (x << __builtin_ctz(run)) & run;
        x = __builtin_amdgcn_alignbit(0u, x, (uint32_t)__builtin_popcount(run));
    }
    return acc;
}

}  // namespace dev
}  // namespace ibp
