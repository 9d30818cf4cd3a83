// gfx950 row gather of clustered-scheme streams whose clusters have compact metadata slots:
// packed rows in device memory (the payload, or a staged chunk of it), and, for rows of at
// most 128 words, read in place from pinned host memory, directly or behind the compressed
// row cache.
//
// What bounds it: HBM, once the instructions per row are few enough. A packed row is ~200
// bytes, and a wave that finds its words' bits row by row (k_gather_rows: ~100 vector and ~80
// scalar instructions per 100-word row, four cycles each on a SIMD) spends more issue time
// than the bytes take to move: 164k of those rows, 130 MB of traffic, issued for 27 of the
// 33.7 us they took. So everything that depends only on a cluster is computed for several
// rows at once, and everything that depends only on a lane is a constant:
//
//   * A wave takes 64/P work items per pass (P = 8 or 16 lanes, at least the pairs of a slot;
//     an item is a row, or a tile of 64K words of a wider row). Lane l holds pair l mod P of item l / P: one
//     load fetches every item's pairs, one pass over the lanes turns each pair into its
//     deposit (where up to four runs of variant bits go and how far they shift), and one
//     16-byte LDS write per lane publishes them.
//   * Lane l owns the K consecutive words K*l .. K*l + K-1 of an item. It reads their 4-bit
//     pair indices with one load, their widths from the LDS table, and one scan per item
//     gives its first bit. Two neighbouring words share a window of three dwords.
//   * A word is then rebuilt from its LDS entry: a shift and a bit-select per run, one more
//     to merge Bitval. Words of more than four runs take the holes deposit.
//   * Rows of more than 256 words are tiles of 256 words, each starting at the bit that the
//     cluster's tile table gives, so the tiles of a row decode independently.
//   * Loads past a row's end and stores past an output row's end are dropped by the range
//     check of a buffer descriptor per row, not by branches; the only branch per item picks
//     the deposit of up to two or up to four runs.
//
// Measured (us, row-at-a-time kernel -> this one): 53k Zipf lookups of 512-B rows 14.3 -> 9.5,
// 164k sorted 400-B rows of 2.4M 33.7 -> 25.6 (130 MB of HBM traffic: 5.1 TB/s, a large
// copy's rate), 1.5M shuffled 512-B rows of 3M 293 -> 235, 16k random 4-KB rows 230 -> 19.4
// (there each row's 8 KB of Mask/Bitval words are replaced by its cluster's 640-byte slot).
// From pinned host memory, us: 82k sorted 400-B rows 486 -> 468 (their distinct 128-B lines at
// the link's 57 GB/s take 469), 53k Zipf lookups behind a cache that misses 16% 62.2 -> 61.2
// (lines of the misses: 50). Measured and not kept: half the items in flight (+1-8%), plain stores (+6-24%), one
// 12-byte load per window for K <= 2 (+4-5%) and three 4-byte ones for K = 4 (+17%).
#include <algorithm>
#include <type_traits>

#include "ibp_cache.hpp"
#include "ibp_device.hpp"
#include "ibp_wave.hpp"

namespace ibp {
namespace dev {

namespace {

// A pair's deposit, as published in LDS. Byte fields of p0: left shift of run 1, left shift
// of run 2, first bit of run 2, variant bits (0-32); of p1: shift and first bit of run 3,
// of run 4. A run that is not there repeats the one before it.
struct PairDeposit {
    uint32_t nm, bv, p0, p1;
};

__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

__device__ __forceinline__ uint32_t first_bit(uint32_t v) { return (uint32_t)__builtin_ctz(v | 0x80000000u); }

// The lane's number, opaque: an address of a uniform base and this offset is then one
// instruction's scalar base and 32-bit vector offset, not a 64-bit sum kept per base.
__device__ __forceinline__ uint32_t own_lane() {
    uint32_t l = lane_id();
    asm("" : "+v"(l));
    return l;
}

// f(integral_constant<int, i>) for i in [A, B): every index a constant, so that what is
// kept per item stays in registers.
template <int A, int B, class F>
__device__ __forceinline__ void for_items(F &&f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        for_items<A + 1, B>(f);
    }
}

// Packed bits x (bit 0 = the word's first variant bit) to their places, Bitval elsewhere.
// MANY: runs 3 and 4 too.
template <bool MANY>
__device__ __forceinline__ uint32_t deposit(const PairDeposit &e, uint32_t x) {
    uint32_t y = x << (e.p0 & 31u);
    y = bfi(0xFFFFFFFFu << ((e.p0 >> 16) & 31u), x << ((e.p0 >> 8) & 31u), y);
    if constexpr (MANY) {
        y = bfi(0xFFFFFFFFu << ((e.p1 >> 8) & 31u), x << (e.p1 & 31u), y);
        y = bfi(0xFFFFFFFFu << ((e.p1 >> 24) & 31u), x << ((e.p1 >> 16) & 31u), y);
    }
    return bfi(e.nm, y, e.bv);
}

enum { kFromIds = 0, kFromStage = 1, kFromCache = 2 };   // where an item's row is found

// SPLIT: a window as separate dword loads. `blocks`, `block_waves`: the launch's blocks and waves
// per block, as arguments: read from the launch they would bring 256 bytes of implicit ones.
template <int K, int P, int SRC, bool TILED, bool SPLIT>
__device__ __forceinline__ void gather_slots(const DevStream &s, const CacheView &c, const uint8_t *__restrict__ pay,
                                             const int64_t *__restrict__ ids, const uint32_t *__restrict__ sg,
                                             const uint32_t *__restrict__ soff, uint64_t n_items, uint32_t tiles,
                                             uint32_t blocks, uint32_t block_waves, uint64_t tiles_magic,
                                             uint32_t *__restrict__ out,
                                             unsigned long long *err) {
    constexpr int IT = kWave / P;                       // items of the wave
    constexpr int GROUP = K <= 2 || IT < 4 ? IT : 4;    // items whose windows are in flight together
    constexpr int H = (K + 1) / 2;                      // windows per lane: one per two words
    constexpr int D = K == 1 ? 2 : 3;                   // dwords per window
    __shared__ PairDeposit s_tab[kBlock];
    const uint32_t l = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    PairDeposit *__restrict__ tab = s_tab + wave * kWave;
    const uint64_t base = ((uint64_t)xcd_block(blockIdx.x, blocks) * block_waves + wave) * IT;
    if (base >= n_items) return;
    const uint32_t W = s.W;
    const uint32_t cnt = (uint32_t)min((uint64_t)IT, n_items - base);
    const uint32_t own = l / P;
    const uint32_t pair_at = P == 8 ? l % 8 : l & (s.slot_pairs - 1);   // (P 16 also takes slots of 8 pairs)
    const uint64_t item = base + min(own, cnt - 1);   // lanes past the end repeat the last item
    uint64_t r = item;
    uint32_t t = 0;
    if constexpr (TILED) {
        r = __umul64hi(item, tiles_magic);
        t = (uint32_t)(item - r * tiles);
    }
    bool valid = true, hit = false;
    uint64_t g, byte;
    uint32_t len;
    const uint8_t *slot_l;
    uint2 pair;
    uint64_t uid = 0;
    [[maybe_unused]] CacheProbe probe;
    if constexpr (SRC == kFromStage) {
        g = sg[r];
        byte = soff[r];
        len = soff[r + 1] - (uint32_t)byte;
        slot_l = s.slots + g * s.slot_bytes;
        pair = reinterpret_cast<const uint2 *>(slot_l)[pair_at];
    } else {
        const int64_t id = ids[r];
        valid = id >= 0 && (uint64_t)id < s.n_rows;
        uid = valid ? (uint64_t)id : 0;
        if constexpr (SRC == kFromCache) probe = cache_probe_begin(c, uid);
        g = s.G == 1 ? uid : __umul64hi(uid, s.g_magic);
        slot_l = s.slots + g * s.slot_bytes;
        pair = reinterpret_cast<const uint2 *>(slot_l)[pair_at];
        const GroupInfo gi = s.groups[g];
        byte = valid ? gi.off + (uint64_t)(uint32_t)(uid - g * s.G) * gi.stride : 0;
        len = valid ? gi.stride : 0u;   // (an invalid id reads nothing)
    }
    // every item's pair indices of the lane's words, 4 bits each
    const uint8_t *const idx_l = slot_l + (P == 8 ? 64u : 8u * s.slot_pairs) + (TILED ? t * (32u * K) : 0u);
    uint32_t idx[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const GlobalBytes p = lane_ptr(idx_l, i * P);
        if constexpr (K == 1) idx[i] = p[own_lane() >> 1];
        else if constexpr (K == 2) idx[i] = p[own_lane()];
        else idx[i] = *(const __attribute__((address_space(1))) uint16_t *)(p + 2u * own_lane());
    }
    if constexpr (SRC == kFromCache) {
        keep_order();   // the probe's loop is entered with the loads above in flight
        hit = valid && cache_probe_end(c, uid, probe, byte);
    }
    uint32_t start = 0;
    if constexpr (TILED) start = s.tile_bits[g * s.tiles128 + t * (K / 2)];
    // where each item's bits are: the dword its row starts in, the dwords of the row, the
    // first bit of the item
    const uint8_t *const row_l = (SRC == kFromCache && hit ? c.slab : pay) + (byte & ~3ull);
    const uint32_t bit0 = ((uint32_t)byte & 3u) * 8u;
    // (at least 12 bytes, readable past any row (kReadPast), so that a window's split loads stay ordered
    // against the range)
    const uint32_t range_l = max(((bit0 + len * 8u + 31u) >> 5) * 4u, 12u);
    const uint32_t first_l = bit0 + start;
    const uint64_t okm = __ballot(valid && own < cnt);
    const uint64_t badm = __ballot(!valid && own < cnt);
    if constexpr (SRC == kFromCache) {
        const uint64_t hits = __ballot(hit && own < cnt && l % P == 0);
        const uint64_t misses = __ballot(valid && !hit && own < cnt && l % P == 0);
        if (l == 0) cache_count(c, (uint32_t)__popcll(hits), (uint32_t)__popcll(misses));
    }

    // the deposit of this lane's pair
    const uint32_t nm = ~pair.x;
    const uint32_t lo1 = first_bit(nm);
    const uint32_t m2 = nm & (nm + (nm & (0u - nm)));
    uint32_t n1 = (uint32_t)__builtin_popcount(nm ^ m2);
    const uint32_t lo2 = m2 ? first_bit(m2) : lo1, sh2 = m2 ? lo2 - n1 : lo1;
    const uint32_t m3 = m2 & (m2 + (m2 & (0u - m2)));
    const uint64_t many = __ballot(m3 != 0);   // pairs of more than two runs
    uint64_t more = 0;                         // of more than four
    PairDeposit e;
    e.nm = nm;
    e.bv = pair.y;
    e.p0 = lo1 | sh2 << 8 | lo2 << 16 | (uint32_t)__builtin_popcount(nm) << 24;
    e.p1 = 0;
    if (many) {
        n1 += (uint32_t)__builtin_popcount(m2 ^ m3);
        const uint32_t lo3 = m3 ? first_bit(m3) : lo2, sh3 = m3 ? lo3 - n1 : sh2;
        const uint32_t m4 = m3 & (m3 + (m3 & (0u - m3)));
        n1 += (uint32_t)__builtin_popcount(m3 ^ m4);
        const uint32_t lo4 = m4 ? first_bit(m4) : lo3, sh4 = m4 ? lo4 - n1 : sh3;
        e.p1 = sh3 | lo3 << 8 | sh4 << 16 | lo4 << 24;
        more = __ballot((m4 & (m4 + (m4 & (0u - m4)))) != 0);
    }
    tab[l] = e;
    wave_lds_fence();

    // every item's first bit of the lane's windows
    uint32_t row_mask[K];   // all ones for the lane's words inside the row
#pragma unroll
    for (int j = 0; j < K; ++j) row_mask[j] = K * l + j < W ? ~0u : 0u;
    auto entry = [&](uint32_t bits, int j, uint32_t i) {   // the table entry of the lane's word j of item i
        return ((K == 1 ? bits >> ((l & 1u) * 4u) : bits >> (4 * j)) & 15u) + i * P;
    };
    auto first_bits = [&](uint32_t bits, uint32_t i, uint32_t (&first)[H]) {
        uint32_t width[K], sum = 0;
        const uint32_t words = TILED ? W - (uint32_t)__builtin_amdgcn_readlane((int)t, (int)(i * P)) * (64u * K) : W;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            // (a mask, not a branch: the table reads of all items stay in flight)
            const uint32_t in_row = TILED ? (K * l + j < words ? ~0u : 0u) : row_mask[j];
            width[j] = reinterpret_cast<const uint8_t *>(&tab[entry(bits, j, i)].p0)[3] & in_row;
            sum += width[j];
        }
        first[0] = wave_incl_scan(sum) - sum + (uint32_t)__builtin_amdgcn_readlane((int)first_l, (int)(i * P));
        if constexpr (H == 2) first[1] = first[0] + width[0] + width[1];
    };
    auto row_of = [&](uint32_t i) {
        return row_rsrc(reinterpret_cast<const uint32_t *>(lane_u64(reinterpret_cast<uint64_t>(row_l), i * P)),
                        (uint32_t)__builtin_amdgcn_readlane((int)range_l, (int)(i * P)));
    };
    auto windows = [&](uint32_t i, const uint32_t (&first)[H], uint32_t (&d)[H][D]) {
        const __amdgpu_buffer_rsrc_t rr = row_of(i);
#pragma unroll
        for (int h = 0; h < H; ++h) row_window<D, SPLIT>(rr, first[h], d[h]);
    };
    auto words_of = [&](auto how, uint32_t bits, uint32_t i, const uint32_t (&first)[H], const uint32_t (&d)[H][D],
                        uint32_t (&v)[K]) {
        constexpr int HOW = decltype(how)::value;
        auto word = [&](const PairDeposit &p, uint32_t x) {
            if constexpr (HOW < 2) {
                return deposit<HOW == 1>(p, x);
            } else {
                const uint32_t most = wave_max(run_count(p.nm));
                return word_deposit(p.bv, p.nm, x, most ? most - 1u : 0u);
            }
        };
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const PairDeposit e0 = tab[entry(bits, 2 * h, i)];
            const uint32_t lo = __builtin_amdgcn_alignbit(d[h][1], d[h][0], first[h]);
            v[2 * h] = word(e0, lo);
            if constexpr (K > 1) {
                const PairDeposit e1 = tab[entry(bits, 2 * h + 1, i)];
                const uint32_t hi = __builtin_amdgcn_alignbit(d[h][2], d[h][1], first[h]);
                v[2 * h + 1] = word(e1, (uint32_t)((((uint64_t)hi << 32) | lo) >> (e0.p0 >> 24)));
            }
        }
    };
    // An item's words through a buffer descriptor over its output: the range check drops the
    // lanes (and the words of the last lane) past the row's end, and, with an empty range,
    // the whole item of an out-of-range id, without a branch.
    const uint64_t out_w = reinterpret_cast<uint64_t>(out + base * W);
    auto store = [&](uint32_t i, bool on, const uint32_t (&v)[K]) {
        uint64_t to = out_w + (uint64_t)(i * W * 4u);
        uint32_t bytes = W * 4u;
        if constexpr (TILED) {
            const uint32_t tu = (uint32_t)__builtin_amdgcn_readlane((int)t, (int)(i * P)) * (64u * K);
            bytes = (W - tu) * 4u;
            to = reinterpret_cast<uint64_t>(out) + (lane_u64(r, i * P) * W + tu) * 4u;
        }
        store_words<K>(row_rsrc(reinterpret_cast<const uint32_t *>(to), on ? bytes : 0u), l * (4u * K), v);
    };

    // groups of items: all their first bits, all their windows, then their words
    for_items<0, IT / GROUP>([&](auto gg) {
        constexpr int i0 = decltype(gg)::value * GROUP;
        uint32_t first[GROUP][H], d[GROUP][H][D];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) first_bits(idx[i0 + i], i0 + i, first[i]);
#pragma unroll
        for (int i = 0; i < GROUP; ++i) windows(i0 + i, first[i], d[i]);
        keep_order();
        for_items<0, GROUP>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            constexpr uint64_t kPairs = ((1ull << P) - 1ull) << ((i0 + i) * P);
            const bool on = ((okm >> ((i0 + i) * P)) & 1ull) && !(more & kPairs);
            uint32_t v[K];
            if (!(many & kPairs)) words_of(std::integral_constant<int, 0>{}, idx[i0 + i], i0 + i, first[i], d[i], v);
            else words_of(std::integral_constant<int, 1>{}, idx[i0 + i], i0 + i, first[i], d[i], v);
            store(i0 + i, on, v);
        });
    });
    if (more) {
        // items with words of more than four runs: the holes deposit, one item at a time
        for (uint32_t i = 0; i < cnt; ++i) {
            if (!((okm >> (i * P)) & 1ull) || !((more >> (i * P)) & ((1ull << P) - 1ull))) continue;
            const GlobalBytes p = lane_ptr(idx_l, i * P);
            uint32_t bits, f[H], w[H][D], v[K];
            if constexpr (K == 1) bits = p[l >> 1];
            else if constexpr (K == 2) bits = p[l];
            else bits = *(const __attribute__((address_space(1))) uint16_t *)(p + 2u * l);
            first_bits(bits, i, f);
            windows(i, f, w);
            words_of(std::integral_constant<int, 2>{}, bits, i, f, w, v);
            store(i, true, v);
        }
    }
    if (badm) {
        // zero the rows of out-of-range ids, each counted once (by its first tile)
        for (int i = 0; i < IT; ++i) {
            if (!((badm >> (i * P)) & 1ull)) continue;
            const uint32_t tu = (uint32_t)__builtin_amdgcn_readlane((int)t, i * P) * (64u * K);
            uint32_t *orow = out + lane_u64(r, i * P) * W;
            for (uint32_t w = tu + l; w < min(W, tu + 64u * K); w += kWave) orow[w] = 0u;
        }
        const uint64_t counted = __ballot(!valid && own < cnt && l % P == 0 && t == 0);
        if (l == 0 && counted) atomicAdd(err, (unsigned long long)__popcll(counted));
    }
}

template <int K, int P, int SRC, bool TILED, bool SPLIT>
__global__ __launch_bounds__(kBlock, K <= 2 ? 8 : 5) void k_gather_slots(DevStream s, const uint8_t *__restrict__ pay,
                                                                         const int64_t *__restrict__ ids,
                                                                         const uint32_t *__restrict__ sg,
                                                                         const uint32_t *__restrict__ soff,
                                                                         uint64_t n_items, uint32_t tiles,
                                                                         uint32_t blocks, uint32_t block_waves,
                                                                         uint64_t tiles_magic,
                                                                         uint32_t *__restrict__ out,
                                                                         unsigned long long *err) {
    gather_slots<K, P, SRC, TILED, SPLIT>(s, CacheView{}, pay, ids, sg, soff, n_items, tiles, blocks, block_waves,
                                          tiles_magic, out, err);
}

template <int K, int P>
__global__ __launch_bounds__(kBlock, 8) void k_cache_gather_slots(DevStream s, CacheView c,
                                                                  const int64_t *__restrict__ ids, uint64_t n_items,
                                                                  uint32_t blocks, uint32_t block_waves,
                                                                  uint32_t *__restrict__ out,
                                                                  unsigned long long *err) {
    gather_slots<K, P, kFromCache, false, false>(s, c, c.host_payload, ids, nullptr, nullptr, n_items, 1, blocks,
                                                 block_waves, 0, out, err);
}

// Per cluster: where its rows start, their distance, and the bit at which every 128-word
// tile of a row starts. A wave per cluster, the clusters in strides of the grid.
__global__ __launch_bounds__(kBlock) void k_group_info(DevStream s, GroupInfo *__restrict__ groups,
                                                       uint32_t *__restrict__ tile_bits) {
    const uint32_t l = lane_id(), W = s.W;
    for (uint64_t g = wave_slot(); g < s.n_groups; g += (uint64_t)gridDim.x * kWavesPerBlock) {
        const uint32_t *__restrict__ mg = s.meta + g * 2ull * W;
        uint32_t bits = 0;
        for (uint32_t w0 = 0, t = 0; w0 < W; w0 += 128, ++t) {
            if (tile_bits && l == 0) tile_bits[g * s.tiles128 + t] = bits;
            uint32_t n = 0;
            for (uint32_t w = w0 + l; w < min(W, w0 + 128u); w += kWave) n += (uint32_t)__builtin_popcount(~mg[w]);
            bits += wave_sum(n);
        }
        if (groups && l == 0)
            groups[g] = GroupInfo{s.index[g], (uint32_t)row_stride((bits + 7u) >> 3, s.row_align)};
    }
}

}  // namespace

hipError_t launch_group_info(const DevStream &s, GroupInfo *groups, uint32_t *tile_bits, hipStream_t stream) {
    if (s.n_groups == 0) return hipSuccess;
    hipLaunchKernelGGL(k_group_info, dim3((unsigned)cluster_blocks(s.n_groups)), dim3(kBlock), 0, stream, s, groups,
                       tile_bits);
    return hipGetLastError();
}

hipError_t launch_gather_slots(const DevStream &s, const CacheView *cache, const uint8_t *payload, const int64_t *ids,
                               const uint32_t *sg, const uint32_t *soff, uint64_t n, void *out,
                               unsigned long long *err, hipStream_t stream) {
    auto *o = static_cast<uint32_t *>(out);
    const uint32_t tiles = s.W <= 256 ? 1u : (s.W + 255u) / 256u;
    const uint64_t items = n * tiles;
    // Few items: 16 lanes each also where slots hold 8 pairs (four items per wave instead of eight,
    // which follow one another at several points), and a wave per block, so that they spread over
    // the CUs. us on the GPU, 8 lanes and 4 waves per block / 16 and 4 / 16 and 1, clusters of at
    // most 8 pairs in device memory:
    //   rows of 100 words  100: 4.08 / 3.20 / 3.09   4,000: 4.33 / 3.46 / 3.43   8,000: 4.54 / 3.85 / 3.94
    //                      16,000: 4.91 / 4.55 / 4.85
    //   rows of 300 words  100: 5.42 / 3.93 / 3.82   4,000 (8,000 items): 5.84 / 4.86 / 4.87
    //   rows of 1,000 words  4,000 (16,000 items): 7.27 / 6.81 / 7.10   8,000: 10.88 / 11.03 / 11.05
    // in host memory, 100 words, 400 rows 7.54 / 6.77 / 6.63; 520 of 100 words behind a cache that
    // misses most 8.62 / 8.10 / 5.84.
    const bool pairs16 = s.slot_pairs == 16 || items <= 16384;
    const uint32_t per = pairs16 ? 4 : 8;
    const uint64_t waves = (items + per - 1) / per;
    const uint32_t block_waves = waves <= 1024 ? 1 : kWavesPerBlock;
    const uint64_t blocks = (waves + block_waves - 1) / block_waves;
    if (too_many_blocks(blocks, n))
        return in_halves(n, [&](uint64_t i, uint64_t count) {
            return launch_gather_slots(s, cache, payload, from(ids, i), from(sg, i), from(soff, i), count, o + i * s.W,
                                       err, stream);
        });
    const dim3 grid((unsigned)blocks), block(kWave * block_waves);
    auto go = [&](auto k, auto tiled, auto src, auto split) {
        constexpr int K = decltype(k)::value, SRC = decltype(src)::value;
        constexpr bool T = decltype(tiled)::value, SP = decltype(split)::value;
        auto pairs = [&](auto p) {
            constexpr int P = decltype(p)::value;
            if constexpr (SRC == kFromCache)
                hipLaunchKernelGGL((k_cache_gather_slots<K, P>), grid, block, 0, stream, s, *cache, ids, items,
                                   (uint32_t)blocks, block_waves, o, err);
            else
                hipLaunchKernelGGL((k_gather_slots<K, P, SRC, T, SP>), grid, block, 0, stream, s, payload, ids, sg,
                                   soff, items, tiles, (uint32_t)blocks, block_waves, div_magic(tiles),
                                   o, err);
        };
        if (pairs16) pairs(std::integral_constant<int, 16>{});
        else pairs(std::integral_constant<int, 8>{});
    };
    // A window of device memory is read as separate dwords at one or two words per lane (4-5%
    // faster than one load) and as one load at four (17% faster). From host memory always as
    // one: its reads bypass the L2, so that every load of a line is a read over PCIe.
    auto narrow = [&](auto k) {
        if (cache) go(k, std::false_type{}, std::integral_constant<int, kFromCache>{}, std::false_type{});
        else if (s.payload_host) go(k, std::false_type{}, std::integral_constant<int, kFromIds>{}, std::false_type{});
        else if (soff) go(k, std::false_type{}, std::integral_constant<int, kFromStage>{}, std::true_type{});
        else go(k, std::false_type{}, std::integral_constant<int, kFromIds>{}, std::true_type{});
    };
    auto wide = [&](auto tiled) {
        constexpr std::integral_constant<int, 4> k{};
        if (soff) go(k, tiled, std::integral_constant<int, kFromStage>{}, std::false_type{});
        else go(k, tiled, std::integral_constant<int, kFromIds>{}, std::false_type{});
    };
    if (s.W <= 64) narrow(std::integral_constant<int, 1>{});
    else if (s.W <= 128) narrow(std::integral_constant<int, 2>{});
    else if (cache || s.payload_host) return hipErrorInvalidValue;   // (they have lane-order slots)
    else if (s.W <= 256) wide(std::false_type{});
    else wide(std::true_type{});
    return hipGetLastError();
}

}  // namespace dev
}  // namespace ibp
