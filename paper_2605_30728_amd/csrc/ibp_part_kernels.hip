// gfx950 decode of thresholded-scheme rows (participation bits, stream flags = 1) of at most
// 128 words, contiguous or gathered.
//
// Which chunks of a row are compressed differs from row to row, so its word offsets are a
// scan per row: a word's width is popcount(~Mask) when its chunk is compressed and 32
// otherwise. What a wave does per row is therefore kept short:
//
//   * lane i first locates item i (its row's bytes) and fetches the row's participation
//     dwords (at most 128 chunks: one, two or four) in the same round trip; a row's values
//     are then read from its lane where needed;
//   * lane l owns the K consecutive words K*l .. K*l + K - 1: one scan per row, and one
//     window of three dwords and one store for two words;
//   * a word's participation bit becomes an all-ones or all-zeros lane mask (a sign-extended
//     bit-field extract), which selects its width and then its rebuilt or raw value by
//     bit-field insert: no compare and no branch per row;
//   * loads past a row's packed bytes and stores past its output are dropped by the range
//     check of a buffer descriptor per row.
//
// Measured (us, strided words with a scan and a store per word -> this): a 134 MB bf16 KV
// layer (524k rows of 64 words, 259 MB of HBM traffic) 50.2 -> 45.2, 82k sorted 400-B rows of
// 1.2M 17.4 -> 13.8 (108 -> ~55 vector instructions per row; HBM bounds both now), 145k rows
// of 60 words 14.5 -> 14.2, 82k rows under per-cluster Masks 30.0 -> 23.8.
//
// Under one Mask for the whole stream (ONE, the scheme as published) its words are set up
// once per wave. Otherwise a batch of rows that share a cluster reuses its setup, and a
// batch of rows from different clusters loads every row's Mask/Bitval words.
#include <algorithm>
#include <type_traits>

#include "ibp_device.hpp"
#include "ibp_tile.hpp"
#include "ibp_wave.hpp"

namespace ibp {
namespace dev {

namespace {

enum { kSrcRange = 0, kSrcIds = 1, kSrcStaged = 2 };

// A row of a batch between its loads and its rebuild.
template <int K>
struct PartRow {
    uint32_t d[K + 1];   // the lane's window
    uint32_t first;      // its first bit (the low five bits count)
    uint32_t sel[K];     // all ones for a word of a compressed chunk
    uint32_t width;      // of the lane's first word
};

// PRE: participation dwords per row (1, 2 or 4). SPLIT: a window as separate dword loads.
template <int K, int MAXR, int SRC, int PRE, bool ONE, bool SPLIT>
__global__ __launch_bounds__(kBlock, K == 1 ? 8 : (!ONE ? 5 : (PRE == 2 ? 8 : 7))) void k_part_narrow(DevStream s, const uint8_t *__restrict__ pay,
                                                           uint64_t pay_base, const int64_t *__restrict__ ids,
                                                           const uint32_t *__restrict__ sg,
                                                           const uint32_t *__restrict__ soff, uint64_t first,
                                                           uint64_t n, uint32_t *__restrict__ out, uint32_t seg,
                                                           uint32_t block_waves, unsigned long long *err) {
    constexpr int RB = K == 1 ? 8 : 4;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint64_t i0 = ((uint64_t)blockIdx.x * block_waves + wave) * seg;
    if (i0 >= n) return;
    const uint32_t cnt = (uint32_t)min((uint64_t)seg, n - i0);
    const uint32_t l = lane_id();
    const uint32_t W = s.W, m = s.part_m, C = W / m;
    const uint32_t li = min(l, cnt - 1);   // lanes past the end repeat the last item
    uint64_t g_l, byte_l;
    uint32_t size_l;
    bool valid = true;
    if constexpr (SRC == kSrcStaged) {
        g_l = sg[i0 + li];
        byte_l = soff[i0 + li];
        size_l = soff[i0 + li + 1] - (uint32_t)byte_l;
    } else {
        uint64_t r;
        if constexpr (SRC == kSrcIds) {
            const int64_t id = ids[i0 + li];
            valid = id >= 0 && (uint64_t)id < s.n_rows;
            r = valid ? (uint64_t)id : 0u;
        } else {
            r = first + i0 + li;
        }
        g_l = s.G == 1 ? r : __umul64hi(r, s.g_magic);
        uint64_t o0, o1;
        row_span(s, r, o0, o1);
        byte_l = valid ? o0 - pay_base : 0u;
        size_l = valid ? (uint32_t)(o1 - o0) : 0u;   // (an invalid id reads nothing)
    }
    const uint8_t *const row_l = pay + (byte_l & ~3ull);
    const uint32_t bit0 = ((uint32_t)byte_l & 3u) * 8u;
    uint32_t pdw[PRE];
    {
        const uint32_t *__restrict__ p = reinterpret_cast<const uint32_t *>(row_l);
        uint32_t q[PRE + 1];
#pragma unroll
        for (int k = 0; k <= PRE; ++k) q[k] = p[k];
#pragma unroll
        for (int k = 0; k < PRE; ++k) pdw[k] = __builtin_amdgcn_alignbit(q[k + 1], q[k], bit0);
    }
    const bool raw_l = size_l == 4u * W;   // no chunk of a raw row is compressed
    if (raw_l) {
#pragma unroll
        for (int k = 0; k < PRE; ++k) pdw[k] = 0u;
    }
    const uint32_t first_l = bit0 + (raw_l ? 0u : C);
    const uint32_t range_l = max(((bit0 + size_l * 8u + 31u) >> 5) * 4u, 12u);   // (see row_window)
    const uint64_t okm = __ballot(l < cnt && valid);
    const uint64_t badm = __ballot(l < cnt && !valid);

    // lane constants of the lane's words: width when raw, and where its chunk's bit is
    uint32_t full[K], bit[K], dw[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const uint32_t w = K * l + j, c = (w < W ? w : 0u) / m;
        full[j] = w < W ? 32u : 0u;
        bit[j] = c & 31u;
        dw[j] = c >> 5;
    }
    auto load = [&](uint32_t i, const uint32_t (&pk)[K], PartRow<K> &row) {
        uint32_t p[PRE], width[K], sum = 0;
#pragma unroll
        for (int k = 0; k < PRE; ++k) p[k] = (uint32_t)__builtin_amdgcn_readlane((int)pdw[k], (int)i);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            uint32_t x = p[0];
            if constexpr (PRE == 2) x = dw[j] ? p[1] : p[0];
            if constexpr (PRE == 4) x = dw[j] & 2u ? (dw[j] & 1u ? p[3] : p[2]) : (dw[j] & 1u ? p[1] : p[0]);
            row.sel[j] = (uint32_t)__builtin_amdgcn_sbfe((int)x, bit[j], 1u);
            width[j] = bit_select(row.sel[j], pk[j], full[j]);
            sum += width[j];
        }
        row.width = width[0];
        row.first = wave_incl_scan(sum) - sum + (uint32_t)__builtin_amdgcn_readlane((int)first_l, (int)i);
        row_window<K + 1, SPLIT>(row_rsrc(reinterpret_cast<const uint32_t *>(lane_u64(reinterpret_cast<uint64_t>(row_l), i)),
                                          (uint32_t)__builtin_amdgcn_readlane((int)range_l, (int)i)),
                                 row.first, row.d);
    };
    uint32_t *const out_seg = out + i0 * W;
    auto store = [&](uint32_t i, bool on, const uint32_t (&v)[K]) {
        store_words<K>(row_rsrc(out_seg + i * W, on ? 4u * W : 0u), l * (4u * K), v);
    };
    // the word's packed bits x, rebuilt by `word` when its chunk is compressed
    auto rebuild = [&](PartRow<K> &row, auto word, uint32_t (&v)[K]) {
        if constexpr (PRE == 4) {
            // the window is needed from here on: shifted earlier, to save registers, every row's
            // load was waited for before the next one was issued (100 rows of 104 words in host
            // memory, four-byte chunks, 9.5 us on the GPU; in flight together 5.9)
#pragma unroll
            for (int k = 0; k <= K; ++k) asm volatile("" : "+v"(row.d[k]));
        }
        const uint32_t lo = __builtin_amdgcn_alignbit(row.d[1], row.d[0], row.first);
        v[0] = bit_select(row.sel[0], word(0, lo), lo);
        if constexpr (K == 2) {
            const uint32_t hi = __builtin_amdgcn_alignbit(row.d[2], row.d[1], row.first);
            const uint32_t x = (uint32_t)((((uint64_t)hi << 32) | lo) >> row.width);
            v[1] = bit_select(row.sel[1], word(1, x), x);
        }
    };
    // RB rows from i on that share the cluster of tile t
    Tile<K, MAXR> t;
    auto batch = [&](auto nr, uint32_t i) {
        constexpr int NR = decltype(nr)::value;
        PartRow<K> row[RB];
#pragma unroll
        for (int u = 0; u < RB; ++u) load(min(i + u, cnt - 1), t.pk, row[u]);
        keep_order();
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            uint32_t v[K];
            rebuild(row[u], [&](int j, uint32_t x) {
                if constexpr (NR >= 0) return word_fast<NR>(t, j, x);
                else return word_generic(t.bv[j], t.nm[j], x);
            }, v);
            store(i + u, ((okm >> (i + u)) & 1ull) && i + u < cnt, v);
        }
    };
    auto with_runs = [&](auto f) {   // f(the tile's run count, a constant)
        switch (t.nr) {   // wave-uniform
        case 0: f(std::integral_constant<int, 0>{}); break;
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        default: f(std::integral_constant<int, -1>{}); break;
        }
    };
    if constexpr (ONE) {
        tile_setup<true>(t, s.meta, W, 0, 0);
        with_runs([&](auto nr) {
            for (uint32_t i = 0; i < cnt; i += RB) batch(nr, i);
        });
    } else {
        const uint32_t src = (l ? l - 1u : 0u) * 4u;
        const uint32_t gp_lo = (uint32_t)__builtin_amdgcn_ds_bpermute((int)src, (int)(uint32_t)g_l);
        const uint32_t gp_hi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)src, (int)(uint32_t)(g_l >> 32));
        const uint64_t samep = __ballot((((uint64_t)gp_hi << 32) | gp_lo) == g_l);   // as the item before
        uint64_t cached_g = ~0ull;
        for (uint32_t i = 0; i < cnt; i += RB) {
            const uint64_t tail = ((1ull << (RB - 1)) - 1ull) << (i + 1);   // i + RB <= seg <= 64
            if ((samep & tail) == tail) {
                const uint64_t g = lane_u64(g_l, i);
                if (g != cached_g) {
                    tile_setup<true>(t, s.meta + g * 2ull * W, W, 0, 0);
                    cached_g = g;
                }
                with_runs([&](auto nr) { batch(nr, i); });
                continue;
            }
            // rows of different clusters, half a batch at a time (every row's Mask/Bitval
            // words are live): the holes deposit, since a setup of runs per row would cost
            // more than it saves
#pragma unroll 1
            for (uint32_t h = i; h < i + RB && h < cnt; h += RB / 2) {
                uint32_t nm[RB / 2][K], bv[RB / 2][K];
                PartRow<K> row[RB / 2];
#pragma unroll
                for (int u = 0; u < RB / 2; ++u) {
                    const uint32_t *__restrict__ mg = s.meta + lane_u64(g_l, min(h + u, cnt - 1)) * 2ull * W;
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        const uint32_t w = K * l + j, wc = w < W ? w : 0u;
                        nm[u][j] = mg[wc];
                        bv[u][j] = mg[W + wc];
                    }
                }
#pragma unroll
                for (int u = 0; u < RB / 2; ++u) {
                    uint32_t pk[K];
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        nm[u][j] = K * l + j < W ? ~nm[u][j] : 0u;
                        pk[j] = (uint32_t)__builtin_popcount(nm[u][j]);
                    }
                    load(min(h + u, cnt - 1), pk, row[u]);
                }
                keep_order();
#pragma unroll
                for (int u = 0; u < RB / 2; ++u) {
                    uint32_t runs = 0, v[K];
#pragma unroll
                    for (int j = 0; j < K; ++j) runs = max(runs, run_count(nm[u][j]));
                    const uint32_t most = wave_max(runs);
                    rebuild(row[u], [&](int j, uint32_t x) {
                        return word_deposit(bv[u][j], nm[u][j], x, most ? most - 1u : 0u);
                    }, v);
                    store(h + u, ((okm >> (h + u)) & 1ull) && h + u < cnt, v);
                }
            }
        }
    }
    if (badm) {
        for (uint32_t i = 0; i < cnt; ++i)
            if ((badm >> i) & 1ull)
                for (uint32_t w = l; w < W; w += kWave) out_seg[(uint64_t)i * W + w] = 0u;
        if (l == 0) atomicAdd(err, (unsigned long long)__popcll(badm));
    }
}

template <int K, int MAXR>
hipError_t launch_narrow_k(const DevStream &s, const uint8_t *payload, uint64_t pay_base, const int64_t *ids,
                           const uint32_t *sg, const uint32_t *soff, uint64_t first, uint64_t n, uint32_t *o,
                           unsigned long long *err, hipStream_t stream) {
    // Batches of RB rows, two per wave when that leaves 8k waves (K = 2: 4k), else one: a wave
    // sets its Mask words up once, but its batches follow one another. Measured at 400-B rows
    // (K = 2): 82k gathered rows 15.9 us with one batch, 13.8 with two; 40k 9.7 and 8.3;
    // 200k contiguous 512-B rows 39 us with two, 41.6 with four. K = 1: 100k contiguous 256-B
    // rows 10.8 us with one, 11.5 with two; 524k 51 us with one, 45 with two, 55 with four.
    // Under per-cluster Masks two batches rarely share a setup: 300k contiguous 256-B rows of
    // 32-row clusters 28.3 us with one, 29.1 with two (82k gathered 400-B rows: 26.0 and 23.8).
    constexpr int RB = K == 1 ? 8 : 4;
    const bool one = (uint64_t)s.G >= s.n_rows;   // a single cluster
    const uint32_t nb = n / ((K == 1 ? 16384ull : 8192ull) * RB) >= 1 && (K == 2 || one) ? 2 : 1;
    // Requests under per-cluster Masks from pinned host memory, one word per lane: half a batch per
    // wave, since a wave decodes its halves one after the other, a round trip over PCIe each (us on
    // the GPU, 100 rows of 20 words 10.6 -> 6.6, 1,000 14.1 -> 9.2).
    const uint32_t seg = K == 1 && !one && ids && s.payload_host ? RB / 2 : RB * nb;
    const uint64_t waves = (n + seg - 1) / seg;
    // few waves spread over the CUs, except where neighbours share lines that cross PCIe (1,000
    // contiguous rows of 72 words in host memory 14.2 us in blocks of four waves, 15.8 of one)
    const uint32_t block_waves = waves <= 1024 && (!s.payload_host || ids) ? 1 : kWavesPerBlock;
    const uint64_t blocks = (waves + block_waves - 1) / block_waves;
    if (too_many_blocks(blocks, n))
        return in_halves(n, [&](uint64_t i, uint64_t count) {
            return launch_narrow_k<K, MAXR>(s, payload, pay_base, from(ids, i), from(sg, i), from(soff, i), first + i,
                                            count, o + i * s.W, err, stream);
        });
    const dim3 grid((unsigned)blocks), block(kWave * block_waves);
    const uint32_t chunks = s.W / s.part_m;
    auto go = [&](auto pre, auto one_tag, auto src) {
        constexpr int P = decltype(pre)::value, S = decltype(src)::value;
        constexpr bool O = decltype(one_tag)::value;
        // windows as separate dword loads at K = 1 (524k rows: 45.2 us, 50.1 as one 8-byte
        // load; from pinned host memory too: 9,879 rows of 16 words 15.1 and 16.2, 28,882 of 12
        // words 27.7 and 28.7, rows of 40 words and more alike), as one 12-byte load at K = 2
        // (200k contiguous 512-B rows: 39 us, 48 split)
        hipLaunchKernelGGL((k_part_narrow<K, MAXR, S, P, O, K == 1>), grid, block, 0, stream, s, payload, pay_base,
                           ids, sg, soff, first, n, o, seg, block_waves, err);
    };
    auto go_src = [&](auto pre, auto one_tag) {
        if (ids) go(pre, one_tag, std::integral_constant<int, kSrcIds>{});
        else if (sg) go(pre, one_tag, std::integral_constant<int, kSrcStaged>{});
        else go(pre, one_tag, std::integral_constant<int, kSrcRange>{});
    };
    auto go_one = [&](auto pre) {
        if (one) go_src(pre, std::true_type{});
        else go_src(pre, std::false_type{});
    };
    if (chunks <= 32u) go_one(std::integral_constant<int, 1>{});
    else if (chunks <= 64u) go_one(std::integral_constant<int, 2>{});
    else if constexpr (K == 2) go_one(std::integral_constant<int, 4>{});
    else return hipErrorInvalidValue;   // 64 words: at most 64 chunks
    return hipGetLastError();
}

}  // namespace

hipError_t launch_part_narrow(const DevStream &s, const uint8_t *payload, uint64_t pay_base, const int64_t *ids,
                              const uint32_t *sg, const uint32_t *soff, uint64_t first, uint64_t n, void *out,
                              unsigned long long *err, hipStream_t stream) {
    auto *o = static_cast<uint32_t *>(out);
    if (s.W <= 64) return launch_narrow_k<1, 4>(s, payload, pay_base, ids, sg, soff, first, n, o, err, stream);
    if (s.W <= 128) return launch_narrow_k<2, 4>(s, payload, pay_base, ids, sg, soff, first, n, o, err, stream);
    return hipErrorInvalidValue;
}

}  // namespace dev
}  // namespace ibp
