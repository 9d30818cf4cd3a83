// gfx950 kernel of the compressed device-resident row cache (the paper's cache
// compression, Sec. 5): a static set of rows is kept, in packed form, back to back in a
// device slab; a lookup table maps a row id to a 64-bit entry (slab byte offset in bits
// 0-39, slab id in bits 40-42, compressed-form flag in bit 43). A gather resolves every
// requested id against the table: hits are decoded from the slab in HBM, misses from the
// stream's payload in pinned host memory, read in place over PCIe.
//
// Rows of at most 128 words whose clusters have metadata slots are decoded by the gather of
// ibp_gather_kernels.hip, which finds a row here before its payload offset. The others by the
// kernel below, as the row-at-a-time gather: one wave per batch of RB requests, each row
// decoded on its own (its cluster's Mask/Bitval, a scan of popcount(~Mask), the holes
// deposit), all loads of the batch issued before any word is rebuilt. The only change is
// that a row's packed bytes are located by an absolute address chosen per request.
#include <type_traits>

#include "ibp_cache.hpp"
#include "ibp_device.hpp"
#include "ibp_wave.hpp"

namespace ibp {
namespace dev {

namespace {

template <int K, int RB, int FORM>
__global__ __launch_bounds__(kBlock) void k_cache_gather(DevStream s, CacheView c, const int64_t *__restrict__ ids,
                                                          uint64_t n, uint32_t *__restrict__ out,
                                                          unsigned long long *err) {
    const uint64_t slot = (uint64_t)xcd_block(blockIdx.x, gridDim.x) * kWavesPerBlock +
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint64_t i0 = slot * RB;
    if (i0 >= n) return;
    const uint32_t cnt = (uint32_t)min((uint64_t)RB, n - i0);
    const uint32_t l = lane_id();
    const uint32_t W = s.W;
    // lane l < cnt resolves request l: cluster, row inside it, and where its bytes are
    const int64_t id = l < cnt ? ids[i0 + l] : -1;
    const bool valid = l < cnt && id >= 0 && (uint64_t)id < s.n_rows;
    const uint64_t uid = valid ? (uint64_t)id : 0;
    const uint64_t g_l = s.G == 1 ? uid : __umul64hi(uid, s.g_magic);
    const uint32_t r_l = (uint32_t)(uid - g_l * s.G);
    // byte address of the row's packed bits: the slab entry for a hit; for a miss the
    // cluster's payload offset, to which the row's index times its packed size is added
    // once the size is known from the Mask
    const CacheProbe probe = cache_probe_begin(c, uid);
    uint64_t off_l = s.index[g_l];
    const bool hit = valid && cache_probe_end(c, uid, probe, off_l);
    const uint32_t mul_l = hit ? 0u : r_l;
    const uint64_t nhit = __ballot(valid && hit), nmiss = __ballot(valid && !hit);
    const uint64_t bad = __ballot(l < cnt && !valid);
    if (l == 0) {
        cache_count(c, (uint32_t)__popcll(nhit), (uint32_t)__popcll(nmiss));
        if (bad) atomicAdd(err, (unsigned long long)__popcll(bad));
    }
    uint32_t *__restrict__ out_seg = out + i0 * W;
    if (bad) {
        for (uint32_t i = 0; i < cnt; ++i)
            if ((bad >> i) & 1ull)
                for (uint32_t w = l; w < W; w += kWave) out_seg[(uint64_t)i * W + w] = 0u;
    }
    auto rd64 = [](uint64_t v, uint32_t i) -> uint64_t {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)i) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)i);
    };
    auto slot_of = [&](uint32_t i) { return i < cnt ? i : cnt - 1; };
    RowMeta<K, FORM> meta[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
        const uint64_t g = rd64(g_l, slot_of(u));
        load_row_meta<K, FORM>(meta[u], s.meta + g * 2ull * W, s.slots + g * s.slot_bytes, s.slot_pairs, W);
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) hold_row_meta(meta[u]);
    uint32_t nm[RB][K], bv[RB][K], ofs[RB][K], d0[RB][K], d1[RB][K], nh[RB], bit0[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
        const uint32_t i = slot_of(u);
        uint32_t cntw[K], runs = 0, mw[K], bw[K];
        expand_row_meta(meta[u], mw, bw);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool in_row = l + kWave * j < W;
            nm[u][j] = in_row ? ~mw[j] : 0u;
            bv[u][j] = in_row ? bw[j] : 0u;
            cntw[j] = (uint32_t)__builtin_popcount(nm[u][j]);
            if constexpr (FORM == kMetaRaw) runs = max(runs, run_count(nm[u][j]));
        }
        const uint32_t tot = row_offsets<K>(cntw, ofs[u]);
        uint32_t max_runs;
        if constexpr (FORM == kMetaSlots) max_runs = slot_max_runs(meta[u], s.slot_pairs);
        else max_runs = wave_max(runs);
        nh[u] = max_runs ? max_runs - 1u : 0u;
        const uint64_t rb = (tot + 7u) >> 3;
        // a select of the two buffers, not an integer address, keeps the loads global
        // (not flat) and the choice free of branches
        const uint8_t *__restrict__ buf = ((nhit >> i) & 1ull) ? c.slab : c.host_payload;
        const uint64_t addr = rd64(off_l, i) + (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mul_l, (int)i) * rb;
        const uint32_t *__restrict__ p = reinterpret_cast<const uint32_t *>(buf + (addr & ~3ull));
        bit0[u] = ((uint32_t)addr & 3u) * 8u;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint32_t q = (ofs[u][j] + bit0[u]) >> 5;
            d0[u][j] = p[q];
            d1[u][j] = p[q + 1];
        }
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) {
        const uint32_t i = u;
        const bool row_ok = i < cnt && !((bad >> i) & 1ull);
        uint32_t *__restrict__ orow = out_seg + (uint64_t)slot_of(i) * W;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint32_t x = __builtin_amdgcn_alignbit(d1[u][j], d0[u][j], ofs[u][j] + bit0[u]);
            const uint32_t v = word_deposit(bv[u][j], nm[u][j], x, nh[u]);
            const uint32_t w = l + kWave * j;
            if (row_ok && w < W) store_out(&orow[w], v);
        }
    }
}

}  // namespace

hipError_t launch_cache_gather(const DevStream &s, const CacheView &c, const int64_t *ids, uint64_t n, void *out,
                               unsigned long long *err, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (s.slots && s.word_order)
        return launch_gather_slots(s, &c, c.host_payload, ids, nullptr, nullptr, n, out, err, stream);
    auto *o = static_cast<uint32_t *>(out);
    const uint32_t rb_sel = s.W <= 64 ? 8 : (s.W <= 128 ? 4 : (s.W <= 256 ? 2 : 1));
    const uint64_t blocks = blocks_of_waves((n + rb_sel - 1) / rb_sel);
    if (too_many_blocks(blocks, n))
        return in_halves(n, [&](uint64_t i, uint64_t count) {
            return launch_cache_gather(s, c, ids + i, count, o + i * s.W, err, stream);
        });
    const dim3 grid((unsigned)blocks);
    auto go = [&](auto kk, auto rb) {
        constexpr int KK = decltype(kk)::value, R = decltype(rb)::value;
        if (s.slots) {   // (lane order: rows of more than 128 words)
            if constexpr (KK >= 4) hipLaunchKernelGGL((k_cache_gather<KK, R, kMetaSlots>), grid, dim3(kBlock), 0, stream, s, c, ids, n, o, err);
        } else hipLaunchKernelGGL((k_cache_gather<KK, R, kMetaRaw>), grid, dim3(kBlock), 0, stream, s, c, ids, n, o, err);
    };
    if (s.W <= 64) go(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
    else if (s.W <= 128) go(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    else if (s.W <= 256) go(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    else if (s.W <= 512) go(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{});
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace dev
}  // namespace ibp
