// How a call's rows are shared out over the waves of a launch: plain arithmetic that the
// launchers and the kernels share and that also compiles without HIP.
#pragma once

#include <algorithm>
#include <cstdint>

#ifdef __HIPCC__
#define IBP_HD __host__ __device__ __forceinline__
#else
#define IBP_HD inline
#endif

namespace ibp {
namespace dev {

inline constexpr int kWave = 64;
inline constexpr int kWavesPerBlock = 4;
inline constexpr int kBlock = kWave * kWavesPerBlock;

// Blocks of one launch: a grid's threads are counted in 32 bits, and one of 2^32 or more runs
// short without an error. A launcher halves a call that has more (in_halves).
inline constexpr uint64_t kMaxBlocks = 0xFFFFFFFFull / kBlock;

// kMaxBlocks, or less while the library was loaded with the environment variable
// IBP_TEST_MAX_BLOCKS set: a test hook, with which small calls take several launches too.
uint64_t max_blocks();

// Whether a call of n rows has to be halved: its launch would have too many blocks.
inline bool too_many_blocks(uint64_t blocks, uint64_t n) { return blocks > max_blocks() && n > 1; }

// A call of n rows as two: part(first row, rows) for each half, to the first that fails.
template <class Part>
auto in_halves(uint64_t n, const Part &part) -> decltype(part(n, n)) {
    const uint64_t h = n / 2;
    const auto e = part(0, h);
    return e != decltype(e){} ? e : part(h, n - h);
}

// An optional array from its i-th element on.
template <class T>
T *from(T *p, uint64_t i) {
    return p ? p + i : nullptr;
}

inline uint64_t blocks_of_waves(uint64_t waves) { return (waves + kWavesPerBlock - 1) / kWavesPerBlock; }

// The slices (at most `rows` rows of one cluster each) that hold rows [first, first + n): only
// those, whatever the clusters' nominal size, so that n bounds their number.
struct RowSlices {
    uint64_t g0;          // first cluster
    uint32_t rows;        // rows per slice
    uint32_t per_group;   // slices of a whole cluster
    uint32_t skip;        // slices of the first cluster before the range
    uint64_t count;
};

// Rows [first, first + n) as the places of the first and the last in their clusters.
// n >= 1, G >= 1.
struct RowRange {
    uint64_t g0, g1;       // clusters
    uint32_t row0, row1;   // rows inside them
};

inline RowRange row_range(uint64_t first, uint64_t n, uint32_t G) {
    const uint64_t last = first + n - 1, g0 = first / G, g1 = last / G;
    return {g0, g1, (uint32_t)(first - g0 * G), (uint32_t)(last - g1 * G)};
}

// rows >= 1.
inline RowSlices row_slices(const RowRange &r, uint32_t G, uint32_t rows) {
    RowSlices u;
    u.g0 = r.g0;
    u.rows = rows;
    u.per_group = (G - 1) / rows + 1;
    u.skip = r.row0 / rows;
    u.count = (r.g1 - r.g0) * u.per_group + r.row1 / rows - u.skip + 1;
    return u;
}

// Cluster and slice of unit i (below count, and below 2^32: one launch has fewer waves).
IBP_HD void slice_of(const RowSlices &u, uint32_t i, uint64_t &group, uint32_t &slice) {
    const uint32_t head = u.per_group - u.skip;
    if (i < head) {
        group = u.g0;
        slice = u.skip + i;
    } else {
        const uint32_t q = (i - head) / u.per_group;
        group = u.g0 + 1 + q;
        slice = i - head - q * u.per_group;
    }
}

// The slices of a contiguous decompress of rows of W words, each decoded by `tiles` waves of K
// words per lane. A slice repeats its cluster's setup, so it should hold many rows; but many
// rows per wave leave few waves, whose loads have to hide one another's latency. So a slice is
// a whole cluster (at most 64 rows), halved in whole batches while the launch has too few waves.
// Measured, us:
//   W <= 32  the setup weighs most (a row is little work): down to 16 rows for 16k waves, to 8
//            for 4k. 134 MB out of 64-B rows 110 with 8 rows, 78 with 16, 65 with 32; of
//            128-B rows 55, 41 and 38; 31k rows of 128 B 4.3 with 8 and 4.7 with 32
//   W <= 48  16 rows for 8k waves, else 8: 134 MB out of 160-B rows 46, 40 and 43 with 8, 16, 32
//   W <= 64  8 rows: 524k rows of 256 B 40.5, 42.4 with 32
//   W <= 128 8 rows for 2k waves, else 4: 134 MB out of 400-B rows 38 with 4, 34.5 with 8, 38
//            with 16; 5k rows 3.6 with 4 and 3.75 with 8
//   tiles    down to 4 rows for 16k waves (50k rows of 600 words 45.4, 47.9 for 32k waves)
// From pinned host memory neighbouring rows share the lines that a wave reads over PCIe: 16k
// waves at any width but 13 to 64 words, there 512 (20,000 rows of 256 B 79.8 us in slices
// of 8 rows and 71.9 in whole clusters of 32, 93,750 rows 334 and 325; 20,000 of 128 B 46.4 and
// 40.7; 2,000 rows of 256 B 11.9 in 8 and 12.7 in 32). A few rows of up to 12 words fit one line
// as it is: bf16 rows of 32 B, 163,840 of them 98.8 in 8 rows and 104.5 in 32; of 40 B, 131,072
// 97.3 and 100.1; of 48 B 96.5 and 98.9; but of 56 B 58.3 and 55.3 (56,173 rows).
inline RowSlices decompress_slices(uint64_t first, uint64_t n, uint32_t G, uint32_t W, int K, uint32_t tiles,
                                   bool host) {
    const uint32_t batch = K == 1 ? 8 : (K == 2 ? 4 : (K == 4 ? 2 : 1));
    const RowRange range = row_range(first, n, G);
    uint32_t rows = std::min<uint32_t>(G, 64);
    auto few = [&](uint32_t r, uint64_t waves) { return row_slices(range, G, r).count * tiles < waves; };
    auto halve = [&](uint32_t least, uint64_t waves) {
        if (rows > least && few(least, waves)) rows = least;   // (a small call: no steps to it)
        while (rows > least && few(rows, waves)) rows = ((rows + 1) / 2 + batch - 1) / batch * batch;
    };
    if (host || tiles > 1) {
        halve(batch, host && K == 1 && W > 12 ? 512 : 16384);
    } else if (W <= 32) {
        halve(16, 16384);
        halve(8, 4096);
    } else if (W <= 48) {
        rows = std::min(rows, 16u);
        halve(8, 8192);
    } else if (W <= 64) {
        rows = std::min(rows, 8u);
    } else {
        rows = std::min(rows, 8u);
        halve(4, 2048);
    }
    return row_slices(range, G, rows);
}

// The waves of a kernel that takes a stream's clusters in strides of the grid: one per cluster,
// up to what fills the chip many times over.
inline uint64_t cluster_blocks(uint64_t n_groups) {
    return std::min<uint64_t>(blocks_of_waves(n_groups), 1u << 18);
}

}  // namespace dev
}  // namespace ibp
