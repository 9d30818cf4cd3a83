"""How calls are shared out over launches, on the CPU: the arithmetic of ibp_grid.hpp, built
with the host compiler. Every row of a range lies in exactly one unit, and a launch's blocks
follow from the rows asked for, not from the clusters' nominal size (a grid of 2^32 threads or
more runs short without an error)."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_30728_amd", "csrc")
SHIM = r"""
#include "ibp_grid.hpp"
using namespace ibp::dev;
extern "C" {
uint64_t max_blocks() { return kMaxBlocks; }
uint64_t decompress_blocks(uint64_t first, uint64_t n, uint32_t G, uint32_t W, int K, uint32_t tiles, int host) {
    return blocks_of_waves(decompress_slices(first, n, G, W, K, tiles, host).count * tiles);
}
uint64_t cluster_grid(uint64_t n_groups) { return cluster_blocks(n_groups); }
uint64_t slices(uint64_t first, uint64_t n, uint32_t G, uint32_t rows) { return row_slices(row_range(first, n, G), G, rows).count; }
uint64_t decompress_rows(uint64_t first, uint64_t n, uint32_t G, uint32_t W, int K, uint32_t tiles, int host) {
    return decompress_slices(first, n, G, W, K, tiles, host).rows;
}
// first row of unit i, which ends at the slice's, the cluster's or the range's end
uint64_t unit_row(uint64_t first, uint64_t n, uint32_t G, uint32_t rows, uint32_t i) {
    const RowSlices u = row_slices(row_range(first, n, G), G, rows);
    uint64_t g; uint32_t s;
    slice_of(u, i, g, s);
    return g * G + (uint64_t)s * rows;
}
}
"""


@pytest.fixture(scope="module")
def grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "grid.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "shim.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    u64, u32, i32 = ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int
    for name, args in {"max_blocks": [], "cluster_grid": [u64], "decompress_blocks": [u64, u64, u32, u32, i32, u32, i32], "slices": [u64, u64, u32, u32],
                       "decompress_rows": [u64, u64, u32, u32, i32, u32, i32], "unit_row": [u64, u64, u32, u32, u32]}.items():
        getattr(lib, name).argtypes = args
        getattr(lib, name).restype = u64
    return lib


def test_units_cover_a_range_once(grid):
    rng = random.Random(1)
    for _ in range(3000):
        G = rng.choice([1, 2, 7, 8, 32, 63, 64, 65, 200, 1000, 1 << 29, 0xFFFFFFFF, rng.randint(1, 300)])
        rows = min(G, rng.choice([1, 2, 4, 8, 16, 33, 64]))
        first = rng.choice([0, rng.randint(0, 500), rng.randint(0, 1 << 36)])
        n = rng.randint(1, 400)
        count, at = grid.slices(first, n, G, rows), first
        assert count <= n
        for i in range(count):
            lo = grid.unit_row(first, n, G, rows, i)
            hi = min(lo + rows, (lo // G + 1) * G, first + n)
            assert max(lo, first) == at < hi, (first, n, G, rows, i)
            at = hi
        assert at == first + n, (first, n, G, rows)


@pytest.mark.parametrize("host", [0, 1])
@pytest.mark.parametrize("W", [16, 100, 256, 1024, 2048])
@pytest.mark.parametrize("G", [1 << 20, 1 << 28, 1 << 29, 1 << 31, (1 << 32) - 1])
def test_decompress_blocks_follow_the_rows(grid, W, G, host):
    K, tiles = (1, 1) if W <= 64 else (2, 1) if W <= 128 else (4 if W <= 256 else 8, 1) if host else (2, (W + 127) // 128)
    for first, n in ((0, 1000), (5, 900), (0, 1), (999, 1), (0, 50_000_000)):
        blocks = grid.decompress_blocks(first, n, G, W, K, tiles, host)
        rows = grid.decompress_rows(first, n, G, W, K, tiles, host)
        assert 1 <= blocks <= ((n - 1) // rows + 2) * tiles // 4 + 1, (first, n, rows)
    # halving a call reaches one launch's blocks, wherever a whole table starts
    n = 1 << 36
    while grid.decompress_blocks(3, n, G, W, K, tiles, host) > grid.max_blocks():
        n //= 2
    assert n >= 1 << 20


@pytest.mark.parametrize("W,n,rows", [(16, 2_000_000, 32), (16, 300_000, 16), (16, 30_000, 8), (32, 1_000_000, 32),
                                      (32, 200_000, 16), (32, 60_000, 8), (33, 1_000_000, 16), (48, 1_000_000, 16),
                                      (48, 100_000, 8), (49, 1_000_000, 8), (64, 3_000, 8), (65, 20_000, 8),
                                      (128, 300_000, 8), (128, 10_000, 4)])
def test_narrow_rows_keep_their_setup(grid, W, n, rows):
    """Rows per slice of a payload in device memory: a narrow row is too little work to repeat
    its cluster's setup every 8 rows, except where whole clusters leave few waves."""
    assert grid.decompress_rows(0, n, 32, W, 1 if W <= 64 else 2, 1, 0) == rows


@pytest.mark.parametrize("W,n,rows", [(1, 100_000, 8), (12, 100_000, 8), (12, 1_000_000, 32), (13, 100_000, 32),
                                      (13, 10_000, 16), (64, 100_000, 32), (65, 20_000, 4)])
def test_rows_in_host_memory_share_their_lines(grid, W, n, rows):
    assert grid.decompress_rows(0, n, 32, W, 1 if W <= 64 else 2, 1, 1) == rows


@pytest.mark.parametrize("n", [1, 4, 5, 1 << 20, (1 << 26) - 1, 1 << 26, (1 << 26) + 1, 1 << 33])
def test_cluster_grid_is_bounded(grid, n):
    assert 1 <= grid.cluster_grid(n) <= min((n + 3) // 4, grid.max_blocks())
