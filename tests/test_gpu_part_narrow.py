"""GPU parity of thresholded-scheme rows of at most 128 words at the sizes where their decode
can go wrong: one and two words per lane to either side of a boundary, chunks of 1 to W words
(one, two and four participation dwords, and chunks that end inside a lane's two words), one
Mask and per-cluster Masks (batches of one cluster and of several), rows stored raw, calls
that end inside a batch and take one or two batches per wave, ids outside the table. Expected
rows are the rows themselves (the scheme is lossless), compressed by the CPU oracle; exact."""
import sys

import numpy as np
import pytest

import oracle
import paper_2605_30728_amd as ibp
from workloads import structured_rows

pytestmark = pytest.mark.gpu

FLAGS = {"device": ibp.IBP_OPEN_PAYLOAD_DEVICE, "staged": ibp.IBP_OPEN_PAYLOAD_HOST,
         "zero_copy": ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    ibp.lib()
    return t


def take(torch, call, n, L):
    out = torch.full((n * L + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    call(out)
    torch.cuda.synchronize()
    assert (out[n * L:].cpu().numpy() == 0xA5).all(), "wrote past the output"
    return out[:n * L].cpu().numpy().reshape(n, L)


@pytest.mark.parametrize("placement", sorted(FLAGS))
@pytest.mark.parametrize("W,m", [(1, 1), (3, 1), (32, 1), (33, 1), (64, 1), (64, 2), (65, 1), (66, 3), (96, 1), (97, 1),
                                 (100, 2), (126, 7), (127, 127), (128, 1), (128, 2), (128, 4)])
def test_narrow_rows(torch, W, m, placement):
    n, L = 83, 4 * W
    print(f"[part narrow] W={W} m={m} {placement}", file=sys.stderr, flush=True)
    for kind in ("floats", "sparse", "random", "identical", "specials"):
        rows = structured_rows(kind, n, L, seed=W)
        for G in (9, 1000):
            stream = oracle.compress(rows, G, chunk_bytes=4 * m, threshold=(4, 5))
            rng = np.random.default_rng(W * G)
            with ibp.ibp_open(stream, 0, FLAGS[placement]) as h:
                for first, count in ((0, n), (7, 33), (n - 1, 1)):
                    got = take(torch, lambda o: ibp.ibp_decompress(h, first, count, o, out_cap=count * L), count, L)
                    assert np.array_equal(got, rows[first:first + count]), (kind, G, first, count)
                ids = np.concatenate([rng.integers(0, n, size=60), np.sort(rng.integers(0, n, size=41))]).astype(np.int64)
                if placement == "staged":
                    got = take(torch, lambda o: ibp.ibp_gather_decompress(h, ids, o, out_cap=ids.size * L), ids.size, L)
                    assert np.array_equal(got, rows[ids]), (kind, G)
                    continue
                bad = rng.random(ids.size) < 0.1
                d_ids = torch.from_numpy(np.where(bad, np.where(ids % 2, -1 - ids, n + ids), ids)).cuda()
                got = take(torch, lambda o: ibp.ibp_gather_decompress_device(h, d_ids, o, out_cap=ids.size * L), ids.size, L)
                want = rows[ids].copy()
                want[bad] = 0
                assert np.array_equal(got, want), (kind, G)
                assert ibp.ibp_device_errors(h) == bad.sum()


@pytest.mark.parametrize("G", [40, 1 << 20])
@pytest.mark.parametrize("W", [20, 64, 100])
def test_two_batches_per_wave(torch, W, G):
    """Calls large enough for two batches per wave, ending inside the second, and the largest
    that take one."""
    L = 4 * W
    edge = 131072 if W <= 64 else 32768
    n = edge + 5
    rows = structured_rows("floats", n, L, seed=W)
    stream = ibp.ibp_compress_ex(rows, G, 4, (4, 5))
    ids = np.random.default_rng(W).integers(0, n, size=n).astype(np.int64)
    with ibp.ibp_open(stream, 0) as h:
        for count in (edge - 1, edge, n):
            got = take(torch, lambda o: ibp.ibp_decompress(h, n - count, count, o, out_cap=count * L), count, L)
            assert np.array_equal(got, rows[n - count:]), count
            got = take(torch, lambda o: ibp.ibp_gather_decompress(h, ids[:count], o, out_cap=count * L), count, L)
            assert np.array_equal(got, rows[ids[:count]]), count


@pytest.mark.parametrize("G", [40, 1 << 20])
@pytest.mark.parametrize("placement", sorted(FLAGS))
@pytest.mark.parametrize("W,m", [(20, 1), (64, 2), (100, 1), (100, 2)])
def test_blocks_of_one_wave(torch, W, m, placement, G):
    """The most rows whose waves are a block each (1,024 waves) and the fewest whose are not; from
    host memory under per-cluster Masks half as many rows per wave at one word per lane."""
    L = 4 * W
    rows = structured_rows("floats", 8201, L, seed=W)
    stream = ibp.ibp_compress_ex(rows, G, 4 * m, (4, 5))
    rng = np.random.default_rng(W)
    with ibp.ibp_open(stream, 0, FLAGS[placement]) as h:
        for count in (4096, 4097, 8192, 8201):
            got = take(torch, lambda o: ibp.ibp_decompress(h, 8201 - count, count, o, out_cap=count * L), count, L)
            assert np.array_equal(got, rows[8201 - count:]), count
            ids = rng.integers(0, 8201, size=count).astype(np.int64)
            got = take(torch, lambda o: ibp.ibp_gather_decompress(h, ids, o, out_cap=count * L), count, L)
            assert np.array_equal(got, rows[ids]), count
