"""GPU parity of the gathers that read word-order metadata slots (payload or stage in device
memory, or rows of at most 128 words in place in host memory), at the sizes where their tiling can go wrong: one, two and four words per lane and
rows of several 256-word tiles, one word to either side of each boundary; slots of 8 and 16
pairs (8 and 4 items per wave); words of one, two, three, four and more runs of variant bits,
mixed within one wave; batches that end inside a wave; ids outside the table. Expected rows
are the rows themselves (the scheme is lossless), compressed by the CPU oracle; exact."""
import sys

import numpy as np
import pytest

import oracle
import paper_2605_30728_amd as ibp

pytestmark = pytest.mark.gpu

# masks of the invariant bits of a word, by the runs of variant bits they leave
RUNS = {0: 0xFFFFFFFF, 1: 0xFF80007F, 2: 0x7F00FFFF, 3: 0x0F0FF0FF, 4: 0xF00FF00F, 5: 0x33333FFF, 16: 0x55555555,
        32: 0x00000000}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    ibp.lib()
    return t


def rows_of_runs(W, n, G, kinds, seed):
    """n rows of W words; cluster c's words cycle through the masks of kinds[c % len(kinds)]."""
    rng = np.random.default_rng(seed)
    out = np.empty((n, W), np.uint32)
    for c in range((n + G - 1) // G):
        r0, r1 = c * G, min(n, c * G + G)
        masks = np.array([RUNS[k] for k in kinds[c % len(kinds)]], np.uint32)[np.arange(W) % len(kinds[c % len(kinds)])]
        value = rng.integers(0, 1 << 32, size=len(masks), dtype=np.uint64).astype(np.uint32)
        value = value[np.arange(W) % len(kinds[c % len(kinds)])]    # few distinct (Mask, Bitval) pairs
        noise = rng.integers(0, 1 << 32, size=(r1 - r0, W), dtype=np.uint64).astype(np.uint32)
        if r1 - r0 < G:
            noise[:] = 0                       # few rows would agree on random bits
        out[r0:r1] = (value & masks) | (noise & ~masks)
    return out.view(np.uint8).reshape(n, 4 * W)


KINDS = {"two": [(1,), (2, 0, 1), (0,)],                      # up to two runs, and rows of no bits
         "four": [(1, 2), (3, 1), (4, 2, 0), (2,)],           # three and four in some items
         "any": [(1,), (5, 2), (16, 32, 3), (32,)]}           # the holes deposit in some items


@pytest.mark.parametrize("placement", ["device_ids", "host_ids", "staged"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("W", [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 768, 769, 1025])
def test_word_order_slots(torch, W, kind, placement):
    G = 40                                     # noise bits then vary in every cluster
    n = G * len(KINDS[kind]) * 2 + 3           # a ragged last cluster
    L = 4 * W
    rows = rows_of_runs(W, n, G, KINDS[kind], seed=W)
    stream = oracle.compress(rows, G)
    rng = np.random.default_rng(W)
    flags = ibp.IBP_OPEN_PAYLOAD_HOST if placement == "staged" else ibp.IBP_OPEN_PAYLOAD_DEVICE
    print(f"[gather tiles] W={W} {kind} {placement}", file=sys.stderr, flush=True)
    with ibp.ibp_open(stream, 0, flags) as h:
        k = 1 if W <= 64 else 2 if W <= 128 else 4 * ((W + 255) // 256)
        assert ibp.ibp_get_stats(h)["gather_meta_bytes"] == (8 * 8 + 32 * k + 127) // 128 * 128
        for count in (1, 5, 8, 9, 3 * n):      # inside a wave, a whole one, one past it
            ids = rng.integers(0, n, size=count).astype(np.int64)
            ids[-1] = n - 1
            out = torch.full((count * L + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            if placement == "device_ids":
                bad = rng.random(count) < 0.1
                sent = np.where(bad, np.where(rng.random(count) < 0.5, -1 - ids, n + ids), ids)
                ibp.ibp_gather_decompress_device(h, torch.from_numpy(sent).cuda(), out, out_cap=count * L)
            else:
                bad = np.zeros(count, bool)
                ibp.ibp_gather_decompress(h, ids, out, out_cap=count * L)
            torch.cuda.synchronize()
            got = out[:count * L].cpu().numpy().reshape(count, L)
            want = rows[ids].copy()
            want[bad] = 0
            assert np.array_equal(got, want), (count, np.flatnonzero((got != want).any(1))[:8])
            assert (out[count * L:].cpu().numpy() == 0xA5).all(), "wrote past the output"
            assert ibp.ibp_device_errors(h) == bad.sum()


@pytest.mark.parametrize("W", [48, 100, 200, 600])
def test_sixteen_pairs(torch, W):
    """Slots of 16 pairs: four items per wave, and a cluster of exactly 16."""
    G, n = 32, 32 * 9 + 1
    rng = np.random.default_rng(W)
    masks = np.array([RUNS[k] for k in (1, 2, 3, 4)], np.uint32)
    rows = np.empty((n, W), np.uint32)
    for c in range(0, n, G):
        p = 1 + (c // G * 7) % 16 if c else 16
        m = masks[np.arange(p) % 4]
        v = np.arange(p, dtype=np.uint32) * np.uint32(0x11111111)
        m = m | np.uint32(0xF) if p > 4 else m
        pat = np.arange(W) % p
        noise = rng.integers(0, 1 << 32, size=(min(G, n - c), W), dtype=np.uint64).astype(np.uint32)
        rows[c:c + G] = (v & m)[pat] | (noise & ~m[pat])
    rows[-1] = 0
    L = 4 * W
    rows = rows.view(np.uint8).reshape(n, L)
    ids = rng.integers(0, n, size=2001).astype(np.int64)
    with ibp.ibp_open(oracle.compress(rows, G), 0) as h:
        k = 1 if W <= 64 else 2 if W <= 128 else 4 * ((W + 255) // 256)
        assert ibp.ibp_get_stats(h)["gather_meta_bytes"] == (8 * 16 + 32 * k + 127) // 128 * 128
        out = torch.empty(ids.size * L, dtype=torch.uint8, device="cuda")
        ibp.ibp_gather_decompress_device(h, torch.from_numpy(ids).cuda(), out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().reshape(-1, L), rows[ids])


def test_host_ids_in_place_and_copied(torch):
    """Host ids read in their pinned slot (at most 65,536) or copied to the device first, in
    calls that follow one another without a wait, so that each slot is taken again while
    earlier calls may still read it."""
    n, L, G = 5000, 64, 32
    rows = rows_of_runs(L // 4, n, G, KINDS["two"], seed=5)
    rng = np.random.default_rng(5)
    counts = [3, 65536, 65537, 1, 40000, 65535, 70000, 8, 9]
    with ibp.ibp_open(oracle.compress(rows, G), 0) as h:
        calls = []
        for c in counts:
            ids = rng.integers(0, n, size=c).astype(np.int64)
            out = torch.empty(c * L, dtype=torch.uint8, device="cuda")
            sent = ids.copy()
            ibp.ibp_gather_decompress(h, sent, out)
            sent[:] = -1                       # read before the call returned
            calls.append((ids, out))
        torch.cuda.synchronize()
        for ids, out in calls:
            assert np.array_equal(out.cpu().numpy().reshape(-1, L), rows[ids]), ids.size


@pytest.mark.parametrize("placement", ["zero_copy", "zero_copy_aligned", "cache"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("W", [1, 2, 31, 63, 64, 65, 127, 128, 129, 200])
def test_host_memory_in_place(torch, W, kind, placement):
    """The same gather with the packed rows in pinned host memory (rows of at most 128 words;
    wider ones take the row-at-a-time kernel), and behind the row cache: hits, misses and ids
    outside the table mixed within a wave, and counted."""
    G = 40
    n, L = G * len(KINDS[kind]) * 2 + 3, 4 * W
    rows = rows_of_runs(W, n, G, KINDS[kind], seed=W + 1)
    rng = np.random.default_rng(W)
    flags = (ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY_ALIGNED if placement == "zero_copy_aligned"
             else ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY)
    with ibp.ibp_open(oracle.compress(rows, G), 0, flags) as h:
        held = rng.permutation(n)[:n // 3]
        cache = ibp.ibp_cache_create(h, held) if placement == "cache" else None
        for count in (1, 8, 9, 2 * n + 1):
            ids = rng.integers(0, n, size=count).astype(np.int64)
            bad = rng.random(count) < 0.1
            sent = torch.from_numpy(np.where(bad, np.where(ids % 2, -1 - ids, n + ids), ids)).cuda()
            out = torch.full((count * L + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            if cache is not None:
                ibp.ibp_cache_reset_stats(cache)
                ibp.ibp_cache_gather(cache, sent, out, out_cap=count * L)
                st = ibp.ibp_cache_get_stats(cache)
                hits = int(np.isin(ids[~bad], held).sum())
                assert (st["hits"], st["misses"]) == (hits, int((~bad).sum()) - hits)
            else:
                ibp.ibp_gather_decompress_device(h, sent, out, out_cap=count * L)
            torch.cuda.synchronize()
            want = rows[ids].copy()
            want[bad] = 0
            assert np.array_equal(out[:count * L].cpu().numpy().reshape(count, L), want), count
            assert (out[count * L:].cpu().numpy() == 0xA5).all(), "wrote past the output"
            assert ibp.ibp_device_errors(h) == bad.sum()
        if cache is not None:
            ibp.ibp_cache_destroy(cache)


@pytest.mark.parametrize("W", [20, 100, 200, 600])
def test_output_at_any_byte(torch, W):
    """An output that starts off a word boundary (a view into a larger buffer): every kernel
    that stores through a descriptor over its output row, and not a byte beside the output."""
    G = 40
    n, L = G * 6 + 3, 4 * W
    rows = rows_of_runs(W, n, G, KINDS["any"], seed=W + 2)
    ids = np.random.default_rng(W).integers(0, n, size=301).astype(np.int64)
    d_ids = torch.from_numpy(ids).cuda()
    clustered, one_mask = oracle.compress(rows, G), oracle.compress(rows, n, chunk_bytes=4, threshold=(4, 5))

    def check(call, want):
        for at in (1, 2, 3):
            buf = torch.full((want.size + 256,), 0xA5, dtype=torch.uint8, device="cuda")
            call(buf[64 + at:64 + at + want.size])
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            assert np.array_equal(got[64 + at:64 + at + want.size], want.reshape(-1)), at
            assert (got[:64 + at] == 0xA5).all() and (got[64 + at + want.size:] == 0xA5).all(), at

    for stream in (clustered, one_mask):
        for flags in (ibp.IBP_OPEN_PAYLOAD_DEVICE, ibp.IBP_OPEN_PAYLOAD_HOST, ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY):
            with ibp.ibp_open(stream, 0, flags) as h:
                check(lambda o: ibp.ibp_decompress(h, 3, n - 3, o), rows[3:])
                check(lambda o: ibp.ibp_gather_decompress(h, ids, o), rows[ids])
    if W <= 512:
        with ibp.ibp_open(clustered, 0, ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY) as h:
            cache = ibp.ibp_cache_create(h, np.arange(0, n, 3))
            check(lambda o: ibp.ibp_cache_gather(cache, d_ids, o), rows[ids])
            ibp.ibp_cache_destroy(cache)


def test_more_rows_than_one_launch(torch):
    """At 8 rows per wave, 2^29 rows are 2^32 threads, one more than a launch may have."""
    n, G, count = 4000, 32, (1 << 29) + 5
    if torch.cuda.mem_get_info()[0] < 16 << 30:
        pytest.skip("needs 16 GB of device memory")
    rows = rows_of_runs(1, n, G, KINDS["two"], seed=6)
    table = torch.from_numpy(rows.view(np.int32).reshape(-1).copy()).cuda()
    with ibp.ibp_open(oracle.compress(rows, G), 0) as h:
        ids = torch.randint(0, n, (count,), device="cuda")
        out = torch.zeros(count, dtype=torch.int32, device="cuda")
        ibp.ibp_gather_decompress_device(h, ids, out)
        torch.cuda.synchronize()
        for lo in range(0, count, 1 << 27):
            assert torch.equal(out[lo:lo + (1 << 27)], table[ids[lo:lo + (1 << 27)]]), lo


def test_more_clusters_than_one_launch(torch):
    """At a wave per cluster, 2^26 clusters are 2^32 threads: the clusters' places in the
    payload have to be there for the last ones too."""
    n = (1 << 27) + 9
    if torch.cuda.mem_get_info()[0] < 32 << 30:
        pytest.skip("needs 32 GB of device memory")
    rows = np.random.default_rng(7).integers(0, 1 << 32, size=n, dtype=np.uint32)
    ids = np.concatenate([np.random.default_rng(8).integers(0, n, size=4000), np.arange(n - 900, n)]).astype(np.int64)
    with ibp.ibp_open(ibp.ibp_compress(rows.view(np.uint8).reshape(n, 4), 2), 0) as h:
        out = torch.empty(ids.size, dtype=torch.int32, device="cuda")
        ibp.ibp_gather_decompress_device(h, torch.from_numpy(ids).cuda(), out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), rows[ids])


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("W,where", [(1, "device"), (64, "device"), (65, "device"), (128, "device"), (129, "device"),
                                     (256, "device"), (257, "device"), (1025, "device"), (64, "zero_copy"),
                                     (65, "zero_copy"), (128, "zero_copy"), (33, "cache"), (100, "cache")])
def test_small_and_large_calls(torch, W, kind, where):
    """The two lane counts per item under slots of 8 pairs and the two sizes of a block, to either
    side of both lines (4,096 and 16,384 items), with ids outside the table among the last."""
    G, L = 40, 4 * W
    n = G * len(KINDS[kind]) * 3 + 3
    rows = rows_of_runs(W, n, G, KINDS[kind], seed=W + 7)
    rng = np.random.default_rng(W)
    tiles = (W + 255) // 256
    flags = ibp.IBP_OPEN_PAYLOAD_DEVICE if where == "device" else ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY
    print(f"[gather tiles] small and large W={W} {kind} {where}", file=sys.stderr, flush=True)
    with ibp.ibp_open(oracle.compress(rows, G), 0, flags) as h:
        cache = ibp.ibp_cache_create(h, rng.permutation(n)[:n // 2].astype(np.int64)) if where == "cache" else None
        call = (lambda i, o, c: ibp.ibp_cache_gather(cache, i, o, out_cap=c)) if cache else \
            (lambda i, o, c: ibp.ibp_gather_decompress_device(h, i, o, out_cap=c))
        total = 0
        for items in (4096, 4100, 16384, 16393):
            count = -(-items // tiles)
            ids = rng.integers(0, n, size=count).astype(np.int64)
            sent = ids.copy()
            sent[-7:-3] = (-1, n, 1 << 40, -(1 << 40))
            out = torch.full((count * L + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            call(torch.from_numpy(sent).cuda(), out, count * L)
            torch.cuda.synchronize()
            want = rows[ids].copy()
            want[-7:-3] = 0
            got = out[:count * L].cpu().numpy().reshape(count, L)
            assert np.array_equal(got, want), (count, np.flatnonzero((got != want).any(1))[:8])
            assert (out[count * L:].cpu().numpy() == 0xA5).all(), "wrote past the output"
            total += 4
        assert cache or ibp.ibp_device_errors(h) == total
        if cache:
            ibp.ibp_cache_destroy(cache)
