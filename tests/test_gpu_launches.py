"""GPU parity of calls that take several launches. A launch may have fewer than 2^32 threads,
and every launcher halves a call that asks for more; here a second copy of the library, loaded
with the limit at three blocks (IBP_TEST_MAX_BLOCKS), takes every launcher's halving at a few
hundred rows. Expected rows are the rows
themselves (the scheme is lossless); exact."""
import os
import shutil
import sys

import numpy as np
import pytest

import oracle
import paper_2605_30728_amd as ibp
from workloads import structured_rows

pytestmark = pytest.mark.gpu

DEVICE, STAGED, ZERO_COPY = (ibp.IBP_OPEN_PAYLOAD_DEVICE, ibp.IBP_OPEN_PAYLOAD_HOST,
                             ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    ibp.lib()
    return t


@pytest.fixture(scope="module")
def three_blocks(torch, tmp_path_factory):
    """The package over a copy of the library whose launches have at most three blocks."""
    copy = str(tmp_path_factory.mktemp("launches") / "libibp_three_blocks.so")
    shutil.copy(ibp.LIB_PATH, copy)
    whole, path = ibp.lib(), ibp.LIB_PATH
    os.environ["IBP_TEST_MAX_BLOCKS"] = "3"
    ibp._lib, ibp.LIB_PATH = None, copy
    try:
        ibp.lib()
        del os.environ["IBP_TEST_MAX_BLOCKS"]
        yield
    finally:
        os.environ.pop("IBP_TEST_MAX_BLOCKS", None)
        ibp._lib, ibp.LIB_PATH = whole, path


def take(torch, call, n, L):
    out = torch.full((n * L + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    call(out)
    torch.cuda.synchronize()
    assert (out[n * L:].cpu().numpy() == 0xA5).all(), "wrote past the output"
    return out[:n * L].cpu().numpy().reshape(n, L)


# "floats": clusters with metadata slots; "random": more than 16 pairs, so none
@pytest.mark.parametrize("kind", ["floats", "random"])
@pytest.mark.parametrize("flags", [DEVICE, STAGED, ZERO_COPY])
@pytest.mark.parametrize("scheme", ["clusters", "one_mask", "masks"])
@pytest.mark.parametrize("W", [20, 100, 200, 300, 600])
def test_every_launcher_in_parts(torch, three_blocks, W, scheme, flags, kind):
    n, L = 401, 4 * W
    print(f"[launches] W={W} {scheme} flags={flags} {kind}", file=sys.stderr, flush=True)
    rows = structured_rows(kind, n, L, seed=W)
    stream = (oracle.compress(rows, 24) if scheme == "clusters" else
              oracle.compress(rows, 24 if scheme == "masks" else n, chunk_bytes=8, threshold=(4, 5)))
    rng = np.random.default_rng(W)
    ids = rng.integers(0, n, size=777).astype(np.int64)
    bad = rng.random(ids.size) < 0.1
    want = rows[ids].copy()
    with ibp.ibp_open(stream, 0, flags) as h:
        for first, count in ((0, n), (5, 300)):
            got = take(torch, lambda o: ibp.ibp_decompress(h, first, count, o, out_cap=count * L), count, L)
            assert np.array_equal(got, rows[first:first + count])
        got = take(torch, lambda o: ibp.ibp_gather_decompress(h, ids, o, out_cap=ids.size * L), ids.size, L)
        assert np.array_equal(got, want)
        if flags == STAGED:
            return
        want[bad] = 0
        sent = torch.from_numpy(np.where(bad, np.where(ids % 2, -1 - ids, n + ids), ids)).cuda()
        got = take(torch, lambda o: ibp.ibp_gather_decompress_device(h, sent, o, out_cap=ids.size * L), ids.size, L)
        assert np.array_equal(got, want)
        assert ibp.ibp_device_errors(h) == bad.sum()
        if flags == ZERO_COPY and scheme == "clusters" and W <= 512:
            held = np.arange(0, n, 3)
            cache = ibp.ibp_cache_create(h, held)
            got = take(torch, lambda o: ibp.ibp_cache_gather(cache, sent, o, out_cap=ids.size * L), ids.size, L)
            assert np.array_equal(got, want)
            hits = int(np.isin(ids[~bad], held).sum())
            st = ibp.ibp_cache_get_stats(cache)
            assert (st["hits"], st["misses"]) == (hits, int((~bad).sum()) - hits)
            assert ibp.ibp_device_errors(h) == bad.sum()
            ibp.ibp_cache_destroy(cache)
