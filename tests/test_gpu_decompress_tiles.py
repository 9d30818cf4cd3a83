"""GPU parity of the contiguous decompress where its split of the rows can go wrong: rows of
several 128-word tiles (one word to either side of a boundary) from device memory and from a
stage, whole rows from pinned host memory, clusters whose rows are not whole batches, ranges
that start and end inside clusters, and enough rows that a wave takes more than one batch.
Expected rows are the rows themselves (the scheme is lossless), compressed by the CPU oracle;
exact."""
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


def check(torch, h, rows, first, n):
    L = rows.shape[1]
    out = torch.full((n * L + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    ibp.ibp_decompress(h, first, n, out, out_cap=n * L)
    torch.cuda.synchronize()
    got = out[:n * L].cpu().numpy().reshape(n, L)
    assert np.array_equal(got, rows[first:first + n]), (first, n, np.flatnonzero((got != rows[first:first + n]).any(1))[:8])
    assert (out[n * L:].cpu().numpy() == 0xA5).all(), "wrote past the output"


@pytest.mark.parametrize("placement", sorted(FLAGS))
@pytest.mark.parametrize("G", [1, 13, 32, 200])
@pytest.mark.parametrize("W", [63, 64, 65, 128, 129, 255, 256, 257, 384, 385, 512, 513, 641])
def test_tiles_and_ranges(torch, W, G, placement):
    n = 147
    print(f"[decompress tiles] W={W} G={G} {placement}", file=sys.stderr, flush=True)
    for kind in ("floats", "specials", "alternating", "identical", "random"):   # 0 runs to 16, and all bits
        rows = structured_rows(kind, n, 4 * W, seed=W)
        with ibp.ibp_open(oracle.compress(rows, G), 0, FLAGS[placement]) as h:
            for first, count in ((0, n), (5, n - 5), (12, 1), (31, 34), (n - 1, 1)):
                check(torch, h, rows, first, count)


@pytest.mark.parametrize("W,n,G", [(40, 300000, 100), (64, 140001, 24), (96, 90001, 40), (200, 40003, 64)])
def test_many_batches_per_wave(torch, W, n, G):
    """Launches with enough waves that slices keep several batches and a rest."""
    rows = structured_rows("floats", n, 4 * W, seed=W)
    with ibp.ibp_open(ibp.ibp_compress(rows, G), 0) as h:
        check(torch, h, rows, 0, n)
        check(torch, h, rows, 17, n - 40)


@pytest.mark.parametrize("placement", sorted(FLAGS))
@pytest.mark.parametrize("W", [20, 100, 256, 1000, 2048])
@pytest.mark.parametrize("G", [1 << 29, 1 << 31, (1 << 32) - 1])
def test_one_mask_for_everything(torch, W, G, placement):
    """A nominal cluster far larger than the table (one Mask for all rows): a launch's blocks
    follow from the rows of the range."""
    n = 300
    rows = structured_rows("floats", n, 4 * W, seed=W)
    with ibp.ibp_open(ibp.ibp_compress(rows, G), 0, FLAGS[placement]) as h:
        for first, count in ((0, n), (7, 200), (n - 1, 1)):
            check(torch, h, rows, first, count)
