"""The compressor's two row packers (bit extraction, and run by run on CPUs without it) give
the oracle's stream, byte for byte: odd and even word counts, rows of no variant bits and of
all of them, widths whose packed bits end on and around the 64-bit accumulator's edge."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2605_30728_amd as ibp
from workloads import structured_rows

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_30728_amd", "csrc")


@pytest.fixture(scope="module")
def by_runs(tmp_path_factory):
    """The host half of the library built without bit extraction."""
    so = str(tmp_path_factory.mktemp("pack") / "host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-DIBP_NO_BMI2", f"-I{os.path.join(ROOT, 'include')}",
                    f"-I{CSRC}", os.path.join(CSRC, "ibp_host.cpp"), "-o", so, "-lpthread"], check=True)
    lib = ctypes.CDLL(so)
    lib.ibp_compress.argtypes = ibp._SIGS["ibp_compress"]

    def compress(rows, G):
        n, L = rows.shape
        out = np.zeros(64 + (n // G + 1) * (2 * L + 8) + n * L + 8, np.uint8)
        got = ctypes.c_uint64(0)
        assert lib.ibp_compress(rows.ctypes.data, n, L, G, 3, out.ctypes.data, out.size, ctypes.byref(got)) == 0
        return out[:got.value]
    return compress


@pytest.mark.parametrize("W", [1, 2, 3, 4, 7, 8, 31, 64, 65, 100, 127])
def test_both_packers_match_the_oracle(by_runs, W):
    rng = np.random.default_rng(W)
    for kind in ("random", "floats", "alternating", "identical", "ones", "onebit", "specials", "sparse"):
        rows = structured_rows(kind, 41, 4 * W, seed=W)
        for G in (1, 2, 16, 41):
            want = oracle.compress(rows, G)
            assert np.array_equal(ibp.ibp_compress(rows, G), want), (kind, G)
            assert np.array_equal(by_runs(rows, G), want), (kind, G)
    for variant in (0, 1, 31, 32, 33, 63, 64, 65, 127, 128):   # variant bits of a row, at random places
        if variant > 32 * W:
            continue
        bits = np.zeros(32 * W, np.uint8)
        bits[rng.permutation(32 * W)[:variant]] = 1
        mask = np.packbits(bits, bitorder="little")
        rows = rng.integers(0, 256, size=(40, 4 * W), dtype=np.uint8) & mask
        rows[0], rows[1] = 0, mask          # every chosen bit does vary
        want = oracle.compress(rows, 40)
        assert np.array_equal(ibp.ibp_compress(rows, 40), want), variant
        assert np.array_equal(by_runs(rows, 40), want), variant
