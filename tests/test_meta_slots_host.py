"""The metadata slots' host builder on the CPU: it allocates nothing on the pool's threads (an
exception there would end the process, not the call), whatever the rows' width, and tells pairs
of one 32-bit tag apart."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_30728_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <new>
#include "ibp_internal.hpp"

static thread_local bool caller = false;
static bool failing = false;
void *operator new(std::size_t n) {   // no memory for any thread but the caller's
    if (failing && !caller) throw std::bad_alloc();
    if (void *p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main(int argc, char **argv) {
    caller = true;
    const uint32_t W = (uint32_t)std::atoi(argv[1]);
    const bool word_order = argv[2][0] == '1';
    const bool tagged = argv[3][0] == '1';   // every pair's tag is 0
    const uint64_t groups = 64;
    std::vector<uint32_t> meta(groups * 2 * W);
    for (uint64_t g = 0; g < groups; ++g)
        for (uint32_t w = 0; w < W; ++w) meta[(2 * g) * W + w] = w % 11, meta[(2 * g + 1) * W + w] = tagged ? (w % 11) * 0x9E3779B1u : 0;
    ibp::Pool pool(4);
    std::vector<uint8_t> slots;
    failing = true;
    const uint32_t P = ibp::build_meta_slots(reinterpret_cast<const uint8_t *>(meta.data()), groups, W,
                                             W <= 64 ? 1 : 8, pool, slots, word_order);
    failing = false;
    if (P != 16) return 1;
    const uint64_t S = slots.size() / groups;
    for (uint64_t g = 0; g < groups; ++g)
        for (uint32_t w = 0; w < W; ++w) {
            const uint64_t at = word_order ? w : (uint64_t)(W <= 64 ? 1 : 8) * (w % 64) + w / 64;
            if (slots[g * S + 8 * (w % 11)] != w % 11) return 3;
            if (((slots[g * S + 8 * P + at / 2] >> (4 * (at % 2))) & 15) != w % 11) return 2;
        }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", str(d / "main.cpp"),
                    *(os.path.join(CSRC, f) for f in ("ibp_meta_slots.cpp", "ibp_pool.cpp", "ibp_host.cpp")),
                    "-o", str(d / "slots"), "-lpthread"], check=True)
    return str(d / "slots")


@pytest.mark.parametrize("tagged", [0, 1])
@pytest.mark.parametrize("W,word_order", [(11, 0), (64, 1), (500, 0), (512, 1), (513, 1), (20_000, 1)])
def test_no_memory_on_the_pool_threads(program, W, word_order, tagged):
    assert subprocess.run([program, str(W), str(word_order), str(tagged)]).returncode == 0
