"""How much the idle compute units of an attention launch read ahead (csrc/read_ahead.h, plain C++), on the CPU."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_30010_amd", "csrc")

SHIM = """
#include "read_ahead.h"
extern "C" void ahead(const uint32_t *bytes, int idle, int tiles, uint32_t *out, int *same_ptr) {
  et::WarmRanges w;
  for (int i = 0; i < 4; ++i) { w.ptr[i] = bytes + i; w.bytes[i] = bytes[i]; }
  const et::WarmRanges r = et::read_ahead_of(w, idle, tiles);
  *same_ptr = 1;
  for (int i = 0; i < 4; ++i) { out[i] = r.bytes[i]; *same_ptr &= !out[i] || r.ptr[i] == w.ptr[i]; }
}
"""


@pytest.fixture(scope="module")
def ahead(tmp_path_factory):
    d = tmp_path_factory.mktemp("read_ahead")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    fn = C.CDLL(lib).ahead

    def call(ranges, idle, tiles):
        out, same = (C.c_uint32 * 4)(), C.c_int(0)
        fn((C.c_uint32 * 4)(*ranges), idle, tiles, out, C.byref(same))
        assert same.value
        return list(out)
    return call


def test_a_unit_reads_no_more_than_fits_beside_the_attention(ahead):
    rng = random.Random(2)
    block = lambda d, m: [2 * d * d, 2 * d * m, 2 * d * m, 6 * d * d]
    cases = [(block(1152, 4352), i, t) for i in (0, 1, 15, 16, 32, 40, 48, 64, 112, 224) for t in (1, 2, 3, 6)]
    cases += [(block(64 * rng.randint(1, 64), 64 * rng.randint(1, 256)), rng.randint(-300, 255), rng.randint(1, 12)) for _ in range(3000)]
    cases += [(block(768, 3072)[:3] + [0], i, 1) for i in (16, 64, 200)]                     # the last block: nothing behind it
    for ranges, idle, tiles in cases:
        got = ahead(ranges, idle, tiles)
        assert all(g <= r and g % 16 == 0 for g, r in zip(got, ranges)), (ranges, idle, tiles, got)
        short = next((i for i in range(4) if got[i] < ranges[i]), 4)
        assert not any(got[short + 1:]), (ranges, idle, tiles, got)                          # in the order of use
        limit = 768 if tiles >= 3 else 512
        if idle < 16:
            assert sum(got) == 0
        elif sum(ranges) <= idle * 1024 * limit:
            assert got == ranges
        else:
            assert sum(got) == min(sum(ranges), idle * 1024 * 192)


def test_read_ahead_at_measured_sizes(ahead):
    block = [2654208, 10027008, 10027008, 7962624]                   # a width of 1152, an MLP of 4352
    assert ahead(block, 64, 1) == ahead(block, 64, 3) == block       # 16 heads, 1 x 729, 4 x 169, 2 x 361
    assert ahead(block, 40, 3) == block                              # 12 heads of 96, 6 x 361
    assert sum(ahead(block, 40, 1)) == 40 * 196608                   # 18 heads, 6 x 100: all of it costs more than it gives
    assert ahead(block, 16, 3) == [2654208, 491520, 0, 0]            # 16 heads, 5 x 361: the block took 122 us instead of 104
