"""Where the lanes of a 16 x 16 matrix instruction read their share of a K-step (csrc/fragments.h, compiled for the host): every code once, the same quarter of K for all
rows of a lane group, and 16-byte reads without bank conflicts.  The hardware's counters gave the order in which a read takes its lanes: with quarter q as lane group
q's own, 48 % of the LDS cycles of the int8 kernels were conflicts and 40 % of the E2M3 ones', which is what `conflicts` says of it."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21302_amd", "csrc")
DRIVER = r"""
#include "fragments.h"
#include <cstdio>
#include <initializer_list>
using namespace qvggt;
int main()
{
    for (int q = 0; q < 4; ++q) for (int c = 0; c < 16; ++c) std::printf("%d ", i8_place(c, q));
    for (int tile : {24576, 1536, 768}) for (int q = 0; q < 4; ++q) for (int c = 0; c < 16; ++c) std::printf("%d %d ", e2m3_place(c, q, tile), e2m3_place(c, q, tile) + e2m3_rest(q));
}
"""
GOES = [[*range(0, 4), *range(12, 16), *range(20, 28)], [*range(4, 12), *range(16, 20), *range(28, 32)]]       # of the lower half of a wave; the upper one alike


def conflicts(places, size):
    """Cycles that a read of a wave takes beyond those without conflicts: 64 banks of 4 bytes, 16-byte reads in four goes, 8-byte ones by halves."""
    extra = 0
    for half in (0, 32):
        for go in GOES if size == 16 else [range(32)]:
            banks = [(places[half + lane] // 4 + w) % 64 for lane in go for w in range(size // 4)]
            extra += max(banks.count(b) for b in set(banks)) - 1
    return extra


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    tmp = tmp_path_factory.mktemp("fragments")
    (tmp / "d.cpp").write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp / "d", tmp / "d.cpp"], check=True)
    v = [int(x) for x in subprocess.run([tmp / "d"], capture_output=True, text=True, check=True).stdout.split()]
    return v[:64], {tile: (v[64 + 128 * i: 192 + 128 * i: 2], v[65 + 128 * i: 192 + 128 * i: 2]) for i, tile in enumerate((24576, 1536, 768))}


def test_int8_fragments(places):
    straight = [c * 64 + ((q ^ (c >> 2)) << 4) for q in range(4) for c in range(16)]
    assert conflicts(straight, 16) == 4                      # of 8 cycles
    at, _ = places
    assert conflicts(at, 16) == 0
    assert sorted(at) == [16 * i for i in range(64)]
    for q in range(4):                                       # the chunk of row c that lies in slot s of it is s ^ (c >> 2)
        assert len({at[16 * q + c] % 64 // 16 ^ c >> 2 for c in range(16)}) == 1 and [at[16 * q + c] // 64 for c in range(16)] == list(range(16))


@pytest.mark.parametrize("tile", [24576, 1536, 768])
def test_e2m3_fragments(places, tile):
    straight = [(q >> 1) * tile + c * 48 + (q & 1) * 16 for q in range(4) for c in range(16)]
    assert (conflicts(straight, 16), conflicts([p + 32 - 8 * (i >> 4 & 1) for i, p in enumerate(straight)], 8)) == (4, 0)      # of 10 cycles
    first, rest = places[1][tile]
    assert (conflicts(first, 16), conflicts(rest, 8)) == (0, 2)                                                              # of 8
    seen = set()
    for q in range(4):
        where = {((first[16 * q + c] - 48 * c) // tile, (first[16 * q + c] - 48 * c) % tile // 16, (rest[16 * q + c] - 48 * c) % tile) for c in range(16)}
        assert len(where) == 1
        k_tile, blob, behind = where.pop()
        assert behind == 32 + 8 * blob and blob in (0, 1) and k_tile in (0, 1)
        seen.add((k_tile, blob))
    assert len(seen) == 4
