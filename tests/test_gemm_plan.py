"""The int8-instruction GEMM without a GPU: the plan (csrc/gemm_plan.h, compiled for the host), and what the compiler says of its kernels."""
import math
import os
import random
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21302_amd", "csrc")
DRIVER = r"""
#include "gemm_plan.h"
#include <cstdio>
int main()
{
    int M, N, K, bits, affine, dump;
    while (std::scanf("%d %d %d %d %d %d", &M, &N, &K, &bits, &affine, &dump) == 6) {
        const qvggt::GemmPlan p = qvggt::int8_instruction_gemm_plan(M, N, K, bits, affine, dump);
        std::printf("%s %d\n", p.shape == p.kBig ? "big" : p.shape == p.kSmall ? "small" : p.shape == p.kDeep ? "deep" : "big+deep", p.rows_main);
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans([(M, N, K, bits, affine, dump), ...]) -> [(shape, rows of the big tiles), ...]"""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    folder = tmp_path_factory.mktemp("gemm_plan")
    src, exe = folder / "driver.cpp", folder / "driver"
    src.write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", exe, src], check=True)

    def ask(problems):
        text = "\n".join(" ".join(str(int(v)) for v in p) for p in problems)
        lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
        assert len(lines) == len(problems)
        return [(s, int(r)) for s, r in (line.split() for line in lines)]
    return ask


# one round of 256 big tiles holds them, and one of 512 small tiles does not quite: measured 1.1 to 1.5 times slower in small tiles
@pytest.mark.parametrize("M,N,K,bits", [(9591, 896, 4096, 8), (22039, 304, 4096, 8), (6388, 1376, 2048, 8), (2247, 4256, 2048, 8), (20356, 400, 2048, 8),
                                        (9214, 1120, 1280, 8), (39144, 160, 5120, 4)])
def test_just_past_a_round_of_small_tiles(plans, M, N, K, bits):
    assert plans([(M, N, K, bits, 0, 0)]) == [("big", 0)]


# few tiles: the deep ring only where a tile's chain is long enough to pay for filling it (measured 3 to 7 % slower on the left ones)
@pytest.mark.parametrize("M,N,K,bits,affine,want", [
    (1422, 192, 512, 4, 0, "small"), (18, 768, 1024, 4, 0, "small"), (211, 144, 1536, 4, 0, "small"), (19930, 64, 256, 8, 0, "small"),
    (1600, 432, 512, 8, 0, "small"), (30, 64, 768, 8, 0, "small"), (953, 2896, 3584, 4, 0, "deep"), (125, 80, 3072, 4, 0, "small"), (68, 3456, 4096, 4, 0, "small"), (21, 16, 6144, 4, 0, "deep"), (2048, 2048, 4096, 4, 0, "deep"),
    (372, 1312, 4096, 4, 1, "deep"), (20, 464, 1024, 4, 1, "deep"), (1374, 1024, 4096, 8, 0, "deep"), (360, 3696, 1024, 8, 0, "deep")])
def test_deep_ring_needs_a_long_chain(plans, M, N, K, bits, affine, want):
    assert plans([(M, N, K, bits, affine, 0)]) == [(want, 0)]


# whole rounds in big tiles and the rest in deep ones, where that measured faster than one configuration for all rows (by 5 to 19 %)
@pytest.mark.parametrize("M,N,K,bits,affine", [(17354, 1184, 4096, 4, 0), (34003, 480, 2048, 8, 0), (46628, 736, 1024, 8, 0), (49610, 1952, 1024, 4, 0),
                                               (113324, 672, 768, 4, 0), (90930, 192, 4096, 4, 1),
                                               (4298, 4864, 3584, 4, 1)])
def test_rows_are_divided(plans, M, N, K, bits, affine):
    (shape, rows), = plans([(M, N, K, bits, affine, 0)])
    assert shape == "big+deep" and rows % 256 == 0 and 0 < rows < M


def test_deep_ring_never_with_fewer_than_four_k_tiles(plans):
    """The eight-stage ring's waits cover a tile's scales from three K-tiles on.  Rows that a plan divides are whole 256-row tiles that
    leave some over."""
    rng = random.Random(3)
    sizes = [128, 256, 384, 512, 768, 1024, 1280, 1536, 1792, 2048, 2560, 3072, 3584, 4096, 5120, 6144, 8192]
    problems = []
    for i in range(200000):
        K = rng.choice(sizes[:5] if i % 2 else sizes)
        bits = rng.choice((4, 8))
        problems.append((int(math.exp(rng.uniform(0, math.log(1 << 21)))), 16 * int(math.exp(rng.uniform(0, math.log(4096)))), K, bits,
                         bits == 4 and rng.random() < 0.3, rng.random() < 0.1))
    seen = set()
    for (M, N, K, bits, _, _), (shape, rows) in zip(problems, plans(problems)):
        if "deep" in shape:
            assert K * bits // 512 >= 4, (M, N, K, bits, shape)
        assert (rows % 256 == 0 and 0 < rows < M) if shape == "big+deep" else rows == 0
        seen.add(shape)
    assert seen == {"big", "small", "deep", "big+deep"}


def test_no_kernel_uses_scratch_memory(tmp_path):
    """Every instantiation fits its registers: a kernel that spills pays for its scratch memory in every wave's start."""
    from paper_2509_21302_amd import build as B
    if not os.path.exists(B.HIPCC) and shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc is not installed")
    r = subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(CSRC, "gemm_w4a4.hip"),
                        "-o", str(tmp_path / "gemm.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    names, scratch = re.findall(r"Function Name: (\S+)", r.stderr), re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)
    assert len(names) == len(scratch) and sum("w4a4_gemm" in n for n in names) >= 24
    assert not [n for n, b in zip(names, scratch) if int(b)]


def test_gpu_tests_reach_the_plans_they_are_named_for(plans):
    """A change of the plan must not leave a GPU test on another kernel than its table says."""
    from tests.test_gpu_asym import ASYM_PLANS
    from tests.test_gpu_gemm import ROWS_SPLIT, TILE_PLANS
    from tests.test_gpu_int8_blocks import BOTH_TILE_SHAPES
    cases = [((M, N, K, 8 if wide else 4, 0, 1), want) for M, N, K, wide, want in ROWS_SPLIT]
    cases += [((M, N, K, 4 if kind == "packed" else 8, 0, 0), want) for M, N, K, kind, want in TILE_PLANS]
    cases += [((M, N, K, 8, 0, 0), want) for M, N, K, want in BOTH_TILE_SHAPES] + [((M, N, K, 4, 1, 0), want) for M, N, K, want in ASYM_PLANS]
    for (problem, want), (shape, rows) in zip(cases, plans([c[0] for c in cases])):
        assert shape == want, (problem, shape)
        if want == "big+deep":          # the seam the tests look at
            M, N = problem[:2]
            tiles_n = (N + 255) // 256
            assert rows == ((M + 255) // 256 * tiles_n // 256 * 256 // tiles_n) * 256
    for plan in ("big", "small", "deep", "big+deep"):
        assert any(want == plan for _, _, _, want in ASYM_PLANS) and any(p[4] == plan for p in TILE_PLANS)
        assert any(p[4] == plan and p[3] == "blocks" and p[2] != 1024 for p in TILE_PLANS)       # K = 1024: registers hold the weights, but for the dump
    assert {p[3] for p in BOTH_TILE_SHAPES if p[2] != 1024} == {p[3] for p in BOTH_TILE_SHAPES}


def test_gpu_tests_reach_several_big_tiles_per_block(plans, tiles256):
    """int8 blocks: more than one tile for each of 256 blocks, none of the last ones whole, at K of either body of the tiles."""
    from tests.test_gpu_int8_blocks import BIG_TILES
    for (M, N, K, want), (shape, rows) in zip(BIG_TILES, plans([(*p[:3], 8, 0, 0) for p in BIG_TILES])):
        main = M if want == "big" else rows
        assert shape == want and K != 1024 and N % 256 and M % 128 and (main + 255) // 256 * ((N + 255) // 256) > 264, (M, N, K, shape)
    assert [t[3] for t in tiles256([(*p[:3], 0) for p in BIG_TILES])] == [p[2] >= 768 for p in BIG_TILES]
    assert {(K < 768, want) for _, _, K, want in BIG_TILES} == {(True, "big"), (False, "big"), (True, "big+deep"), (False, "big+deep")}


E2M3_DRIVER = r"""
#include "gemm_plan.h"
#include <cstdio>
int main()
{
    int M, N, K;
    const char *names[] = {"256", "192", "128", "64", "32x64", "32"};
    while (std::scanf("%d %d %d", &M, &N, &K) == 3) {
        const qvggt::E2m3Plan p = qvggt::e2m3_gemm_plan(M, N, K);
        std::printf("%s %s %d\n", names[p.shape], names[p.rest], p.rows_main);
    }
}
"""


def test_e2m3_plans(tmp_path):
    """The GPU test's table reaches the tile shapes it names; every plan of 100000 random problems is one of them, and one that divides the rows
    gives whole blocks of the operand format to the first launch and leaves some to the second."""
    from tests.test_gpu_e2m3 import E2M3_PLANS
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(E2M3_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)

    def ask(problems):
        lines = subprocess.run([tmp_path / "d"], input="\n".join("%d %d %d" % p for p in problems), capture_output=True, text=True, check=True).stdout.split()
        return [(lines[i], lines[i + 1], int(lines[i + 2])) for i in range(0, len(lines), 3)]
    for (M, N, K, want), (shape, rest, rows) in zip(E2M3_PLANS, ask([p[:3] for p in E2M3_PLANS])):
        assert (shape if rows == M else f"{shape}+{rest}") == want, (M, N, K)
    rng = random.Random(5)
    problems = [(int(math.exp(rng.uniform(0, math.log(1 << 21)))), 16 * int(math.exp(rng.uniform(0, math.log(4096)))),
                 rng.choice([128, 256, 512, 768, 1024, 1280, 1792, 2048, 3584, 4096, 6144, 8192])) for _ in range(100000)]
    divided = 0
    for (M, N, K), (shape, rest, rows) in zip(problems, ask(problems)):
        if rows != M:
            divided += 1
            assert shape == "256" and rows % 256 == 0 and 0 < rows < M
    assert divided > 100
    assert {p[3].split("+")[0] for p in E2M3_PLANS} == {"256", "192", "128", "64", "32x64", "32"}


FEW_DRIVER = r"""
#include "gemm_plan.h"
#include <cstdio>
int main()
{
    int M, N, K, bits, blocks;
    const char *names[] = {"none", "64", "32x64", "32"};
    while (std::scanf("%d %d %d %d %d", &M, &N, &K, &bits, &blocks) == 5) std::printf("%s\n", names[(int)qvggt::int8_instruction_few_tiles(M, N, K, bits, blocks)]);
}
"""


def test_few_tiles(tmp_path):
    """The GPU test's table reaches the shapes it names; no problem of more than 256 tiles of 128 x 128 is one of few."""
    from tests.test_gpu_gemm import FEW_TILES
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(FEW_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)

    def ask(problems):
        return subprocess.run([tmp_path / "d"], input="\n".join("%d %d %d %d %d" % p for p in problems), capture_output=True, text=True, check=True).stdout.split()
    bits = {"packed": (4, 0), "affine": (4, 0), "int8": (8, 0), "blocks": (8, 1)}
    for (M, N, K, kind, want), got in zip(FEW_TILES, ask([p[:3] + bits[p[3]] for p in FEW_TILES])):
        assert got == want, (M, N, K, kind)
    rng = random.Random(7)
    problems = [(int(math.exp(rng.uniform(0, math.log(1 << 21)))), 16 * int(math.exp(rng.uniform(0, math.log(4096)))), rng.choice([128, 768, 1024, 4096, 8192]),
                 *rng.choice([(4, 0), (8, 0), (8, 1)])) for _ in range(20000)]
    for (M, N, *_), got in zip(problems, ask(problems)):
        assert got == "none" or (M + 127) // 128 * ((N + 127) // 128) <= 256


# problems whose shapes were measured far enough apart to say which it has to be (with kernel 1, us, the shape that a wrong price takes / this one):
# 27.4 / 24.9, 62.6 / 56.0, 112.5 / 103.6, 73.6 / 69.8; 128s 97.6 / 192s 81.9; 192s 151.9 / 256s and a rest 142.1
@pytest.mark.parametrize("M,N,K,plan", [(6715, 3072, 1024, "128"), (13091, 4096, 1024, "128"), (50838, 1024, 1024, "128"),
                                        (10992, 1024, 4096, "192"), (21984, 1024, 4096, "192"), (32976, 1024, 4096, "256+32")])
def test_e2m3_plan_where_the_shapes_differ(tmp_path, M, N, K, plan):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(E2M3_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)
    shape, rest, rows = subprocess.run([tmp_path / "d"], input=f"{M} {N} {K}", capture_output=True, text=True, check=True).stdout.split()
    assert (shape if int(rows) == M else f"{shape}+{rest}") == plan


TILES256_DRIVER = r"""
#include "gemm_plan.h"
#include <cstdio>
using namespace qvggt;
int main()
{
    int M, N, K, shifted;
    while (std::scanf("%d %d %d %d", &M, &N, &K, &shifted) == 4) {
        const E2m3Plan p = e2m3_gemm_plan(M, N, K);
        std::printf("%d %d %d %d\n", p.shape == E2m3Plan::k256 && !e2m3_resident(M, N, K, shifted != 0), e2m3_tiles256(p.rows_main, N, K), e2m3_streams_y(p.rows_main, N),
                    i8b_tiles256(M, N, K));
    }
}
"""


@pytest.fixture(scope="module")
def tiles256(tmp_path_factory):
    """tiles256([(M, N, K, shifted), ...]) -> [(in 256-row E2M3 tiles, on the 16 x 16 instructions, Y past the caches, int8 tiles on the 16 x 16 ones), ...]"""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    tmp = tmp_path_factory.mktemp("tiles256")
    (tmp / "d.cpp").write_text(TILES256_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp / "d", tmp / "d.cpp"], check=True)

    def ask(problems):
        out = subprocess.run([tmp / "d"], input="\n".join("%d %d %d %d" % p for p in problems), capture_output=True, text=True, check=True).stdout.split()
        return [tuple(int(v) for v in out[i:i + 4]) for i in range(0, len(out), 4)]
    return ask


def test_256_row_tiles_where_the_instructions_differ(tiles256):
    """us, 32 x 32 / 16 x 16: few tiles or short K are the former's (10.7 / 12.0, 10.9 / 11.6, 16.8 / 18.0, 17.0 / 18.2; int8 13.0 / 15.2, 15.2 / 17.5), many of long K the latter's."""
    e2m3 = [(16381, 1024, 128, 0), (16381, 1024, 256, 0), (25447, 480, 1280, 0), (4102, 2912, 1536, 0), (32976, 2048, 4096, 0), (9000, 1552, 8192, 0), (137400, 1024, 4096, 0)]
    int8 = [(16381, 1024, 128, 0), (11660, 736, 768, 0), (12870, 768, 1024, 0), (32976, 1024, 4096, 0), (65550, 2048, 2048, 0), (24705, 1056, 8192, 0)]
    assert [t[1] for t in tiles256(e2m3)] == [0, 0, 0, 0, 1, 1, 1]
    assert [t[3] for t in tiles256(int8)] == [0, 0, 0, 1, 1, 1]


def test_256_row_tiles_keep_their_least_k(tiles256):
    """The ring of stages and the one set of scales of affine codes want K of 768 and more."""
    rng = random.Random(5)
    problems = [(int(math.exp(rng.uniform(0, math.log(1 << 21)))), 16 * int(math.exp(rng.uniform(0, math.log(4096)))), K, 0) for K in (128, 256, 512) for _ in range(3000)]
    assert not any(t[1] or t[3] for t in tiles256(problems))


def test_gpu_tests_reach_every_256_row_kernel(tiles256):
    """Plain codes and affine ones, without the dump: both instructions, each with both kinds of store."""
    from tests.test_gpu_e2m3 import CACHED_PLANS, CALL_PLANS, E2M3_PLANS, SHIFTED_SHORT_K, SHORT_K
    for shifted, problems in ((0, E2M3_PLANS + CACHED_PLANS + CALL_PLANS + SHORT_K), (1, CACHED_PLANS + CALL_PLANS + SHIFTED_SHORT_K)):
        assert {t[1:3] for t in tiles256([(*p[:3], shifted) for p in problems]) if t[0]} == {(0, 0), (0, 1), (1, 0), (1, 1)}
    assert all(t[0] for t in tiles256([(*p, 0) for p in SHORT_K] + [(*p, 1) for p in SHIFTED_SHORT_K]))


VARIANT_DRIVER = r"""
#include "gemm_plan.h"
#include <cstdio>
int main()
{
    int M, N, K;
    const char *names[] = {"256", "192", "128", "64", "32x64", "32"};
    while (std::scanf("%d %d %d", &M, &N, &K) == 3) {
        const qvggt::E2m3Plan p = qvggt::e2m3_gemm_plan(M, N, K);
        std::printf("%s %d %d %d %d %d\n", names[p.shape], p.rows_main, qvggt::e2m3_streams_y(p.rows_main, N),
                    qvggt::e2m3_128_tokens_first((p.rows_main + 127) / 128, (N + 127) / 128, N, K), qvggt::e2m3_resident(M, N, K, false),
                    qvggt::e2m3_resident(M, N, K, true));
    }
}
"""


def test_gpu_tests_reach_every_variant_of_the_e2m3_tiles(tmp_path):
    """Plain codes and shifted ones, as calls run them (without the dump, whose kernels are others): both kinds of store of the 256- and 192-row tiles, both
    orders of the 128-row ones, and a divided plan with either store.  What the kernel with the weights in registers takes does not count."""
    from tests.test_gpu_e2m3 import CACHED_PLANS, CALL_PLANS, E2M3_PLANS
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(VARIANT_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)

    def variants(problems, affine):
        lines = subprocess.run([tmp_path / "d"], input="\n".join("%d %d %d" % p[:3] for p in problems), capture_output=True, text=True, check=True).stdout.split()
        found = set()
        for p, shape, rows, streams, tokens, *resident in zip(problems, *(lines[i::6] for i in range(6))):
            assert shape == p[3].split("+")[0] and (int(rows) != p[0]) == ("+" in p[3]), p
            if resident[affine] == "1":
                assert p not in CALL_PLANS
                continue
            if shape in ("256", "192"):
                found.add((shape, "streams" if streams == "1" else "caches"))
            elif shape == "128":
                found.add((shape, "tokens first" if tokens == "1" else "channels first"))
            if int(rows) != p[0]:
                found.add(("divided", "streams" if streams == "1" else "caches"))
        return found
    every = {("256", "streams"), ("256", "caches"), ("192", "streams"), ("192", "caches"), ("128", "channels first"), ("128", "tokens first"),
             ("divided", "streams"), ("divided", "caches")}
    shifted = [p for p in E2M3_PLANS if p[2] in (1024, 2048, 4096) and p[0] < 12000 or "+" in p[3]]
    assert variants(E2M3_PLANS + CACHED_PLANS + CALL_PLANS, False) == every and variants(shifted + CACHED_PLANS + CALL_PLANS, True) == every


RESIDENT_DRIVER = r"""
#include "gemm_plan.h"
#include <cstdio>
int main()
{
    int M, N, K, shifted;
    while (std::scanf("%d %d %d %d", &M, &N, &K, &shifted) == 4)
        std::printf("%d %d %d\n", qvggt::e2m3_resident(M, N, K, shifted != 0), qvggt::resident_groups(N) * qvggt::resident_ranges(M, N), qvggt::i8b_resident(M, N, K));
}
"""


# problems that one kernel had measured far enough ahead to say which it has to be (us in front of a copy of the codes or behind kernel 1, tiles / weights in
# registers), most of them with rows of Y in 64-byte pieces
@pytest.mark.parametrize("M,N,K,int8,resident", [
    (2796, 4576, 1024, True, False), (3383, 3680, 1024, True, False), (5567, 2080, 1024, True, False), (6278, 1888, 1024, True, False), (9968, 1248, 1024, True, False),
    (23358, 1360, 1024, True, True), (117758, 3648, 1024, True, True), (10993, 3056, 1024, True, True),      # 63.1 / 57.3, 529 / 453
    (13740, 800, 1280, False, False), (13119, 1056, 1280, False, False), (37024, 224, 1280, False, False),   # 23.2 / 26.2, 25.4 / 27.4, 27.6 / 29.6
    (3617, 3648, 2048, False, False), (3693, 3392, 2048, False, False), (3725, 3200, 1792, False, False),       # 28.8 / 30.0, 28.7 / 29.5, 31.4 / 32.1
    (48869, 160, 1024, False, True), (23603, 288, 1024, False, True), (19952, 416, 1024, False, True),      # 47.0 / 42.8, 33.4 / 31.5, 30.3 / 28.9
    (10992, 4096, 1024, False, True), (32976, 4096, 2048, False, True), (10992, 3072, 768, False, True)])
def test_resident_weights_where_the_kernels_differ(tmp_path, M, N, K, int8, resident):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(RESIDENT_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)
    out = subprocess.run([tmp_path / "d"], input=f"{M} {N} {K} 0", capture_output=True, text=True, check=True).stdout.split()
    assert int(out[2 if int8 else 0]) == resident


def test_resident_weights_where_affine_codes_differ(tmp_path):
    """K = 2048, us behind kernel 1, tiles / weights in registers: 64.0 / 58.0, 61.7 / 54.2."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(RESIDENT_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)
    out = subprocess.run([tmp_path / "d"], input="18571 1248 2048 1\n15510 1504 2048 1", capture_output=True, text=True, check=True).stdout.split()
    assert out[::3] == ["1", "1"]


def test_resident_weights_of_128_channels_a_wave(tmp_path):
    """The GPU test's table reaches them, and its other rows do not; they come with full ranges and more of Y than goes through the caches."""
    from tests.test_gpu_e2m3 import RESIDENT, RESIDENT_WIDE
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text('#include "gemm_plan.h"\n#include <cstdio>\nint main() { int M, N; while (std::scanf("%d %d", &M, &N) == 2) '
                                    'std::printf("%d %d\\n", qvggt::resident_wide(M, N), qvggt::resident_groups(N, 8) * qvggt::resident_ranges(M, N, 8)); }\n')
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)

    def ask(problems):
        out = subprocess.run([tmp_path / "d"], input="\n".join("%d %d" % p for p in problems), capture_output=True, text=True, check=True).stdout.split()
        return [(int(out[i]), int(out[i + 1])) for i in range(0, len(out), 2)]
    assert all(wide for wide, _ in ask([p[:2] for p in RESIDENT_WIDE])) and not any(wide for wide, _ in ask([p[:2] for p in RESIDENT]))
    rng = random.Random(3)
    problems = [(int(math.exp(rng.uniform(0, math.log(1 << 21)))), 16 * int(math.exp(rng.uniform(0, math.log(8192))))) for _ in range(20000)]
    for (M, N), (wide, blocks) in zip(problems, ask(problems)):
        if wide: assert 2 * M * N > 130e6 and 224 < blocks <= 256, (M, N)


def test_resident_weights(tmp_path):
    """The GPU test's table reaches the kernel with every K it takes; no other K does, nor affine codes with those that kernel 1 does not write; the
    blocks of a launch have a compute unit each unless there are more groups of channels than that."""
    from tests.test_gpu_e2m3 import RESIDENT
    from tests.test_gpu_large_offsets import M_BIG
    from tests.test_gpu_int8_blocks import RESIDENT as INT8
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "d.cpp").write_text(RESIDENT_DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-o", tmp_path / "d", tmp_path / "d.cpp"], check=True)

    def ask(problems):
        out = subprocess.run([tmp_path / "d"], input="\n".join("%d %d %d %d" % p for p in problems), capture_output=True, text=True, check=True).stdout.split()
        return [(int(out[i]), int(out[i + 1]), int(out[i + 2])) for i in range(0, len(out), 3)]
    problems = [(*p, 0) for p in RESIDENT] + [(*p, 1) for p in RESIDENT if p[2] in (1024, 2048)]
    for p, (resident, _, _) in zip(problems, ask(problems)):
        assert resident, p
    assert {p[2] for p in RESIDENT} == {512, 768, 1024, 1280, 1536, 1792, 2048}
    assert all(int8 for _, _, int8 in ask([(*p, 1024, 0) for p in INT8]))
    assert M_BIG * 4096 > 1 << 31 and ask([(M_BIG, 4096, 512, 0)])[0][0] and ask([(M_BIG, 4096, 1024, 0)])[0][2]
    rng = random.Random(9)
    problems = [(int(math.exp(rng.uniform(0, math.log(1 << 21)))), 16 * int(math.exp(rng.uniform(0, math.log(8192)))),
                 rng.choice([128, 256, 512, 768, 1024, 1280, 1536, 1792, 2048, 2560, 3584, 4096, 6144, 8192]), rng.randrange(2)) for _ in range(20000)]
    for (M, N, K, shifted), (resident, blocks, int8) in zip(problems, ask(problems)):
        assert not resident or K in ((1024, 2048) if shifted else (512, 768, 1024, 1280, 1536, 1792, 2048))
        assert not int8 or K == 1024
        assert blocks <= max(256, (N + 255) // 256)
