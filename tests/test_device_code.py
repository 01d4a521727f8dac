"""What the compiled kernels have to keep to and no run shows: wait states behind instructions in asm blocks, which the compiler does not see, LDS reads that
a barrier in an asm block has to wait for, and registers without scratch memory.  The sources are compiled to assembly here as the library is built."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2509_21302_amd import build as B

SOURCES = tuple(s for s in B.SOURCES if s.startswith(("gemm_resident", "gemm_e2m3")))


def _compile(source, out):
    subprocess.run([B.HIPCC, *B.FLAGS, *B.FLAGS_OF.get(source, []), "--cuda-device-only", "-S", os.path.join(B.CSRC, source), "-o", out],
                   check=True, capture_output=True)
    kernels, scratch, name = {}, {}, None
    for line in out.read_text().splitlines():
        line = line.split(";")[0].strip()
        m = re.fullmatch(r"(_Z\w+):", line)
        if m: name = m[1]
        m = re.fullmatch(r"\.amdhsa_kernel (\w+)", line)
        if m: described = m[1]
        m = re.fullmatch(r"\.amdhsa_private_segment_fixed_size (\d+)", line)
        if m: scratch[described] = int(m[1])
        if line.startswith(".section"): name = None
        if name and (re.match(r"[a-z]", line) or re.fullmatch(r"\.L\w+:", line)): kernels.setdefault(name, []).append(line)
    return kernels, scratch


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """source -> ({kernel: its lines of instructions and labels}, {kernel: bytes of scratch memory a lane}); the sources compile side by side."""
    if shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc is not installed")
    tmp = tmp_path_factory.mktemp("asm")
    with ThreadPoolExecutor(len(SOURCES)) as ex:
        return dict(zip(SOURCES, ex.map(lambda s: _compile(s, tmp / (s + ".s")), SOURCES)))


def registers(operand):
    """{("v", 3), ...} of an operand."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    return {(m[1], n) for n in range(int(m[2] or m[3]), int(m[2] or m[4]) + 1)} if m else set()


def overwritten_stores(lines):
    """Stores of more than 8 bytes whose data registers a vector instruction writes with fewer than two wait states between them."""
    bad = []
    for i, line in enumerate(lines):
        m = re.match(r"(?:global|flat|buffer|scratch)_store_(?:dwordx[34]|b96|b128)\s+(.*)", line)
        if not m: continue
        data = max((registers(o) for o in m[1].split(",")), key=len)
        states = 0
        for after in lines[i + 1:]:
            if after.endswith(":"): continue
            op, _, rest = after.partition(" ")
            if states >= 2 or op.startswith("s_branch") or op == "s_endpgm": break
            if op.startswith("v_") and data & registers(rest.split(",")[0]): bad.append((line, after))
            states += int(rest) + 1 if op == "s_nop" else 1
    return bad


def test_wide_stores_keep_their_data(assembly):
    """First the rule above on stores that are overwritten too early and on ones that are not."""
    store = "global_store_dwordx4 v207, v[138:141], s[16:17] nt"
    for between, bad in (([], 1), (["s_nop 0"], 1), (["s_add_u32 s0, s0, s1"], 1), (["s_nop 1"], 0), (["s_nop 0", "s_add_u32 s0, s0, s1"], 0)):
        assert len(overwritten_stores([store, *between, "v_add_u32_e32 v138, s42, v208"])) == bad
        assert len(overwritten_stores([store, *between, "v_mfma_f32_16x16x128_f8f6f4 v[140:143], v[0:5], a[30:35], 0"])) == bad
    assert not overwritten_stores([store, "v_add_u32_e32 v142, s42, v138"])
    kernels = assembly["gemm_resident_1024_wide.hip"][0]
    assert kernels and sum("store_dwordx4" in l for k in kernels.values() for l in k) >= 8
    assert not [(k, *s) for k, lines in kernels.items() for s in overwritten_stores(lines)]


def scales_read_across_barriers(lines, stage_bytes):
    """LDS reads of token scales (the 512 bytes behind the `stage_bytes` of tokens of a ring stage) that have not come back at a barrier: behind it another wave's transfer
    writes their place.  They come back in order, so waiting for all but n leaves the last n."""
    label = {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}
    bad = []

    def of_scales(line):
        offset = re.search(r"offset:(\d+)", line)
        return line.startswith("ds_read") and offset and int(offset[1]) % (stage_bytes + 512) >= stage_bytes

    def walk(i, flying, jumps):
        for i in range(i, len(lines)):
            op, _, rest = lines[i].partition(" ")
            if op.startswith("ds_"): flying = flying + [(i, lines[i])]
            elif op == "s_waitcnt" and "lgkmcnt" in rest:
                n = int(re.search(r"lgkmcnt\((\d+)\)", rest)[1])
                flying = flying[-n:] if n else []
            elif op == "s_barrier":
                bad.extend(r for r in flying if of_scales(r[1]))
                if not jumps: return
                flying = []
            elif op.startswith(("s_cbranch", "s_branch")):
                if jumps: walk(label[rest], flying, False)           # to the first barrier there
                if op == "s_branch":
                    if not jumps: return walk(label[rest], flying, False) if label[rest] > i else None
                    flying = []
            elif op == "s_endpgm":
                if not jumps: return
                flying = []
    walk(0, [], True)
    return sorted(set(bad))


# the sizes of one stage per step: source, arguments of the kernel's name, tokens of a step times 48 bytes times K / 64
@pytest.mark.parametrize("source,kernel,stage_bytes", [("gemm_resident_1024_wide.hip", "16ELi1ELi8ELb0", 12288), ("gemm_resident_1280_2048.hip", "20ELi1ELi4ELb0", 30720),
                                                       ("gemm_resident_affine.hip", "16ELi1ELi4ELb1", 24576)])
def test_barriers_wait_for_the_scales(assembly, source, kernel, stage_bytes):
    """First the rule above on a loop of its own."""
    loop = [".L0:", "s_waitcnt lgkmcnt(%d)", "s_barrier", "ds_read_b128 v[0:3], v9 offset:128", "ds_read_b128 v[4:7], v8 offset:12288", "ds_read_b64 v[0:1], v9 offset:32",
            "s_cbranch_scc1 .L0", "s_endpgm"]
    for n, bad in ((0, 0), (1, 0), (2, 1), (3, 1)):
        assert len(scales_read_across_barriers([l % n if "%d" in l else l for l in loop], 12288)) == bad
    kernels = [lines for name, lines in assembly[source][0].items() if "resident_gemm_kernel" in name and kernel in name]
    assert kernels
    for lines in kernels:
        assert sum("offset:%d" % stage_bytes in l for l in lines) >= 3 and sum(l == "s_barrier" for l in lines) >= 4
        assert not scales_read_across_barriers(lines, stage_bytes)


def test_no_kernel_uses_scratch_memory(assembly):
    """The weights in registers, 256 x 256 tiles and the rest of the E2M3 GEMM: several are at the last register."""
    scratch = {k: b for _, sizes in assembly.values() for k, b in sizes.items()}
    assert sum("resident_gemm_kernel" in k for k in scratch) >= 21 and sum("e2m3_256_kernel" in k for k in scratch) == 5 and sum("e2m3_gemm" in k for k in scratch) >= 20
    assert not {k: b for k, b in scratch.items() if b}
