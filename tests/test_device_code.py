"""What the compiled kernels have to keep to and no run shows: wait states behind instructions in asm blocks, which the compiler does not see.  The sources are
compiled to assembly here as the library is built."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_21302_amd import build as B

_ASSEMBLY = {}


def assembly(source, tmp_path_factory):
    """{kernel: its lines of instructions and labels} of a source."""
    if shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc is not installed")
    if source not in _ASSEMBLY:
        out = tmp_path_factory.mktemp("asm") / "k.s"
        subprocess.run([B.HIPCC, *B.FLAGS, *B.FLAGS_OF.get(source, []), "--cuda-device-only", "-S", os.path.join(B.CSRC, source), "-o", out],
                       check=True, capture_output=True)
        kernels, name = {}, None
        for line in out.read_text().splitlines():
            line = line.split(";")[0].strip()
            m = re.fullmatch(r"(_Z\w+):", line)
            if m: name = m[1]
            if line.startswith(".end_amdhsa_kernel") or line.startswith(".section"): name = None
            if name and (re.match(r"[a-z]", line) or re.fullmatch(r"\.L\w+:", line)): kernels.setdefault(name, []).append(line)
        _ASSEMBLY[source] = kernels
    return _ASSEMBLY[source]


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


def test_wide_stores_keep_their_data(tmp_path_factory):
    """First the rule above on stores that are overwritten too early and on ones that are not."""
    store = "global_store_dwordx4 v207, v[138:141], s[16:17] nt"
    for between, bad in (([], 1), (["s_nop 0"], 1), (["s_add_u32 s0, s0, s1"], 1), (["s_nop 1"], 0), (["s_nop 0", "s_add_u32 s0, s0, s1"], 0)):
        assert len(overwritten_stores([store, *between, "v_add_u32_e32 v138, s42, v208"])) == bad
        assert len(overwritten_stores([store, *between, "v_mfma_f32_16x16x128_f8f6f4 v[140:143], v[0:5], a[30:35], 0"])) == bad
    assert not overwritten_stores([store, "v_add_u32_e32 v142, s42, v138"])
    kernels = assembly("gemm_resident_1024_wide.hip", tmp_path_factory)
    assert kernels and sum("store_dwordx4" in l for k in kernels.values() for l in k) >= 8
    assert not [(k, *s) for k, lines in kernels.items() for s in overwritten_stores(lines)]
