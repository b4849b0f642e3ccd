"""The K-split convolution writes its pipelined k-loop's MFMAs as inline assembly, which the compiler's
hazard recogniser does not look into.  What the source relies on is checked in the assembly this
compiler makes of it: between the two fences around the loop nothing but those MFMAs touches an
accumulator register, and what wrote their operands last is an LDS read that has been waited for, never
a vector instruction that an MFMA would have to keep a distance from."""
import os
import re
import subprocess

import pytest

from paper_2406_09425_amd import build

KERNEL = re.compile(r"^(_ZN5sgprs18conv_ksplit_kernel\w+):.*?^\.Lfunc_end", re.S | re.M)
MFMA = re.compile(r"v_mfma_\S+ a\[(\d+):(\d+)\], (v\d+|v\[\d+:\d+\]), (v\d+|v\[\d+:\d+\]), a\[(\d+):(\d+)\]$")


def registers(text, kind="v"):
    """Numbers of the vector (v) or accumulation (a) registers that operands name: v7, a[4:7]."""
    found = set()
    for m in re.finditer(rf"\b{kind}(?:(\d+)|\[(\d+):(\d+)\])", text):
        found |= {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))
    return found


def instructions(text):
    """(written as inline assembly, instruction) in text order."""
    inline = False
    for line in text.split("\n"):
        line = line.strip()
        if line.startswith(";;#ASM"):
            inline = line.startswith(";;#ASMSTART")
        elif line and not line.startswith((";", ".")):
            yield inline, line.split(";")[0].strip()


def check(text):
    """Number of inline MFMAs of one kernel; 0 for a kernel without the pipelined loop."""
    code = list(instructions(text))
    mfmas = [i for i, (inline, t) in enumerate(code) if inline and t.startswith("v_mfma")]
    if not mfmas:
        return 0
    first = [i for i, (inline, t) in enumerate(code) if inline and t == "s_nop 7"]
    last = [i for i, (inline, t) in enumerate(code) if inline and t == "s_nop 15"]
    assert len(first) == 1 and len(last) == 2, (first, last)
    assert first[0] < mfmas[0] and mfmas[-1] < last[0]
    loop = code[first[0] + 1:last[0]]
    accumulators = set().union(*(registers(t, "a") for inline, t in loop if inline))
    writer = {}                                           # vector register -> what wrote it last
    for inline, t in loop:
        name, _, operands = t.partition(" ")
        if inline:
            m = MFMA.match(t)
            assert m and m[1] == m[5] and m[2] == m[6], t     # accumulates in place
            for r in registers(m[3]) | registers(m[4]):
                assert writer.get(r) in (None, "waited for"), (t, writer[r])
            continue
        assert not registers(operands, "a") & accumulators, t
        if name == "s_waitcnt" and "lgkmcnt(0)" in operands:
            writer = {r: "waited for" if w.startswith("ds_read") else w for r, w in writer.items()}
        if name.startswith(("v_", "ds_read")):
            writer.update(dict.fromkeys(registers(operands.split(",")[0]), t))
    return len(mfmas)


def test_inline_mfmas_keep_their_distance(tmp_path):
    out = str(tmp_path / "conv_ksplit.s")
    subprocess.run([build.hipcc()] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S",
                   os.path.join(build.CSRC, "conv_ksplit.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        kernels = {m.group(1): m.group(0) for m in KERNEL.finditer(f.read())}
    assert len(kernels) == 8 * 3                          # eight tiles: fp32 with two and four sets, bf16
    pipelined = [k for k, text in kernels.items() if check(text)]
    assert len(pipelined) == 8 * 2 + 4                    # all of fp32, the bf16 tiles of eight and more MFMAs a half k-tile


def test_the_check_sees_what_it_looks_for():
    fence = [";;#ASMSTART\ns_nop 7\n;;#ASMEND", ";;#ASMSTART\ns_nop 15\ns_nop 15\n;;#ASMEND"]
    mfma = ";;#ASMSTART\nv_mfma_f32_16x16x4_f32 a[0:3], v9, v[10:10], a[0:3]\n;;#ASMEND"
    ok = "v_mov_b32_e32 v9, v3\nds_read_b128 v[8:11], v2\ns_waitcnt lgkmcnt(0)\nv_add_u32_e32 v12, v9, v9"
    assert check("\n".join([fence[0], ok, mfma, fence[1]])) == 1
    assert check(ok) == 0
    for bad in ("v_accvgpr_read_b32 v1, a0", "v_mov_b32_e32 v9, v3", "v_accvgpr_mov_b32 a4, a0", "v_accvgpr_write_b32 a3, v1", "ds_read_b128 v[8:11], v2"):
        with pytest.raises(AssertionError):
            check("\n".join([fence[0], mfma, bad, mfma, fence[1]]))
