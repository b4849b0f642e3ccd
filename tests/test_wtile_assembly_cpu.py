"""The kernel whose weights go from the L2 to registers writes its MFMAs as inline assembly, which the compiler's
hazard recogniser does not look into.  What the source relies on is checked in the assembly this compiler makes
of it: after an MFMA nothing touches an accumulator register before the fence of 16 wait states, and what wrote
an MFMA's operands last is a load, never a vector instruction that it would have to keep a distance from."""
import os
import re
import subprocess

import pytest

from paper_2406_09425_amd import build

from test_ksplit_assembly_cpu import instructions, registers

KERNEL = re.compile(r"^(_ZN5sgprs20conv3x3_wtile_kernel\w+):.*?^\.Lfunc_end", re.S | re.M)
MFMA = re.compile(r"v_mfma_f32_16x16x32_bf16 a\[(\d+):(\d+)\], (v\[\d+:\d+\]), (v\[\d+:\d+\]), (0|a\[(\d+):(\d+)\])$")


def check(text):
    """Number of inline MFMAs."""
    code = list(instructions(text))
    accumulators = set().union(*(registers(t.split(",")[0], "a") for inline, t in code if inline and t.startswith("v_mfma")))
    count, fenced, writer = 0, True, {}
    for inline, t in code:
        name, _, operands = t.partition(" ")
        if inline and name == "v_mfma_f32_16x16x32_bf16":
            m = MFMA.match(t)
            assert m and (m[5] == "0" or (m[1], m[2]) == (m[6], m[7])), t  # starts from zero or accumulates in place
            for r in registers(m[3]) | registers(m[4]):
                assert writer.get(r, "ds_read").startswith(("ds_read", "buffer_load")), (t, writer[r])
            count, fenced = count + 1, False
        elif inline and t == "s_nop 15":
            fenced = True
        elif registers(operands, "a") & accumulators:
            assert fenced, t
        if not inline and name.startswith(("v_", "ds_read", "buffer_load", "global_load")):
            writer.update(dict.fromkeys(registers(operands.split(",")[0]), t))
    return count


def test_inline_mfmas_keep_their_distance(tmp_path):
    out = str(tmp_path / "conv_wtile.s")
    subprocess.run([build.hipcc()] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S",
                   os.path.join(build.CSRC, "conv_wtile.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        kernels = {m.group(1): m.group(0) for m in KERNEL.finditer(f.read())}
    assert len(kernels) == 3                                     # 1, 2 or 4 wavefronts share a tile
    for name, text in kernels.items():
        assert check(text) == 2 * 18 * 28, name                  # the first chunk of an item and the others
        assert "scratch_" not in text, name                      # a spill to memory would join the counted loads


def test_the_check_sees_what_it_looks_for():
    mfma = ";;#ASMSTART\nv_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3]\n;;#ASMEND"
    fence = ";;#ASMSTART\ns_nop 15\n;;#ASMEND"
    ok = "v_add_u32_e32 v1, v2, v3\nds_read_b128 v[8:11], v1\ns_waitcnt lgkmcnt(0)\nv_accvgpr_write_b32 a9, v7"
    assert check("\n".join([ok, mfma, ok, mfma, fence, "v_accvgpr_read_b32 v1, a0"])) == 2
    for bad in ("v_accvgpr_read_b32 v1, a0", "v_accvgpr_mov_b32 a4, a1", "v_mov_b32_e32 v9, v3"):
        with pytest.raises(AssertionError):
            check("\n".join([mfma, bad, mfma, fence]))
