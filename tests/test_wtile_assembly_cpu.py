"""The kernel whose weights go from the L2 to registers writes its MFMAs as inline assembly, which the compiler's
hazard recogniser does not look into.  What the source relies on is checked in the assembly this compiler makes
of it: after an MFMA nothing touches an accumulator register before the fence of 16 wait states, and what wrote
an MFMA's operands last is a load, never a vector instruction that it would have to keep a distance from.  The waits
for a patch count the weights requested after it: that the compiler leaves that many loads behind the patch's last
request, and nothing of the patch's behind them, is checked here too."""
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


def patch_waits(text):
    """For every wait that the source counts, the loads to registers between the last request of a patch and it."""
    counts, loads, mfmas = [], None, 0
    for line in (t.strip() for t in text.split("\n")):
        if line.startswith("buffer_load") and " lds" in line:
            loads = 0
        elif line.startswith(("buffer_load", "global_load")) and loads is not None:
            loads += 1
        elif line.startswith((".LBB", "s_cbranch", "s_branch", "s_barrier")):
            loads = loads and None  # ways part or meet among the loads: the count is not the text's
        elif re.match(r"s_waitcnt vmcnt\(20\)", line) and loads is not None:
            counts.append(loads)
            loads = None
    return counts


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
        waits = patch_waits(text)                                # before the first chunk, behind the first and the others
        assert len(waits) == 3 and waits[0] == 20 and min(waits[1:]) >= 20, (name, waits)


def test_the_check_sees_what_it_looks_for():
    mfma = ";;#ASMSTART\nv_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3]\n;;#ASMEND"
    fence = ";;#ASMSTART\ns_nop 15\n;;#ASMEND"
    ok = "v_add_u32_e32 v1, v2, v3\nds_read_b128 v[8:11], v1\ns_waitcnt lgkmcnt(0)\nv_accvgpr_write_b32 a9, v7"
    assert check("\n".join([ok, mfma, ok, mfma, fence, "v_accvgpr_read_b32 v1, a0"])) == 2
    patch, weights, wait = ["buffer_load_dwordx4 v1, s[0:3], 0 offen lds"], ["buffer_load_dwordx4 v[0:3], v1, s[0:3], 0 offen"], ["s_waitcnt vmcnt(20)"]
    assert patch_waits("\n".join(patch + weights * 20 + wait + patch + weights * 27 + wait)) == [20, 27]
    assert patch_waits("\n".join(patch + weights * 19 + wait + weights)) == [19]
    assert patch_waits("\n".join(weights * 4 + patch * 2 + weights * 16 + patch + weights * 4 + wait)) == [4]
    assert patch_waits("\n".join(patch + [".LBB0_1:"] + weights * 20 + wait)) == [20]
    assert patch_waits("\n".join(patch + weights * 10 + [".LBB0_1:"] + weights * 10 + wait)) == []
    for bad in ("v_accvgpr_read_b32 v1, a0", "v_accvgpr_mov_b32 a4, a1", "v_mov_b32_e32 v9, v3"):
        with pytest.raises(AssertionError):
            check("\n".join([mfma, bad, mfma, fence]))
