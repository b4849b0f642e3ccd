"""The bf16 stem kernel writes its MFMAs as inline assembly, which the compiler's hazard recogniser does not look into.
What the source relies on is checked in the assembly: between the last MFMA that writes a register and whatever else touches it
lie two more MFMAs or the fence of wait states, around the loops too; operands come from LDS; what an inline maximum reads from
the lane before was not written by the two instructions in front of it; nothing is spilled; and the waits for input rows are those
that the source counts."""
import os
import re
import subprocess

from paper_2406_09425_amd import build

from test_ksplit_assembly_cpu import instructions, registers

KERNEL = re.compile(r"^_ZN5sgprs23stem_pool_packed_kernel\w+:.*?^\.Lfunc_end", re.S | re.M)
MFMA = re.compile(r"v_mfma_f32_32x32x16_bf16 (v\[\d+:\d+\]), (a\[\d+:\d+\]), (a\[\d+:\d+\]), (?:0|\1)$")


def unrolled(text):
    """The text with each loop's body once more behind its end, inner loops first."""
    lines = text.split("\n")
    i = 0
    while i < len(lines):
        m = re.match(r"\s+s_c?branch\w* (\.LBB\w+)", lines[i])
        head = [k for k, l in enumerate(lines[:i]) if m and l.startswith(m[1] + ":")]
        if head:
            body = [l for l in lines[head[0] + 1:i]]
            lines[i:i + 1] = [l for l in body if not l.startswith(".LBB")]
            i = head[0] + 1 + 2 * len(body)
        else:
            i += 1
    return "\n".join(lines)


def check(text):
    """Number of inline MFMAs in the order of the text."""
    count, fence, written, loaded, recent = 0, 0, {}, {}, [set(), set()]
    for inline, t in instructions(text):
        name, _, operands = t.partition(" ")
        if inline and name.endswith("_dpp"):
            assert not registers(operands.partition(",")[2]) & (recent[0] | recent[1]), t
        recent = [recent[1], registers(operands.partition(",")[0]) if name.startswith("v_") and not name.startswith("v_mfma") else set()]
        if inline and name.startswith("v_mfma"):
            m = MFMA.match(t)
            assert m, t  # starts from zero or accumulates in place
            for r in registers(m[2], "a") | registers(m[3], "a"):
                assert loaded[r].startswith("ds_read"), (t, loaded[r])
            written.update(dict.fromkeys(registers(m[1]), count))
            count += 1
        elif inline and t == "s_nop 15":
            fence += 1
            if fence % 2 == 0:
                written.clear()
        else:
            for r in registers(operands) & written.keys():
                assert count - 1 - written[r] >= 2, (t, count, written[r])
        if name.startswith(("v_accvgpr_write", "ds_read", "buffer_load")):
            loaded.update(dict.fromkeys(registers(operands.split(",")[0], "a"), t))
    return count


def test_inline_mfmas_and_counted_waits(tmp_path):
    out = str(tmp_path / "stem_pool.s")
    subprocess.run([build.hipcc()] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S",
                   os.path.join(build.CSRC, "stem_pool.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        text, = KERNEL.findall(f.read())
    assert check(text) == 6 * 22                         # two of the first row, four of the loop over row pairs
    assert check(unrolled(text)) > 10 * 22
    assert "scratch_" not in text and "v_accvgpr" not in text
    waits = re.findall(r"s_waitcnt vmcnt\((\d+)\)(.*)", text)
    assert sorted(waits) == [("0", "")] * 2 + [("0", " expcnt(0) lgkmcnt(0)"), ("6", ""), ("6", ""), ("9", "")], waits


def test_the_check_sees_what_it_looks_for():
    mfma = lambda d: f"\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 v[{d}:{d + 15}], a[0:3], a[4:7], 0\n\t;;#ASMEND\n"
    load, use = "\tds_read_b128 a[0:3], v99\n\tds_read_b128 a[4:7], v99\n", "\tv_add_f32_e32 v98, v97, v3\n"
    assert check(load + mfma(0) + mfma(16) + mfma(32) + use) == 3
    shifted = "\t;;#ASMSTART\n\tv_max_f32_dpp v96, v98, v98 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t;;#ASMEND\n"
    assert check(use + "\ts_add_u32 s0, s0, s1\n" * 2 + shifted) == 0
    loop = load + ".LBB0_1:\n" + mfma(0) + mfma(16) + mfma(32) + "\ts_cbranch_scc1 .LBB0_1\n" + mfma(16) + use
    assert unrolled(loop).count("v_mfma") == 7 and check(unrolled(loop)) == 7
    for bad in (load + mfma(0) + mfma(16) + use, load + use + mfma(0) + mfma(16) + "\tv_accvgpr_write_b32 a1, v3\n" + mfma(32),
                unrolled(load + ".LBB0_1:\n" + use + mfma(16) + mfma(0) + "\ts_cbranch_scc1 .LBB0_1\n"), use + "\ts_add_u32 s0, s0, s1\n" + shifted):
        try:
            check(bad)
        except (AssertionError, KeyError):
            continue
        raise RuntimeError("not seen: " + bad)
