"""The stride-2 pair kernel whose weights go from the L2 to registers writes its MFMAs as inline assembly and counts the
weights requested after a patch in its waits.  As for the stride-1 kernel of that kind, what the source relies on is
checked in the assembly: accumulators are left alone until the fence, an MFMA's operands come from loads, nothing
is spilled, and behind a patch's last request lie at least as many loads of weights as its wait leaves in flight."""
import os
import re
import subprocess

from paper_2406_09425_amd import build

from test_wtile_assembly_cpu import check

KERNEL = re.compile(r"^(_ZN5sgprs18conv_s2tile_kernelILi(\d)ELi(\d)E\w+):.*?^\.Lfunc_end", re.S | re.M)


def patch_waits(text, left):
    """Of every barrier behind a wait that leaves `left` requests: the loads to registers between a patch's last request and it."""
    counts, loads, waited = [], None, False
    for line in (t.strip() for t in text.split("\n")):
        if line.startswith("buffer_load") and " lds" in line:
            loads, waited = 0, False
        elif line.startswith(("buffer_load", "global_load")):
            loads, waited = None if loads is None else loads + 1, False
        elif re.match(rf"s_waitcnt vmcnt\({left}\)", line):
            waited = True
        elif line.startswith("s_barrier"):
            if waited and loads is not None:
                counts.append(loads)
            loads = None
        elif line.startswith((".LBB", "s_cbranch", "s_branch")):
            loads = loads and None  # ways part or meet among the loads: the count is not the text's
    return counts


def test_inline_mfmas_and_counted_waits(tmp_path):
    out = str(tmp_path / "conv_s2tile.s")
    subprocess.run([build.hipcc()] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S",
                   os.path.join(build.CSRC, "conv_s2tile.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        kernels = {(int(m.group(2)), int(m.group(3))): m.group(0) for m in KERNEL.finditer(f.read())}
    assert sorted(kernels) == [(4, 1), (4, 2), (7, 1), (7, 2)]
    for (tm, ks), text in kernels.items():
        assert check(text) == 2 * 10 * tm * 4, (tm, ks)          # the first stage of an item and the others
        assert "scratch_" not in text, (tm, ks)                  # a spill to memory would join the counted loads
        left = 8 if (tm, ks) == (4, 1) else 20
        waits = patch_waits(text, left)
        assert len(waits) == 2 and min(waits) >= left, (tm, ks, waits)


def test_the_count_sees_what_it_looks_for():
    patch, weights, end = ["buffer_load_dwordx4 v1, s[0:3], 0 offen lds"], ["buffer_load_dwordx4 v[0:3], v1, s[0:3], 0 offen"], ["s_waitcnt vmcnt(8)", "s_barrier"]
    assert patch_waits("\n".join(patch + weights * 9 + end + patch + weights * 4 + end), 8) == [9, 4]
    assert patch_waits("\n".join(weights * 4 + patch * 2 + weights * 3 + patch + weights * 4 + end[:1] + weights * 4 + end), 8) == [8]
    assert patch_waits("\n".join(patch + weights * 9 + end[:1] + weights + end[1:]), 8) == []
