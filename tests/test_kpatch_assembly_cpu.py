"""The kernel that keeps a tile's pixels in LDS waits for them by counting what was requested after them: the
weights' second half and the epilogue's operands.  The compiler may merge, move or sink the latter; that
it emits as many as the source counts, between the last pixel request and the barrier, is checked here, and
that the planner keeps the kernel to bf16 launches of at most one tile per CU."""
import os
import re
import subprocess

import pytest

import paper_2406_09425_amd as S
from paper_2406_09425_amd import build

KERNEL = re.compile(r"^_ZN5sgprs21conv3x3_kpatch_kernelILi(\d)ELi(\d)ELi(\d)E\w+:.*?^\.Lfunc_end", re.S | re.M)


def test_operands_that_the_pixel_wait_counts(tmp_path):
    out = str(tmp_path / "conv_kpatch.s")
    subprocess.run([build.hipcc()] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S",
                   os.path.join(build.CSRC, "conv_kpatch.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        kernels = {tuple(map(int, m.groups())): m.group(0) for m in KERNEL.finditer(f.read())}
    assert len(kernels) == 5
    for (tm, tn, h), text in kernels.items():
        lines = [t.strip() for t in text.split("\n")]
        assert not any(t.startswith(("scratch_", "flat_")) for t in lines)
        operands = [i for i, t in enumerate(lines) if re.match(r"(global|buffer)_load", t) and " lds" not in t]
        assert len(operands) == 2 + -(-(16 * tm * 4 * tn) // 512), (tm, tn, h)
        barrier = next(i for i, t in enumerate(lines) if t == "s_barrier")
        # the pixels' loop, and the weights' second half behind it, lie before the operands (rare branches of
        # the weights' requests are placed behind the kernel's end and jump back before them)
        loop = max(i for i, t in enumerate(lines[:operands[0]]) if t.startswith("buffer_load") and " lds" in t)
        assert loop < operands[0] and operands[-1] < barrier
        between = lines[operands[0]:operands[-1]]
        assert not any(t.startswith(("s_cbranch", "s_branch", ".LBB")) for t in between)
        waits = [int(m[1]) for t in lines[operands[-1]:barrier] for m in [re.match(r"s_waitcnt vmcnt\((\d+)\)", t)] if m]
        assert max(waits) == h * 2 * tn + len(operands)


TILE = [(16, 16), (32, 16), (32, 32), (64, 32), (64, 64)]  # output pixels, channels


@pytest.mark.parametrize("h,c", [(56, 64), (28, 128), (14, 256), (7, 512)])
@pytest.mark.parametrize("n", [1, 2, 3, 8])
def test_planner_takes_it_for_one_tile_per_cu(n, h, c):
    for cus in (8, 32, 64, 128, 256):
        family, detail = S.sgprs_conv2d_plan(S.ConvDesc(n, h, h, c, c, 3, 3, 1, 1, S.SGPRS_BF16, 1), cus)
        if family == 0 and detail >= 16:
            pixels, channels = TILE[detail - 16]
            assert -(-n * h * h // pixels) * (c // channels) <= cus
        for d in (S.ConvDesc(n, h, h, c, c, 3, 3, 1, 1, S.SGPRS_F32, 1), S.ConvDesc(n, h, h, c, c, 3, 3, 2, 1, S.SGPRS_BF16, 1),
                  S.ConvDesc(n, h, h, c, c, 1, 1, 1, 0, S.SGPRS_BF16, 1)):
            family, detail = S.sgprs_conv2d_plan(d, cus)
            assert family != 0 or detail < 16
    if (n, h) == (1, 7):  # 49 pixels, 2 x 32 tiles
        assert S.sgprs_conv2d_plan(S.ConvDesc(1, 7, 7, 512, 512, 3, 3, 1, 1, S.SGPRS_BF16, 1), 64) == (0, 17)


@pytest.mark.parametrize("n,h,w,cout,cus", [(3, 24, 15, 64, 248), (2, 12, 14, 192, 224), (8, 5, 6, 64, 32)])
def test_planner_leaves_it_where_a_share_ends_inside_a_half(n, h, w, cout, cus):
    """384 channels are 54 k-tiles, 7 in a wavefront's share, 3 in half a ring."""
    assert S.sgprs_conv2d_plan(S.ConvDesc(n, h, w, 384, cout, 3, 3, 1, 1, S.SGPRS_BF16, 1), cus, True) != (0, 17)
