"""The fp32 kernel on the bf16 matrix cores waits for a k-tile's pixels by counting what was requested after them: the
next k-tile's weights, 3 TN loads to registers.  That the compiler leaves them all between those pixels' requests
and the wait, in both k-tiles of a loop trip, is checked here."""
import os
import re
import subprocess

from paper_2406_09425_amd import build

KERNEL = re.compile(r"^_ZN5sgprs17conv_split_kernelILi(\d)ELi(\d)ELi(\d)E\w+:.*?^\.Lfunc_end", re.S | re.M)


def test_weights_that_the_pixel_wait_counts(tmp_path):
    out = str(tmp_path / "conv_split.s")
    subprocess.run([build.hipcc()] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-S",
                   os.path.join(build.CSRC, "conv_split.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        kernels = {tuple(map(int, m.groups())): m.group(0) for m in KERNEL.finditer(f.read())}
    assert len(kernels) == 4
    for (tm, tn, nw), text in kernels.items():
        assert "scratch_" not in text
        tiles = 0
        events = []  # since the last request of pixels, in text order: the weights
        for line in (t.strip() for t in text[:text.index("v_mfma_f32_16x16x4")].split("\n")):
            if line.startswith("buffer_load") and " lds" in line:
                events = []
            elif line.startswith("buffer_load"):
                events.append("w")
            elif re.match(rf"s_waitcnt vmcnt\({3 * tn}\) lgkmcnt\(0\)$", line):
                assert events == ["w"] * (3 * tn), (tm, tn, nw, events)
                tiles, events = tiles + 1, []
        assert tiles == 2, (tm, tn, nw)
