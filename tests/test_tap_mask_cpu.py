"""Host logic of the K-split convolution kernel: the masks of filter taps inside the image (a header
the kernel includes), checked on the CPU against their definition, wide padding included."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tap_masks_match_their_definition(tmp_path):
    exe = str(tmp_path / "tap_mask_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2406_09425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "tap_mask_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr
    assert int(r.stdout.split()[1]) > 25000
