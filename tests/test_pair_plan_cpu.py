"""Where the planner takes the stride-2 pair kernel (conv_s2tile.hip) for a bf16 task's down-sampling blocks, and where it leaves them to
the implicit GEMM: sizes at which both were timed inside the network, with inputs that change."""
import os
import subprocess

from paper_2406_09425_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BLOCK = {2: (56, 64), 3: (28, 128), 4: (14, 256)}
TILES = ((7, 1), (7, 2), (4, 1), (4, 2))

# block, images, CUs: us per launch of the implicit GEMM and of the best tile of the other kernel
SLOWER = [  # a little beyond whole rounds of items, or few items beside the chip's clock
    (2, 25, 96, 17.2, 20.5), (2, 9, 32, 17.8, 18.2), (2, 29, 96, 20.2, 22.2), (2, 34, 128, 20.0, 21.0), (2, 42, 160, 20.4, 21.6),
    (2, 51, 192, 21.1, 22.7), (2, 59, 224, 22.4, 23.7), (2, 68, 256, 23.3, 24.8), (2, 77, 256, 24.5, 25.4),
    (3, 22, 64, 20.3, 21.8), (3, 24, 64, 20.9, 22.3), (3, 36, 96, 22.2, 23.9), (3, 44, 128, 22.0, 23.7), (3, 87, 256, 23.4, 24.8)]
FASTER = [  # ... and which
    (2, 32, 128, 21.2, 17.0, (4, 1)), (2, 64, 256, 22.8, 19.6, (4, 1)), (2, 128, 256, 39.0, 37.8, (7, 1)),
    (3, 4, 32, 12.1, 11.0, (4, 2)), (3, 64, 256, 20.8, 17.8, (7, 2)), (3, 128, 256, 29.2, 26.0, (7, 1)),
    (4, 16, 64, 20.1, 14.4, (4, 2)), (4, 64, 256, 28.1, 18.6, (4, 2)), (4, 128, 256, 33.0, 25.9, (7, 2))]


def test_the_pair_kernel_is_chosen_where_it_is_faster(tmp_path):
    exe = str(tmp_path / "pair_plan_check")
    subprocess.run([build.hipcc()] + build.COMMON + [os.path.join(ROOT, "tests", "cpp", "pair_plan_check.cpp"), "-o", exe, "-L", build.PKG, "-lsgprs",
                    f"-Wl,-rpath,{build.PKG}"], check=True, capture_output=True)
    asked = "".join("%d %d %d %d\n" % (*BLOCK[c[0]], c[1], c[2]) for c in SLOWER + FASTER)
    r = subprocess.run([exe], input=asked, capture_output=True, text=True, check=True)
    plans = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    assert len(plans) == len(SLOWER) + len(FASTER)
    for case, (kind, variant) in zip(SLOWER + FASTER, plans):
        got = TILES[variant] if kind == 8 else None
        assert got == (case[5] if len(case) > 5 else None), (case, kind, variant)
