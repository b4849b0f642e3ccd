"""Host logic of the static executor: whose turn it is (a header that sgprs_pool_run_static includes),
driven on the CPU over pools of 1..9 partitions, gates 0..9 and 1..100 rounds."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_turns_keep_the_gate_and_starve_nobody(tmp_path):
    exe = str(tmp_path / "static_turns_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2406_09425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "static_turns_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr
    assert int(r.stdout.split()[1]) == 9 * 10 * 8
