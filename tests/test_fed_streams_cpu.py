"""Host logic behind graph replay on pools of one partition: whether a thread feeds one stream or several."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_one_stream_or_several(tmp_path):
    exe = str(tmp_path / "fed_streams_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2406_09425_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "fed_streams_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
