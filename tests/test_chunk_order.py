"""The scheduling order of chunks (longest remaining chain first, equal ones in their order), on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_longest_first_matches_a_stable_sort(tmp_path):
    exe, src = str(tmp_path / "sort_check"), os.path.join(ROOT, "paper_2205_03251_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", src, "-o", exe, os.path.join(ROOT, "tests", "csrc", "sort_check.cpp"),
                           os.path.join(src, "prep.cpp"), "-lpthread"])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.split()[0] == "224"
