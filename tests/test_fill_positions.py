"""Output positions of the fill kernels' sample lists, on the host: the walk
over whole blocks of 64 positions up to the last one a 32-bit index can name
(2^31 - 1 samples are accepted, a list's blocks must not pass them)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lists_end_inside_the_output(tmp_path):
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-O1", "-fwrapv", "-std=c++17", "-Wall", "-Wextra", "-o", exe,
                    "-I", os.path.join(ROOT, "paper_2210_04847_amd", "csrc"),
                    os.path.join(ROOT, "tests", "fill_list_walk.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
