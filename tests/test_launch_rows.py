"""Launches of more workgroups than one dimension holds (2^32 threads), on
the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_in_rows(tmp_path):
    exe = str(tmp_path / "rows")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-o", exe,
                    "-I", os.path.join(ROOT, "paper_2210_04847_amd", "csrc"),
                    os.path.join(ROOT, "tests", "launch_rows.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
