"""A cluster that keeps its centroid while that is being posted (csrc/lc_rounds_planes.h), played through on the host by a small C++
program: no order of the wavefronts posts a word that is not the standing centroid's, and the orders drawn are ones that one plane
number to a cluster does not survive."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_standing_centroid_in_any_order(tmp_path):
    exe = tmp_path / "rounds_planes_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_08453_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "rounds_planes_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout + out.stderr
    orders, faults = map(int, out.stdout.split()[1:])
    assert orders == 20000 and faults > 0
