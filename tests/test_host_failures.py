"""The host side of the entry points that share pinned memory with kernels, when the HIP runtime reports errors: built
with the host compiler over a stand-in of the runtime (tests/cpp/fake_hip) and run through every failing call."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_memory_of_kernels_in_flight_is_left_alone(tmp_path):
    exe = tmp_path / "host_failures"
    cpp = os.path.join(ROOT, "tests", "cpp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-subobject-linkage", "-I", os.path.join(cpp, "fake_hip"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2603_08453_amd", "csrc"),
                    "-x", "c++", os.path.join(cpp, "host_failures.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout + out.stderr
    assert int(out.stdout.split()[1]) >= 100
