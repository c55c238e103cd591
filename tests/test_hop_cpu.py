"""The stopping rule of the pointer-doubling loops (csrc/hop.hpp, host and
device code) on the CPU: valid lists are ranked, and lanes end within a bounded
number of hops whatever the records hold. Cases in tests/hop_mock.cpp, compiled
here with g++."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_lane_ends(tmp_path):
    exe = str(tmp_path / "hop_mock")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2606_09318_amd", "csrc"),
                    os.path.join(ROOT, "tests", "hop_mock.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
