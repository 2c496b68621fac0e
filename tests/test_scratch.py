"""Scratch growth of the reverse mode where the device has little room, on the host (scratch_logic.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_reverse_mode_takes_fewer_segments_when_memory_is_short(tmp_path):
    exe = tmp_path / "scratch_logic"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2501_19042_amd", "csrc"), "-o", str(exe),
                    os.path.join(ROOT, "tests", "scratch_logic.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip().splitlines()[-1] == "0", r.stdout
