"""fp32 drift bounds of the FP64 solve and of the reverse sweep over many iterations, on the host (drift_logic.cpp)."""
import os
import subprocess

from paper_2501_19042_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_drift_bounds_hold_over_many_steps(tmp_path):
    exe = tmp_path / "drift_logic"
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-o", str(exe),
                    os.path.join(ROOT, "tests", "drift_logic.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip().splitlines()[-1] == "0", r.stdout
