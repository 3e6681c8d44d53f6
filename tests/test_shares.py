"""Where the vocabulary strips of a sweep and the pieces of a contraction begin: the kernels form the quotients
from a factor that the host takes (host code; nothing is launched)."""
import os
import subprocess

from paper_2605_28396_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_shares_are_spread_evenly(tmp_path):
    exe = str(tmp_path / "shares")
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                        "-I", build.CSRC, os.path.join(ROOT, "tests", "shares_main.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok "), (r.returncode, r.stdout, r.stderr)
