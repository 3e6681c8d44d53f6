"""Small host programs that call the library's own functions, compiled with the library's headers."""
import os
import subprocess

from paper_2605_28396_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, name, link=False, timeout=60):
    """Compiles tests/<name>.cpp (host code only), runs it and returns its exit status and output."""
    exe = str(tmp_path / name)
    cmd = [build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-ffp-contract=off",
           "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe]
    if link:
        cmd[-2:-2] = ["-x", "none", build.LIB, "-Wl,-rpath," + os.path.dirname(build.LIB)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=timeout)
    return r.returncode, r.stdout + r.stderr
