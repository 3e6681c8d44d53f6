"""What the launchers check of their argument blocks before they launch anything (host code): the first launch of a call holds
a fixed number of arrays to clear, and one more is refused instead of being written past the end; the gradient GEMM
stores rows by eights."""
import os
import shutil
import subprocess

import pytest

from paper_2605_28396_amd import binding
from tests import host_program

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_one_array_too_many_is_refused(tmp_path):
    exe = str(tmp_path / "setup_args")
    lib = os.path.dirname(binding.LIB_PATH)
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2605_28396_amd", "csrc"),
                        os.path.join(ROOT, "tests", "setup_args_main.cpp"), binding.LIB_PATH,
                        "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                        f"-Wl,-rpath,{lib}:{os.path.join(ROCM, 'lib')}", "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "kept refused", (r.returncode, r.stdout, r.stderr)


def test_gradient_rows_that_are_no_multiple_of_eight_are_refused(tmp_path):
    status, out = host_program.run(tmp_path, "grad_args_main", link=True)
    assert status == 0 and out.strip() == "refused", (status, out)
