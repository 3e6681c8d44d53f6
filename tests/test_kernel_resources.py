"""Scratch memory of the built kernels.  Every one of them is written to hold its state in registers
and LDS; a spill, or an array that the compiler puts into memory, is a cost that no parity test sees."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_28396_amd import binding

LLVM = "/opt/rocm/llvm/bin"
# bytes per lane
ALLOWED = {
    # 75 + 36 vectors of a row held in registers: four of them do not fit
    "logits_row_resident_kernelILb0EE": 20,
}


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")), reason="no ROCm LLVM tools")
def test_no_kernel_uses_scratch(tmp_path):
    lib = shutil.copy(binding.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(lib)], cwd=tmp_path, check=True,
                   capture_output=True)
    seen = {}
    for f in tmp_path.glob("lib.so.*gfx950"):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(f)], check=True,
                               capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\w+)\n.*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            seen[name] = int(size)
    assert any("grad_gemm_kernel" in n for n in seen) and any("logit_pass_dma_kernel" in n for n in seen)
    over = {n: s for n, s in seen.items() if s > max([b for k, b in ALLOWED.items() if k in n], default=0)}
    assert not over, over
