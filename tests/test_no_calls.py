"""The refinement kernels hold no calls: a call makes a recursion that takes all
registers save the caller's through scratch memory, and values kept in lanes of vector
registers across calls once came back wrong.  Disassembles the library built here (no
GPU) and looks for call instructions."""
import os
import shutil
import subprocess

import pytest

from paper_2606_05687_amd import build as b

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_refinement_kernels_make_no_calls(tmp_path):
    lib = shutil.copy(b.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    seen = 0
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / name)],
                              check=True, capture_output=True, text=True).stdout
        if "refine_kernel" not in text and "refine_wide_kernel" not in text:
            continue
        seen += 1
        assert "s_endpgm" in text
        assert "s_swappc" not in text and "s_call" not in text
    assert seen == 2   # one code object per source
