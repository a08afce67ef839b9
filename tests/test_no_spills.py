"""No kernel of the built library keeps registers in scratch memory (no GPU:
the resource counts in the metadata of its gfx950 code object). A spill in the
decode loop costs a memory round trip a step."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2502_00922_amd", "libhufflm.so")
LLVM = "/opt/rocm/llvm/bin"


def test_no_register_spills(tmp_path):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout  # noqa: E731
    fat, obj = str(tmp_path / "fat"), str(tmp_path / "gfx950.o")
    run(f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", LIB, str(tmp_path / "copy"))
    run(f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={obj}",
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950")
    notes = run(f"{LLVM}/llvm-readelf", "--notes", obj)
    kernels = re.findall(r"\.name:\s+(\S+).*?\.sgpr_spill_count:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)", notes, re.S)
    assert len(kernels) > 100, len(kernels)
    spilled = {name: int(v) for name, s, v in kernels if int(v)}
    assert not spilled, spilled
