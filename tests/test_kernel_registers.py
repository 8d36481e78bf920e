"""Kernels whose running sums have to stay in registers: the compiler spills none of them.  Read from the
objects that the build leaves."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJ = os.path.join(ROOT, "paper_1601_06767_amd", "_build", "pair_transform.o")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def _spills(tmp_path):
    fat, dev = str(tmp_path / "fat.bin"), str(tmp_path / "dev.o")
    run = lambda tool, *a: subprocess.run([os.path.join(LLVM, tool), *a], check=True, capture_output=True, text=True).stdout
    run("llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", OBJ, str(tmp_path / "copy.o"))
    run("clang-offload-bundler", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}",
        f"--output={dev}", "--unbundle")
    notes = run("llvm-readelf", "--notes", dev)
    return {m[1]: int(m[2]) for m in re.finditer(r"\.name: +(_Z\S+).*?\.vgpr_spill_count: +(\d+)", notes, re.S)}


@pytest.mark.skipif(not (os.path.exists(OBJ) and shutil.which("llvm-readelf", path=LLVM)),
                    reason="no built objects, or no LLVM tools to read them")
def test_line_sums_of_the_last_stage_stay_in_registers(tmp_path):
    finish = {n: s for n, s in _spills(tmp_path).items() if "k_pair_finish" in n}
    assert len(finish) == 60, len(finish)   # max|n_chi| 1 .. 15, two precisions, rows in LDS or not
    assert not [n for n, s in finish.items() if s > 0]
