"""CPU test of the built kernels' registers (the code objects' own notes): the
passes with staged records, held to a number of wavefronts per SIMD, keep what
their loops use in registers."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1107_2619_amd", "libmdeam.so")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def _kernels(tmp_path):
    """{mangled name: VGPRs spilled} of every gfx950 kernel of the library."""
    lib = str(tmp_path / "lib.so")
    shutil.copy(LIB, lib)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True)
    out = {}
    for name in os.listdir(tmp_path):
        if not name.endswith("gfx950"):
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(tmp_path / name)], check=True,
                               capture_output=True, text=True).stdout
        for block in notes.split("- .agpr_count")[1:]:
            symbol = re.search(r"\.name:\s*(\S+)", re.sub(r"\.args:.*?(?=\n    \.\w)", "", block, flags=re.S))
            spills = re.search(r"\.vgpr_spill_count:\s*(\d+)", block)
            out[symbol.group(1)] = int(spills.group(1))
    return out


def test_staged_passes_do_not_spill(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("the built library or llvm-readelf is missing")
    kernels = _kernels(tmp_path)
    # the last template argument: staged records
    staged = {k: v for k, v in kernels.items() if re.search(r"k_(force|density)I\w*Lb1EEEvNS_", k)}
    assert len(staged) > 50
    assert [k for k, v in staged.items() if v] == []
