"""What the built kernels keep in scratch memory: nothing in those that score, cut and gather."""
import os
import re
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_00194_amd", "libfamilyseer.so")
LLVM = "/opt/rocm/llvm/bin/"


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="needs the tools that read the library's own kernels")
def test_scoring_kernels_use_no_scratch(tmp_path):
    here = tmp_path / "lib.so"
    here.symlink_to(LIB)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", str(here)], check=True, capture_output=True, cwd=tmp_path)
    scratch = {}
    for code in tmp_path.glob("lib.so.*gfx950"):
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(code)], check=True, capture_output=True, text=True).stdout
        names = re.findall(r"^\s+\.name:\s+(_Z\S+)$", notes, re.M)
        sizes = re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
        assert len(names) == len(sizes)
        scratch.update(zip(names, map(int, sizes)))
    assert len(scratch) > 30
    assert {name: n for name, n in scratch.items() if n and "train" not in name} == {}
