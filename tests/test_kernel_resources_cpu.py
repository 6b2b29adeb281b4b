"""What the host assumes about the built kernels' own LDS, read from the notes of the built library: the fused kernels' dynamic
share of a compute unit's 160 KB is sized with an upper bound of their static LDS, and the grid with the workgroups that then fit."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2601_16986_amd import ckv

LLVM = "/opt/rocm/llvm/bin"


def _tool(name):
    path = os.path.join(LLVM, name)
    path = path if os.path.exists(path) else shutil.which(name)
    if not path:
        pytest.skip(f"{name} not found")
    return path


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: {field: number}} of the library's kernels."""
    tmp = tmp_path_factory.mktemp("co")
    fat, co = str(tmp / "fat"), str(tmp / "co")
    subprocess.run([_tool("llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", ckv.LIB_PATH, str(tmp / "copy.so")], check=True)
    subprocess.run([_tool("clang-offload-bundler"), "--type=o", "--unbundle", f"--input={fat}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={co}"], check=True)
    notes = subprocess.run([_tool("llvm-readelf"), "--notes", co], check=True, capture_output=True, text=True).stdout
    got = {}
    for block in re.split(r"\n  - ", notes):
        name = re.search(r"\.name:\s+(_Z\S+)", block)
        if name:
            got[name.group(1)] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)$", block, re.M)}
    return got


# 160 KB / 2 and / 4, less these, are the fused kernels' dynamic LDS (ckv_init)
@pytest.mark.parametrize("waves,bound", [(4, 11 * 1024), (2, 6 * 1024)])
def test_static_lds_of_the_fused_kernels(kernels, waves, bound):
    name = [n for n in kernels if f"unit_kernelILi{waves}E" in n]
    assert len(name) == 1, name
    assert 0 < kernels[name[0]]["group_segment_fixed_size"] <= bound


def test_static_lds_of_kernels_that_hold_a_value_per_entry(kernels):
    """Their dynamic LDS takes 4 bytes per entry and a bit, up to 132 KB; 12 KB are left for what they declare."""
    names = [n for n in kernels if "finish_kernel" in n or "seed_hits_kernelILi0E" in n or "layer_step_kernel" in n]
    assert len(names) == 3 + 6
    assert all(kernels[n]["group_segment_fixed_size"] <= 12 * 1024 for n in names)
