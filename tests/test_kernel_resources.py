"""Private memory of the built kernels, from the code objects inside the library
this repository builds: a sweep whose context is passed to a call keeps it in
memory, and at orders 12 (d 32) and 16-24 the checkpointing sweep ran 1.6-3 times
slower for it."""
import os
import re
import subprocess

import pytest

from paper_2502_20392_amd import _lib, build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLER = "/opt/rocm/llvm/bin/clang-offload-bundler"


def kernels_of(obj, tmp_path):
    """{kernel<args>: (private bytes, spilled vector registers)} of one unit."""
    co = tmp_path / (os.path.basename(obj) + ".co")
    fat = tmp_path / (os.path.basename(obj) + ".fat")
    subprocess.run(["objcopy", "--dump-section", f".hip_fatbin={fat}", obj, str(tmp_path / "o")],
                   check=True)
    subprocess.run([BUNDLER, "--type=o", f"--input={fat}", "--unbundle", f"--output={co}",
                    f"--targets=hipv4-amdgcn-amd-amdhsa--{build.ARCH}"], check=True)
    notes = subprocess.run([READELF, "--notes", str(co)], capture_output=True, text=True,
                           check=True).stdout
    out = {}
    for block in notes.split("- .agpr_count")[1:]:
        def field(k):
            return int(re.search(rf"\.{k}:\s+(\d+)", block).group(1))
        m = re.search(r"\.symbol:\s+_ZN4sigk\d+(\w+?_kernel)I((?:L[ib]\d+E)+)E", block)
        if m:
            args = ",".join(re.findall(r"L[ib](\d+)E", m.group(2)))
            out[f"{m.group(1)}<{args}>"] = (field("private_segment_fixed_size"),
                                            field("vgpr_spill_count"))
    return out


@pytest.mark.parametrize("order,d", [(12, 32), (16, 8), (16, 32), (20, 16), (20, 32), (24, 8),
                                     (24, 32)])
def test_checkpointing_sweeps_keep_their_context_in_registers(order, d, tmp_path):
    obj = os.path.join(build.BUILD, f"bwd_{order}_{d}.o")
    if not os.path.exists(READELF) or not os.path.exists(BUNDLER):
        pytest.skip("no tools to read the code objects")
    if not os.path.exists(obj):
        pytest.skip("the objects of this build are not kept here")
    got = kernels_of(obj, tmp_path)
    for name in ("ckpt_kernel", "lines_kernel"):
        assert got[f"{name}<{order},{d}>"][0] == 0, got
