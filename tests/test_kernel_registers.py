"""Registers of the built walk kernels, from the code object's metadata: at least two waves of every one fit a SIMD (512
registers a lane), whatever the number of values its threads hold."""
import os
import re
import subprocess

import pytest

from paper_2205_03251_amd import gpeval as g

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """Kernel name -> registers a lane (architectural and accumulation), from the built library's own code objects."""
    for tool in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf"):
        if not os.path.exists(f"{LLVM}/{tool}"):
            pytest.skip(f"{tool} is not installed")
    d = tmp_path_factory.mktemp("code")
    obj = os.path.join(os.path.dirname(g.LIB_PATH), "_build", "kernels.o")
    if not os.path.exists(obj):
        pytest.skip("the library's object files are not here")
    fat, co = str(d / "fat.bin"), str(d / "kernels.co")
    subprocess.check_call([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, str(d / "rest.o")])
    subprocess.check_call([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={co}",
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
    out, name, regs = subprocess.check_output([f"{LLVM}/llvm-readelf", "--notes", co], text=True), None, {}
    for block in out.split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block)[1]
        regs[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", block)[1])       # the unified count
    return regs


def test_walks_keep_two_waves_resident(registers):
    walks = {n: r for n, r in registers.items() if "k_walk" in n or "k_coeval" in n}
    assert len(walks) >= 22
    assert {n: r for n, r in walks.items() if r > 256} == {}
