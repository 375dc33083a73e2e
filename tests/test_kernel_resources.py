"""What the compiler gave the kernels of this build: those whose time is the
number of waves in flight keep their values in registers."""
import os
import re
import subprocess

import pytest

from helpers import ROOT

LLVM = "/opt/rocm/llvm/bin"
BUILD = os.path.join(ROOT, "paper_2303_07030_amd", "_build")


def kernels(source, tmp_path):
    """{kernel symbol: bytes of scratch per thread} of one compiled source."""
    obj = os.path.join(BUILD, source + ".o")
    if not os.path.exists(obj) or not os.path.exists(os.path.join(LLVM, "clang-offload-bundler")):
        pytest.skip("no object file of this build, or no LLVM tools")
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")

    def run(tool, *args):
        return subprocess.run([os.path.join(LLVM, tool), *args], check=True, capture_output=True,
                              text=True).stdout

    run("llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", obj, str(tmp_path / "obj"))
    run("clang-offload-bundler", "--type=o", "--unbundle",
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={code}")
    notes = run("llvm-readelf", "--notes", code)
    sizes = re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
    names = re.findall(r"\.symbol:\s+'?([^'\s]+)", notes)
    assert len(sizes) == len(names) > 0
    return dict(zip(names, map(int, sizes)))


@pytest.mark.parametrize("source, kernel", [("build.hip", "radix_scatter_kernel")])
def test_no_scratch(source, kernel, tmp_path):
    found = {n: s for n, s in kernels(source, tmp_path).items() if kernel in n}
    assert found
    assert not {n: s for n, s in found.items() if s}
