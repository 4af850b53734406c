"""Vector registers of the scan kernels, read from the built library's code-object metadata.

A SIMD holds 512 registers per lane: the FP32 scan in the uniform field (workgroups of 4
waves) keeps to 128, so that four workgroups fit a CU where the LDS allows; adaptive steps
run with 4-step blocks.
"""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    from paper_1908_01949_amd import rknscan
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
    if not all(shutil.which(t) for t in tools):
        pytest.skip("no LLVM tools")
    d = tmp_path_factory.mktemp("co")
    subprocess.run([tools[0], f"--dump-section=.hip_fatbin={d}/fat", rknscan.LIB_PATH, f"{d}/x.so"], check=True)
    out = {}
    # the section holds one bundle per source file
    fat = (d / "fat").read_bytes()
    starts = [m.start() for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", fat)] + [len(fat)]
    for k, (a, b) in enumerate(zip(starts, starts[1:])):
        (d / f"b{k}").write_bytes(fat[a:b])
        subprocess.run([tools[1], "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                        f"--input={d}/b{k}", f"--output={d}/c{k}"], check=True)
        notes = subprocess.run([tools[2], "--notes", f"{d}/c{k}"], capture_output=True, text=True, check=True).stdout
        for part in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name: +(_Z\S+)", part)
            if name:
                out[name.group(1)] = {f: int(re.search(rf"\.{f}: +(\d+)", part).group(1))
                                      for f in ("vgpr_count", "vgpr_spill_count")}
    return out


@pytest.mark.parametrize("block,var", [(4, 0), (4, 1), (4, 2), (6, 0), (6, 1), (8, 0), (8, 1)])
def test_uniform_fp32_scan_fits_four_workgroups(kernels, block, var):
    k = [v for n, v in kernels.items() if f"scan_kernelIfLi0ELi{block}ELi4ELi0ELi{var}ELb0E" in n]
    assert len(k) == 1
    assert k[0]["vgpr_count"] <= 128 and k[0]["vgpr_spill_count"] == 0
