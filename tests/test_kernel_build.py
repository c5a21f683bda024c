"""What the compiler is told and what it makes of the kernels (no GPU: hipcc cross-compiles)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1204_6367_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")


def device_compile(tmp_path, header, *options):
    """Compiles the kernels that `use` names from one header; the compiler's messages and the output file."""
    src = tmp_path / "unit.hip"
    src.write_text(header)
    out = tmp_path / "unit.out"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run(["hipcc", *flags, "--cuda-device-only", "-I", os.path.join(build.ROOT, "include"),
                        "-I", os.path.join(build.HERE, "csrc"), *options, str(src), "-o", str(out)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stderr, out


def test_lanes_of_a_ray_share_their_slots_in_order(tmp_path):
    """With several lanes per ray one lane reads LDS slots that another wrote: four places where
    the source has to order them (after the clearing, before and after a cell of several
    materials for each lane, before the sums).  One lane per ray needs none."""
    use = "\n".join(f"template __global__ void gdrr::raytrace_kernel<{g}, false, true>(gdrr::RtParams);" for g in (1, 4, 16))
    _, out = device_compile(tmp_path, '#include "gdrr.h"\n#include "gdrr_raytrace.h"\n' + use, "-S", "-emit-llvm")
    fences = {}
    for name, body in re.findall(r"^define[^\n]*raytrace_kernelILi(\d+)E[^\n]*\{\n(.*?)^\}", out.read_text(), re.M | re.S):
        fences[int(name)] = len(re.findall(r'fence syncscope\("wavefront"\)', body))
    assert fences[1] == 0 and fences[4] >= 2 + 2 * 4 and fences[16] >= 2 + 2 * 16, fences


def test_whole_images_of_64_and_256_columns_are_held_without_spills(tmp_path):
    """A whole image in the registers of one workgroup (128 a lane) leaves none over: what the loads
    and stores around the sweeps take decides whether any are spilled."""
    use = "\n".join(f"template __global__ void gdrr::denoise_tile_kernel<{k}, false, {s}>(gdrr::DnParams);"
                    for k in ("4, 12, 6", "1, 48, 24") for s in ("false", "true"))
    said, _ = device_compile(tmp_path, '#include "gdrr_denoise.h"\n' + use, "-S", "-Rpass-analysis=kernel-resource-usage")
    spills = re.findall(r"Function Name: \S*denoise_tile_kernel\S*.*?VGPRs Spill: (\d+)", said, re.S)
    assert spills == ["0"] * 4, said[-3000:]
