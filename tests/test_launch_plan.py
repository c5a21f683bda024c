"""The LDS of a transport launch (csrc/gdrr_plan.h, plain C++), compiled for the host."""
import os
import shutil
import subprocess

import pytest

from paper_1204_6367_amd import build

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")


def run_cpp(tmp_path, body):
    src = tmp_path / "plan.cpp"
    src.write_text('#include <cstdio>\n#include "gdrr_plan.h"\nusing namespace gdrr;\nint main() {\n' + body + "\n}\n")
    exe = tmp_path / "plan"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", str(exe)], check=True)
    return [[int(x) for x in line.split()] for line in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines()]


def test_started_photons_take_a_kilobyte_a_wavefront(tmp_path):
    """Half a wavefront of started photons fits the 16 bytes a lane that drawing them ahead took, in
    every kind of launch, so that none loses workgroups to them; wavefronts' slots stay 16-byte aligned."""
    rows = run_cpp(tmp_path, 'for (int k = 0; k <= 5; ++k) std::printf("%d %d\\n", kMinSlots, (int)slot_bytes(k));')
    for n, size in rows:
        assert n >= 32 and n * size <= 16 * 64
        assert n * size % 16 == 0 and 64 * size % 16 == 0
