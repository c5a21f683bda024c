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


@pytest.mark.parametrize("words, waves, most, slot, least_rows", [
    (1960, 8, 4, 24, 6), (1960, 4, 8, 24, 6), (3 * 1960, 8, 4, 24, 6), (3 * 1960, 16, 2, 24, 6),     # one and three phantoms, 40 mm cubes
    (3564, 4, 8, 28, 2), (3564, 8, 4, 28, 6), (3564, 16, 2, 28, 6), (1960, 16, 1, 24, 6),     # (28 bytes: screened)
    (28000, 16, 2, 24, 0), (40, 1, 32, 24, 0)])
def test_rows_before_slots_before_workgroups(tmp_path, words, waves, most, slot, least_rows):
    """4 materials on 299 energies (rows of 2392 bytes, 11 sets): room for half of the sets at the
    price of slots, then of at most half of the workgroups (for two of them if a screened launch
    would be left with fewer than 24 wavefronts); what is planned fits."""
    row, lds = 299 * 8, 160 * 1024
    fixed = 4 * row + 4 * words
    for wanted in (0, 1, 2, 64):
        (slots, rows, per_cu, size), = run_cpp(tmp_path, f"""
            const LdsPlan p = plan_lds({fixed}, {row}, 11, {slot} == 28, {waves}, {slot}, {lds}, {most}, {wanted});
            std::printf("%d %d %d %d\\n", p.slots, p.rows, p.per_cu, (int)p.bytes);""")
        assert slots in (32, 64) and 0 <= rows <= 11 and 1 <= per_cu <= most
        assert size == (fixed + rows * row + 15) // 16 * 16 + waves * slots * slot
        assert per_cu * ((size + 1279) // 1280) <= 128
        if wanted in (0, 1):
            assert rows >= least_rows
        if wanted == 0:
            alone = (fixed + 15) // 16 * 16 + waves * 32 * slot
            assert 2 * per_cu >= min(most, 128 // ((alone + 1279) // 1280))


def test_what_does_not_fit_is_not_planned(tmp_path):
    (slots, rows, per_cu, size), = run_cpp(tmp_path, """
        const LdsPlan p = plan_lds(163000, 2392, 11, false, 4, 24u, 163840, 8, 0);
        std::printf("%d %d %d %d\\n", p.slots, p.rows, p.per_cu, (int)p.bytes);""")
    assert per_cu == 0 and size > 163840


@pytest.mark.parametrize("msy, msz", [(2, 4), (2, 6), (3, 9), (7, 49), (14, 140), (21, 462), (61, 4331), (514, 1028), (2, 1026), (14000, 28000)])
def test_cube_numbers_from_float_reciprocals(msy, msz):
    """A cube without a row finds its grid place by two divisions in float32: exact for every
    word of a 112 KiB grid, with reciprocals up to 2 ulp off."""
    import numpy as np
    c = np.arange(28672)
    f = np.float32
    for ulp in (-2, -1, 0, 1, 2):
        def quotient(n, d):
            r = (np.array([f(1) / f(d)], f).view(np.int32) + np.int32(ulp)).view(f)[0]
            return ((n.astype(f) + f(0.5)) * r).astype(np.int64)
        z = quotient(c, msz)
        y = quotient(c - z * msz, msy)
        assert (z == c // msz).all() and (y == (c % msz) // msy).all()


def test_default_tuning_is_a_shape_for_every_launch():
    """What gdrr_default_tuning returns may be passed to any call: not the shape of one kind of launch."""
    import ctypes as C

    from paper_1204_6367_amd import _abi
    if not os.path.exists(_abi.LIB_PATH):
        build.build()
    t = _abi.Tuning()
    assert _abi.lib().gdrr_default_tuning(C.byref(t)) == 0
    assert (t.block, t.blocks_per_cu, t.chunk, t.defer, t.coll_defer) == (256, 0, 0, 32, 0)
