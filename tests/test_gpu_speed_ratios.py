"""Kernel times against each other, where a path was once far slower than its neighbour.
Bounds lie between the two, and times are the shortest of several."""
import pytest

from paper_1204_6367_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    api.enable_timing(True)
    yield api
    api.enable_timing(False)


def shortest(gpu, call, n=5):
    call()
    times = []
    for _ in range(n):
        call()
        times.append(gpu.last_kernel_ms())
    return min(times)


def rays(gpu, shape, n_images, noise):
    """16 or more images of 256 x 192 (one lane per ray) of an ellipsoid phantom, a share of its materials at random."""
    import torch
    nz, ny, nx = shape
    ph = W.ellipsoid_phantom(shape, (400.0 / nz, 500.0 / ny, 500.0 / nx), 5, n_inner=6)
    geom = W.Geometry()
    vol, phys, src = gpu.upload(W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1))
    g = torch.Generator(device="cuda").manual_seed(1)
    at = torch.rand(vol.material.shape, device="cuda", generator=g) < noise
    some = (torch.rand(vol.material.shape, device="cuda", generator=g) * len(ph.materials)).to(torch.uint8)
    vol.material = torch.where(at, some, vol.material).contiguous()
    return gpu.Batch([vol], phys, [src], [gpu.JobSpec(geom.replace(phi_rad=0.37 * k), 0, k) for k in range(n_images)])


def test_cells_of_several_materials(gpu):
    """Rays through noise take 1.6 times as long as through the phantom; 7.8 times with materials
    read from the voxels one by one."""
    clean, noisy = (rays(gpu, (160, 256, 256), 16, p) for p in (0.0, 1.0))
    assert shortest(gpu, noisy.primary) < 3.5 * shortest(gpu, clean.primary)


def test_nearest_voxel_rays(gpu):
    """The nearest voxel's density costs no more than the interpolated one; 1.5 times as much
    when the wavefronts lie across the voxel rows."""
    b = rays(gpu, (64, 64, 64), 16, 0.0)
    assert shortest(gpu, lambda: b.primary(interp=False)) < 1.25 * shortest(gpu, b.primary)


def test_single_majorant_of_nine_materials(gpu):
    """A single majorant of more than 8 materials is screened too: 1.4 times as long as with 4, 3.2 times
    when every cube of several materials had its points tested."""
    import numpy as np
    import torch
    shape = (160, 256, 256)
    ph = W.ellipsoid_phantom(shape, (2.5, 1.95, 1.95), 5, n_inner=6)
    geom = W.Geometry()
    prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1)
    vol, phys, src = gpu.upload(prob)
    n = len(ph.materials)
    few = gpu.Batch([vol], phys, [src], [gpu.JobSpec(geom, 6_000_000, 0)])
    more = W.Physics(np.concatenate([prob.physics.mu_mass] * 3)[:9], prob.physics.grid, None)
    prob9 = W.Problem(ph, more, prob.source, geom, 1)
    vol9, phys9, src9 = gpu.upload(prob9)
    layer = (torch.arange(shape[2], device="cuda") // 8 % 3).to(torch.uint8) * n
    vol9.material = ((vol9.material + layer) % 9).to(torch.uint8).contiguous()
    many = gpu.Batch([vol9], phys9, [src9], [gpu.JobSpec(geom, 6_000_000, 0)])
    times = [shortest(gpu, lambda b=b: b.project(seed=1, sumsq=False)) for b in (few, many)]
    print(times)
    assert times[1] < 2.2 * times[0]


def test_majorant_of_a_tall_volume(gpu):
    """200000 voxels on top of each other cost what they cost in a row (5.4 times as much with one column
    of cells per lane and the other lanes idle)."""
    import torch
    ph = W.ellipsoid_phantom((4, 4, 4), (10.0, 10.0, 10.0), 5, n_inner=1)
    geom = W.Geometry()
    _, phys, _ = gpu.upload(W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1))
    times = []
    for shape in ((1, 1, 200_000), (200_000, 1, 1)):
        vol = gpu.DeviceVolume(torch.rand(shape, device="cuda"), torch.ones(shape, dtype=torch.uint8, device="cuda"), (1.0, 1.0, 1.0))
        ms = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                gpu.majorant(vol, phys)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        times.append(min(ms))
    assert times[1] < 2.5 * times[0], times


def test_majorant_of_the_voxels_themselves(gpu):
    """Without interpolation the maximum needs one read of each voxel: half of the time of the
    neighbourhoods' maximum for a large volume, no less than it when every cell read its corners."""
    import torch
    ph = W.ellipsoid_phantom((4, 4, 4), (10.0, 10.0, 10.0), 5, n_inner=1)
    geom = W.Geometry()
    _, phys, _ = gpu.upload(W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1))
    shape = (256, 512, 512)
    vol = gpu.DeviceVolume(torch.rand(shape, device="cuda"), torch.ones(shape, dtype=torch.uint8, device="cuda"), (1.0, 1.0, 1.0))
    times = []
    for interp in (True, False):
        ms = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                gpu.majorant(vol, phys, interp)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        times.append(min(ms))
    assert times[1] < 0.8 * times[0], times
