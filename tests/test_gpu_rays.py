"""The ray tracer's images do not depend on how many lanes trace a ray."""
import numpy as np
import pytest

from paper_1204_6367_amd import workloads as W

from test_gpu_raytrace import check_image

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_6367_amd import api
    return api


@pytest.mark.parametrize("interp", [True, False])
@pytest.mark.parametrize("n_mat, shape", [(3, (1, 1, 1)), (4, (21, 30, 33)), (15, (9, 8, 7)), (16, (70, 12, 11))])
def test_lanes_per_ray(gpu, n_mat, shape, interp):
    """One, four and sixteen lanes per ray (more than 512, up to 512 and up to 64 tiles in the
    call) give the same bits: noisy materials (most cells mixed), blocks of one material (the
    last one's number is the mark of cells to look up), detectors of one pixel to odd tiles,
    a joint source."""
    import torch
    rng = np.random.default_rng(n_mat)
    names = [["air", "soft_tissue", "bone", "lung", "aluminium", "water"][k % 6] for k in range(n_mat)]
    mat = rng.integers(0, n_mat, shape).astype(np.uint8)
    mat[: (shape[0] + 1) // 2] = n_mat - 1
    dens = rng.uniform(0.0, 2.0, shape).astype(np.float32)
    dens.flat[:: 5] = rng.choice(np.array([0.0, -0.0, -1.0, np.nan], np.float32), dens.flat[:: 5].shape)
    ph = W.Phantom(dens, mat, (150.0 / shape[2], 140.0 / shape[1], 130.0 / shape[0]), names)
    for nu, nv in ((1, 1), (17, 31), (45, 40)):
        geom = W.Geometry(nu=nu, nv=nv, du_mm=240.0 / nu, dv_mm=200.0 / nv)
        prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom, joint=nu > 1), geom, 1)
        vol, phys, src = gpu.upload(prob)
        tiles = ((nu + 15) // 16) * ((nv + 15) // 16)
        jobs = [gpu.JobSpec(geom.replace(phi_rad=0.11 * k, theta_rad=0.02 * (k % 3)), 0, k)
                for k in range(513 // tiles + 1)]
        many = gpu.Batch([vol], phys, [src], jobs).primary(interp=interp)              # one lane
        some = gpu.Batch([vol], phys, [src], jobs[: 65 // tiles + 1]).primary(interp=interp)   # four
        assert 64 < tiles * len(some) <= 512 < tiles * len(many)
        for k in range(len(some)):
            assert torch.equal(some[k], many[k]), (nu, k)
        for k in (0, 7):
            one = gpu.Batch([vol], phys, [src], [jobs[k]]).primary(interp=interp)      # sixteen
            assert torch.equal(one[0], many[k]), (nu, k)
        assert float(sum(m.sum() for m in many)) > 0


def test_records_with_rows_beyond_24_bits(gpu):
    """A volume whose rows of plane records are 2^24 apart takes the full products: the oracle's
    image, and with one, four and sixteen lanes per ray the same bits."""
    import oracle
    import torch
    names = ["air", "soft_tissue", "bone"]
    geom = W.Geometry(nu=9, nv=7, du_mm=40.0, dv_mm=40.0)
    z, y, x = np.ogrid[0:4100, 0:2, 0:4100]
    mat = (1 + ((z // 100 + x // 70 + y) % 2)).astype(np.uint8)
    dens = np.broadcast_to(0.2 + 0.1 * np.sin(x / 300.0) + 0.05 * y, mat.shape).astype(np.float32)
    ph = W.Phantom(dens, mat, (0.1, 150.0, 0.1), names)
    prob = W.Problem(ph, W.physics_for(ph), W.pelvis_source(geom), geom, 1)
    vol, phys, src = gpu.upload(prob)
    images = []
    for n_jobs in (1, 100, 600):
        jobs = [gpu.JobSpec(geom.replace(phi_rad=geom.phi_rad + 0.01 * k), 0, k) for k in range(n_jobs)]
        images.append(gpu.Batch([vol], phys, [src], jobs).primary()[0].clone())
    assert torch.equal(images[0], images[1]) and torch.equal(images[0], images[2])
    check_image(images[0].cpu().numpy(), oracle.primary_raytrace(oracle.Problem.from_workload(prob)), "rows beyond 2^24")


def test_more_cell_rows_than_a_launch_has_workgroups(gpu):
    """2^24 rows of cells, a tile of plane records each: a launch of that many workgroups would
    have 2^32 lanes.  Density linear in y, which 300 rows of 1 mm interpolate as well; float32 sums
    of about 600 intervals (2^-24 each) over an optical depth of 4 differ by less than 2e-4."""
    import torch
    geom = W.Geometry(nu=17, nv=3, du_mm=20.0, dv_mm=20.0)
    images = []
    for ny in (300, 1 << 24):
        dy = 300.0 / ny
        y = (torch.arange(ny, device="cuda", dtype=torch.float64) + 0.5) * dy
        dens = (0.5 + y / 300.0).float().reshape(1, ny, 1)
        mat = torch.ones((1, ny, 1), dtype=torch.uint8, device="cuda")
        small = W.Phantom(np.ones((1, 1, 1), np.float32), np.ones((1, 1, 1), np.uint8), (1.0, 1.0, 1.0), ["air", "soft_tissue"])
        _, phys, src = gpu.upload(W.Problem(small, W.physics_for(small), W.pelvis_source(geom), geom, 1))
        vol = gpu.DeviceVolume(dens, mat, (150.0, dy, 200.0))
        images.append(gpu.Batch([vol], phys, [src], [gpu.JobSpec(geom, 0, 0)]).primary(step_mm=0.25)[0].clone())
    assert float(images[0].min()) > 0
    assert float(((images[1] - images[0]) / images[0]).abs().max()) < 2e-4
